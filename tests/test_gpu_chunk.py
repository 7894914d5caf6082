"""Steps of more than 32 query rows per KV head (T > 1) against the oracle:
edges of the query tiles and key tiles, every pair of head sizes, ragged,
empty and clipped lengths, items cut over many workgroups and items that may
not be cut, and values that need care as 16-bit operands: magnitudes far from
1, growing and falling ones, infinities and NaN.  The small shapes stay with
the decode kernels; the ones after them take the chunk kernels.

Tolerance: 1e-5 of V's largest magnitude, as for the other decodes at N(0, 1)
(values of about 4: the fp32 sums of at most a few thousand terms and the
products that are left out, at most 2^-24 of each term, stay below 1e-6 of
it)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_19456_amd import binding
from paper_2607_19456_amd.workloads import normal

pytestmark = pytest.mark.gpu


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def inputs(B, h_q, h_kv, d_k, d_v, n_max, T, lens, seed=5):
    q = normal(seed, 1, (B, h_q, T, d_k))
    K = normal(seed, 2, (B, h_kv, n_max, d_k))
    V = normal(seed, 3, (B, h_kv, n_max, d_v))
    kn = normal(seed, 4, (B, h_kv, T, d_k))
    vn = normal(seed, 5, (B, h_kv, T, d_v))
    for b, n in enumerate(lens):
        K[b, :, max(n, 0):] = np.nan
        V[b, :, max(n, 0):] = np.nan
    return q, K, V, kn, vn, np.array(lens, np.int32)


def check(got, ref, scale, what):
    got = got.cpu().numpy().astype(np.float64)
    same = np.isnan(ref) == np.isnan(got)
    assert same.all(), f"{what}: NaN where there is none, or none where there is one"
    err = float(np.nanmax(np.abs(got - ref))) if np.isfinite(ref).any() else 0.0
    print(f"  {what}: max-abs-err {err:.3e}", flush=True)
    assert err <= 1e-5 * scale, f"{what}: {err:.3e}"


def run_both(B, h_q, h_kv, d_k, d_v, n_max, T, lens, change=None, vscale=1.0):
    q, K, V, kn, vn, ln = inputs(B, h_q, h_kv, d_k, d_v, n_max, T, lens)
    if change:
        change(q, K, V, kn, vn)
    sc = np.float32(d_k ** -0.5)
    print("chunk", B, h_q, h_kv, d_k, d_v, n_max, T, list(lens)[:6], flush=True)
    dq, dK, dV, dl = dev(q), dev(K), dev(V), dev(ln)
    ws = binding.alloc_multi_workspace(dq, dK, dV)
    nc = binding.workspace_counter_bytes(B, h_q * T, h_kv, n_max, d_k, d_v)
    ws.fill_(0xFF)
    ws[:nc].zero_()
    with np.errstate(all="ignore"):
        out = binding.decode_multi(dq, dK, dV, dl, float(sc), workspace=ws)
        torch.cuda.synchronize()
        assert not ws[:nc].any()
        check(out, oracle.decode_multi(q, K, V, ln, sc), vscale, "multi")
        out = binding.decode_multi_step(dq, dK, dV, dev(kn), dev(vn), dl, float(sc), workspace=ws)
        torch.cuda.synchronize()
        assert not ws[:nc].any()
        before = ln.copy()
        oracle.append_rows(K, V, kn, vn, ln)
    assert dl.cpu().numpy().tolist() == ln.tolist()
    assert np.array_equal(dK.cpu().numpy().view(np.uint32), K.view(np.uint32))
    assert np.array_equal(dV.cpu().numpy().view(np.uint32), V.view(np.uint32))
    # Where every row fits the step is append, then multi; row r of the
    # others sees min(len + r + 1, n_max) rows (none below zero).
    ref = np.zeros((B, h_q, T, d_v))
    fits = (before >= 0) & (before + T <= n_max)
    with np.errstate(all="ignore"):
        full = oracle.decode_multi(q, K, V, ln, sc)
        ref[fits] = full[fits]
        for b in np.nonzero(~fits)[0]:
            for r in range(T):
                n = min(int(before[b]) + r + 1, n_max) if before[b] >= 0 else 0
                ref[b, :, r] = oracle.decode(np.ascontiguousarray(q[b:b + 1, :, r]), K[b:b + 1],
                                             V[b:b + 1], np.array([n], np.int32), sc)[0]
    check(out, ref, vscale, "step")


SHAPES = [
    # B, h_q, h_kv, d_k, d_v, n_max, T, lens
    (2, 3, 1, 128, 128, 200, 11, [33, 0]),                # 33 rows: the smallest
    (1, 1, 1, 128, 128, 700, 256, [31]),                  # one whole query tile
    (2, 2, 2, 128, 128, 700, 257, [32, 443]),             # one row in the second
    (3, 5, 1, 128, 128, 500, 52, [449, 460, -2]),         # tiles across heads; clipped; negative
    (2, 8, 2, 64, 64, 1000, 100, [0, 900]),
    (2, 4, 1, 64, 128, 400, 20, [129, 77]),
    (2, 4, 1, 128, 64, 400, 20, [128, 380]),
    (1, 4, 2, 64, 256, 400, 33, [300]),
    (1, 4, 2, 256, 64, 400, 33, [301]),
    (1, 4, 2, 128, 256, 400, 33, [95]),
    (1, 4, 2, 256, 128, 400, 33, [96]),
    (2, 4, 2, 256, 256, 900, 70, [640, 1]),
    (300, 2, 2, 64, 64, 90, 40, [(7 * b) % 91 for b in range(300)]),   # items may not be cut
    (1, 4, 1, 64, 64, 40000, 10, [39985]),                # more units than slots
    (1, 2, 1, 64, 64, 3000, 2048, [952]),                 # many query tiles
    # Enough work for the chunk kernels.
    (32, 5, 1, 128, 128, 900, 13, [33, 0, 31, 32, 800, 887, 890, -2] * 4),   # 65 rows: the fewest
    (32, 1, 1, 128, 128, 900, 256, [31, 0, 32, 643, 644, 700, 899, 900] * 4),    # one whole tile
    (16, 4, 2, 128, 128, 800, 129, [32, 443] * 8),        # two rows in the second; across heads
    (32, 2, 1, 64, 64, 1000, 100, [0, 900] * 16),
    (32, 4, 1, 64, 128, 800, 20, [129, 77] * 16),
    (32, 4, 1, 128, 64, 800, 20, [128, 380] * 16),
    (16, 4, 2, 64, 256, 800, 33, [300, 799] * 8),
    (16, 4, 2, 256, 64, 800, 33, [301, 0] * 8),
    (16, 4, 2, 128, 256, 800, 33, [95, 97] * 8),
    (16, 4, 2, 256, 128, 800, 33, [96, 3] * 8),
    (16, 4, 2, 256, 256, 900, 70, [640, 1] * 8),
    (128, 8, 1, 64, 64, 1100, 5, [(9 * b) % 1101 for b in range(128)]),  # two groups, short caches
    (180, 2, 1, 256, 256, 90, 40, [b % 91 for b in range(180)]),  # items may not be cut
    (1, 8, 1, 64, 64, 40000, 128, [39800]),               # more units than slots
]


@pytest.mark.parametrize("shape", SHAPES, ids=[str(i) for i in range(len(SHAPES))])
def test_chunk_shapes(cuda_device, shape):
    run_both(*shape)


# The same step where the decode kernels take it and where the chunk kernels do.
BASE = {"decode": (1, 4, 1, 128, 128, 600, 40, [500]),
        "chunk": (32, 4, 1, 128, 128, 800, 40, [500] * 32)}
# For what must stay with the rows that see it: other sizes, the direct form.
MORE = {"decode_64": (2, 4, 1, 64, 64, 900, 40, [500] * 2),
        "decode_256": (1, 4, 1, 256, 256, 600, 40, [500]),
        "decode_64_256": (1, 4, 1, 64, 256, 600, 40, [500]),
        "decode_direct": (60, 4, 1, 64, 64, 600, 40, [500] * 60),
        "chunk_256": (32, 4, 1, 256, 256, 800, 40, [500] * 32)}


@pytest.fixture(params=BASE)
def base(request):
    return BASE[request.param]


def scaled(kf, qf, vf):
    def change(q, K, V, kn, vn):
        for x, f in ((q, qf), (K, kf), (kn, kf), (V, vf), (vn, vf)):
            x *= np.float32(f)
    return change


@pytest.mark.parametrize("kf,qf,vf", [(1e4, 1e-4, 1e-20), (1e-12, 1e12, 1e20), (3e-30, 3e29, 1.0),
                                      (1e-3, 1.0, 1e-3)])
def test_chunk_magnitudes(cuda_device, base, kf, qf, vf):
    run_both(*base, change=scaled(kf, qf, vf), vscale=vf)


def test_chunk_growing_values(cuda_device, base):
    """V (and K) outgrow the first tile's scale again and again."""
    def change(q, K, V, kn, vn):
        V *= (2.0 ** (np.arange(V.shape[2]) // 50)).astype(np.float32)[None, None, :, None]
        vn *= np.float32(2.0 ** 11)
        K[:, :, 200:] *= 16
        q /= 16
    run_both(*base, change=change, vscale=2.0 ** 11)


@pytest.mark.parametrize("small", ["V", "K"])
def test_chunk_falling_values(cuda_device, base, small):
    """A tile of very large values first, then ordinary ones; q has no part in
    the large keys, so the ordinary ones decide."""
    def change(q, K, V, kn, vn):
        q[..., 0] = 0
        if small == "V":
            K[:, :, :32] = 0
            K[:, :, :32, 1] = -60 * np.sign(q[0, 0, 0, 1])
            q[..., 1] = q[0, 0, 0, 1]
            q[..., 1] = np.sign(q[0, 0, 0, 1]) * 40
            K[:, :, 32:, 1] = 0
            kn[..., 1] = 0
            V[:, :, :32] *= np.float32(1e9)
        else:
            K[:, :, :32] = 0
            K[:, :, :32, 0] = 1e12
    run_both(*base, change=change)


@pytest.mark.parametrize("where", ["k_neg_inf", "k_nan", "v_inf", "v_nan_new", "q_nan", "k_huge"])
@pytest.mark.parametrize("shape", {**BASE, **MORE})
def test_chunk_non_finite(cuda_device, where, shape):
    """A key of -inf has no weight, a NaN or an infinite value reaches the rows
    that see it and no others (rows before it in the chunk stay finite)."""
    def change(q, K, V, kn, vn):
        if where == "k_neg_inf":
            q[..., 5] = np.abs(q[..., 5]) + 0.5
            K[0, 0, 77, 5] = -np.inf
            kn[0, 0, 3, 5] = -np.inf
        elif where == "k_nan":
            kn[0, 0, 20, 9] = np.nan
        elif where == "v_inf":
            vn[0, 0, 20, 9] = np.inf
        elif where == "v_nan_new":
            vn[0, 0, 39] = np.nan
        elif where == "q_nan":
            q[0, 2, 7, 3] = np.nan
        else:
            K[0, 0, 100] = np.float32(3.3e38)
            q[...] = -np.abs(q)
    shape = {**BASE, **MORE}[shape]
    B, h_q, h_kv, d_k, d_v, n_max, T, lens = shape
    q, K, V, kn, vn, ln = inputs(*shape)
    change(q, K, V, kn, vn)
    sc = np.float32(d_k ** -0.5)
    print("chunk non-finite", where, shape[:7], flush=True)
    dq, dK, dV, dl = dev(q), dev(K), dev(V), dev(ln)
    step = binding.decode_multi_step(dq, dK, dV, dev(kn), dev(vn), dl, float(sc))
    multi = binding.decode_multi(dq, dK, dV, dl, float(sc))   # the same positions again
    torch.cuda.synchronize()
    outs = [x.cpu().numpy().astype(np.float64)[0] for x in (step, multi)]
    Kf, Vf = (np.concatenate([x[0, 0, :500], y[0, 0]]).astype(np.float64)
              for x, y in ((K, kn), (V, vn)))
    with np.errstate(all="ignore"):
        for h in range(h_q):
            for r in range(T):
                n = 500 + r + 1
                s = Kf[:n] @ q[0, h, r].astype(np.float64) * sc
                if where == "k_huge":
                    s[100] = -np.inf                       # overflows in 32 bits
                p = np.exp(s - s.max())
                p[s == -np.inf] = 0
                p /= p.sum()
                ref = p @ Vf[:n]
                ok = np.isfinite(ref)
                for got in outs:
                    assert np.array_equal(np.isnan(ref), np.isnan(got[h, r])), (h, r)
                    assert np.array_equal(np.isinf(ref), np.isinf(got[h, r])), (h, r)
                    assert not ok.any() or np.max(np.abs(ref[ok] - got[h, r][ok])) <= 1e-5, (h, r)


def test_chunk_replays_in_a_graph(cuda_device):
    """A captured step, replayed after eager work, equals the eager step."""
    B, h_q, h_kv, d_k, d_v, n_max, T, lens = 2, 8, 2, 128, 128, 700, 30, [100, 333]
    q, K, V, kn, vn, ln = inputs(B, h_q, h_kv, d_k, d_v, n_max, T, lens)
    K, V = np.nan_to_num(K), np.nan_to_num(V)
    sc = float(np.float32(d_k ** -0.5))
    dq, dK, dV, dl, dkn, dvn = dev(q), dev(K), dev(V), dev(ln), dev(kn), dev(vn)
    start = dl.clone()
    ws = binding.alloc_multi_workspace(dq, dK, dV)
    out = torch.empty((B, h_q, T, d_v), device="cuda")
    eager = binding.decode_multi_step(dq, dK, dV, dkn, dvn, dl, sc, workspace=ws).clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dl.copy_(start)
        binding.decode_multi_step(dq, dK, dV, dkn, dvn, dl, sc, out=out, workspace=ws)
    for k in range(4):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), k
        assert dl.tolist() == [n + T for n in lens]
        binding.decode_multi(dq, dK, dV, dl, sc, workspace=ws)
