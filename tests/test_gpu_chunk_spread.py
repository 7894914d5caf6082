"""The chunk kernels (more than 32 query rows per KV head, T > 1) on finite
inputs whose elements differ widely in magnitude within a row, a column or a
tile: every output element is compared by itself, so that a small column, or a
row whose weight lies on small values, counts as much as a large one.

Tolerance, per output element d of a query row, from 32-bit arithmetic alone:
  (16 + 4 S) 2^-24 sum_k a_k |V_kd|,   S = max_k scale sum_j |q_j K_kj|.
A score is off by the roundings of its sum, each at most 2^-24 S: d_k of them
at the very most, of either sign, so that 4 S is seldom reached; every weight is
off by as much.  The weights' exponentials, their sum and the sum over keys add
a few units each (16).  The plain fp32 kernels are held to the same."""
import numpy as np
import pytest
import torch

from paper_2607_19456_amd import binding
from paper_2607_19456_amd.workloads import normal

pytestmark = pytest.mark.gpu

# 32 sequences of 80 query rows on one KV head: enough for the chunk kernels.
B, LEN, T, H, N_MAX = 32, 200, 20, 4, 800


def k_channel(f, g):
    def change(q, K, V):
        K[..., 0] *= np.float32(f)
        q[..., 0] *= np.float32(g)
    return change


def k_mixed(q, K, V):
    """Every channel another power of ten, q the other way."""
    e = np.linspace(-12, 12, K.shape[-1])
    np.random.default_rng(3).shuffle(e)
    K *= (10.0 ** e).astype(np.float32)
    q *= (10.0 ** -e).astype(np.float32)


def v_columns(f):
    def change(q, K, V):
        V[..., 1:] *= np.float32(f)
    return change


def v_column_large(f):
    def change(q, K, V):
        V[..., 5] *= np.float32(f)
    return change


def strong_key(gap, value):
    """The first key stands `gap` powers of two above the others for every row
    and holds only `value` (an attention sink)."""
    def change(q, K, V):
        d = K.shape[-1]
        K[..., :4] = 0
        q[..., :4] = 0
        q[..., 0] = 8
        K[:, :, 0] = 0
        K[:, :, 0, 0] = gap * np.log(2.0) * d ** 0.5 / 8
        V[:, :, 0] = value
    return change


def large_row(gap, value):
    """Key 40, in a tile of ordinary ones, stands `gap` powers of two below them
    and holds values that much larger than its weight is small."""
    def change(q, K, V):
        d = K.shape[-1]
        K[..., :4] = 0
        q[..., :4] = 0
        q[..., 0] = 8
        K[:, :, 40] = 0
        K[:, :, 40, 0] = -gap * np.log(2.0) * d ** 0.5 / 8
        V[:, :, 40] *= np.float32(value)
    return change


def strong_small_key_for_one_row(q, K, V):
    """One query row has all its weight on a key whose values are small in half
    of the columns."""
    d = K.shape[-1]
    K[..., 0] = 0
    K[:, :, 77, 0] = 60
    q[..., 0] = 0
    q[:, 1, 3, 0] = d ** 0.5
    V[:, :, 77, ::2] *= np.float32(1e-9)


CASES = {
    "as_it_is": lambda q, K, V: None,
    "k_channel_1e5": k_channel(1e5, 1e-5),
    "k_channel_1e7": k_channel(1e7, 1e-7),
    "k_channel_1e9_q0": k_channel(1e9, 0),
    "k_channel_1e12_q0": k_channel(1e12, 0),
    "k_mixed": k_mixed,
    "v_columns_2^-22": v_columns(2.0 ** -22),
    "v_columns_2^-37": v_columns(2.0 ** -37),
    "v_columns_1e-30": v_columns(1e-30),
    "v_column_1e7": v_column_large(1e7),
    "v_column_1e30": v_column_large(1e30),
    "sink_24": strong_key(24, 0),
    "sink_34": strong_key(34, 0),
    "sink_100": strong_key(100, 0),
    "sink_small": strong_key(60, 1e-9),
    "large_row_30": large_row(30, 2.0 ** 30),
    "large_row_60": large_row(60, 2.0 ** 62),
    "one_row": strong_small_key_for_one_row,
    "padding_1e-6": lambda q, K, V: (K[:, :, 32:96].__imul__(np.float32(1e-6)),
                                     V[:, :, 32:96].__imul__(np.float32(1e-6))),
    "zero_head": lambda q, K, V: (K[:, :, :64].fill(0), V[:, :, :64].fill(0),
                                  V[:, :, 64:].__imul__(np.float32(100))),
    "zero_q_k": lambda q, K, V: (q.fill(0), K.fill(0)),
    "tiny_k_huge_q": lambda q, K, V: (K.__imul__(np.float32(1e-17)), q.__imul__(np.float32(1e17))),
}


def reference(q, K, V, n, scale):
    """Output and tolerance in 64 bits; q [H, T, d], K [n_max, d]."""
    ref = np.zeros((H, T, V.shape[1]))
    tol = np.zeros_like(ref)
    K, V = K.astype(np.float64), V.astype(np.float64)
    for h in range(H):
        for r in range(T):
            m = n - T + r + 1
            x = q[h, r].astype(np.float64) * scale
            s = K[:m] @ x
            p = np.exp(s - s.max())
            p /= p.sum()
            S = (np.abs(K[:m]) @ np.abs(x)).max()
            ref[h, r] = p @ V[:m]
            tol[h, r] = (16 + 4 * S) * 2.0 ** -24 * (p @ np.abs(V[:m]))
    return ref, tol


@pytest.mark.parametrize("dims", [(128, 128), (64, 64), (256, 256)], ids=["128", "64", "256"])
@pytest.mark.parametrize("case", CASES)
def test_spread(cuda_device, case, dims):
    d_k, d_v = dims
    q = normal(7, 1, (B, H, T, d_k))
    K = normal(7, 2, (B, 1, N_MAX, d_k))
    V = normal(7, 3, (B, 1, N_MAX, d_v))
    CASES[case](q, K, V)
    scale = np.float32(d_k ** -0.5)
    refs = {b: reference(q[b], K[b, 0], V[b, 0], LEN, float(scale)) for b in (0, B - 1)}
    dq, dK, dV = (torch.from_numpy(x).to(cuda_device) for x in (q, K, V))
    ln = torch.full((B,), LEN, dtype=torch.int32, device=cuda_device)
    print("spread", case, dims, flush=True)
    outs = []
    for name, chunk in (("fp32", 768), ("chunk", 0)):
        out = binding.decode_multi(dq, dK, dV, ln, float(scale), chunk_rows=chunk)
        outs.append(out.cpu().numpy())
        for b, (ref, tol) in refs.items():
            err = np.abs(outs[-1][b].astype(np.float64) - ref)
            worst = float(np.max(err / np.maximum(tol, 2.0 ** -149)))
            print(f"  {name}, sequence {b}: {worst:.3f} of the tolerance", flush=True)
            assert worst <= 1, (case, name, b, worst)
    # Other roundings: the second call did take the other kernels.
    assert not np.array_equal(*outs)
