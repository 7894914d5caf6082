"""Small batches, which are cut into scheduling units instead of chunks, and
short slabs that are split although each is a single segment: on both sides of
the lines between the plans, against the oracle (1e-5, as everywhere)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_19456_amd import binding, workloads

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, h_q, h_kv, d_k, d_v, n_max, lens
    (1, 4, 1, 128, 128, 512, [511]),             # the smallest split slab
    (1, 4, 1, 128, 128, 511, [510]),             # the largest direct one of few slabs
    (8, 16, 8, 128, 128, 513, [512, 0, 1, 127, 128, 129, 300, 511]),   # 64 slabs
    (13, 10, 5, 128, 128, 513, [512] * 12 + [7]),                      # 65 slabs
    (2, 32, 1, 128, 128, 700, [699, 255]),       # two column blocks
    (2, 4, 2, 256, 256, 256, [255, 3]),
    (1, 8, 1, 64, 64, 32768, [32767]),           # as many visitors as a slab may have
    # More units in the slab than it has slots: fewer workgroups take part.
    (1, 8, 1, 64, 64, 16384, [16383]),
    (1, 8, 1, 64, 64, 16513, [16512]),
    (1, 4, 1, 256, 256, 16384, [16383]),
    (3, 2, 1, 64, 64, 2000, [0, 0, 1]),          # almost nothing to do
    # All rows in one sequence of many; two column blocks.
    (16, 8, 8, 64, 64, 4096, [4095] + [0] * 15),
    (8, 32, 1, 64, 64, 8192, [0] * 7 + [8190]),
    (8, 32, 1, 64, 64, 2049, [2048, 64, 65, 63, 0, 1, 2000, 1030]),
    # Chunks on two thirds of 256 CUs, and on one more: ranges and chunks.
    (17, 8, 2, 128, 128, 3800, [3799 - 13 * b for b in range(17)]),
    (19, 3, 3, 64, 64, 2000, [1999 - 100 * b for b in range(19)]),
]


@pytest.mark.parametrize("shape", SHAPES, ids=[str(i) for i in range(len(SHAPES))])
def test_small_batches(cuda_device, schedule, shape):
    B, h_q, h_kv, d_k, d_v, n_max, lens = shape
    sh = workloads.custom("small", B=B, h_q=h_q, h_kv=h_kv, d_k=d_k, d_v=d_v, n_max=n_max, steps=1)
    inp = workloads.make(sh, seed=11, lens=np.array(lens, np.int32))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(cuda_device)  # noqa: E731
    q, K, V, ln = dev(inp.q), dev(inp.K), dev(inp.V), dev(inp.lens)
    ws = binding.alloc_workspace(q, K, V)
    nc = binding.workspace_counter_bytes(B, h_q, h_kv, n_max, d_k, d_v)
    ws.fill_(0xFF)
    ws[:nc].zero_()
    sc = sh.scale32()
    print("small batch", shape, flush=True)
    out = binding.decode_attn(q, K, V, ln, float(sc), workspace=ws)
    step = binding.decode_step(dev(inp.q_step[0]), K, V, dev(inp.k_new[0]), dev(inp.v_new[0]), ln,
                               float(sc), workspace=ws)
    torch.cuda.synchronize()
    assert not ws[:nc].any()
    ref = oracle.decode(inp.q, inp.K, inp.V, inp.lens, sc)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-5
    oracle.append(inp.K, inp.V, inp.k_new[0], inp.v_new[0], inp.lens)
    ref = oracle.decode(inp.q_step[0], inp.K, inp.V, inp.lens, sc)
    assert np.max(np.abs(step.cpu().numpy() - ref)) <= 1e-5
    assert ln.tolist() == inp.lens.tolist()
    assert np.array_equal(K.cpu().numpy().view(np.uint32), inp.K.view(np.uint32))


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[4], SHAPES[5]], ids=str)
def test_split_slabs_on_less_workspace(cuda_device, shape):
    """Slabs that are split where the workspace holds the slots: in one of the
    direct form's size, whole calls and the two halves, which may name the
    library's segment rows in one and leave them to it in the other."""
    B, h_q, h_kv, d_k, d_v, n_max, lens = shape
    sh = workloads.custom("small", B=B, h_q=h_q, h_kv=h_kv, d_k=d_k, d_v=d_v, n_max=n_max, steps=1)
    inp = workloads.make(sh, seed=11, lens=np.array(lens, np.int32))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(cuda_device)  # noqa: E731
    q, K, V, ln = dev(inp.q), dev(inp.K), dev(inp.V), dev(inp.lens)
    sc = float(sh.scale32())
    rows = binding.chunk_rows(B, h_q, h_kv, n_max, d_k, d_v)
    size = binding.workspace_bytes(B, h_q, h_kv, n_max, d_k, d_v, rows)
    assert size < binding.workspace_bytes(B, h_q, h_kv, n_max, d_k, d_v)
    nc = binding.workspace_counter_bytes(B, h_q, h_kv, n_max, d_k, d_v)
    full = torch.full((size + 4096,), 0xFF, dtype=torch.uint8, device=cuda_device)
    ws = full[:size]
    ws[:nc].zero_()
    ref = oracle.decode(inp.q, inp.K, inp.V, inp.lens, sh.scale32())
    print("less workspace", shape, flush=True)
    outs = [binding.decode_attn(q, K, V, ln, sc, workspace=ws)]
    for first, second in ((0, rows), (rows, 0), (0, 0)):
        binding.decode_partial(q, K, V, ln, sc, ws, first)
        outs.append(binding.decode_merge(torch.empty_like(outs[0]), ws, B, h_q, h_kv, n_max, d_k,
                                         d_v, second))
    step = binding.decode_step(dev(inp.q_step[0]), K, V, dev(inp.k_new[0]), dev(inp.v_new[0]), ln,
                               sc, workspace=ws)
    torch.cuda.synchronize()
    assert not ws[:nc].any() and bool((full[size:] == 0xFF).all())
    for out in outs:
        assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-5
    oracle.append(inp.K, inp.V, inp.k_new[0], inp.v_new[0], inp.lens)
    ref = oracle.decode(inp.q_step[0], inp.K, inp.V, inp.lens, sh.scale32())
    assert np.max(np.abs(step.cpu().numpy() - ref)) <= 1e-5
    assert ln.tolist() == inp.lens.tolist()
