"""Both forms of the T-row append (one launch for few 16-byte pieces per
sequence, copies spread over the chip and a second launch for many), around
the line between them and at remainders of a workgroup's pieces: bit-exact
against the oracle, near capacity, full, empty and negative lengths included."""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_19456_amd import binding
from paper_2607_19456_amd.workloads import normal

pytestmark = pytest.mark.gpu

CASES = [
    # B, h_kv, d_k, d_v, n_max, T      pieces per sequence
    (3, 1, 4, 4, 40, 1),               # 2
    (5, 8, 128, 128, 40, 8),           # 4096: the last one-launch size
    (5, 8, 128, 128, 40, 9),           # 4608
    (5, 1, 64, 128, 200, 86),          # 4128; 1024 * 4 + 32 per slab
    (4, 3, 12, 20, 700, 171),          # 4104: head sizes off the vector widths
    (6, 2, 256, 64, 900, 333),         # 53280, odd rows
]


@pytest.mark.parametrize("B,h_kv,d_k,d_v,n_max,T", CASES)
def test_append_forms_bit_exact(cuda_device, B, h_kv, d_k, d_v, n_max, T):
    K = normal(3, 1, (B, h_kv, n_max, d_k))
    V = normal(3, 2, (B, h_kv, n_max, d_v))
    kn = normal(3, 3, (B, h_kv, T, d_k))
    vn = normal(3, 4, (B, h_kv, T, d_v))
    kn[0, 0, 0, 0] = np.nan
    lens = np.array([0, n_max - T, n_max - 1, n_max, -1, n_max - T // 2][:B], np.int32)
    dev = [torch.from_numpy(x.copy()).to(cuda_device) for x in (K, V, kn, vn, lens)]
    print("append forms", B, h_kv, d_k, d_v, n_max, T, flush=True)
    binding.kv_append_rows(*dev)
    torch.cuda.synchronize()
    oracle.append_rows(K, V, kn, vn, lens)
    for got, ref in ((dev[0], K), (dev[1], V)):
        assert np.array_equal(got.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    assert np.array_equal(dev[4].cpu().numpy(), lens)
