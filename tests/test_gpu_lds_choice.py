"""One or two frames per workgroup in the LDS-resident decoder (GPU), where a CU
holds one, two, three or more workgroups: every frame against the streaming
path, some against the oracle, at batches on either side of the choice."""
import numpy as np
import pytest

from paper_2507_10424_amd import workloads as wl
from parity import assert_parity, note, oracle_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [800, 1000, 1200, 2500])  # four, three, two workgroups of one frame per CU, one
def test_either_side(n):
    import torch
    from paper_2507_10424_amd import ldpc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    H = wl.random_irregular_code(n, n // 2, seed=7, dv_choices=(2, 3, 3), max_row_degree=8)
    g = ldpc.build_graph(torch.from_numpy(H).to(dev))
    for B in (255, 257, 2049, 6145, 8300):
        llr = wl.bpsk_awgn_llr_torch(None, 2.5, 0.5, B, dev, n=n, batch=B)
        note(f"[lds choice] n={n} B={B}")
        out = ldpc.minsum_decode(g, llr, 12)
        ref = ldpc.minsum_decode(g, llr, 12, flags=ldpc.LDPC_FORCE_STREAM)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, ref)), B
        some = np.r_[0:6, B - 6:B]
        assert_parity(tuple(t.cpu().numpy()[some] for t in out), oracle_decode(H, llr.cpu().numpy()[some], 12), f"B={B}")
