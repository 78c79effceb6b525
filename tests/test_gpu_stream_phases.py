"""Streaming batches decoded in phases (GPU) against the CPU oracle: plans that
pack the frames, plans that do not, tiles and whole batches that end early, and
iteration limits around the plans."""
import pytest

from paper_2507_10424_amd import workloads as wl
from parity import assert_parity, note, oracle_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [0, 1, 6, 7, 10, 11, 13, 14, 17, 50])
@pytest.mark.parametrize("ebn0,period", [(1.0, 1), (2.0, 1), (4.5, 1), (2.5, 3)])
def test_phases(L, ebn0, period):
    import torch
    from paper_2507_10424_amd import ldpc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    H = wl.regular_ldpc(96, 48, 3, 6, seed=1)
    g = ldpc.build_graph(torch.from_numpy(H).to(dev))
    flags = ldpc.check_period(period)
    for B, chunk in ((65, -1), (960, -1), (700, 1), (500, 3), (4200, 2)):  # 2 to 66 tiles in chunks of fewer than 16
        llr = wl.bpsk_awgn_llr(None, ebn0, 0.5, seed=B, n=96, batch=B)
        if ebn0 == 4.5:  # all but the frames of one tile start as codewords
            llr[:64 * (B // 128)] = 3.0
            llr[64 * (B // 128) + 64:] = 3.0
        note(f"[phases] L={L} ebn0={ebn0} period={period} B={B} chunk={chunk}")
        ldpc.set_tuning(g, 2, stream_chunk=chunk)
        out = ldpc.minsum_decode(g, torch.from_numpy(llr).to(dev), L, flags=flags)
        torch.cuda.synchronize()
        assert_parity(tuple(t.cpu().numpy() for t in out), oracle_decode(H, llr, L, flags), f"B={B} chunk={chunk}")
