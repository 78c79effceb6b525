"""Row degrees of the streaming check kernels (GPU) against the CPU oracle: the
form with rows of up to 16 edges unrolled, the one with rows of up to 32, and
the loop for the degrees that neither unrolls, alone and beside unrolled ones."""
import numpy as np
import pytest

from paper_2507_10424_amd import workloads as wl
from parity import assert_parity, note, oracle_decode

pytestmark = pytest.mark.gpu

DEGREES = {
    "to_16": list(range(2, 17)),
    "unrolled_to_32": [2, 15, 16, 20, 24, 28, 32],
    "loop_17_to_31": [2, 9, 16, 17, 18, 19, 20, 21, 23, 24, 25, 28, 31, 32],
    "loop_33": [33],
    "loop_beside_short": [2, 6, 16, 20, 32, 33, 40, 64, 65],
}


@pytest.mark.parametrize("learned", [False, True])
@pytest.mark.parametrize("name", sorted(DEGREES))
def test_row_degrees(name, learned):
    import torch
    from paper_2507_10424_amd import ldpc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(4)
    degrees = [d for d in DEGREES[name] for _ in range(3)]
    n, B, L = 150, 70, 7
    H = np.zeros((len(degrees), n), np.uint8)
    for i, d in enumerate(degrees):
        H[i, rng.choice(n, size=d, replace=False)] = 1
    llr = wl.bpsk_awgn_llr(None, 4.0, 0.7, seed=9, n=n, batch=B)
    C = len(set(degrees))
    alpha = rng.uniform(0.6, 1.1, size=(L, C)).astype(np.float32) if learned else None
    beta = rng.uniform(0.0, 0.3, size=(L, C)).astype(np.float32) if learned else None
    note(f"[stream rows] {name} learned={learned}")
    g = ldpc.build_graph(torch.from_numpy(H).to(dev))
    x = torch.from_numpy(llr).to(dev)
    for flags in (0, ldpc.LDPC_NO_EARLY_EXIT):
        if learned:
            out = ldpc.nms_decode(g, x, L, torch.from_numpy(alpha).to(dev), torch.from_numpy(beta).to(dev),
                                  flags=flags | ldpc.LDPC_FORCE_STREAM)
            ref = oracle_decode(H, llr, L, flags, alpha, beta)
        else:
            out = ldpc.minsum_decode(g, x, L, flags=flags | ldpc.LDPC_FORCE_STREAM)
            ref = oracle_decode(H, llr, L, flags)
        torch.cuda.synchronize()
        assert_parity(tuple(t.cpu().numpy() for t in out), ref, f"{name} flags {flags}")


@pytest.mark.parametrize("B", [1, 15, 16, 17, 33, 64, 81])
@pytest.mark.parametrize("code", ["regular", "mixed"])
def test_partial_rows(code, B):
    """The last tile's frames end at any lane, and frames stop lane by lane."""
    import torch
    from paper_2507_10424_amd import ldpc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    H = (wl.regular_ldpc(120, 60, 3, 6, seed=2) if code == "regular" else
         wl.random_irregular_code(130, 60, seed=3, dv_choices=(2, 3, 4), max_row_degree=12))
    n, L = H.shape[1], 20
    llr = wl.bpsk_awgn_llr(None, 2.5, 0.5, seed=20 + B, n=n, batch=B)
    g = ldpc.build_graph(torch.from_numpy(H).to(dev))
    out = ldpc.minsum_decode(g, torch.from_numpy(llr).to(dev), L, flags=ldpc.LDPC_FORCE_STREAM)
    torch.cuda.synchronize()
    assert_parity(tuple(t.cpu().numpy() for t in out), oracle_decode(H, llr, L), f"{code} B={B}")
