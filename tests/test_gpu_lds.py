"""The LDS-resident decoder (codes that no on-chip variant takes) against the
CPU oracle, at the edges of its ranges: one and two frames per workgroup, rows
of up to 8, 16 and 32 edges, 4, 8 and 16 bits per thread, more frames than the
grid, and every decode option."""
import numpy as np
import pytest

from paper_2507_10424_amd import workloads as wl
from parity import assert_parity, note, oracle_decode

pytestmark = pytest.mark.gpu


def _no_empty(H):
    return H[H.sum(1) > 0]


CODES = {
    # rows of 32 in one wavefront group and a remainder: one frame per workgroup
    "wide_rows": lambda: wl.regular_ldpc(520, 65, 4, 32, seed=3),
    "paper_8176": lambda: wl.regular_ldpc(8176, 1022, 4, 32, seed=2),
    # rows of at most 8, 2 and 3 groups per wavefront, 4 bits per thread
    "regular_4096": lambda: wl.regular_ldpc(4096, 2048, 3, 6, seed=9),
    "regular_4098": lambda: wl.regular_ldpc(4098, 2049, 3, 6, seed=9),  # 8 bits per thread
    # 16 bits per thread (n > 8192)
    "long_9000": lambda: wl.regular_ldpc(9000, 4500, 2, 4, seed=4),
    # mixed degrees with rows above 16 and columns of 0 and above 8
    "mixed_rows": lambda: wl.random_irregular_code(700, 130, seed=21, dv_choices=(0, 1, 2, 3, 9), max_row_degree=27),
    # mixed rows of at most 16, too many rows for the on-chip variants
    "irregular_2600": lambda: wl.random_irregular_code(2600, 1201, seed=5, dv_choices=(1, 2, 3, 4, 12),
                                                       max_row_degree=16),
}


def decode(H, llr, L, flags=0, alpha=None, beta=None):
    import torch
    from paper_2507_10424_amd import ldpc
    dev = torch.device("cuda:0")
    g = ldpc.build_graph(torch.from_numpy(np.ascontiguousarray(H)).to(dev))
    x = torch.from_numpy(llr).to(dev)
    with pytest.raises(ldpc.LdpcError) as e:  # not a graph of the on-chip path
        ldpc.minsum_decode(g, x, L, flags=ldpc.LDPC_FORCE_ONCHIP)
    assert e.value.status == -6
    out = ldpc._outputs(llr.shape[0], g.n, dev, True)
    for t, v in zip(out, (7, float("nan"), -7, 9)):
        t.fill_(v)
    if alpha is None:
        ldpc.minsum_decode(g, x, L, flags=flags, out=out)
    else:
        ldpc.nms_decode(g, x, L, torch.from_numpy(alpha).to(dev), torch.from_numpy(beta).to(dev), flags=flags, out=out)
    torch.cuda.synchronize()
    got = tuple(t.cpu().numpy() for t in out)
    s = (ldpc.minsum_decode(g, x, L, flags=flags | ldpc.LDPC_FORCE_STREAM) if alpha is None else
         ldpc.nms_decode(g, x, L, torch.from_numpy(alpha).to(dev), torch.from_numpy(beta).to(dev),
                         flags=flags | ldpc.LDPC_FORCE_STREAM))
    torch.cuda.synchronize()
    for a, b in zip(got, s):  # every frame, bit for bit
        assert np.array_equal(a, b.cpu().numpy())
    return got


def frames(H, B, seed):
    m, n = H.shape
    rate = max(0.3, 1.0 - m / n)
    return wl.bpsk_awgn_llr(None, 2.0 + 5.5 * max(0.0, rate - 0.5), rate, seed=seed, n=n, batch=B)


@pytest.mark.parametrize("B", [1, 3, 700])
@pytest.mark.parametrize("name", sorted(CODES))
def test_codes(name, B):
    H = _no_empty(CODES[name]())
    llr = frames(H, B, seed=50 + B)
    note(f"[lds] {name} m={H.shape[0]} n={H.shape[1]} B={B}")
    got = decode(H, llr, 20)
    some = slice(0, B) if H.shape[1] < 1000 else slice(0, min(B, 12))  # the oracle's share of the long ones
    assert_parity(tuple(t[some] for t in got), oracle_decode(H, llr[some], 20), name)


@pytest.mark.parametrize("name", ["wide_rows", "mixed_rows", "irregular_2600"])
@pytest.mark.parametrize("L,flags", [(0, 0), (1, 0), (9, 1), (14, 6 << 8), (25, 3 << 8)])
def test_options(name, L, flags):
    H = _no_empty(CODES[name]())
    llr = frames(H, 300, seed=7)
    note(f"[lds] {name} L={L} flags={flags}")
    got = decode(H, llr, L, flags)
    some = slice(0, 40)
    assert_parity(tuple(t[some] for t in got), oracle_decode(H, llr[some], L, flags), name)


@pytest.mark.parametrize("name", sorted(CODES))
def test_learned(name):
    H = _no_empty(CODES[name]())
    T, C = 7, np.unique(H.sum(1)).size
    rng = np.random.default_rng(3)
    alpha = rng.uniform(0.6, 1.1, size=(T, C)).astype(np.float32)
    beta = rng.uniform(0.0, 0.3, size=(T, C)).astype(np.float32)
    for B in (5, 290):
        llr = frames(H, B, seed=70 + B)
        note(f"[lds] learned {name} B={B}")
        got = decode(H, llr, T, 0, alpha, beta)
        some = slice(0, 10)
        assert_parity(tuple(t[some] for t in got), oracle_decode(H, llr[some], T, 0, alpha, beta), name)


@pytest.mark.parametrize("learned", [False, True])
def test_two_frames_with_long_rows(learned):
    """Rows of up to 16 edges take two frames per workgroup from 8 frames per
    resident workgroup on."""
    H = _no_empty(CODES["irregular_2600"]())
    llr = frames(H, 2600, seed=15)
    note(f"[lds] two frames, long rows, learned={learned}")
    a = b = None
    if learned:
        C, rng = np.unique(H.sum(1)).size, np.random.default_rng(3)
        a = rng.uniform(0.6, 1.1, size=(9, C)).astype(np.float32)
        b = rng.uniform(0.0, 0.3, size=(9, C)).astype(np.float32)
    got = decode(H, llr, 9, 0, a, b)
    some = slice(2000, 2010)
    assert_parity(tuple(t[some] for t in got), oracle_decode(H, llr[some], 9, 0, a, b), "long rows")


def test_more_frames_than_the_grid():
    """Frames beyond the first ones of every workgroup come from a counter."""
    H = CODES["wide_rows"]()
    llr = frames(H, 9000, seed=11)
    note("[lds] 9000 frames")
    got = decode(H, llr, 15)
    some = slice(8000, 8200)
    assert_parity(tuple(t[some] for t in got), oracle_decode(H, llr[some], 15), "late frames")


def test_non_finite_frames_stay_apart():
    H = CODES["irregular_2600"]()
    llr = frames(H, 600, seed=12)
    clean = llr.copy()
    bad = np.arange(0, 600, 3)
    llr[bad, ::5] = np.inf
    llr[bad[::2], 1::7] = np.nan
    import torch
    from paper_2507_10424_amd import ldpc
    dev = torch.device("cuda:0")
    g = ldpc.build_graph(torch.from_numpy(H).to(dev))
    note("[lds] non-finite frames")
    a = ldpc.minsum_decode(g, torch.from_numpy(llr).to(dev), 12)
    b = ldpc.minsum_decode(g, torch.from_numpy(clean).to(dev), 12)
    torch.cuda.synchronize()
    good = np.setdiff1d(np.arange(600), bad)
    for x, y in zip(a, b):
        assert np.array_equal(x.cpu().numpy()[good], y.cpu().numpy()[good])
    assert int(a[0].max()) <= 1 and 0 <= int(a[2].min()) and int(a[2].max()) <= 12
