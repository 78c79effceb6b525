"""The training kernels at the edges of their ranges: state in LDS (rows of at
most 8, 16 and 32 edges, 4, 8 and 16 bits per thread, one and several degree
classes) and in device memory (unrolled rows, rows of more than 16 edges, the
streaming row order), transmitted codewords, and batches trained in passes."""
import numpy as np
import pytest

import oracle
from paper_2507_10424_amd import workloads as wl
from parity import note
from test_gpu_nms import assert_grad_parity

pytestmark = pytest.mark.gpu


def _classes(H, most=8):
    """H with whole rows left out until at most `most` row degrees remain."""
    d = H.sum(1)
    degs, count = np.unique(d, return_counts=True)
    keep = degs[np.argsort(-count)][:most]
    return H[np.isin(d, keep) & (d > 1)]


CODES = {
    "lds_8": lambda: _classes(wl.random_irregular_code(700, 390, seed=2, dv_choices=(1, 2, 3, 4), max_row_degree=8)),
    "lds_16": lambda: _classes(wl.random_irregular_code(1500, 400, seed=3, dv_choices=(1, 2, 3, 9), max_row_degree=16)),
    "lds_32": lambda: wl.regular_ldpc(544, 68, 4, 32, seed=3),
    "lds_two_groups": lambda: wl.regular_ldpc(4200, 2100, 3, 6, seed=5),
    "lds_long": lambda: wl.regular_ldpc(9000, 4500, 2, 4, seed=4),
    "stream_10": lambda: wl.regular_ldpc(9000, 4500, 5, 10, seed=6),
    "stream_ordered": lambda: wl.regular_ldpc(16500, 8250, 3, 6, seed=7),
    "stream_wide": lambda: _classes(wl.random_irregular_code(900, 66, seed=8, dv_choices=(2, 3), max_row_degree=45)),
    "stream_row_70": lambda: wl.regular_ldpc(700, 20, 2, 70, seed=9),
}


def _run(H, llr, a, b, K, target=None, grad_loss=1.0):
    import torch
    from paper_2507_10424_amd import ldpc
    dev = torch.device("cuda:0")
    g = ldpc.build_graph(torch.from_numpy(np.ascontiguousarray(H)).to(dev))
    at, bt, lt = (torch.from_numpy(x).to(dev) for x in (a, b, llr))
    tg = None if target is None else torch.from_numpy(target).to(dev)
    ws = torch.empty(ldpc.train_workspace_bytes(g, llr.shape[0], a.shape[0], K), dtype=torch.uint8, device=dev)
    ws.fill_(255)  # NaNs
    loss, post = ldpc.nms_train_forward(g, lt, at, bt, K, ws, target=tg, want_post=True)
    ga, gb, gl = ldpc.nms_train_backward(g, lt, at, bt, K, ws, target=tg, want_llr_grad=True, grad_loss=grad_loss)
    torch.cuda.synchronize()
    return float(loss), post.cpu().numpy(), ga.cpu().numpy(), gb.cpu().numpy(), gl.cpu().numpy()


def _weights(T, C, seed):
    rng = np.random.default_rng(seed)
    return (rng.uniform(0.6, 1.05, size=(T, C)).astype(np.float32),
            rng.uniform(0.0, 0.3, size=(T, C)).astype(np.float32))


@pytest.mark.parametrize("name", sorted(CODES))
def test_gradient(name):
    H = CODES[name]()
    m, n = H.shape
    T, B = 4, 3 if n > 5000 else 70
    a, b = _weights(T, oracle.check_degrees(H).size, 2)
    llr = wl.bpsk_awgn_llr(None, 2.0, max(0.3, 1 - m / n), seed=4, n=n, batch=B)
    note(f"[train] {name} m={m} n={n} classes={a.shape[1]} B={B}")
    loss, post, ga, gb, gl = _run(H, llr, a, b, 2)
    ref = oracle.nms_train_grad_f32_forward(H, llr, a, b, llr_grad=True)
    assert np.array_equal(post.astype(np.float64), ref["post"])
    assert abs(loss - ref["loss"]) <= 2e-5 * abs(ref["loss"])
    assert_grad_parity(H, T, B, {"galpha": ga, "gbeta": gb, "gllr": gl}, ref, name)


@pytest.mark.parametrize("name", ["lds_32", "stream_row_70"])
def test_transmitted_codewords(name):
    """Min-Sum is symmetric: the frames r (1 - 2c) with targets c have the loss
    and weight gradients of r with the zero codeword, and gllr (1 - 2c)."""
    H = CODES[name]()
    n, B, T = H.shape[1], 67, 5
    a, b = _weights(T, 1, 5)
    llr = wl.bpsk_awgn_llr(None, 3.0, 0.8, seed=6, n=n, batch=B)
    c = wl.gf2_encoder(H).random_codewords(B, seed=7)
    s = (1.0 - 2.0 * c).astype(np.float32)
    note(f"[train] codewords {name}")
    p = _run(H, llr, a, b, 1)
    q = _run(H, llr * s, a, b, 1, target=c)
    assert p[0] == q[0] and np.array_equal(p[1] * s, q[1])
    for k, sign in ((2, 1.0), (3, 1.0), (4, s)):
        assert np.array_equal(p[k] * sign, q[k])


@pytest.mark.parametrize("name,B,T,K", [("lds_32", 8200, 300, 300), ("stream_10", 2048, 100, 10)])
def test_batches_in_passes(name, B, T, K):
    """Batches whose records exceed the workspace's bound are trained in passes,
    the backward running each pass's forward again: the same posteriors and LLR
    gradients as in small batches, frame by frame, and the mean of their loss
    and weight gradients."""
    import torch
    from paper_2507_10424_amd import ldpc
    H = CODES[name]()
    n = H.shape[1]
    dev = torch.device("cuda:0")
    g = ldpc.build_graph(torch.from_numpy(H).to(dev))
    a, b = (torch.from_numpy(x).to(dev) for x in _weights(T, 1, 8))
    llr = ldpc.awgn_llr(B, n, 0.6, (1.0, 3.0), 11, dev)
    need = ldpc.train_workspace_bytes(g, B, T, K)
    note(f"[train] passes {name} B={B} T={T} workspace {need / 2**30:.2f} GiB")
    assert need < 1.2 * 2**33 and ldpc.train_workspace_bytes(g, B // 2, T, K) > need // 2  # bounded: not all kept
    ws = torch.empty(need, dtype=torch.uint8, device=dev)
    loss, post = ldpc.nms_train_forward(g, llr, a, b, K, ws, want_post=True)
    ga, gb, gl = ldpc.nms_train_backward(g, llr, a, b, K, ws, want_llr_grad=True)
    parts = []
    for h in range(2):
        x = llr[h * B // 2:(h + 1) * B // 2].contiguous()
        l2, p2 = ldpc.nms_train_forward(g, x, a, b, K, ws, want_post=True)
        ga2, gb2, gl2 = ldpc.nms_train_backward(g, x, a, b, K, ws, want_llr_grad=True)
        rows = slice(h * B // 2, (h + 1) * B // 2)
        assert torch.equal(p2, post[rows])
        # 1 / (B n) against 2 / (B n): powers of two apart
        assert torch.equal(gl2 * 0.5, gl[rows])
        parts.append((l2, ga2, gb2))
    for x, y, z in zip((loss, ga, gb), *parts):
        want = 0.5 * (y.double() + z.double())
        # (the magnitudes of the code with columns of 5 overflow after 80 iterations)
        fine = torch.isfinite(want)
        assert torch.equal(fine, torch.isfinite(x)) and bool(fine.any())
        # B frames in another order: (B + T m) roundings of sums whose terms may cancel
        scale = float(torch.maximum(y.abs(), z.abs())[fine].max())
        assert float((x.double() - want)[fine].abs().max()) <= 2e-5 * scale


STREAM_IRREGULAR = {
    "rows_16_columns_12": lambda: _classes(wl.random_irregular_code(9001, 5500, seed=12, dv_choices=(2, 3, 12),
                                                                   max_row_degree=16)),
    "rows_8": lambda: _classes(wl.random_irregular_code(17003, 8500, seed=13, dv_choices=(1, 2, 3, 4),
                                                        max_row_degree=8)),
}


@pytest.mark.parametrize("name", sorted(STREAM_IRREGULAR))
def test_gradient_of_irregular_codes_in_device_memory(name):
    """State in device memory with several row degrees, columns of more than 8
    checks, a number of bits that is no multiple of 4 and one frame in the last
    tile of 64 (the lanes without a frame hold NaNs in the workspace)."""
    H = STREAM_IRREGULAR[name]()
    m, n = H.shape
    T, B = 3, 65
    C = oracle.check_degrees(H).size
    assert C > 1 and n % 4
    a, b = _weights(T, C, 14)
    llr = wl.bpsk_awgn_llr(None, 2.0, 0.4, seed=15, n=n, batch=B)
    note(f"[train] {name} m={m} n={n} classes={C} B={B}")
    loss, post, ga, gb, gl = _run(H, llr, a, b, 2)
    ref = oracle.nms_train_grad_f32_forward(H, llr, a, b, llr_grad=True)
    assert np.array_equal(post.astype(np.float64), ref["post"])
    assert abs(loss - ref["loss"]) <= 2e-5 * abs(ref["loss"])
    assert_grad_parity(H, T, B, {"galpha": ga, "gbeta": gb, "gllr": gl}, ref, name)
