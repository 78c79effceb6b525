"""The training workspace (GPU): bounded by the checkpoint interval, not falling
with the batch or the iterations, and the same loss and gradients, bit for bit,
with the records kept and in passes."""
import pytest

from paper_2507_10424_amd import workloads as wl

pytestmark = pytest.mark.gpu

MIB = 1 << 20


@pytest.fixture(scope="module")
def graph():
    import torch
    from paper_2507_10424_amd import ldpc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch, ldpc, ldpc.build_graph(torch.from_numpy(wl.regular_ldpc(1026, 513, 3, 6, seed=2)).to("cuda:0"))


def sums(B, T):
    """Bytes of the per-frame sums of the loss and of one class's weight gradients, and the alignment's slack."""
    return 4 * B * (1 + 2 * T) + MIB


def test_interval_bounds_the_workspace(graph):
    _, ldpc, g = graph
    state = 4 * (g.n + g.E)  # of one frame's checkpoint
    for B in (4096, 20000, 300000):
        for T, K in ((10, 10), (10, 5), (10, 3), (30, 100)):
            checkpoints = -(-T // K) * B * state
            assert ldpc.train_workspace_bytes(g, B, T, K) <= max(256 * MIB, checkpoints) + sums(B, T)
        for K in (1, 2):
            assert ldpc.train_workspace_bytes(g, B, 10, K) <= max(8192 * MIB, -(-10 // K) * B * state) + sums(B, 10)


def test_size_does_not_fall(graph):
    _, ldpc, g = graph
    for K in (2, 7):
        for B in (3, 4096, 100000):
            sizes = [ldpc.train_workspace_bytes(g, B, T, K) for T in range(1, 120)]
            assert sizes == sorted(sizes), (K, B)
        for T in (10, 100):
            sizes = [ldpc.train_workspace_bytes(g, B, T, K) for B in range(1, 200000, 997)]
            assert sizes == sorted(sizes), (K, T)


def test_passes_give_the_kept_result(graph):
    torch, ldpc, g = graph
    B, T = 8000, 10
    gen = torch.Generator().manual_seed(1)
    a = (0.75 + 0.2 * torch.rand((T, 1), generator=gen)).to("cuda:0")
    b = (0.1 * torch.rand((T, 1), generator=gen)).to("cuda:0")
    llr = ldpc.awgn_llr(B, g.n, 0.5, (1.0, 3.0), 3, torch.device("cuda:0"))
    results = []
    for K in (2, 10):
        ws = torch.empty(ldpc.train_workspace_bytes(g, B, T, K), dtype=torch.uint8, device="cuda:0")
        ws.fill_(0xFF)  # NaNs
        loss, post = ldpc.nms_train_forward(g, llr, a, b, K, ws, want_post=True)
        results.append((loss, post, *ldpc.nms_train_backward(g, llr, a, b, K, ws, want_llr_grad=True)))
        assert (ws.numel() > 512 * MIB) == (K == 2)
    assert all(torch.isfinite(x).all() for x in results[0])
    assert all(torch.equal(x, y) for x, y in zip(*results))
