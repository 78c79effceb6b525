"""Training loss and gradients of very sure bits (GPU): softplus and sigmoid
down to the smallest subnormal number, in both forms of the training kernels.

With alpha = beta = 0 every message is 0, so the posterior of a bit is its LLR
z, the loss of its iteration log1p(exp(-z)) and its gradient -sigmoid(-z)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

UNIT = 2.0 ** -149
Z = [0.25, 20.0, 86.5, 87.2, 87.4, 88.0, 90.0, 95.5, 100.0, 102.0, 103.5, 103.9, 104.2, 120.0, 3e38]


@pytest.mark.parametrize("n", [4, 33])  # state in LDS; in device memory (a row of 33 edges)
def test_small_losses_and_gradients(n):
    import torch
    from paper_2507_10424_amd import ldpc
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    g = ldpc.build_graph(torch.ones((1, n), dtype=torch.uint8, device=dev))
    zero = torch.zeros((1, 1), dtype=torch.float32, device=dev)
    ws = torch.empty(ldpc.train_workspace_bytes(g, 1, 1, 1), dtype=torch.uint8, device=dev)
    for z in Z:
        llr = torch.full((1, n), z, dtype=torch.float32, device=dev)
        x = float(llr[0, 0])
        loss, _ = ldpc.nms_train_forward(g, llr, zero, zero, 1, ws)
        _, _, gl = ldpc.nms_train_backward(g, llr, zero, zero, 1, ws, grad_loss=float(n), want_llr_grad=True)
        for got, want in ((float(loss[0]), np.log1p(np.exp(-x))), (-float(gl[0, 0]), np.exp(-x) / (1.0 + np.exp(-x)))):
            # 6 units of the last place for the function, 2 for the mean over n bits; below 2^-126 the function and
            # the mean round to multiples of 2^-149 (a unit each for the former, half of one for the latter)
            assert abs(got - want) <= 8 * 2.0 ** -24 * want + 1.5 * UNIT, (n, z, got, want)
        assert torch.equal(gl, gl[:, :1].expand(1, n))
