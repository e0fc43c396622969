"""The network gradient kernel at the edges of its tiles (32 samples per
workgroup, at most 256 workgroups), with inputs that are only 4-byte aligned,
against the FP64 oracle.

Tolerance: the longest chain of rounded operations is the two forward
products (120 + 64 terms), two backward ones (20 + 64) and the sum over n
samples; with unit roundoff 6e-8 and errors that add like a random walk the
relative 2-norm error stays below 6e-8 sqrt(300 + n) <= 6e-6 for n <= 8,225;
1e-5 is asked for."""
import numpy as np
import pytest

from oracle import closure as oc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", (1, 31, 32, 33, 8191, 8192, 8193, 8225))
def test_gradient_at_tile_edges(n):
    from paper_1409_0405_amd import frlib
    print(f"mlp gradient n={n}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.normal(0, 1.5, (n + 5, oc.N_IN)).astype(np.float32)
    t = rng.normal(0, 0.1, (n + 5, oc.N_OUT)).astype(np.float32)
    idx = rng.permutation(n + 5)[:n].astype(np.int32)
    theta = np.concatenate([rng.normal(0, s, c) for s, c in (
        (0.1, 64 * 120), (0.1, 64), (0.1, 64 * 64), (0.1, 64), (0.1, 20 * 64), (0.1, 20))]).astype(np.float32)
    net = frlib.MLP(0)
    net.set_params(theta)
    # arrays that start 4 bytes after a 16-byte boundary
    xd = torch.zeros(x.size + 1, device="cuda")
    td = torch.zeros(t.size + 1, device="cuda")
    xd[1:] = torch.as_tensor(x.ravel(), device="cuda")
    td[1:] = torch.as_tensor(t.ravel(), device="cuda")
    idd = torch.as_tensor(idx, device="cuda")
    want_loss, want = oc.mlp_loss_grad(theta.astype(np.float64), x[idx].astype(np.float64), t[idx].astype(np.float64))
    loss = net.grad(xd[1:].data_ptr(), td[1:].data_ptr(), n, idx_ptr=idd.data_ptr())
    g = net.get_grad().astype(np.float64)
    assert abs(loss - want_loss) < 1e-5 * want_loss
    assert np.linalg.norm(g - want) < 1e-5 * np.linalg.norm(want)
    again = net.grad(xd[1:].data_ptr(), td[1:].data_ptr(), n, idx_ptr=idd.data_ptr())
    assert again == loss and np.array_equal(net.get_grad().astype(np.float64), g)
