"""The network's gradient at batch sizes around the 32-sample blocks of the
training kernel and the sixteen slices of the update kernel's sum, against the
float64 gradient of the reference."""
import numpy as np
import pytest

from oracle.learned import bf16_round, bf16_weights, mlp_init, mlp_loss_grad

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2601_16911_amd import cvw  # noqa: E402


@pytest.mark.parametrize("batch", [1, 31, 32, 33, 511, 513, 1100])
def test_gradient(batch):
    rng = np.random.default_rng(batch)
    P = mlp_init(3)
    P["b1"], P["b2"], P["b3"] = rng.normal(size=64) * 0.2, rng.normal(size=64) * 0.2, np.array([0.3])
    P = cvw.unpack_params(cvw.pack_params(P))
    X = bf16_round(rng.normal(size=(700, 48)))
    t = rng.uniform(size=700).astype(np.float32).astype(np.float64)
    idx = rng.integers(0, 700, batch)
    feat = torch.from_numpy((X.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16).view(np.int16)).cuda()
    net = cvw.Mlp(cvw.pack_params(P))
    grad = torch.zeros(cvw.MLP_NPARAM, device="cuda")
    net.train_step(feat, torch.from_numpy(t.astype(np.float32)).cuda(), torch.from_numpy(idx.astype(np.int32)).cuda(),
                   0.0, cvw.Mlp.train_workspace(batch), grad_out=grad)
    G = cvw.unpack_params(grad.cpu().numpy())
    _, Go = mlp_loss_grad(bf16_weights(P), X[idx], t[idx])
    # activations and errors carry 2^-16 (two bfloat16 terms), through three layers and the float32 GELU (1.5e-7)
    for k in Go:
        assert np.abs(G[k] - Go[k]).max() <= 2e-4 * np.abs(Go[k]).max(), k
