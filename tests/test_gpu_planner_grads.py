"""A caller's gradient buffer holds the gradients and nothing else: with grads
given, planner_train_step writes the parameters' gradients and leaves what
lies behind them alone (exact comparison), and returns the loss and gradients
of the update form's first moment, (1 - beta1) g after one step from zero:
equal but for one FP32 rounding of the product, 2^-23 relative."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 5, 17, 64, 100, 512])
def test_gradients_stay_in_their_buffer(batch):
    import paper_2012_00506_amd as fb
    print(f"planner grads batch={batch}", flush=True)
    nw = fb.planner_bytes() // 4
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    w = 0.05 * torch.randn(nw, device="cuda", generator=gen)
    X = torch.randn(batch, 80, device="cuda", generator=gen)
    T = torch.rand(batch, 64, device="cuda", generator=gen)
    buf = torch.full((nw + 4096,), 7.25, device="cuda")
    loss = fb.planner_train_step(w.clone(), None, X, T, 0.0, 0, grads=buf[:nw])
    assert bool((buf[nw:] == 7.25).all())
    opt = torch.zeros(2 * nw, device="cuda")
    loss2 = fb.planner_train_step(w.clone(), opt, X, T, 1e-3, 1)
    assert loss == loss2
    g, m = buf[:nw].double().cpu().numpy(), opt[:nw].double().cpu().numpy()
    c = float(np.float32(1.0) - np.float32(0.9))
    assert np.all(np.abs(m - c * g) <= 2.0 ** -23 * np.abs(c * g) + 1e-37)
