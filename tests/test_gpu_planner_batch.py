"""The network's forward pass by large batches, whose layers take the form with
fewer loads in flight from 2 048 waves on (more than 2 048 rows in the hidden layers,
8 192 in the last): every row equals, bit for bit, what a small batch gives."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [2048, 2049, 8192, 8209])
def test_large_batches_equal_small_ones(batch):
    import paper_2012_00506_amd as fb
    print(f"planner batch={batch}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    w = 0.05 * torch.randn(fb.planner_bytes() // 4, device="cuda", generator=gen)
    X = torch.randn(batch, 80, device="cuda", generator=gen)
    out = fb.planner_forward(w, X)
    for r in range(0, batch, 500):
        assert bool((fb.planner_forward(w, X[r:r + 500]) == out[r:r + 500]).all())
