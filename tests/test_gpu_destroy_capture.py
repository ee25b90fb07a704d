"""A model that is destroyed while a graph is being captured (Python may collect
it there at any time) leaves the capture as it is, and the pinned blocks that
models' scalars come through are given back and may run out."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _model():
    from paper_2410_05902_amd import Model
    X = torch.randn(512, 16, generator=torch.Generator().manual_seed(1)).cuda()
    m = Model(X, k=4, b_max=64, window=2, kernel="gauss", kernel_param=32.0)
    m.init_centers(torch.arange(4, dtype=torch.int32, device="cuda"))
    m.step(torch.arange(64, dtype=torch.int32, device="cuda"), want_objective=True)
    return m


def test_destroy_during_capture():
    m = _model()
    y = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        y.add_(1.0)
        m.close()
        y.add_(1.0)
    for i in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert y.tolist() == [2.0 * (i + 1)] * 8
    del g
    _model().close()  # the next one works as the first did


def test_more_models_than_blocks():
    ref = _model()
    idx = torch.arange(512, dtype=torch.int32, device="cuda")
    f = ref.objective(idx[:64])
    for _ in range(2):  # 64 blocks, given back in between
        many = [_model() for _ in range(70)]
        assert [m.objective(idx[:64]) for m in many] == [f] * 70
        for m in many[::2] + many[1::2]:
            m.close()
    with pytest.raises(RuntimeError):  # (a raised flag is reported and cleared)
        ref.assign(torch.full((3,), 512, dtype=torch.int32, device="cuda"))
    assert ref.objective(idx[:64]) == f
