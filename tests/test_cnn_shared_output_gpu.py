"""lbm_cnn_forward with its output in memory that the pass still reads or writes
elsewhere: y the input itself (three channels) or within it (more, one sample),
or in the first hidden activations' memory.  Equal bit for bit to the call with
memory of its own, on fields of several tiles."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from test_cnn_gpu import setup  # noqa: E402


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


@pytest.mark.parametrize("n,cin,where", [(5, 3, "x"), (1, 4, "x"), (1, 7, "inside x"), (4, 4, "a1")])
def test_output_in_shared_memory(L, n, cin, where):
    h, w = 70, 83
    _, _, _, g, shape, params, ws = setup(L, n=n, cin=cin, h=h, w=w, seed=cin)
    a1, a2 = (torch.empty((n, 32, h, w), device="cuda") for _ in range(2))
    y = torch.empty((n, 3, h, w), device="cuda")

    def forward(x, to):
        L.lbm_cnn_forward(shape, params, x.data_ptr(), a1.data_ptr(), a2.data_ptr(), to.data_ptr(), ws.data_ptr(),
                          ws.numel(), torch.cuda.current_stream().cuda_stream)

    forward(g["x"], y)
    hidden = a1.clone(), a2.clone()
    x = g["x"].clone()
    to = {"x": x, "inside x": x[:, 3:], "a1": a1}[where].reshape(-1)[:y.numel()]
    forward(x, to)
    assert torch.equal(to.view_as(y), y)
    assert torch.equal(a2, hidden[1])
    if where != "a1":
        assert torch.equal(a1, hidden[0])
