"""The binding refuses a tensor with the error that names what is wrong with it,
and passes the pointers of right ones."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_06763_amd import gdn_tree as G
    G.lib()
    return G


@pytest.mark.parametrize("what,exc,text", [
    ("none", ValueError, "q is required"), ("list", TypeError, "q: expected a torch.Tensor"),
    ("cpu", ValueError, "q: must be a device tensor"),
    ("dtype", ValueError, "q: dtype torch.float16, expected torch.float32"),
    ("shape", ValueError, "q: shape (2, 8, 4), expected (2, 4, 8)"),
    ("rank", ValueError, "q: shape (1, 2, 4, 8), expected (2, 4, 8)"),
    ("strides", ValueError, "q: must be contiguous"), ("offset", ValueError, "q: must be 16-byte aligned"),
])
def test_refused(G, what, exc, text):
    import torch
    x = torch.zeros(2, 4, 8, device="cuda")
    bad = {"none": None, "list": [0.0], "cpu": x.cpu(), "dtype": x.half(), "shape": torch.zeros(2, 8, 4, device="cuda"),
           "rank": x[None], "strides": torch.zeros(2, 8, 4, device="cuda").transpose(1, 2),
           "offset": torch.zeros(65, device="cuda")[1:].view(2, 4, 8)}[what]
    with pytest.raises(exc) as e:
        G._ptrs(((x, (2, 4, 8), torch.float32, "k"), (bad, (2, 4, 8), torch.float32, "q")))
    assert str(e.value) == text


def test_passed(G):
    import torch
    x = torch.nn.Parameter(torch.zeros(2, 4, device="cuda"))
    e = torch.zeros(0, 4, device="cuda")
    args = ((x, (2, 4), torch.float32, "x"), (None, (2,), torch.int32, "status", None), (e, (0, 4), torch.float32, "e"))
    assert G._ptrs(args) == [x.data_ptr(), None, 0]
    side = torch.cuda.Stream()
    assert G._stream(side) == side.cuda_stream and G._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert G._stream(None) == side.cuda_stream
