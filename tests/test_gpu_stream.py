"""The stream that the binding passes on: the current one, wherever it was made
current, and the outputs it makes when it is given none."""
import pytest

from paper_2301_13016_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)


def test_handle_is_the_current_stream():
    side = torch.cuda.Stream()
    assert (B._stream_handle(None).value or 0) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert B._stream_handle(None).value == side.cuda_stream
    assert B._stream_handle(side).value == side.cuda_stream


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64, torch.bfloat16])
def test_new_outputs_equal_given_ones_on_a_side_stream(dtype):
    nx, ny, nz = 66, 5, 3
    odt = torch.float64 if dtype == torch.float64 else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    x = [(torch.rand((nz + 2, ny + 2, nx + 2), device="cuda", generator=gen) - 0.5).to(dtype) for _ in range(3)]
    c = B.Coeffs(0.25, 0.5, *[torch.rand(nz, device="cuda", generator=gen).to(odt) for _ in range(4)])
    want = [torch.empty((nz, ny, nx), dtype=odt, device="cuda") for _ in range(3)]
    B.advect(*x, c, out=want)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        got = B.advect(*x, c)
    side.synchronize()
    assert all(a.is_contiguous() and a.dtype == odt and torch.equal(a, b) for a, b in zip(got, want))
    assert len({a.data_ptr() for a in got}) == 3
