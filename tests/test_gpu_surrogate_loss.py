"""The loss of large planes: an increment that is the same everywhere, against
its value in 64 bits.  Summed in FP32, a thousand equal squares per thread
were 1.5e-5 off."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nx,ny", [(1, 2048, 2048), (3, 256, 256), (2, 256, 16), (1, 4096, 2064)])
def test_loss_of_a_constant_increment(n, nx, ny):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    print(f"case loss N={n} {nx}x{ny}", flush=True)
    s = mlfilm.Surrogate(n, nx, ny, width=64, blocks=0, batch=1, scale=1e-2)
    s.set_params(np.zeros(s.param_count, np.float32))   # predicts no change
    h0 = torch.ones((1, n, ny, nx), device="cuda")
    h1 = torch.full_like(h0, 1.01321)
    inc = (np.float32(1.01321) - np.float32(1.0)) * np.float32(100.0)  # as the network scales it, FP32
    want = float(inc) ** 2
    # one FP32 rounding of the square
    assert abs(s.loss(h0, h1) - want) <= 2.0 ** -23 * want
    loss, g = s.gradient(h0, h1)
    assert abs(loss - want) <= 2.0 ** -23 * want
