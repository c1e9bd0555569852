"""Launches of one step have strips and shapes of their own: a film stepped
one step at a time, in pairs with a step left over, and in a fixed shape has
the same bits, on both sides of each line of the default shapes (both
buffers within 256 MiB or not, short segments of FP64 films, FP32 films from
1 GiB on, 16-bit films)."""
import numpy as np
import pytest

from paper_2409_16659_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nx,ny,prec,tau", [
    (2, 121, 65, "f32", 1.0), (3, 109, 200, "f16mix", 1.0), (4, 700, 300, "f16", 1.0), (2, 240, 61, "bf16", 1.3),
    (3, 700, 900, "f64", 1.0), (2, 1700, 700, "f64", 1.0), (3, 1500, 1400, "f32", 1.3), (1, 4000, 3800, "f32", 1.0),
    (4, 1300, 1500, "f16mix", 1.0), (3, 170, 5200, "f64", 1.3)])
def test_single_steps_in_their_own_shape(n, nx, ny, prec, tau):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    gam = [1.0e-2, 0.7e-2, 0.6e-2, 0.5e-2][:n]
    film = inputs.film_params(n, nx, ny, gamma=gam, mu=[1e-3] * n, hstar=0.1, tau=tau,
                              spread={(l, 1): inputs.young_spreading(gam[l], 20.0) for l in range(n)})
    g = torch.Generator("cuda").manual_seed(nx)
    h0 = torch.rand((n, ny, nx), dtype=torch.float64, device="cuda", generator=g).mul_(2e-3)
    h0 += torch.tensor([1.0, 0.8, 0.6, 0.4][:n], dtype=torch.float64, device="cuda")[:, None, None]
    print(f"case single steps {prec} N={n} {nx}x{ny} tau={tau}", flush=True)
    states = []
    for shape, calls in (((128, 12), (5,)), ((0, 0), (1, 1, 1, 1, 1)), ((0, 0), (5,)), ((0, 0), (2, 3))):
        f = mlfilm.Film(film, prec)
        f.set_launch(*shape)
        f.init(h0)
        for c in calls:
            f.step(c)
        states.append(f.read_device())
        del f
    for s in states[1:]:
        for a, b in zip(states[0], s):
            assert torch.equal(a, b)
