"""Graph replays after calls that leave the populations in either buffer: a
film and a batch whose launches take two steps, against ones stepped without
a graph."""
import numpy as np
import pytest

from paper_2409_16659_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps,calls", [(8, (2, 8, 8, 1, 8, 10, 3, 24)), (6, (6, 2, 6, 1, 6, 7, 18))])
def test_replays_from_either_buffer(steps, calls):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    film = inputs.film_params(2, 70, 40, gamma=[1e-2, 7e-3], mu=[2e-3, 3e-3], hstar=0.15,
                              spread={(l, 1): inputs.young_spreading(1e-2, 20.0) for l in range(2)})
    rng = np.random.default_rng(3)
    h0 = np.stack([v + 1e-3 * rng.uniform(-1, 1, (40, 70)) for v in (1.0, 0.8)])
    a = mlfilm.Film(film, "f32", check_every=5, stream=torch.cuda.Stream())
    e = mlfilm.Film(film, "f32", check_every=5)
    b = mlfilm.Batch([film, film], "f32", stream=torch.cuda.Stream())
    for g in (a, e):
        g.set_launch(64, 20)
        g.init(h0)
    b.set_launch(64, 20)
    for f in range(2):
        b.init(f, h0)
    a.capture(steps)
    b.capture(steps)
    for n in calls:
        print(f"case graph of {steps}, call of {n}", flush=True)
        a.step(n)
        e.step(n)
        b.step(n)
        want = e.populations()
        torch.cuda.synchronize()
        assert a.steps_done == e.steps_done == b.steps_done
        assert np.array_equal(a.populations(), want)
        for got, ref in zip(b.read(1), e.read()):
            assert np.array_equal(got, ref)
