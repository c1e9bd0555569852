"""The step kernel's launches of two time steps against its launches of one,
and the oracle: pairs of steps, odd remainders and every tiling must give
the same bits, since the intermediate state is rounded as its storage would
round it.  Sizes sit at the edges of the tiles: strips of 54 columns, narrow
and short films whose halos wrap around them several times, segments of odd
height and a last segment shorter than the others."""
import numpy as np
import pytest

from paper_2409_16659_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mlf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    mlfilm.load_library()
    return mlfilm


def _film(n, nx, ny, seed):
    rng = np.random.default_rng(seed)
    gam = [1.0e-2, 0.7e-2, 0.6e-2, 0.5e-2][:n]
    spread = {(l, 1): inputs.young_spreading(gam[l], 20.0) for l in range(n)}
    for l in range(n):
        for k in range(2, n - l + 1):
            spread[(l, k)] = rng.uniform(-2e-3, 2e-3)
    film = inputs.film_params(n, nx, ny, gamma=gam, mu=[1e-3] * n, hstar=0.1, spread=spread)
    h0 = np.stack([(1.0, 0.8, 0.6, 0.4)[i] + 1e-3 * rng.uniform(-1, 1, (ny, nx)) for i in range(n)])
    return film, h0


@pytest.mark.parametrize("prec", ["f32", "f16mix", "bf16mix", "f16"])
@pytest.mark.parametrize("n,nx,ny,seg", [(1, 54, 20, 20), (2, 55, 41, 17), (3, 109, 37, 16), (4, 63, 33, 33),
                                         (3, 1, 40, 20), (4, 2, 3, 3), (2, 7, 1, 1), (3, 300, 50, 23)])
def test_two_steps_equal_two_single_steps(mlf, oracle_mod, prec, n, nx, ny, seg):
    film, h0 = _film(n, nx, ny, 40 + n + nx + ny)
    steps = 7
    print(f"case two-step {prec} N={n} {nx}x{ny} seg={seg}", flush=True)
    states = []
    # pairs (segments of at least 16 rows), single steps, and another tiling
    for shape, calls in [((64, seg), [steps]), ((256, seg), [1] * steps), ((512, 1), [steps]),
                         ((128, max(16, ny)), [2, 1, 4])]:
        g = mlf.Film(film, prec)
        g.init(h0)
        g.set_launch(*shape)
        for c in calls:
            g.step(c)
        assert g.steps_done == steps
        states.append(g.populations())
    for s in states[1:]:
        assert np.array_equal(states[0], s)
    if prec == "f32":
        ref = oracle_mod.Oracle(film)
        ref.init(h0)
        ref.step(steps)
        h, _, _ = ref.read()
        # FP32 deviations of 1e-3: about 1e-10 a step on heights near 1
        assert np.max(np.abs(states[0].sum(axis=1) - h)) <= 1e-8


@pytest.mark.parametrize("where", [(0, 0), (19, 53), (20, 54), (39, 99)])
def test_guard_in_every_tile(mlf, where):
    """A height that turns non-positive trips the guard whichever tile holds
    it; a healthy film does not."""
    film, h0 = _film(2, 100, 40, 5)
    g = mlf.Film(film, "f32")
    g.init(h0)
    g.set_launch(64, 20)
    g.step(4)
    f = g.populations()
    f[1, 0, where[0], where[1]] = -3.0
    g.set_populations(f)
    with pytest.raises(mlf.MlfError) as e:
        g.step(2)
    assert e.value.status in ("ENONPOSITIVE", "ENONFINITE")
    ok = mlf.Film(film, "f32")
    ok.init(h0)
    ok.set_launch(64, 20)
    ok.step(64)


@pytest.mark.parametrize("prec", ["f32", "f16mix", "f64"])
@pytest.mark.parametrize("tau", [1.0, 1.3])
@pytest.mark.parametrize("nx,ny", [(600, 2440), (600, 2450), (4, 3000)])
def test_default_shapes_of_tall_films(mlf, prec, tau, nx, ny):
    """The default launch on both sides of the line between one and two
    wavefronts per SIMD: the same bits as in a fixed shape."""
    film, h0 = _film(2, nx, ny, nx + ny)
    film["tau"] = tau
    print(f"case default shape {prec} tau={tau} {nx}x{ny}", flush=True)
    a, b = mlf.Film(film, prec), mlf.Film(film, prec)
    b.set_launch(128, 12)
    for f in (a, b):
        f.init(h0)
        f.step(5)
    assert np.array_equal(a.populations(), b.populations())
