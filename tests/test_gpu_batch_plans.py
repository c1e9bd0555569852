"""A batch keeps a table and a work list for launches of two steps and others
for single steps: calls that mix both, with a graph, after films were given
new heights, in default and fixed shapes, give each film the bits that it has
when stepped alone.  Films are ragged, some one row or a few rows high."""
import numpy as np
import pytest

from paper_2409_16659_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [(2, 130, 70), (3, 61, 33), (1, 54, 1), (4, 100, 18), (2, 300, 5), (3, 230, 120)]


def _film(n, nx, ny, tau=1.0):
    gam = [1.0e-2, 0.7e-2, 0.6e-2, 0.5e-2][:n]
    return inputs.film_params(n, nx, ny, gamma=gam, mu=[1e-3] * n, hstar=0.1, tau=tau,
                              spread={(l, 1): inputs.young_spreading(gam[l], 20.0) for l in range(n)})


def _heights(n, nx, ny, seed):
    rng = np.random.default_rng(seed)
    return np.stack([v + 1e-3 * rng.uniform(-1, 1, (ny, nx)) for v in (1.0, 0.8, 0.6, 0.4)[:n]])


@pytest.mark.parametrize("prec,tau", [("f32", 1.0), ("f16mix", 1.0), ("f16", 1.0), ("f64", 1.0), ("f32", 1.3)])
@pytest.mark.parametrize("shape", [(0, 0, 0), (64, 20, 0), (256, 16, 1), (128, 3, 0)])
def test_mixed_calls_match_films_stepped_alone(prec, tau, shape):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    print(f"case batch plans {prec} tau={tau} shape={shape}", flush=True)
    films = [_film(*s, tau=tau) for s in SIZES]
    b = mlfilm.Batch(films, prec, stream=torch.cuda.Stream())
    b.set_launch(*shape)

    def start(seed):
        for f, s in enumerate(SIZES):
            b.init(f, _heights(*s, seed + f))

    def check(steps, seed):
        for f, s in enumerate(SIZES):
            g = mlfilm.Film(films[f], prec)
            g.set_launch(64, 1)  # single steps in short segments
            g.init(_heights(*s, seed + f))
            g.step(steps)
            for got, want in zip(b.read(f), g.read()):
                assert np.array_equal(got, want), (f, steps)

    start(10)
    for n in (1, 2, 3, 1):
        b.step(n)
    check(7, 10)
    start(30)            # new reference heights: both tables are out of date
    b.step(1)
    b.step(4)
    check(5, 30)
    b.capture(6)
    start(50)            # the graph's launches read the new tables
    b.step(6)
    b.step(1)
    b.step(13)
    check(20, 50)
    assert b.steps_done == 32


def test_default_shape_of_a_batch_on_both_sides_of_the_cache():
    """Films that together fit the Infinity Cache and films that do not, wide
    ones and narrow ones, take different defaults and the same bits."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    for prec, sizes in (("f64", [(2, 900, 500), (2, 800, 700)]), ("f32", [(1, 200, 300)] * 3),
                        ("f64", [(3, 300, 300)] * 8), ("f16mix", [(2, 1500, 1400)])):
        films = [_film(*s) for s in sizes]
        out = []
        for shape in ((0, 0, 0), (128, 12, 0)):
            b = mlfilm.Batch(films, prec)
            b.set_launch(*shape)
            print(f"case default batch {prec} {sizes[0]} x {len(sizes)} {b.get_launch()}", flush=True)
            for f, s in enumerate(sizes):
                b.init(f, _heights(*s, f))
            b.step(1)
            b.step(4)
            out.append([b.read(f) for f in range(len(sizes))])
            del b
        for x, y in zip(*out):
            for p, q in zip(x, y):
                assert np.array_equal(p, q)
