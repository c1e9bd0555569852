"""Films one row high in 16-bit storage, which the step kernel holds by lane
shifts without marching, against the same film repeated over two rows, which
it marches: heights differ by roundings of the storage only (at most one unit
of the rest plane's deviation per step), and a film alone, in a batch and with
stochastic rounding draws the same bits."""
import numpy as np
import pytest

from paper_2409_16659_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f16", "bf16", "f16mix", "bf16mix"])
@pytest.mark.parametrize("n,nx", [(1, 1), (2, 5), (3, 60), (4, 61), (2, 250)])
@pytest.mark.parametrize("tau", [1.0, 1.3])
def test_one_row_against_two(prec, n, nx, tau):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    gam = [1.0e-2, 0.7e-2, 0.6e-2, 0.5e-2][:n]
    films = [inputs.film_params(n, nx, ny, gamma=gam, mu=[1e-3] * n, hstar=0.1, tau=tau,
                                spread={(l, 1): inputs.young_spreading(gam[l], 20.0) for l in range(n)})
             for ny in (1, 2)]
    rng = np.random.default_rng(n + nx)
    row = np.stack([v + 1e-3 * rng.uniform(-1, 1, (1, nx)) for v in (1.0, 0.8, 0.6, 0.4)[:n]])
    steps = 6
    print(f"case one row {prec} N={n} nx={nx} tau={tau}", flush=True)
    h = []
    for film, h0 in zip(films, (row, np.repeat(row, 2, axis=1))):
        f = mlfilm.Film(film, prec)
        f.init(h0)
        f.step(steps)
        h.append(f.read()[0])
        if film["ny"] == 1:
            alone = f.populations()
    unit = 2.0 ** (-10 if prec.startswith("f16") else -7)
    dev = max(np.abs(row - row.mean(axis=2, keepdims=True)).max(), 1e-12)
    assert np.abs(h[1] - h[0]).max() <= steps * unit * dev + 1e-7
    for sr in ((False, True) if prec in ("f16", "bf16") else (False,)):
        b = mlfilm.Batch([films[1], films[0]], prec)
        g = mlfilm.Film(films[0], prec)
        b.set_rounding(sr) if sr else None
        g.set_rounding(sr) if sr else None
        b.init(0, np.repeat(row, 2, axis=1))
        b.init(1, row)
        g.init(row)
        b.step(steps)
        for _ in range(steps):
            g.step(1)
        if not sr:
            assert np.array_equal(g.populations(), alone)
        for x, y in zip(b.read(1), g.read()):
            assert np.array_equal(x, y)
