"""FP64 films of three layers: workgroups of up to 256 lanes and of 512 run
separate compilations of the step kernel (with and without a row loaded
ahead); both must give the same bits, and the oracle's heights."""
import numpy as np
import pytest

from paper_2409_16659_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau,slip,exps", [(1.0, None, (9, 3)), (1.0, [0.05] * 3, (4, 3)), (1.3, None, (9, 3))])
@pytest.mark.parametrize("nx,ny", [(61, 7), (500, 33)])
def test_three_layers_in_both_compilations(oracle_mod, tau, slip, exps, nx, ny):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    gam = [1.0e-2, 0.7e-2, 0.5e-2]
    film = inputs.film_params(3, nx, ny, gamma=gam, mu=[2e-3, 3e-3, 4e-3], hstar=0.15, tau=tau, slip=slip,
                              exp_a=exps[0], exp_b=exps[1],
                              spread={(l, 1): inputs.young_spreading(gam[l], 20.0) for l in range(3)})
    rng = np.random.default_rng(nx)
    h0 = np.stack([v + 1e-3 * rng.uniform(-1, 1, (ny, nx)) for v in (1.0, 0.8, 0.6)])
    print(f"case three FP64 layers {nx}x{ny} tau={tau} exps={exps}", flush=True)
    out = []
    for shape in ((64, 6), (192, 4), (256, 33), (512, 6), (512, 33), (0, 0)):
        f = mlfilm.Film(film, "f64")
        f.init(h0)
        f.set_launch(*shape)
        f.step(6)
        out.append(f.populations())
    for o in out[1:]:
        assert np.array_equal(out[0], o)
    ref = oracle_mod.Oracle(film)
    ref.init(h0)
    ref.step(6)
    h, _, _ = ref.read()
    # a few hundred FP64 operations on numbers near 1
    assert np.max(np.abs(out[0].sum(axis=1) - h)) <= 1e-13
