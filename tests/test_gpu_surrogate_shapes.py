"""The surrogate's launch shapes against each other: the patch layers have a
form for small batches and one for large ones, the convolutions groups of
32, 64 or all channels.  All add in the same order, so a film's prediction
has the same bits whatever batch it comes in (batches around every switch),
and the gradient of a batch is the mean of its parts' gradients up to the
FP32 order of the sums over films."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,N,batches", [(128, 3, (1, 7, 8, 9, 15, 16, 17)), (64, 4, (1, 15, 16, 17, 31, 32, 33)),
                                         (128, 1, (3, 8, 9)), (64, 2, (16, 17))])
def test_prediction_is_the_same_in_every_batch(C, N, batches):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    rng = np.random.default_rng(C + N)
    top = max(batches)
    s = mlfilm.Surrogate(N, 256, 256, width=C, blocks=1, batch=top, scale=1e-2)
    s.set_params(rng.normal(0, 0.03, s.param_count).astype(np.float32))
    h = torch.from_numpy((1.0 + 1e-2 * rng.normal(size=(top, N, 256, 256))).astype(np.float32)).cuda()
    h1 = h + 1e-3 * torch.randn(h.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    want = torch.cat([s.predict(h[i:i + 1]) for i in range(top)])
    one = [s.gradient(h[i:i + 1], h1[i:i + 1]) for i in range(min(9, top))]
    for b in batches:
        print(f"case C={C} N={N} batch {b}", flush=True)
        assert torch.equal(s.predict(h[:b]), want[:b])
        if b <= len(one):
            loss, g = s.gradient(h[:b], h1[:b])
            ref = np.mean([v[1].astype(np.float64) for v in one[:b]], axis=0)
            assert abs(loss - np.mean([v[0] for v in one[:b]])) <= 1e-5 * loss
            assert np.linalg.norm(g - ref) <= 1e-4 * np.linalg.norm(ref)


@pytest.mark.parametrize("C", [64, 128])
def test_weight_gradient_slices(C):
    """Slices of one chunk of pixels (one film) against slices of one or two,
    two or three, three or four, and five or six: odd and even counts and the
    repeated last chunk of the loads issued two ahead.  At most 2^13 FP32
    additions in another order, tolerance as above."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    rng = np.random.default_rng(C)
    s = mlfilm.Surrogate(1, 256, 256, width=C, blocks=2, batch=7, scale=1e-2)
    s.set_params(rng.normal(0, 0.03, s.param_count).astype(np.float32))
    h = torch.from_numpy((1.0 + 1e-2 * rng.normal(size=(7, 1, 256, 256))).astype(np.float32)).cuda()
    h1 = h + 1e-3 * torch.randn(h.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    one = [s.gradient(h[i:i + 1], h1[i:i + 1])[1].astype(np.float64) for i in range(7)]
    for b in (2, 3, 4, 7):
        print(f"case C={C} batch {b}", flush=True)
        g, ref = s.gradient(h[:b], h1[:b])[1], np.mean(one[:b], axis=0)
        assert np.linalg.norm(g - ref) <= 1e-4 * np.linalg.norm(ref)
