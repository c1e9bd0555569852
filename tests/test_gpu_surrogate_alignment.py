"""Heights that start at any element of an allocation: prediction, loss and
gradient take tensors whose address is a multiple of 4 only, and give what
they give for a copy on a 16-byte boundary, up to the order in which the
plane means are summed."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 24])   # both forms of the patch layers
@pytest.mark.parametrize("off0,off1", [(1, 0), (0, 3), (2, 1)])
def test_heights_at_any_element(batch, off0, off1):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    print(f"case surrogate batch {batch} offsets {off0}, {off1}", flush=True)
    rng = np.random.default_rng(batch)
    s = mlfilm.Surrogate(2, 256, 128, width=128, blocks=1, batch=batch, scale=1e-2)
    s.set_params(rng.normal(0, 0.03, s.param_count).astype(np.float32))
    h0 = torch.from_numpy((1.0 + 1e-2 * rng.normal(size=(batch, 2, 128, 256))).astype(np.float32)).cuda()
    h1 = h0 + 1e-3 * torch.from_numpy(rng.normal(size=h0.shape).astype(np.float32)).cuda()

    def at(t, off):
        buf = torch.empty(t.numel() + 4, dtype=torch.float32, device="cuda")
        v = buf[off:off + t.numel()].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16 == 4 * off
        return v

    a0, a1 = at(h0, off0), at(h1, off1)
    p, q = s.predict(h0), s.predict(a0)
    # means of 32768 values near 1 differ by some 2^-24 each way, increments by
    # that over the scale times the network's gain
    assert float((p - q).abs().max()) <= 1e-6
    assert abs(s.loss(a0, a1) - s.loss(h0, h1)) <= 1e-4 * s.loss(h0, h1)
    (l, g), (m, k) = s.gradient(h0, h1), s.gradient(a0, a1)
    assert abs(l - m) <= 1e-4 * l
    assert np.linalg.norm(g - k) <= 1e-3 * np.linalg.norm(g)
