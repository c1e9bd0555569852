"""Heights that start at any element of an allocation.  Addresses that are not
multiples of 16 all take the same order of sums, so tensors one, two and three
elements off give the same bits, in prediction, loss and gradient; the
gradient is held against the FP64 reference with the tolerances of
test_gpu_surrogate_backward.py."""
import numpy as np
import pytest

from oracle import nop

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,ny", [(1, 64), (24, 128)])   # both forms of the patch layers
def test_heights_at_any_element(batch, ny):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_16659_amd import mlfilm

    rng = np.random.default_rng(batch)
    vec = nop.init_params(rng, 2, 128, 1)
    vec = (vec + rng.normal(0, 0.01, vec.size)).astype(np.float32)
    s = mlfilm.Surrogate(2, 256, ny, width=128, blocks=1, batch=batch, scale=1e-2)
    s.set_params(vec)
    n0 = (1.0 + 1e-2 * rng.normal(size=(batch, 2, ny, 256))).astype(np.float32)
    n1 = (n0 + 1e-3 * rng.normal(size=n0.shape)).astype(np.float32)
    h0, h1 = torch.from_numpy(n0).cuda(), torch.from_numpy(n1).cuda()

    def at(t, off):
        buf = torch.empty(t.numel() + 4, dtype=torch.float32, device="cuda")
        v = buf[off:off + t.numel()].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16 == 4 * off
        return v

    out = []
    for off0, off1 in ((1, 0), (2, 3), (3, 1)):
        print(f"case surrogate batch {batch} offsets {off0}, {off1}", flush=True)
        a0, a1 = at(h0, off0), at(h1, off1)
        out.append((s.predict(a0), s.loss(a0, a1), *s.gradient(a0, a1)))
    for p, l, m, g in out[1:]:
        assert torch.equal(p, out[0][0]) and (l, m) == out[0][1:3] and np.array_equal(g, out[0][3])
    assert out[0][1] == out[0][2]
    if batch == 1:
        ref_loss, ref = nop.Net(2, 128, 1, 1e-2, use_bf16=True).gradient(vec.astype(np.float64),
                                                                         n0.astype(np.float64), n1.astype(np.float64))
        assert abs(out[0][1] - ref_loss) <= 2e-3 * ref_loss
        for name, (o, size) in nop.layout(2, 128, 1)[0].items():
            e = np.linalg.norm(out[0][3][o:o + size] - ref[o:o + size]) / max(np.linalg.norm(ref[o:o + size]), 1e-300)
            assert e <= 1e-2, (name, e)
