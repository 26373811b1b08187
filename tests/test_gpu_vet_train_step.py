"""Gradients of the vetting network at batch sizes around the kernels' tiles: the mean of the patches' own gradients."""
import numpy as np
import pytest
import torch as _torch  # imported at collection: the first import on a fresh box is slow

from oracle import vet_oracle as vo
from tests.gpu_util import note

pytestmark = pytest.mark.gpu


# around the 16 patches of a head tile and of a bias partial sum (and the first split of the
# convolutions' weight sums); around the 64 of a product's tile; parts of the positions that end
# inside a patch (1040 of them at 259); dW5 in parts (4099)
@pytest.mark.parametrize("n", [2, 15, 16, 17, 63, 65, 259, 4099])
def test_gradient_is_the_mean_of_single_patches(n):
    from paper_1410_3677_amd import fstat as F
    if not _torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(300 + n)
    theta = vo.init_params(rng)
    theta += 0.02 * rng.standard_normal(theta.size)
    x = _torch.as_tensor((rng.chisquare(4, size=(n, vo.PATCH)) * rng.uniform(1.0, 6.0, size=(n, 1))).astype(np.float32),
                         device="cuda")
    y = _torch.as_tensor((rng.uniform(size=n) < 0.5).astype(np.float32), device="cuda")
    v = F.Vetter(n)
    v.set_params(theta.astype(np.float32))
    out = _torch.full((vo.N_PARAMS + 1,), 7.5, device="cuda")
    loss = _torch.empty(1, device="cuda")
    v.gradient(x, y, loss, out[:-1])
    got = vo.unflatten(out[:-1].cpu().numpy().astype(np.float64))
    assert float(out[-1]) == 7.5                     # nothing written past the gradient
    again = _torch.empty(vo.N_PARAMS, device="cuda")
    v.gradient(x, y, loss, again)
    assert _torch.equal(again, out[:-1])             # the same again, bit for bit
    batch_loss = float(loss)
    one, mean, loss_mean = _torch.empty(vo.N_PARAMS, device="cuda"), 0.0, 0.0
    for i in range(n):
        v.gradient(x[i:i + 1], y[i:i + 1], loss, one)
        mean = mean + one.double() / n
        loss_mean = loss_mean + loss.double() / n
    # the forward pass of a patch is the same in both (to the order of an FP32 sum); the factor
    # 1/n moves the BF16 roundings of dz5, dz4, dz3 and dz2, each at most 2^-9 of an element in
    # either run, of random sign: sqrt(4 * 2 / 3) 2^-9 of the norm; four times that in all
    assert abs(batch_loss - float(loss_mean)) <= 1e-5 * max(1.0, batch_loss)
    ref = vo.unflatten(mean.cpu().numpy())
    for name, _ in vo.SHAPES:
        rel = float(np.linalg.norm(got[name] - ref[name]) / np.linalg.norm(ref[name]))
        note(f"{n} patches, {name}: rel-L2 {rel:.2e}")
        assert rel <= 4 * (8 / 3) ** 0.5 * 2.0 ** -9, name
