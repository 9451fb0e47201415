"""epic_image on random grids against the FP64 transform, for every compiled side
and two that are no powers of two: one feed and two, fewer and more images than
workgroups, in place and out of place, and a grid tensor that starts 8 bytes off
a 16-byte boundary."""
import numpy as np
import pytest

from helpers import U32
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16, 32, 48, 64, 96, 128])
@pytest.mark.parametrize("n_pol,n_chan,n_time,in_place", [(1, 1, 1, False), (2, 3, 5, True),
                                                          (2, 1, 300, False)])
def test_image(n, n_pol, n_chan, n_time, in_place):
    torch = _torch()
    import paper_2609_03027_amd as E
    rng = np.random.default_rng([n, n_pol, n_time])
    plan = E.Plan(np.zeros((1, 2)), np.full(n_chan, 60e6), np.full(n_chan, n, dtype=np.int32),
                  n_pol, kernel_k=1)
    per_t = plan.info["grid_elems_per_t"]
    g = (rng.standard_normal((n_time, per_t)) + 1j * rng.standard_normal((n_time, per_t)))
    g = g.astype(np.complex64)
    buf = torch.empty(1 + g.size, dtype=torch.complex64, device="cuda")
    src = buf[1:].view(n_time, per_t)
    src.copy_(torch.from_numpy(g))
    dst = src if in_place else torch.empty((n_time, per_t), dtype=torch.complex64, device="cuda")
    _say(f"case image {n}^2, {n_pol} feed(s), {n_chan} channels, {n_time} samples, "
         f"in place {in_place}")
    E.image(plan, src, n_time, dst)
    torch.cuda.synchronize()
    got = dst.cpu().numpy().reshape(-1, n, n)
    x = np.fft.ifftshift(g.reshape(-1, n, n).astype(np.complex128), axes=(-2, -1))
    want = np.fft.fftshift(np.fft.ifft2(x), axes=(-2, -1)) * (n * n)
    # about two roundings per radix-2 level, log2(n^2) levels
    bound = 2.0 * np.log2(float(n) * n) * U32
    err = np.abs(got - want)
    assert np.sqrt(np.mean(err ** 2)) <= bound * np.sqrt(np.mean(np.abs(want) ** 2))
    assert err.max() <= 2.0 * bound * np.abs(want).max()
