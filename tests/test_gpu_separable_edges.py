"""The separable DFT-GEMM at the edges of its sample pipeline and gather lists:
one to three samples (fewer than the pipeline is deep), an odd count in one
slice, one element, element counts around a workgroup's and the largest, and
half the elements in one cell, whose list is then longer than one batch."""
import numpy as np
import pytest

import oracle as O
from helpers import image_errors
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu

FREQ = 60e6
CELL = 0.5 * 299792458.0 / FREQ
# operand rounding: FP16, and BF16 hi + lo without the lo lo product
ROUND = {1: 2.0 ** -11, 3: 2.0 ** -16}


@pytest.mark.parametrize("prec", [1, 3])
@pytest.mark.parametrize("n,aperture,n_ant,n_time,crowd", [
    (128, 64, 1, 1, False),
    (128, 64, 65, 2, False),
    (128, 64, 40, 3, True),
    (128, 64, 513, 5, True),
    (128, 64, 1024, 3, False),
    (128, 30, 64, 1, True),
    (64, 64, 257, 2, True),
    (64, 20, 3, 1, False),
    (32, 32, 16, 3, True),
])
def test_separable_edges(n, aperture, n_ant, n_time, crowd, prec):
    torch = _torch()
    import paper_2609_03027_amd as E
    rng = np.random.default_rng([n, aperture, n_ant, n_time])
    lo = (n - aperture) // 2
    x = rng.integers(lo, lo + aperture - 2, size=(n_ant, 2))
    if crowd:
        x[::2] = lo + aperture // 3
    x = x + 0.5 + rng.uniform(0.0, 0.49, size=(n_ant, 2))       # j0 = floor(x - 1/2), K = 3
    pos = (x - n / 2.0) * CELL
    volt = rng.integers(0, 256, size=(n_time, 2, 2, n_ant), dtype=np.uint8)
    _say(f"case separable edges {n}^2 of {aperture}: {n_ant} elements, {n_time} samples, "
         f"crowded {crowd}, precision {prec}")
    plan = E.Plan(pos, np.full(2, FREQ), np.full(2, n, dtype=np.int32), 2, aperture_n=aperture,
                  precision=prec, xform=E.XFORM_DFT_SEPARABLE)
    acc = E.Accumulator(plan)
    E.accumulate(plan, acc, volt=torch.from_numpy(volt).cuda())
    out = torch.empty(plan.info["image_floats"], dtype=torch.float32, device="cuda")
    autos = torch.empty(plan.info["autos_ints"], dtype=torch.int32, device="cuda")
    acc.export(out, autos)
    torch.cuda.synchronize()
    gx, j0 = O.grid_geometry(pos, FREQ, n, k=3)
    w = O.gaussian_kernel(gx, j0, 3, 0.5)
    # grid, Fa and H are rounded once each: an error of about one rounding in E's
    # RMS, twice that in a product, at most 4.5 standard deviations of it over
    # the image's pixels, against a maximum no smaller than the mean square
    tol = 10 * ROUND[prec]
    for c in range(2):
        e = O.decode_int4(volt[:, c])
        want = O.accumulate(O.sky(O.grid(e, j0, w, n)))
        mx, _ = image_errors(plan.channel_image(out.cpu(), c).numpy(), want)
        assert mx.max() <= tol, (c, mx, tol)
        np.testing.assert_array_equal(autos.cpu().numpy().reshape(2, n_ant, 4)[c],
                                      O.antenna_autos(e))
