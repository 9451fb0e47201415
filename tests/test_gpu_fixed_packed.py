"""The fixed-point kernel's packed 16-bit arithmetic at its edges, bit for bit
against the oracle's integer model: sky values of -32768 in every part (where
the cross product reaches 2^31), differences that round to 32768, every stage
with and without halving, one feed, and element counts around the 512 up to
which the kernel adds the self-term sums itself."""
import dataclasses

import numpy as np
import pytest

import oracle as O
import synth
from test_gpu_fixed import _gpu, _kernels, _oracle, _plan_shifts
from test_gpu_parity import _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tb,mask", [(8, 0x000), (15, 0xFFF), (15, 0x000), (2, 0xAAA)])
@pytest.mark.parametrize("n_pol", [1, 2])
def test_full_scale_values(tb, mask, n_pol):
    # eight elements on one cell, all at the same full-scale code: the cell
    # saturates to +-32768/32767 and its transform keeps the extremes
    codes = np.array([-128, 127], dtype=np.int8)
    wl = dataclasses.replace(synth.workload("aavs2"), n_ant=8, n_pol=n_pol, n_time=16, kernel_k=1)
    pos = np.zeros((8, 2))
    volt = np.empty((16, 1, n_pol, 8, 2), dtype=np.int8)
    for t in range(16):
        for p in range(n_pol):
            volt[t, 0, p, :, 0] = codes[(t >> (2 * p)) & 1]
            volt[t, 0, p, :, 1] = codes[(t >> (2 * p + 1)) & 1]
    ker = [np.ones((8, 1, 1), dtype=np.complex128)]
    _say(f"case fixed full scale: {n_pol} feed(s), twiddle bits {tb}, mask {mask:#05x}")
    plan, got = _gpu(wl, pos, volt, ker, twiddle_bits=tb, stage_shifts=mask, grid_shift=0)
    ref = _oracle(wl, pos, volt, ker, 0, _plan_shifts(wl, pos, ker, 8)[0], 0, tb, mask, 8)
    np.testing.assert_array_equal(got[0], ref["acc32"])
    assert np.abs(ref["sky_int"][0]).max() == 32768 or mask


@pytest.mark.parametrize("n_ant", [1, 511, 513])
def test_element_counts(n_ant):
    import torch

    import paper_2609_03027_amd as E
    wl = dataclasses.replace(synth.workload("aavs2"), n_ant=n_ant, n_time=7, kernel_k=3,
                             min_spacing_m=0.5)
    pos = synth.antenna_layout(wl)
    volt = synth.voltages(wl, pos)
    ker = _kernels(wl, pos, [0], seed=n_ant)
    _say(f"case fixed with {n_ant} elements, K=3")
    plan, got = _gpu(wl, pos, volt, ker, stage_shifts=0x555)
    sw, sg = _plan_shifts(wl, pos, ker, 8)
    ref = _oracle(wl, pos, volt, ker, 0, sw, sg, 8, 0x555, 8)
    np.testing.assert_array_equal(got[0], ref["acc32"])
    acc = E.Accumulator(plan)
    E.accumulate(plan, acc, volt=torch.from_numpy(volt).cuda())
    autos = torch.empty(plan.info["autos_ints"], dtype=torch.int32, device="cuda")
    acc.export(None, autos)
    torch.cuda.synchronize()
    S = O.antenna_autos(O.decode_voltages(volt[:, 0]))
    np.testing.assert_array_equal(autos.cpu().numpy().reshape(n_ant, 4), S)
