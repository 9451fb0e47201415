"""Row-unfolded groups reserve time-slice sets for the workgroups that a CU
really holds: with 2048 elements staged in LDS two of 96 x 96 and four of
48 x 48, with 64 elements four and twelve (registers)."""
import numpy as np
import pytest

from test_gpu_parity import _say, _torch
from test_slices_cpu import HEAD
from test_twiddles_cpu import _compile_and_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,n_ant,per_cu", [(96, 64, 4), (96, 2048, 2), (48, 64, 12), (48, 2048, 4)])
def test_sets_follow_occupancy(side, n_ant, per_cu, tmp_path):
    _torch().zeros(1, device="cuda")
    import paper_2609_03027_amd as E
    n_chan = 8                                     # one channel on each XCD: 24 items
    pos = np.random.default_rng(side).uniform(-0.2 * side, 0.2 * side, size=(n_ant, 2)) * 2.49
    plan = E.Plan(pos, np.full(n_chan, 60e6), np.full(n_chan, side, dtype=np.int32), 2)
    i = plan.info
    floats = i["image_floats"]
    sets = (i["bytes_acc"] - 4 * floats - 4 * i["autos_ints"] - 16 * n_chan * 3 * 25) // (4 * floats)
    want = int(_compile_and_run(
        HEAD + f'int main() {{ printf("%d", reserved_slices(24, {256 * per_cu}, {floats})); }}\n', tmp_path))
    _say(f"case {side}^2, {n_ant} elements: {sets} sets, {want} wanted")
    assert sets == want
