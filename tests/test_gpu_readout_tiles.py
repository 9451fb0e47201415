"""Read-out against the oracle's self terms at the edges of its tiles: sides
that are no multiple of a tile (48, 96 beside 128), one row of tiles or many
(two and eight rows a thread), one feed and two, every kernel side."""
import numpy as np
import pytest

import oracle as O
from test_gpu_parity import _say, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_chan", [3, 176])
@pytest.mark.parametrize("n_pol,k,jones", [(1, 1, False), (1, 3, False), (2, 1, False),
                                           (2, 2, False), (2, 3, False), (2, 2, True),
                                           (2, 3, True)])
def test_readout_tiles(n_chan, n_pol, k, jones):
    torch = _torch()
    import paper_2609_03027_amd as E
    rng = np.random.default_rng([n_chan, n_pol, k])
    A, T = 5, 3
    sides = np.array([96, 48, 128] * 59, dtype=np.int32)[:n_chan]
    freq = 60e6 + 1e4 * np.arange(n_chan)
    pos = rng.uniform(-20.0, 20.0, size=(A, 2))
    shape = (n_chan, A) + ((2, 2) if jones else ()) + (k, k, 2)
    table = rng.standard_normal(shape).astype(np.float32)
    volt = rng.integers(0, 256, size=(T, n_chan, n_pol, A), dtype=np.uint8)
    plan = E.Plan(pos, freq, sides, n_pol, kernel_k=k, kernel_table=table, jones=jones)
    acc = E.Accumulator(plan)
    sums = rng.uniform(0.0, 1e4, size=plan.info["image_floats"]).astype(np.float32)
    S = [O.antenna_autos(O.decode_int4(volt[:, c])) for c in range(n_chan)]
    autos = torch.from_numpy(np.concatenate(S).astype(np.int32).reshape(-1)).cuda()
    acc.import_(torch.from_numpy(sums).cuda(), autos, T)
    out = torch.empty(plan.info["image_floats"], dtype=torch.float32, device="cuda")
    _say(f"case read-out tiles: {n_chan} channels, {n_pol} feed(s), K={k}, jones={jones}")
    E.readout(plan, acc, out)
    torch.cuda.synchronize()
    out = out.cpu()
    for c in sorted({0, 1, 2, n_chan - 1}):
        n = int(sides[c])
        _, j0 = O.grid_geometry(pos, freq[c], n, k=k)
        w = table[c, ..., 0].astype(np.float64) + 1j * table[c, ..., 1]
        auto = (O.auto_term_jones(S[c], O.antenna_beams_jones(j0, w, n)) if jones else
                O.auto_term(S[c], O.antenna_beams(j0, w, n)))
        a = plan.channel_image(torch.from_numpy(sums), c).numpy().astype(np.float64)
        want = (a - auto) / T
        got = plan.channel_image(out, c).numpy()
        # FP64 up to two FP32 roundings (1 / count, the result)
        tol = 2.0 ** -23 * np.abs(want) + 1e-11 * np.abs(auto).max()
        assert np.all(np.abs(got - want) <= tol * 1.01)
