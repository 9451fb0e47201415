"""The rules for time slices, compiled on the host."""
from test_twiddles_cpu import _compile_and_run

HEAD = '#include <cstdio>\n#include "slices.h"\nusing namespace epic;\n'


def test_slice_lengths_of_very_long_calls(tmp_path):
    """Frames may be as long as a call: up to 2^31 - 1 samples, in whole frames."""
    calls = [(2 ** 31 - 1, 1, 1), (2 ** 31 - 1, 64, 1), (2 ** 31 - 1, 1, 2 ** 31 - 1),
             (3 * 2 ** 29, 1, 3 * 2 ** 29), (3 * 2 ** 29, 3, 2 ** 29), (2 ** 30, 7, 2 ** 20),
             (100, 3, 4), (1, 1, 1)]
    out = _compile_and_run(
        HEAD + "int main() {" +
        "".join(f'printf("%lld\\n", (long long)slice_len({n}, {s}, {u}));' for n, s, u in calls) + "}\n",
        tmp_path)
    for (n, s, u), got in zip(calls, map(int, out.split())):
        each = -(-n // s)
        assert got == -(-each // u) * u and 0 < got <= n and got % u == 0, (n, s, u, got)


def test_slice_counts_of_very_long_calls(tmp_path):
    """One frame that long is one slice; eight of 2^28 - 1 samples are eight where
    the chip is idle."""
    out = _compile_and_run(
        HEAD + "int main() {"
        'printf("%d ", pair_slices(2, 256, 2147483647, 64, 65536, 2147483647, true));'
        'printf("%d ", pair_slices(2, 256, 8LL * 268435455, 64, 65536, 268435455, true));'
        'printf("%d", pair_slices(256, 256, 2147483647, 64, 8388608, 2147483647, true)); }\n', tmp_path)
    assert [int(x) for x in out.split()] == [1, 8, 1]


def _rule(items, slots, n_time, s_max, floats, unit, frames):
    """Rounds of (samples a slice + 6), and for integrations the partial sets' traffic."""
    best = cost = None
    for s in range(1, s_max + 1):
        tps = -(-(-(-n_time // s)) // unit) * unit
        if -(-n_time // tps) != s:
            continue
        c = -(-items * s // slots) * (tps + 6.0)
        c += 0.0 if frames or s == 1 else 1.0 + s * floats * 8.0 / 18e6
        if best is None or c < 0.97 * cost:
            best, cost = s, c
    return best


def test_frames_of_any_length_pay_for_no_partial_sets(tmp_path):
    calls = [(2 * c, 256, n // u * u, 64, 65536 * c, u, fr)
             for c in (1, 3, 5, 9, 24, 33, 60, 100, 112) for n in (24, 100, 1000)
             for u, fr in ((1, True), (1, False), (4, True))]
    out = _compile_and_run(
        HEAD + "int main() {" + "".join(
            f'printf("%d\\n", pair_slices({i}, {sl}, {n}, {m}, {f}, {u}, {str(fr).lower()}));'
            for i, sl, n, m, f, u, fr in calls) + "}\n", tmp_path)
    got = list(map(int, out.split()))
    assert got == [_rule(*c) for c in calls]
    # the sets do decide for integrations of these lengths
    assert any(_rule(*c) != _rule(*c[:6], False) for c in calls if c[6] and c[5] == 1)
