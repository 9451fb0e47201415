"""The rules for time slices, compiled on the host."""
from test_twiddles_cpu import _compile_and_run

HEAD = """#include <cstdio>
#include "slices.h"
using namespace epic;
static void best(long long items, long long slots, long long n, int s, long long f, long long u, bool fr) {
    const SliceChoice c = best_slices(items, slots, n, s, f, u, fr);
    printf("%d %d\\n", c.slices, c.len);
}
"""


def _run(calls, tmp_path):
    out = _compile_and_run(HEAD + "int main() {" + "".join(
        "best(%d, %d, %d, %d, %d, %d, %s);" % (*c[:6], str(c[6]).lower()) for c in calls) + "}\n", tmp_path)
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def _cost(items, slots, n, floats, frames, s, length):
    """Time of s slices of `length` samples (the last one the rest), in samples."""
    rest = n - (s - 1) * length
    assert 0 < rest <= length
    sets = 0.0 if frames or s == 1 else 1.0 + s * floats * 8.0 / 18e6
    # a short last slice on what the others leave of the fullest of 32 engines
    spare = slots // 32 - -(-items * (s - 1) // 32)
    if spare > 0 and s > 1:
        return max(length + 6.0, -(--(-items // 32) // spare) * (rest + 6.0)) + sets
    return -(-items * s // slots) * (length + 6.0) + sets


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
    n, u = 2 ** 31 - 1, 2 ** 28 - 1
    assert _run([(2, 256, n, 64, 65536, n, True), (2, 256, 8 * u, 64, 65536, u, True),
                 (256, 256, n, 64, 8388608, n, True)], tmp_path) == [(1, n), (8, u), (1, n)]


def test_slices_cover_the_call_at_the_cost_stated(tmp_path):
    """Whole units that cover every sample once, no set more than allowed, never
    dearer than one slice, and no dearer than 1 / 0.97 of the best equal slices;
    frames of any length, one sample too, pay for no partial sets."""
    calls = [(items, slots, n // u * u, s_max, floats, u, fr)
             for items, slots, floats in ((2, 256, 65536), (6, 256, 196608), (26, 256, 851968),
                                          (96, 256, 3145728), (200, 256, 6553600), (224, 256, 7340032),
                                          (256, 256, 8388608), (300, 256, 9830400), (243, 1024, 2985984))
             for n in (1, 7, 25, 100, 1000, 65536) for u, fr in ((1, True), (1, False), (4, True))
             for s_max in (1, 2, 5, 64) if n >= u]
    for c, (s, length) in zip(calls, _run(calls, tmp_path)):
        items, slots, n, s_max, floats, u, fr = c
        assert 1 <= s <= s_max and length % u == 0 and (s - 1) * length < n <= s * length, (c, s, length)
        got = _cost(items, slots, n, floats, fr, s, length)
        for k in range(1, s_max + 1):
            eq = -(-(-(-n // k)) // u) * u
            if -(-n // eq) == k:
                assert 0.97 * got <= _cost(items, slots, n, floats, fr, k, eq) + 1e-9, (c, s, length, k)
    # without the sets' cost some frame calls take more slices than integrations
    frames = [c for c in calls if c[6] and c[5] == 1]
    assert any(a[0] > b[0] for a, b in zip(_run(frames, tmp_path),
                                           _run([(*c[:6], False) for c in frames], tmp_path)))


def test_reserved_sets_are_bounded(tmp_path):
    """Channels of 128^2 (65536 floats a set each) keep at most 96 MiB of partial sets,
    none where the items alone fill whole rounds, and many for one channel."""
    chans = list(range(1, 129)) + [256, 1024]
    out = _compile_and_run(
        HEAD + "int main() {" + "".join(
            f'printf("%d\\n", reserved_slices({2 * c}, 256, {65536 * c}));' for c in chans) + "}\n", tmp_path)
    got = dict(zip(chans, map(int, out.split())))
    for c in chans:
        assert 1 <= got[c] <= 64 and (got[c] == 1 or got[c] * c / 4.0 <= 96.0), (c, got[c])
    assert got[128] == got[256] == got[1024] == 1 and got[1] >= 32
