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
        'printf("%d ", pair_slices(2, 256, 2147483647, 64, 65536, 2147483647));'
        'printf("%d ", pair_slices(2, 256, 8LL * 268435455, 64, 65536, 268435455));'
        'printf("%d", pair_slices(256, 256, 2147483647, 64, 8388608, 2147483647)); }\n', tmp_path)
    assert [int(x) for x in out.split()] == [1, 8, 1]
