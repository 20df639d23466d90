"""CPU: the search of a sorted list that the sampled estimators share, compiled
for the host over lists that are computed instead of stored: every read inside
the list, and the answer, up to the longest lists and the largest offsets."""
import os
import subprocess

from paper_1011_0468_amd import build

HARNESS = r"""
#include "tc_prefix.h"
#include <cstdio>

struct Spread {  // len ids spread evenly over [0, n), at the places lo .. end - 1 of a column array
    int64_t lo, end, n;
    bool* outside;
    int32_t operator[](int64_t i) const {
        if (i < lo || i >= end) { *outside = true; return 0; }
        return (int32_t)((i - lo) * n / (end - lo));
    }
};

int main() {  // lines "lo end n y": "read-outside found expected" each
    long long lo, end, n, y;
    while (scanf("%lld %lld %lld %lld", &lo, &end, &n, &y) == 4) {
        const int64_t len = end - lo, i = (y * len + n - 1) / n;  // the first id >= y
        bool outside = false;
        const bool got = tc::in_list(Spread{lo, end, n, &outside}, (int32_t)lo, (int32_t)end, (int32_t)y, 1.0f / (float)n);
        printf("%d %d %d\n", outside, got, i < len && i * n / len == y);
    }
}
"""

LAST = (1 << 31) - 2  # the largest number of entries
LENGTHS = [0, 1, 32, 33, 1000, (1 << 24) + 1, (1 << 26) + 5, (1 << 29) + 33, (1 << 30) - 1]


def test_reads_and_answers(tmp_path):
    (tmp_path / "h.hip").write_text(HARNESS)
    subprocess.check_call([build.HIPCC, *build.FLAGS, "-I", build.CSRC, str(tmp_path / "h.hip"), "-o",
                           str(tmp_path / "h")], stderr=subprocess.DEVNULL)
    cases = []
    for end in (LAST, 1 << 30):
        for length in LENGTHS:
            for spare in (1, 3, 1 << 20):
                n = min(length + spare, (1 << 31) - 1)
                ys = {0, 1, n // 3, n // 2, n // 2 + 1, n - 2, n - 1}
                cases += [(end - length, end, n, y) for y in sorted(ys) if 0 <= y < n]
    out = subprocess.run([str(tmp_path / "h")], input="".join("%d %d %d %d\n" % c for c in cases), check=True,
                         capture_output=True, text=True).stdout.splitlines()
    assert len(out) == len(cases)
    for case, line in zip(cases, out):
        outside, got, want = line.split()
        assert (outside, got) == ("0", want), case
