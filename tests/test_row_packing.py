"""CPU check of the packed record rows (pack_row): the search reads the first record of every row it takes off its
queues, so a packed row, an empty one too, must name a record that exists, whatever records precede it."""
from __future__ import annotations

import os
import subprocess

from paper_2104_12911_amd import build as b

PROGRAM = r"""
#include "qdta_internal.h"
#include <cstdio>
int main() {
    long long e0, count;
    while (scanf("%lld %lld", &e0, &count) == 2) printf("%u\n", qdta::pack_row(e0, count));
    printf("%u %d\n", qdta::kNoRow, qdta::kRowCountBits);
}
"""


def test_packed_rows_name_records_that_exist(tmp_path):
    src, exe = tmp_path / "rows.hip", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-std=c++17",
                           "-I", b.INCLUDE, "-I", b.CSRC, "-x", "hip", str(src), "-o", str(exe)])
    cases = [(e0, count) for e0 in (0, 1, 15, 16, 1000, 2**25 - 1, 2**25, 2**30) for count in (0, 1, 4, 63, 64, 5000)]
    out = subprocess.run([str(exe)], input="\n".join(f"{e} {c}" for e, c in cases), capture_output=True, text=True,
                         check=True).stdout.split()
    no_row, bits = int(out[-2]), int(out[-1])
    for (e0, count), word in zip(cases, map(int, out)):
        if word & no_row:
            assert count >= 1 << bits or e0 >= 2**25, (e0, count)
            continue
        first, deg = word >> bits, word & ((1 << bits) - 1)
        assert deg == count
        # total records with this row the last one: e0 + count; the record the row starts at is one of them, or the
        # first of all
        assert first == (e0 if count else 0), (e0, count)
