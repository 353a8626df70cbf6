"""Index arithmetic of the kernels at the largest accepted sizes, on the host:
the functions that the kernels index with are compiled into a small program
and evaluated where 32-bit sums would wrap."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _run(tmp_path, body):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    src = tmp_path / "bounds.hip"
    src.write_text('#include <climits>\n#include <cstdio>\n#include "rs_internal.h"\nusing namespace rs;\n'
                   "static int bad = 0;\n"
                   '#define REQUIRE(c) do { if (!(c)) { printf("line %d: %s\\n", __LINE__, #c); bad = 1; } } while (0)\n'
                   "int main() {\n" + body + "\nreturn bad;\n}\n")
    exe = tmp_path / "bounds"
    inc = os.path.join(ROOT, "paper_2508_01485_amd", "csrc")
    r = subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-I", inc, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("slots", [1, 2047, 2048, 2049, 4096, 1 << 30, 2**31 - 4098, 2**31 - 2050, 2**31 - 2048,
                                   2**31 - 2])
def test_type2_tiles_cover_the_slots(slots, tmp_path):
    """The tiles of a graph with `slots` slots (2^31 - 2 are accepted) take
    every slot once, and their windows stay in range and in the LDS buffer,
    whatever the runs at their ends: short ones, runs of the tile's or the
    window's length, and the longest (2^30 entries)."""
    _run(tmp_path, f"""
    const int slots = (int){slots}ll, tiles = (int)(({slots}ll + kT2Tile - 1) / kT2Tile);
    for (int tile : {{0, 1, tiles / 2, tiles - 2, tiles - 1}}) {{
        if (tile < 0 || tile >= tiles) continue;
        const long long first = type2_first(tile);
        const int n = type2_count(slots, tile);
        REQUIRE(first >= 0 && n >= 1 && n <= kT2Tile && first + n <= slots);
        REQUIRE(tile < tiles - 1 ? n == kT2Tile : first + n == slots);
        for (long long len : {{1ll, 2ll, 1023ll, 1024ll, 1025ll, 2048ll, 4095ll, 4096ll, 4097ll, 1ll << 30}}) {{
            for (long long back : {{0ll, 1ll, 1023ll, 1024ll, 1025ll, 2048ll, (1ll << 30) - 1}}) {{
                if (back > first || back >= len) continue;       // the first slot's run starts `back` before the tile
                for (long long l : {{(long long)n - 1, n - len, n - len / 2 - 1}}) {{  // the last slot's leader
                    if (l >= n || l < -first || first + l + len > slots) continue;
                    const Type2Window w = type2_window(slots, tile, back ? (int)-back : (int)len, (int)l, (int)len);
                    REQUIRE(w.lo <= 0 && w.lo >= -back && first + w.lo >= 0);
                    REQUIRE(w.hi >= n && first + w.hi <= slots && w.hi - w.lo <= kT2Win);
                    if (l + len <= w.lo + kT2Win) REQUIRE(w.hi >= l + len);  // a run that fits is whole
                }}
            }}
        }}
    }}""")


@pytest.mark.parametrize("total", [0, 1, 64, 65, 2**31 - 129, 2**31 - 65, 2**31 - 64, 2**31 - 63, 2**31 - 2, 2**31 - 1,
                                   2**31])
def test_flattened_rows_are_counted_in_32_bits(total, tmp_path):
    """Groups of 64 flattened entries: those counted in 32 bits end after the
    last entry without a wrap, and all totals short of the wrap are."""
    _run(tmp_path, f"""
    const long long total = {total}ll, groups = (total + 63) / 64;
    const bool fits = groups * 64 <= (long long)INT_MAX;  // the group that ends the loop
    REQUIRE(!flat_rows_fit(total) || fits);
    REQUIRE(flat_rows_fit(total) || total > (long long)INT_MAX - 64);""")
