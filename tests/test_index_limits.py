"""Index arithmetic of the sort's tiles and scan at the top of the accepted range.

1D-3V takes up to 2^31 - 2 markers and 2^31 - 3 buckets.  The device helpers that
form a tile's bounds, a thread's items and the scan's loads are compiled into a host
program here and compared with 64-bit arithmetic there: no item is read outside
[first, last), every one is read once, and a tile that rounds a grid up to a multiple
of eight holds nothing.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

SRC = r"""
#include "avl_device.h"
#include <cstdio>
#include <cstdlib>
using namespace avl;
static void need(bool ok, const char* what, long long a, long long b)
{
    if (!ok) { std::printf("%s: %lld %lld\n", what, a, b); std::exit(1); }
}
int main()
{
    const long long ns[] = {1, 63, 2048, 3072, 4096, 100001, 2147483646LL, 2147483645LL, 2147481601LL, 2147475457LL, 2147479551LL};
    for (long long n : ns)
        for (int size : {kSortTile, count_tile_size(0), count_tile_size(1), 256}) {
            const long long tiles = (n + size - 1) / size, rounded = (tiles + 7) / 8 * 8;
            need(tile_count(size, (int)n) == tiles, "tile_count", n, size);
            for (long long t = tiles > 4 ? tiles - 4 : 0; t < rounded; ++t) {
                need(tile_starts((int)t, size, (int)n) == (t * size < n), "tile_starts", n, t);
                if (t * size >= n) continue;
                const long long end = t * size + size < n ? t * size + size : n;
                need(tile_last((int)(t * size), size, (int)n) == end - 1, "tile_last", n, t);
                for (int off = 0; off < size; ++off)
                    need(tile_item((int)(t * size), off) == t * size + off, "tile_item", n, t);
            }
        }
    // one scan tile, all its threads: what they read lies inside, each item once
    const long long nbs[] = {5, 4096, 4097, 98305, 2147483645LL, 2147483644LL, 2147479553LL, 2147455000LL};
    for (long long nbt : nbs) {
        const long long tiles = (nbt + kScanTile - 1) / kScanTile;
        for (long long t = tiles > 2 ? tiles - 2 : 0; t < tiles; ++t) {
            const long long first = t * kScanTile, last = first + kScanTile < nbt ? first + kScanTile : nbt;
            need(tile_last((int)first, kScanTile, (int)nbt) + 1 == last, "scan tile", nbt, t);
            long long seen = 0;
            for (unsigned thread = 0; thread < (unsigned)kScanThreads; ++thread) {
                auto one = [&](unsigned b) {
                    need((long long)b >= first && (long long)b < last, "read outside", nbt, b);
                    return 1;
                };
                auto quad = [&](unsigned b) {
                    need(b % 4 == 0 && (long long)b >= first && (long long)b + 4 <= last, "load outside", nbt, b);
                    return make_int4(1, 1, 1, 1);
                };
                seen += scan_part(quad, one, (unsigned)first, (unsigned)last, thread);
            }
            need(seen == last - first, "items read", nbt, seen);
        }
    }
    std::printf("ok\n");
    return 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc missing")
def test_tile_and_scan_indices(tmp_path):
    src, exe = tmp_path / "limits.hip", tmp_path / "limits"
    src.write_text(SRC)
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-w",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           "-I", os.path.join(ROOT, "paper_1804_03901_amd", "csrc"), str(src), "-o", str(exe)],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
