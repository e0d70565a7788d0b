"""Which chunks the attention kernels read by nontemporal loads, on the CPU: a C++ program runs the kernels' own scan (csrc/kv_stream.h) over whole
batches, all lanes of it, and prints the answer per request and chunk.  No device code runs."""
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08151_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "kv_stream.h"

int main()
{
    int B, max_pages, max_kv_len, asked;
    if (std::scanf("%d %d %d %d", &B, &max_pages, &max_kv_len, &asked) != 4) return 2;
    std::vector<int32_t> lens(B), table((size_t)B * max_pages);
    for (auto& x : lens) if (std::scanf("%d", &x) != 1) return 2;
    for (auto& x : table) if (std::scanf("%d", &x) != 1) return 2;
    for (int q = 0; q < asked; ++q) {
        int i, page;
        if (std::scanf("%d %d", &i, &page) != 2) return 2;
        double keys = 0;
        bool shared = false;
        for (int lane = 0; lane < 64; ++lane) {
            const specv::KvScan s = specv::kv_scan_lane(lens.data(), table.data(), max_pages, B, max_kv_len, i, page, lane);
            keys += s.keys;
            shared = shared || s.shared;
        }
        std::printf("%.0f %d\n", keys, (int)shared);
    }
}
"""


@pytest.fixture(scope="module")
def scan(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("kv")
    (d / "scan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined", "-I", CSRC, str(d / "scan.cpp"), "-o", str(d / "scan")], check=True)

    def run(lens, table, max_kv_len, asked):
        B, max_pages = table.shape
        words = [B, max_pages, max_kv_len, len(asked), *lens, *table.ravel(), *np.ravel(asked)]
        out = subprocess.run([str(d / "scan")], input=" ".join(str(int(w)) for w in words), capture_output=True, text=True, check=True).stdout
        return [(int(a), b == "1") for a, b in (line.split() for line in out.splitlines())]
    return run


def test_the_batch_itself_is_counted_and_not_the_stated_bound(scan):
    table = np.full((5, 4096), -1)
    lens = np.array([100, 7, 0, 333, 16])
    for i in range(5):
        table[i, :(lens[i] + 15) // 16] = np.arange((lens[i] + 15) // 16) + 50 * i
    assert scan(lens, table, 65536, [(0, 0), (3, 2)]) == [(456, False)] * 2
    # lengths that the kernels refuse count as what they can be at most
    assert scan([100, -5, 0, 70000, 16], table, 65536, [(0, 0)]) == [(65652, False)]


def test_pages_of_a_common_prefix_are_found(scan):
    """Requests 0, 2 and 3 share their first 4 pages, 2 and 3 their first 8; request 1 holds the same ids at other places, request 4 behind its end."""
    lens = np.array([200, 200, 200, 200, 30])
    table = np.arange(5 * 16).reshape(5, 16) + 100
    table[[0, 2, 3], :4] = [1, 2, 3, 4]
    table[[2, 3], 4:8] = [5, 6, 7, 8]
    table[1, 8:12] = [1, 2, 3, 4]
    table[4] = table[1]
    asked = [(i, page) for i in range(4) for page in range(12)]
    got = [s for _, s in scan(lens, table, 4096, asked)]
    expect = [(i in (0, 2, 3) and page < 4) or (i in (2, 3) and page < 8) or (i == 1 and page < 1) for i, page in asked]
    assert got == expect                                   # (request 4 has one whole page, and it is request 1's)


@pytest.mark.parametrize("B", [63, 64, 65, 3000])
def test_a_window_of_requests_stands_for_a_large_batch(scan, B):
    """64 requests around a request's own are looked at, their keys times B / 64."""
    table = np.arange(B * 2).reshape(B, 2)
    table[0] = table[31] = table[B - 1] = [7777777, 7777778]
    i = min(B - 2, 64)
    got = scan(np.full(B, 32), table, 64, [(0, 0), (i, 0), (B - 1, 1)])
    assert [s for _, s in got] == [True, False, B <= 95]
    assert all(abs(k - 32 * B) <= 1e-5 * 32 * B for k, _ in got)
