"""Plain arithmetic of the library (csrc/layout.h), compiled with the host
compiler: the working arrays of a context hold every size that reuses them."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2107_12720_amd", "csrc")


def run_cpp(tmp_path, body, headers):
    src = tmp_path / "t.cpp"
    inc = "".join(f'#include "{h}"\n' for h in headers)
    src.write_text("#include <cstdio>\n#include <initializer_list>\n" + inc +
                   "int main() { using namespace trim; long long bad = 0;\n" + body +
                   '\nprintf("%lld\\n", bad); return bad != 0; }\n')
    exe = tmp_path / "t"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-ftrapv", "-I", CSRC, str(src),
                           "-o", str(exe)])
    return subprocess.run([str(exe)], capture_output=True, text=True)


@pytest.mark.parametrize("needs", ["1, 63, 64, 65, 960, 961, 3589, 3590, 4095, 4096, 4097",
                                   "65536, 100000, 1000000, 33554431, 33554432, 536870912"])
def test_arrays_hold_every_size_that_reuses_them(tmp_path, needs):
    # every n up to the capacity of every first call `need` (large ranges: the ends)
    r = run_cpp(tmp_path, """
        for (long long need : {%s}) {
            const long long cap = work_capacity(need), old = need + need / 8 + 64;
            if (cap < need || cap %% 4) ++bad;
            // 8 + 8 + 4 + 12 bytes and more of other arrays per vertex: no more than without
            // the room behind the bitmaps
            if (44 * cap + 4 * work_c_ints(cap) > 48 * old) ++bad;
            for (long long n = 1; n <= cap; n += n < cap - 4096 && n > 8192 ? cap / 4096 + 1 : 1) {
                if (2 * round_bitmap_words(n) > work_c_ints(cap)) ++bad;
                if (n >= kTwoWatchMinN && two_watch_ints(n) > work_c_ints(cap)) ++bad;
                if ((n + 3) / 4 * 4 > cap) ++bad;
            }
        }""" % needs, ["layout.h"])
    assert r.returncode == 0, r.stdout


def test_supports_in_lds_fit_with_every_block(tmp_path):
    # the sizes that go to an array of kWatchLdsN entries (batches, any opts.block; the one
    # wavefront's 4,096) and the largest each block takes
    r = run_cpp(tmp_path, """
        for (int lanes = 64; lanes <= 1024; lanes += 64) {
            int most = 0;
            for (int n = 1; n <= 2 * kWatchLdsN; ++n)
                if (watch_fits(n, lanes, kWatchLdsN)) {
                    most = n;
                    if (watch_padded(n, lanes) < n || watch_padded(n, lanes) > kWatchLdsN) ++bad;
                }
            if ((lanes & (lanes - 1)) ? most < 57344 : most != kWatchLdsN) ++bad;
        }
        if (watch_fits(65536, 768, kWatchLdsN) || watch_fits(61441, 768, kWatchLdsN)) ++bad;
        if (!watch_fits(4096, 64, 4096) || watch_fits(4097, 64, 4096)) ++bad;
        // one workgroup of a small graph (small.hip): half as many lanes as vertices, 256 to 1,024
        for (int n = 0; n <= 8192; ++n) {
            const int b = (n / 2 + 63) / 64 * 64;
            if (!watch_fits(n, b < 256 ? 256 : b > 1024 ? 1024 : b, 8192)) ++bad;
        }""", ["layout.h"])
    assert r.returncode == 0, r.stdout


def test_scans_end_at_the_largest_edge_number(tmp_path):
    # steps of every size over lists that end at 2^31 - 1 (signed overflow
    # traps): each entry once, in order, nothing outside the list
    r = run_cpp(tmp_path, """
        for (int step : {4, 64, 512})
            for (int len : {0, 1, 3, 4, 5, 63, 64, 65, 511, 512, 513, 1500})
                for (int e : {2147483647, 2147483646, 1500}) {
                    const int p0 = e - len;
                    long long next = p0;
                    for (uint32_t p = p0; p < (uint32_t)e; p += step)
                        for (int j = 0; j < step; ++j) {
                            const long long at = step_index(p, j, e);
                            if (at < p0 || at >= e) ++bad;
                            if (p + j < (uint32_t)e ? at != next++ : at != e - 1) ++bad;
                        }
                    if (next != e) ++bad;
                }""", ["layout.h"])
    assert r.returncode == 0, r.stdout


def test_pieces_of_long_lists_fit(tmp_path):
    # n lists of m entries in all make at most n + m / piece pieces, eight bytes each, in three
    # arrays of n ints (n at least 64 of capacity)
    r = run_cpp(tmp_path, """
        for (long long n : {1LL, 2LL, 3LL, 64LL, 100LL, 1000LL, 65536LL, 1LL << 26, 1LL << 29})
            for (long long m : {0LL, 1LL, 511LL, 100000LL, 1LL << 24, (1LL << 31) - 1}) {
                const long long piece = piece_entries(n, m, 512);
                if (piece < 1 || piece > 1 << 30 || (piece % 512 && piece != 1 << 30)) ++bad;
                if (8 * (n + m / piece) > 12 * work_capacity(n)) ++bad;
            }""", ["layout.h"])
    assert r.returncode == 0, r.stdout
