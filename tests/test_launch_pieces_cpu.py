"""Launches of more workgroups than one grid holds, checked on the host: every
piece stays below 2^32 threads, starts at a multiple of eight workgroups, and
the pieces hold every workgroup (every tile and round of chunks) once."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2211_16422_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "launch_pieces.h"
using namespace homs;
typedef long long ll;
static int bad(const char* what, ll a, ll b, int threads)
{
    std::printf("%s: %lld x %lld, %d threads\n", what, a, b, threads);
    return 1;
}
int main()
{
    const ll two32 = 1ll << 32;
    for (int threads : {64, 256, 512}) {
        const ll most = most_workgroups(threads);
        if (most % 8 || most * threads >= two32 || (most + 8) * threads < two32)
            return bad("most", most, 0, threads);
        for (ll n : {0ll, 1ll, 8ll, 1000ll, most - 1, most, most + 1, 3 * most, 5 * most + 7,
                     (ll)0x7FFFFFFF}) {
            ll next = 0;
            in_pieces(n, threads, [&](ll first, ll count) {
                if (first != next || first % 8 || count < 1 || count > most) next = -1;
                else next = first + count;
            });
            if (next != n) return bad("line", n, 0, threads);
        }
        // 100,000 queries of 2^31 rows, 2^31 queries of 2^20 rows, ...
        for (ll tiles : {0ll, 1ll, 64ll, 391ll, 8594ll, most / 8 - 1, most / 8, most / 8 + 1,
                         8388608ll})
            for (ll rounds : {0ll, 1ll, 2ll, 512ll, 2749ll, 131072ll}) {
                ll t_at = 0, r_at = 0, area = 0;  // pieces come rounds first, tiles outer
                bool ok = true;
                in_pieces(tiles, rounds, threads, [&](ll t, ll nt, ll r, ll nr) {
                    ok = ok && nt >= 1 && nr >= 1 && nt * nr * 8 * threads < two32;
                    ok = ok && t == t_at && r == r_at && t + nt <= tiles && r + nr <= rounds;
                    area += nt * nr;
                    r_at = r + nr;
                    if (r_at == rounds) {
                        r_at = 0;
                        t_at = t + nt;
                    }
                });
                if (!ok || area != tiles * rounds) return bad("plane", tiles, rounds, threads);
            }
    }
    std::puts("ok");
    return 0;
}
"""


def test_pieces_cover_the_launch(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not found")
    src, exe = tmp_path / "pieces.cpp", str(tmp_path / "pieces")
    src.write_text(PROGRAM)
    b = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", f"-I{CSRC}", str(src),
                        "-o", exe], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
