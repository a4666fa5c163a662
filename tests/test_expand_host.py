"""The parameters of each layer that a block of the O expansion writes, and the LDS it asks for (csrc/expand.h, compiled for
the host): every parameter of a span belongs to exactly one layer's weights or biases, rows are found by the division that
the kernel uses, and the LDS of a launch is that of the span which needs most, below 128 KB for every network."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <random>
#include "expand.h"
using namespace nqs;
int main()
{
    std::mt19937_64 g(1);
    auto rnd = [&](int64_t lo, int64_t hi) { return lo + (int64_t)(g() % (uint64_t)(hi - lo + 1)); };
    long bad = 0, cases = 0;
    int most = 0;
    for (unsigned in = 1; in <= 8192; ++in)
        for (int t = 0; t < 200; ++t) {
            const unsigned m = (unsigned)rnd(0, 8192), q = t % 4 == 0 ? m * in : t % 4 == 1 ? m * in + in - 1 : (unsigned)rnd(0, 1 << 26);
            bad += expand_div(q, in, 0xFFFFFFFFu / in) != q / in;
        }
    for (int it = 0; it < 3000; ++it) {
        ExpandArgs E{};
        E.L = (int)rnd(1, 8);
        int prev = (int)rnd(2, it % 3 ? 200 : 4096);
        int64_t off = 0;
        for (int l = 0; l < E.L; ++l) {
            const int kind = (int)rnd(0, 5);
            const int out = kind == 0 ? (int)rnd(1, 6) : kind == 1 && it % 3 == 0 ? (int)rnd(1, 8192) : (int)rnd(1, 500);
            E.in[l] = prev;
            E.out[l] = out;
            E.inv[l] = 0xFFFFFFFFu / (unsigned)prev;
            E.offW[l] = off;
            off += (int64_t)out * (prev + 1);
            prev = out;
        }
        E.offW[E.L] = off;
        E.p0 = it % 2 ? 0 : rnd(0, off - 1);
        E.p1 = it % 4 < 2 ? off : rnd(E.p0 + 1, off);
        if ((E.p1 - E.p0) / kExpandSpan > 3000) E.p1 = E.p0 + 3000 * (int64_t)kExpandSpan + 7;
        int need = 0;
        for (int64_t b0 = E.p0; b0 < E.p1; b0 += kExpandSpan) {
            const int64_t b1 = std::min(E.p1, b0 + kExpandSpan);
            int64_t at = b0;
            int words = 0;
            for (int l = 0; l < E.L; ++l) {
                const ExpandPart x = expand_part(E, l, b0, b1);
                if (x.rows > 0) {
                    bad += E.offW[l] + x.q0 != at || x.r0 != x.q0 / E.in[l];
                    bad += (x.q0 + x.count - 1) / E.in[l] != x.r0 + x.rows - 1 || (int)x.r0 + x.rows > E.out[l];
                    at += x.count;
                }
                if (x.nd > 0) {
                    bad += E.offW[l + 1] - E.out[l] + x.d0 != at || x.d0 + x.nd > E.out[l];
                    at += x.nd;
                }
                words += expand_words(E.in[l], x.rows, x.nd);
            }
            bad += at != b1;
            need = std::max(need, words);
        }
        const int got = expand_lds_words(E);
        bad += got < need || 4 * got > 128 * 1024;
        most = std::max(most, got);
        ++cases;
    }
    std::printf("%ld %ld %d\n", bad, cases, 4 * most);
    return bad != 0;
}
"""


def test_parts_and_lds_of_every_span(tmp_path):
    src, exe = tmp_path / "expand.cpp", tmp_path / "expand"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__host__=", "-D__device__=", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2601_20782_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split()[1]) == 3000
