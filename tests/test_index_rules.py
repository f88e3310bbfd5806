"""Index rules of kernels whose rounds run past a bucket (csrc/apic_index.h), compiled for the CPU and gone through at the
counts where they can go wrong: every index that such a round reads lies inside the bucket, every particle is met once."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_15249_amd", "csrc")


def run(tmp_path, body):
    src = tmp_path / "rules.cpp"
    src.write_text('#include "apic_index.h"\n#include <climits>\n#include <cstdint>\n#include <cstdio>\n#include <vector>\n'
                   "using namespace apic;\nint main() {\n" + body + "\nreturn 0;\n}\n")
    exe = tmp_path / "rules"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                           "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("line", [16, 32])
def test_copy_of_a_bucket_stays_inside_it(tmp_path, line):
    """k_page_end: empty buckets and every start inside a line."""
    run(tmp_path, """
    const int width = 4 * 256;
    for (int ahead = 0; ahead < %d; ++ahead)
        for (int count : {0, 1, 15, 16, 17, 31, 32, 33, 127, 128, 1000, 1023, 1024, 1025, 5000}) {
            std::vector<int> met(count, 0);
            const int rounds = copy_rounds(count, ahead, width);
            if (count == 0 && rounds != 0) { std::printf("an empty bucket is read (ahead %%d)\\n", ahead); return 1; }
            for (int q = 0; q < rounds; ++q)
                for (int i = 0; i < width; ++i) {
                    const int k = q * width - ahead + i, s = copy_slot(k, count);
                    if (s < 0 || s >= count) { std::printf("slot %%d of %%d (ahead %%d)\\n", s, count, ahead); return 1; }
                    if (k >= 0 && k < count) {
                        if (s != k) return 1;
                        ++met[k];
                    }
                }
            for (int m : met) if (m != 1) { std::printf("met %%d times\\n", m); return 1; }
        }
    """ % line)


def test_places_ahead_at_the_largest_bucket(tmp_path):
    """Tiled deposit and gather + push: the last rounds of buckets up to the largest particle count, wherever they lie in
    the arrays (places counted in a signed word from the arrays' start wrap there)."""
    run(tmp_path, """
    const unsigned block = 256, per = 4;
    const int most = INT_MAX - 1;
    for (int count : {1, 255, 256, 1023, 1024, 1025, most - 1025, most - 1, most})
        for (int64_t first : {(int64_t)0, (int64_t)(most - count) / 2, (int64_t)most - count})
            for (unsigned thread : {0u, 1u, 255u}) {
                // from a round near the bucket's end on
                const unsigned c = (unsigned)count, ahead = per * block;
                const unsigned from = thread + (c > 3 * ahead ? (c / ahead - 2) * ahead : 0);
                int64_t met = 0;
                for (unsigned k0 = from; k0 < c; k0 += ahead) {
                    if (++met > 8) return 1;   // wrapped
                    for (unsigned j = 0; j < per; ++j) {
                        const int64_t i = ahead_index((int)first, k0 + j * block, c);
                        if (i < first || i >= first + count) { std::printf("%lld\\n", (long long)i); return 1; }
                        if (k0 + j * block < c && i != first + (int64_t)(k0 + j * block)) return 1;
                    }
                }
            }
    """)


def test_work_split_of_the_3d_field_solve(tmp_path):
    """Every power-of-two grid: the splits divide it, the tiles fit 64 KiB of LDS, and no workgroup has fewer than 512 points
    (two per thread) unless sixteen lines (eight on grids up to 32768 nodes) hold no more or the grid has no more."""
    run(tmp_path, """
    auto lines = [](const char *what, int got, int n, int most, int nx, int ny, int nz) {
        const int cap = nx * ny * nz <= 32768 ? 8 : 16, want = 512 / n > cap ? cap : 512 / n;
        const bool ok = got > 0 && most % got == 0 && (got >= want || got == most);
        if (!ok) std::printf("%s: %d lines of %d (%d x %d x %d)\\n", what, got, n, nx, ny, nz);
        return ok;
    };
    for (int nx = 4; nx <= 256; nx *= 2)
        for (int ny = 4; ny <= 256; ny *= 2)
            for (int nz = 4; nz <= 256; nz *= 2) {
                const Split3 s = split3_of(nx, ny, nz);
                const int cap = nx * ny * nz <= 32768 ? 8 : 16;
                if (s.Y % 2 || ny % s.Y || (s.Y < cap && s.Y < ny && s.Y / 2 * nx < 512)) {
                    std::printf("x: %d rows of %d\\n", s.Y, nx);
                    return 1;
                }
                if (!lines("y", s.ZB, ny, nz, nx, ny, nz) || !lines("z", s.KY, nz, ny, nx, ny, nz)) return 1;
                if (16 * s.Y * nx > 65536 || 32 * s.ZB * ny > 65536 || 32 * s.KY * nz > 65536 ||
                    16 * s.Y * (nx + nx / 2 + 1) > 65536)
                    return 1;
            }
    """)
