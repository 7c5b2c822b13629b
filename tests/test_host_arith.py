"""Host arithmetic shared with the kernels, compiled for the host alone: positions of
a read's band on a genome for diagonals up to the ends of 64 bits, where the sums and
products wrap, every block of a genome against its bounds, and grids of more threads
than a dimension holds.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "runtime.hpp"

#define CHECK(c, ...)                                     \
    do {                                                  \
        if (!(c)) {                                       \
            printf("line %d: %s ", __LINE__, #c);         \
            printf(__VA_ARGS__);                          \
            printf("\n");                                 \
            return 1;                                     \
        }                                                 \
    } while (0)

static int diagonals() {
    typedef __int128 i128;
    std::vector<i64> ds;
    for (i64 d = -70000 * 3; d <= 70000 * 3; d += 997) ds.push_back(d);
    for (i64 d = 0; d < 140000; d += 613) {
        ds.push_back(INT64_MIN + d);
        ds.push_back(INT64_MAX - d);
        for (int s = 31; s < 63; s++) {
            ds.push_back((1ll << s) + d);
            ds.push_back(-(1ll << s) - d);
        }
    }
    const int ms[] = {0, 1, 63, 64, 150, 65535}, Es[] = {0, 1, 7, 31, 32, 65534};
    const i64 Ls[] = {0, 1, 64, 100000, 4294901759ll};
    for (i64 d : ds)
        for (int m : ms)
            for (int E : Es)
                for (i64 L : Ls) {
                    const i64 c = near_diag(d);
                    CHECK(window_inside(c, m, E, L) == ((i128)d - E >= 0 && (i128)d + m + E <= L), "%lld %d %d %lld",
                          (long long)d, m, E, (long long)L);
                    // the same columns lie in the genome
                    for (int at : {-E, 0, m + E}) {
                        const i128 p = (i128)d + at, q = (i128)c + at;
                        CHECK((p >= 0 && p < L) == (q >= 0 && q < L), "%lld %d", (long long)d, at);
                        if (p >= 0 && p < L) CHECK(p == q, "%lld", (long long)d);
                    }
                }
    return 0;
}

static int blocks() {
    for (i64 L = 0; L <= 130; L++) {
        const i64 n = (L + 63) / 64;
        // exactly the genome's blocks, so that the address of any other faults
        u64x2 *lohi = (u64x2 *)malloc(n ? n * sizeof(u64x2) : 1);
        u64 *nb = (u64 *)malloc(n ? n * sizeof(u64) : 1);
        for (i64 b = 0; b < n; b++) {
            lohi[b] = u64x2{0x1234u + (u64)b, 0x5678u + (u64)b};
            nb[b] = 0;
        }
        std::vector<i64> bs;
        for (i64 b = -3; b <= n + 3; b++) bs.push_back(b);
        for (int s = 31; s < 63; s++)
            for (i64 o = -2; o <= 2; o++) {
                bs.push_back((1ll << s) + o);
                bs.push_back(-(1ll << s) + o);
            }
        bs.push_back(INT64_MIN);
        bs.push_back(INT64_MAX);
        for (i64 b : bs)
            for (int with_n = 0; with_n < 2; with_n++) {
                const Bits64 r = ref_block(lohi, nb, L, with_n, b);
                if (b < 0 || b >= n) {
                    CHECK(r.nb == ~0ull, "L %lld block %lld", (long long)L, (long long)b);
                } else {
                    const i64 room = L - 64 * b;
                    CHECK(r.lo == 0x1234u + (u64)b && r.nb == (room < 64 ? ~0ull << room : 0ull), "L %lld block %lld",
                          (long long)L, (long long)b);
                }
            }
        free(lohi);
        free(nb);
    }
    return 0;
}

static int grids() {
    const u64 per[] = {1, 4, 8, 16, 64, 256};
    for (u64 p : per)
        for (int s = 0; s < 40; s++)
            for (i64 o = -2; o <= 2; o++) {
                const i64 items = (1ll << s) + o;
                if (items < 0 || items / (i64)p > (1ll << 38)) continue;
                const dim3 g = wide_grid((u64)items, p, 256);
                CHECK((u64)g.x * 256 < (1ull << 32) && g.y <= 65535 && g.z == 1, "%lld", (long long)items);
                CHECK((u64)g.x * g.y >= ((u64)items + p - 1) / p, "%lld", (long long)items);
                CHECK((u64)g.x * (g.y - 1) < ((u64)items + p - 1) / p || g.y == 1, "%lld", (long long)items);
            }
    try {
        wide_grid(~0ull, 1, 1024);
        CHECK(false, "not refused");
    } catch (const Error &e) {
        CHECK(e.status == MT_EINVAL, "%d", e.status);
    }
    return 0;
}

int main(int, char **argv) {
    const std::string what = argv[1];
    if (what == "diagonals") return diagonals();
    if (what == "blocks") return blocks();
    if (what == "grids") return grids();
    return 2;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_arith")
    src, exe = d / "host_arith.hip", d / "host_arith"
    src.write_text(SOURCE)
    subprocess.run(["hipcc", "--offload-host-only", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2311_02029_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("what", ["diagonals", "blocks", "grids"])
def test_arithmetic(program, what):
    r = subprocess.run([program, what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout)
