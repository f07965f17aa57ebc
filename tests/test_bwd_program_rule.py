"""The rule that sends a backward to the programs of long launches (16x16x32 MFMAs), compiled for the CPU: short launches, for
which those programs are the slower ones, keep 32x32x16, long ones change over, more work never goes back, and one packed
document goes where a dense call of the same extents goes (both have to give the same bits)."""
from test_work_split import run_on_host

SRC = r'''
#define __HIP_PLATFORM_AMD__ 1
#include "sp_common.h"
#include <cstdio>
using namespace sp;
static bool dense(int64_t B, int64_t S, int32_t Hq, int32_t D, int32_t Hkv = 1) { return bwd_long_launch(B, S, S, 0, Hq, Hkv, D, 0); }
static bool past(int64_t S, int32_t Hq, int32_t D) { return bwd_long_launch(1, S, S, S, Hq, 1, D, 0); }
static bool packed(int64_t T, int64_t n, int32_t Hq, int32_t D) { return bwd_long_launch(1, T, T, 0, Hq, 1, D, n); }
#define CHECK(c) do { if (!(c)) { printf("failed: %s\n", #c); return 1; } } while (0)
int main() {
    // measured: 16x16x32 is 3 to 12 % slower
    CHECK(!dense(1, 512, 8, 128)); CHECK(!dense(1, 1024, 8, 128)); CHECK(!dense(1, 2048, 4, 128)); CHECK(!dense(1, 4096, 8, 128));
    CHECK(!dense(1, 6000, 2, 64)); CHECK(!dense(1, 10007, 2, 64)); CHECK(!dense(16, 1024, 4, 64)); CHECK(!dense(64, 512, 4, 128));
    CHECK(!past(1000, 32, 128)); CHECK(!past(1000, 32, 64));
    CHECK(!packed(9000, 13, 4, 128)); CHECK(!packed(20000, 27, 4, 64)); CHECK(!packed(20000, 27, 3, 128)); CHECK(!packed(65536, 253, 4, 128));
    CHECK(!packed(131072, 484, 4, 64)); CHECK(!packed(131072, 229, 4, 64)); CHECK(!packed(131072, 81, 4, 64));
    // measured: 3 to 6 % faster
    CHECK(dense(1, 8192, 4, 128)); CHECK(dense(1, 16384, 4, 128)); CHECK(dense(1, 32768, 4, 128)); CHECK(dense(16, 4096, 4, 128));
    CHECK(dense(1, 12288, 4, 64)); CHECK(dense(1, 16384, 4, 64)); CHECK(dense(16, 4096, 4, 64)); CHECK(dense(1, 131072, 4, 128));
    CHECK(past(1660, 24, 128)); CHECK(past(4096, 32, 128)); CHECK(past(2048, 32, 64)); CHECK(past(4096, 32, 64)); CHECK(!past(1470, 24, 128)); CHECK(packed(65536, 18, 4, 128)); CHECK(packed(40000, 6, 4, 64));
    // one round: only where both stages end together
    CHECK(dense(1, 4096, 4, 128)); CHECK(dense(1, 3990, 4, 128)); CHECK(dense(2, 8137, 1, 128)); CHECK(!dense(1, 4096, 4, 64));
    CHECK(!dense(1, 4096, 3, 128)); CHECK(!dense(1, 3000, 4, 128)); CHECK(!dense(2, 2248, 8, 128)); CHECK(!dense(1, 3431, 10, 128, 2)); CHECK(!dense(1, 3000, 8, 128));
    for (int32_t D = 64; D <= 128; D += 64) {
        for (int64_t S = 1; S < 300000; S = S * 9 / 8 + 1)
            for (int32_t Hq = 1; Hq <= 64; Hq *= 2) {
                CHECK(packed(S, 1, Hq, D) == dense(1, S, Hq, D));
                if (past(S, Hq, D) || D == 64) {  // (a full round may be followed by a launch that is one and a quarter)
                    CHECK(dense(1, S, Hq, D) <= dense(1, 2 * S, Hq, D) && dense(1, S, Hq, D) <= dense(2, S, Hq, D) && dense(1, S, Hq, D) <= dense(1, S, 2 * Hq, D));
                    CHECK(dense(1, S, Hq, D) <= past(S, Hq, D));
                }
                for (int64_t n = 2; n <= 64 && n <= S; n *= 2) CHECK(packed(S, 2 * n, Hq, D) <= packed(S, n, Hq, D));
            }
        CHECK(dense(65535, 2147483647, 65535, D) && past(2147483647, 65535, D) && packed(2147483647, 2, 1, D));
        CHECK(!dense(1, 1, 1, D) && !packed(1, 2147483647, 1, D));
    }
    printf("ok\n");
    return 0;
}
'''


def test_short_launches_keep_32x32x16(tmp_path):
    run_on_host(tmp_path, SRC)
