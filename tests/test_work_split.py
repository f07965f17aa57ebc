"""The host-side rules that cut the attention work into workgroups, compiled for the CPU and checked over many extents:
the counts stay inside what the kernels are built for, every step of every key tile belongs to exactly one chunk (the
chunk's tile, its first and its last step, derived from its number as the kernel does), and the partial sums of the
chunks lie side by side in the room the workspace query leaves for them."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r'''
#define __HIP_PLATFORM_AMD__ 1
#include "sp_common.h"
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace sp;
static uint64_t seed = 12345;
static int64_t pick(int64_t lo, int64_t hi) { seed = seed * 6364136223846793005ull + 1442695040888963407ull; return lo + (int64_t)((seed >> 33) % (uint64_t)(hi - lo + 1)); }
#define CHECK(c) do { if (!(c)) { printf("failed: %s (B %ld S %ld Skv %ld off %ld Hq %d Hkv %d D %d)\n", #c, (long)B, (long)S, (long)Skv, (long)off, Hq, Hkv, D); return 1; } } while (0)
int main() {
    long equal = 0, full = 0, cut = 0;
    for (int it = 0; it < 200000; ++it) {
        const int64_t B = it % 3 ? 1 : pick(1, 40);
        int64_t S = it % 5 ? pick(1, 3000) : pick(1, 140000), Skv = S, off = 0;
        const int kind = it % 7;
        if (kind == 1) off = pick(0, S);
        if (kind == 2) { Skv = pick(1, 2 * S); off = Skv > S ? Skv - S + pick(0, 50) : pick(0, Skv); }
        if (kind == 3) { Skv = pick(1, 2 * S); off = Skv; }
        if (off > Skv) off = Skv;
        if (Skv > S + off) continue;
        const int32_t Hkv = (int32_t)pick(1, 8), G = (int32_t)pick(1, 8), Hq = Hkv * G, D = it & 1 ? 64 : 128;
        const int32_t rule = dkdv_split_count(B, S, Skv, Hq, Hkv);
        CHECK(rule >= 1 && rule <= 8);
        int32_t nsplit = rule;
        if (off >= Skv) { nsplit = dkdv_full_splits(B, S, Skv, Hq, Hkv, D, rule); ++full; }
        CHECK(nsplit >= 1 && nsplit <= rule);
        const DkdvChunks c = dkdv_chunks(B, (int32_t)S, (int32_t)Skv, (int32_t)off, Hq, Hkv, D, nsplit, off < Skv);
        CHECK(c.nsplit >= 1 && c.nsplit <= nsplit);
        if (c.nsplit < rule) ++cut;
        const int32_t tiles = order_tiles(Skv);
        if (c.len == 0) CHECK(c.n_chunks == tiles * c.nsplit);
        else {
            ++equal;
            CHECK(c.nsplit > 1 && tiles <= kMaxEqualTiles && c.len % 4 == 0);
            int64_t rows = 0, n = 0;
            for (int32_t t = 0; t < tiles; ++t) {
                const int32_t steps = dkdv_tile_steps(t, (int32_t)S, (int32_t)off, G), k = (steps + c.len - 1) / c.len;
                CHECK(steps >= 1 && k >= 1);
                const int64_t keys = Skv - (int64_t)t * kOrderTile;
                n += k; rows += k * (keys < kOrderTile ? keys : kOrderTile);
            }
            CHECK(n == c.n_chunks && rows <= (int64_t)c.nsplit * Skv);
        }
        CHECK(dkdv_part_bytes(B, Skv, Hkv, D, c.nsplit) <= dkdv_part_bytes(B, Skv, Hkv, D, rule));
        if ((int64_t)c.n_chunks > 20000) continue;
        // as the kernel derives them: a chunk's tile and number in it, its steps, the place of its partial sums (keys)
        std::vector<int64_t> done(tiles, 0);  // steps of a tile that the chunks so far have taken, in order
        int64_t place = 0;                    // end of the last chunk's partial sums
        for (int32_t id = 0; id < c.n_chunks; ++id) {
            int32_t jt = 0, split = 0, tile_chunks = c.nsplit, first = 0;
            if (c.len > 0) {
                for (int32_t upto = 0; jt < tiles; ++jt) {
                    tile_chunks = (dkdv_tile_steps(jt, (int32_t)S, (int32_t)off, G) + c.len - 1) / c.len;
                    first = upto; upto += tile_chunks;
                    if (upto > id) break;
                }
                split = id - first;
            } else { jt = id / c.nsplit; split = id % c.nsplit; first = jt * c.nsplit; }
            CHECK(jt < tiles && split >= 0 && split < tile_chunks);
            const int32_t j0 = jt * kOrderTile, n_it = (int32_t)((S + 31) / 32) - (int32_t)(j0 > off ? j0 - off : 0) / 32;
            const int64_t total = (int64_t)n_it * G, per = (total + tile_chunks - 1) / tile_chunks;
            const int64_t s0 = split * per < total ? split * per : total, s1 = s0 + per < total ? s0 + per : total;
            CHECK(s0 == done[jt] && s1 >= s0);
            done[jt] = s1;
            if (split == tile_chunks - 1) CHECK(s1 == total);
            if (c.nsplit > 1) {
                const int64_t keys = Skv - j0 < kOrderTile ? Skv - j0 : kOrderTile, at = (int64_t)first * kOrderTile + split * keys;
                CHECK(at >= place && at + keys <= (int64_t)c.nsplit * Skv);
                place = at + keys;
            }
        }
        for (int32_t t = 0; t < tiles; ++t) CHECK(done[t] == (int64_t)dkdv_tile_steps(t, (int32_t)S, (int32_t)off, G));
        const int ks = fwd_key_groups(B, S, Skv, off, Hq);
        CHECK(ks == 1 || ks == 2 || ks == 4);
        CHECK(dq_row_blocks(B, S, Hq) == 1 || dq_row_blocks(B, S, Hq) == 2);
    }
    // the most extreme extents end quickly and do not overflow into nonsense
    const int64_t B = 65535, S = 32767, Skv = S, off = S; const int32_t Hq = 65535, Hkv = 1, D = 128;
    CHECK(dkdv_full_splits(B, S, Skv, Hq, Hkv, D, 8) >= 1);
    CHECK(fwd_key_groups(1, (int64_t)1 << 30, (int64_t)1 << 30, 0, 1) == 1);
    // a round and a half of equal workgroups takes two; jobs that fit beside a late round cost nothing
    if (dispatch_end(384, [](int64_t) { return 10.; }) < 19.9 || dispatch_end(384, [](int64_t i) { return i < 128 ? 10. : 5.; }) > 10.1) { printf("dispatch_end\n"); return 1; }
    printf("ok %ld %ld %ld\n", equal, full, cut);
    return equal > 100 && full > 100 && cut > 100 ? 0 : 2;
}
'''


def run_on_host(tmp_path, text):
    src, exe = tmp_path / "split.cpp", tmp_path / "split"
    src.write_text(text)
    inc = os.path.join(ROOT, "paper_2604_27089_amd", "csrc")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-I", inc, "-I", "/opt/rocm/include", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    if r.returncode != 0 and "hip" in r.stderr and "No such file" in r.stderr:
        pytest.skip("HIP headers are not installed")
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


def test_chunks_fit_and_cover(tmp_path):
    run_on_host(tmp_path, SRC)


PACKED = r'''
#define __HIP_PLATFORM_AMD__ 1
#include "sp_common.h"
#include <cstdio>
using namespace sp;
int main() {
    int bad = 0;
    // packed rows, documents, query heads; measured with one group against two or four
    const int one[][3] = {{14272, 56, 4}, {17615, 35, 4}, {5760, 23, 8}, {2482, 10, 20}, {9399, 10, 8}, {10304, 11, 8}, {22338, 44, 4}, {65536, 128, 4}};
    const int more[][3] = {{4032, 13, 4}, {15168, 5, 1}, {6528, 7, 4}, {763, 7, 4}, {10007, 2, 3}};
    for (const auto& x : one) if (packed_key_groups(x[0], x[1], x[2]) != 1) { printf("%d rows, %d documents, %d heads: too many groups\n", x[0], x[1], x[2]); ++bad; }
    for (const auto& x : more) if (packed_key_groups(x[0], x[1], x[2]) < 2) { printf("%d rows, %d documents, %d heads: too few groups\n", x[0], x[1], x[2]); ++bad; }
    uint64_t seed = 7;
    for (int it = 0; it < 100000; ++it) {
        seed = seed * 6364136223846793005ull + 1442695040888963407ull;
        const int64_t T = 1 + (int64_t)((seed >> 33) % 70000);
        const int32_t Hq = 1 + (int32_t)((seed >> 20) % 40), n = 1 + (int32_t)((seed >> 40) % (it & 1 ? 64 : 100000));
        const int ks = packed_key_groups(T, n, Hq), whole = fwd_key_groups(1, T, T, 0, Hq);
        if (ks != 1 && ks != 2 && ks != 4) ++bad;
        if (n == 1 && ks != whole) ++bad;                                        // one document is one sequence
        if ((T + n - 1) / n < 64 && Hq * ((T + 255) / 256) > 512 && ks != 1) ++bad;  // short walks, more than two rounds
    }
    return bad ? 1 : 0;
}
'''


def test_packed_documents_get_groups_for_their_own_length(tmp_path):
    """Key groups of the forward follow the documents' walks, not the length of the whole batch."""
    run_on_host(tmp_path, PACKED)


EVEN = r'''
#define __HIP_PLATFORM_AMD__ 1
#include "sp_common.h"
#include <cmath>
#include <cstdio>
#include <queue>
#include <vector>
using namespace sp;
static uint64_t seed = 99;
static double uniform() { seed = seed * 6364136223846793005ull + 1442695040888963407ull; return (double)(seed >> 11) / 9007199254740992.; }
// Both stages' workgroups in the order of dispatch, dealt to 32 engines of 8 units, each with its own walk.
static double simulate(int64_t B, int S, int Skv, int off, int Hq, int Hkv, int D, int n, bool q_first) {
    const int G = Hq / Hkv, q_rows = 128 * dq_row_blocks(B, S, Hq), ranks = (S + q_rows - 1) / q_rows;
    const double sc = D == 64 ? 2. / 3. : 1.;
    std::vector<double> kv, q, all;
    for (int t = 0; t < order_tiles(Skv); ++t)
        for (int c = 0; c < n; ++c) kv.insert(kv.end(), Hkv * B, sc * 1.5 * dkdv_tile_steps(t, S, off, G) / n + 20.);
    for (int r = ranks - 1; r >= 0; --r) {
        const int last = std::min(S - 1, (r + 1) * q_rows - 1) + off, keys = last < Skv - 1 ? last + 1 : Skv;
        q.insert(q.end(), Hq * B, sc * 0.95 * q_rows / 256. * ((keys + 31) / 32) + 10.);
    }
    const auto& a = q_first ? q : kv; const auto& b = q_first ? kv : q;
    all = a; all.insert(all.end(), b.begin(), b.end());
    double end = 0.;
    for (int e = 0; e < 32; ++e) {
        std::priority_queue<double, std::vector<double>, std::greater<double>> unit;
        for (int i = 0; i < 8; ++i) unit.push(0.);
        for (size_t i = e; i < all.size(); i += 32) { const double t = unit.top() + all[i]; unit.pop(); unit.push(t); end = std::max(end, t); }
    }
    return end + (n > 1 ? 4. + n * (double)B * Skv * Hkv * D * 16. / 12e6 : 0.);
}
int main() {
    const int kv_heads[] = {1, 1, 1, 2, 4, 5, 8}, groups[] = {1, 2, 3, 4, 4, 8}, batch[] = {1, 1, 1, 2, 4, 8};
    int seen = 0, worse = 0, jumps = 0;
    double log_sum = 0.;
    while (seen < 1500) {
        const int Hkv = kv_heads[(int)(uniform() * 7)], G = groups[(int)(uniform() * 6)], Hq = Hkv * G, D = uniform() < .5 ? 64 : 128;
        const int64_t B = batch[(int)(uniform() * 6)];
        const int S = (int)exp(log(1000.) + uniform() * log(20.)), off = S - (int)(S * 2 / 3 * uniform() * uniform());
        const int most = dkdv_split_count(B, S, S, Hq, Hkv);
        if ((double)B * S * S * Hq > 6e9 || most < 2) continue;
        const int q_rows = 128 * dq_row_blocks(B, S, Hq);
        const DkdvChunks c = dense_chunks(B, S, S, off, Hq, Hkv, D);
        if (c.len > 0 || (int64_t)c.n_chunks * Hkv * B + (S + q_rows - 1) / q_rows * Hq * B <= kComputeUnits) continue;
        ++seen;
        const bool q_first = even_dq_first(S, S, off, Hq, Hkv, q_rows, c.nsplit, D);
        const double now = simulate(B, S, S, off, Hq, Hkv, D, c.nsplit, q_first), plain = simulate(B, S, S, off, Hq, Hkv, D, most, false);
        log_sum += log(now / plain);
        if (now > 1.08 * plain) ++worse;
        // an offset that hides one key of one row is no other problem than one that hides none
        if (dense_chunks(B, S, S, S - 1, Hq, Hkv, D).nsplit != dense_chunks(B, S, S, S, Hq, Hkv, D).nsplit) ++jumps;
    }
    printf("of %d: %d worse than every chunk the rule allows, %d jumps, mean %.3f\n", seen, worse, jumps, exp(log_sum / seen));
    return worse <= 3 && jumps <= 3 && log_sum < 0. ? 0 : 1;
}
'''


def test_even_walks_are_split_by_whole_rounds(tmp_path):
    """Blocks that hide little or nothing: the chunk count holds up in a simulation of the dispatch with every workgroup's
    own walk, against the full count with one stage after the other, and does not jump where the offset reaches the
    end of the keys."""
    run_on_host(tmp_path, EVEN)


def test_the_group_counts_that_the_gpu_tests_are_there_for(tmp_path):
    """The tables of test_attn_fwd_groups_gpu.py against the rule that picks the kernel."""
    import test_attn_fwd_groups_gpu as groups
    checks = [(f"fwd_key_groups({B}, {S}, {S}, 0, 1)", ks) for S, row in groups.BATCHES.items() for B, ks in row.items()]
    checks += [(f"fwd_key_groups({B}, {Sq}, {Skv}, {min(off, Skv)}, 1)", ks)
               for (Sq, Skv, off), row in groups.BLOCKS.items() for B, ks in row.items()]
    checks += [(f"packed_key_groups({sum(lengths)}, {len(lengths)}, {Hq})", ks) for lengths, row in groups.PACKED.items() for Hq, ks in row.items()]
    checks += [(f"fwd_key_groups(1, {S}, {S}, 0, 4)", ks) for S, ks in groups.WALKS.items()]
    lines = "\n".join(f'    if ({call} != {ks}) {{ printf("{call} is not {ks}\\n"); ++bad; }}' for call, ks in checks)
    run_on_host(tmp_path, "#define __HIP_PLATFORM_AMD__ 1\n#include \"sp_common.h\"\n#include <cstdio>\nusing namespace sp;\n"
                          "int main() {\n    int bad = 0;\n" + lines + "\n    return bad ? 1 : 0;\n}\n")
    for table in (groups.BATCHES, groups.BLOCKS, {"short": groups.PACKED[groups.SHORT]}, {"walks": groups.WALKS}):
        assert {ks for row in table.values() for ks in row.values()} == {1, 2, 4}
