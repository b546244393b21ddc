"""The writers' copies of rows, lane by lane on the host: the code is taken from the source and its loads and
stores are replaced by records of the chunk they touch.  Every chunk of every listed long row is stored once, in order
of the walk, also where the chunks of a wave's rows are more than 32 bits count; every chunk of every listed row of up to one wave
load is stored, none of a row that is to be skipped, and nothing beside the list."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2210_08804_amd", "csrc", "hps_cache.hip")

BEFORE = """
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <type_traits>
#define __host__
#define __device__
#define __forceinline__ inline
#define __restrict__
constexpr int kWave = 64;
static int the_lane;
static int lane_id() { return the_lane; }
static void wait_vm0() {}
static float *const src0 = (float *)(1ull << 60);
static float *const dst0 = (float *)(1ull << 61);
static uint64_t nt_load(const uint64_t *p) { return (uint64_t)((const char *)p - (const char *)src0) / 8; }
static uint64_t expect, stores, chunks;                       // next chunk this lane has to store
static void shared_st64(uint64_t *p, uint64_t v) {
    const uint64_t c = (uint64_t)((char *)p - (char *)dst0) / 8;
    if (c != v) { std::printf("chunk %llu stored to %llu\\n", (unsigned long long)v, (unsigned long long)c); std::exit(1); }
    if (c == expect) { expect += kWave; ++stores; }
    else if (c >= expect || stores * kWave + (uint64_t)the_lane < chunks) {   // (idle lanes may repeat what is stored)
        std::printf("lane %d: chunk %llu instead of %llu\\n", the_lane, (unsigned long long)c, (unsigned long long)expect);
        std::exit(1);
    }
}
struct u32x4 { uint64_t chunk, rest; };
static uint64_t listed;                                       // chunks of the short rows of a list
static int seen[64 * 64];
static uint64_t chunk16(const u32x4 *p, const float *base) {
    const uint64_t c = (uint64_t)((const char *)p - (const char *)base) / 16;
    if (c >= listed) { std::printf("lane %d: chunk %llu of %llu\\n", the_lane, (unsigned long long)c, (unsigned long long)listed); std::exit(1); }
    return c;
}
static u32x4 nt_load(const u32x4 *p) { return {chunk16(p, src0), 0}; }
static void shared_st128(u32x4 *p, u32x4 v) {
    const uint64_t c = chunk16(p, dst0);
    if (c != v.chunk) { std::printf("chunk %llu stored to %llu\\n", (unsigned long long)v.chunk, (unsigned long long)c); std::exit(1); }
    ++seen[c];
}
#define __builtin_nontemporal_load(p) nt_load(p)
"""

AFTER = """
static int short_rows(uint32_t cnt, uint32_t d) {
    RowGeom g{};
    g.d = d;
    const uint32_t C = g.C = d / 4;
    g.c16 = ChunkStep{C, (65536u + C - 1) / C | (64u / C) << 17 | (64u % C) << 24};
    for (g.LPR = 1; g.LPR < C; g.LPR <<= 1) ++g.lprShift;
    uint32_t from[64];
    uint64_t to[64];
    for (int kind = 0; kind < 3; ++kind) {                    // rows asked for ahead, some of them to be skipped, all in one go
        for (uint32_t i = 0; i < 64; ++i) {
            from[i] = i;
            to[i] = kind == 1 && i % 3 == 1 ? kSkipRow : i;
        }
        listed = (uint64_t)cnt * C;
        for (int &n : seen) n = 0;
        for (the_lane = 0; the_lane < kWave; ++the_lane) {
            if (kind == 2) copy_rows_shared<4, false>(g, src0, dst0, from, to, cnt);
            else {
                RowMover<4, false> rows(g, src0, dst0, from, to);
                rows.start(cnt);
                rows.finish(kind == 0);
            }
        }
        for (uint64_t c = 0; c < listed; ++c)
            if ((to[c / C] == kSkipRow) != (seen[c] == 0)) {
                std::printf("kind %d: chunk %llu stored %d times\\n", kind, (unsigned long long)c, seen[c]);
                return 1;
            }
    }
    return 0;
}

int main(int argc, char **v) {
    const uint32_t cnt = (uint32_t)std::atoll(v[1]), d = (uint32_t)std::atoll(v[2]);
    if (argc > 3) return short_rows(cnt, d);
    RowGeom g{};
    g.d = d;
    const uint32_t C = d / 2, inv = C > 64 ? 0u : (65536u + C - 1) / C;
    g.c8 = ChunkStep{C, inv | (64u / C) << 17 | (64u % C) << 24};
    uint32_t from[64];
    uint64_t to[64];
    for (uint32_t i = 0; i < 64; ++i) to[i] = from[i] = i;
    chunks = (uint64_t)cnt * C;
    for (int kind = 0; kind < 2; ++kind)
        for (int lane : {0, 37, 63}) {
            the_lane = lane;
            expect = (uint64_t)lane;
            stores = 0;
            if (kind) copy_rows_shared<8, true>(g, src0, dst0, from, to, cnt);
            else {
                RowMover<8, true> rows(g, src0, dst0, from, to);
                rows.start(cnt);
                rows.finish(true);
            }
            if (stores != (chunks - lane + kWave - 1) / kWave) {
                std::printf("kind %d lane %d: %llu of %llu chunks\\n", kind, lane, (unsigned long long)stores, (unsigned long long)((chunks - lane + kWave - 1) / kWave));
                return 1;
            }
        }
    return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    with open(SRC) as f:
        s = f.read()
    body = (s[s.index("struct ChunkStep {"):s.index("// Copy `cnt` (> 0) rows listed in LDS")]
            + s[s.index("constexpr uint64_t kSkipRow"):s.index("// Set probe for the first KPW lanes'")]).replace('"+v"', '"+r"')
    src = tmp_path_factory.mktemp("walk") / "walk.cpp"
    src.write_text(BEFORE + body + AFTER)
    exe = src.with_suffix("")
    subprocess.run(["g++", "-O2", "-std=c++17", "-w", str(src), "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("cnt", [1, 2, 3, 7, 8, 16, 31, 63, 64])
@pytest.mark.parametrize("d", [4, 8, 12, 60, 64, 68, 124, 128, 132, 192, 252, 256])
def test_every_chunk_of_short_rows_is_stored(walk, cnt, d):
    r = subprocess.run([walk, str(cnt), str(d), "short"], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("cnt,d", [(1, 132), (3, 132), (8, 132), (16, 516), (64, 260), (5, 1028), (64, 4096),
                                   (16, (1 << 29) - 4), (16, 1 << 29), (16, (1 << 29) + 4)])
def test_every_chunk_of_long_rows_is_stored_once(walk, cnt, d):
    r = subprocess.run([walk, str(cnt), str(d)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
