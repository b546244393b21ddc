"""The launches of hps_expand_rows, over its whole range of n and dim: taken from the source, compiled for the host
with the launch replaced by a record."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2210_08804_amd", "csrc", "hps_cache.hip")

BEFORE = """
#include <cstdint>
#include <cstdio>
#include <cstddef>
#include <initializer_list>
constexpr int kWave = 64;
constexpr uint32_t kMinKeysPerWave = 8;
typedef int hipError_t;
typedef void *hipStream_t;
struct dim3 { uint64_t x; dim3(uint64_t v) : x((uint32_t)v) {} };
struct RowGeom { uint32_t d; };
static RowGeom make_geom(uint32_t d) { return RowGeom{d}; }
static hipError_t hipGetLastError() { return 0; }
static const char *bad = nullptr;
static uint64_t rows_done, the_cus;
static const uint32_t *inv0;
static float *out0;
static void record(dim3 grid, dim3 block, int, hipStream_t, const float *, const uint32_t *inverse, uint32_t n, uint32_t kpw,
                   const RowGeom &g, float *out) {
    const uint64_t waves = block.x / kWave;
    if (grid.x * block.x >= 1ull << 32) bad = "work-items of a launch";
    if (kpw < 1 || kpw > 64) bad = "rows per wave";
    const uint64_t of_a_wave = kpw < n ? kpw : n;
    if (of_a_wave * (g.d / 4) >= (1ull << 32) - 64 * 64) bad = "chunks of a wave, counted in 32 bits";
    if (kpw > 1 && (uint64_t)kpw * g.d * 4 > 49152 && (n + kpw - 1) / kpw < 4ull * the_cus) bad = "long rows in few waves";
    if (grid.x * waves * kpw < n || (grid.x - 1) * waves * kpw >= n) bad = "work-groups for n";
    if ((uintptr_t)inverse - (uintptr_t)inv0 != rows_done * 4 || (uintptr_t)out - (uintptr_t)out0 != rows_done * g.d * 4) bad = "place of a part";
    rows_done += n;
}
#define hipLaunchKernelGGL(kernel, grid, block, ...) record(grid, block, __VA_ARGS__)
"""

AFTER = """
int main() {
    inv0 = (const uint32_t *)0x1000;
    out0 = (float *)0x1000;
    for (uint32_t cus : {256u, 304u, 38u, 1u})
        for (uint64_t d = 4; d < 1ull << 32; d = d < 1024 ? d + 124 : d * 2 + 4)
            for (double x = 0; x <= 32.01; x += 0.05)
                for (int o = -1; o < 2; ++o) {
                    uint64_t n = (uint64_t)__builtin_exp2(x) + o;
                    if (n < 1) continue;
                    if (n >= 1ull << 32) n = (1ull << 32) - 1 - (uint64_t)(o + 1) * 255;
                    if (n * d >= 1ull << 38) continue;                     // a result of 1 TiB
                    rows_done = 0;
                    the_cus = cus;
                    bad = nullptr;
                    hps_launch_expand_rows((const float *)0x1000, inv0, (uint32_t)n, (uint32_t)d, out0, cus, nullptr);
                    if (rows_done != n) bad = "rows of all launches";
                    if (bad) {
                        std::printf("cus %u dim %llu n %llu: %s\\n", cus, (unsigned long long)d, (unsigned long long)n, bad);
                        return 1;
                    }
                }
    return 0;
}
"""


def test_launches_cover_every_row_and_stay_within_the_limits(tmp_path):
    with open(SRC) as f:
        s = f.read()
    start = s.index("hipError_t hps_launch_expand_rows(")
    src = tmp_path / "expand.cpp"
    rule = s.find("uint64_t most_rows(")
    src.write_text(BEFORE + (s[rule:s.index("\n", rule) + 1] if rule >= 0 else "") + s[start:s.index("\n}\n", start) + 3] + AFTER)
    exe = tmp_path / "expand"
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wno-unused", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
