"""Every launch shape that the query's rule can choose is one that the dispatch has a kernel for: the rule is
taken from the source and compiled for the host, the shapes are compared with the dispatch's labels."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2210_08804_amd", "csrc", "hps_cache.hip")

MAIN = """
int main() {
    for (uint64_t cus : {256ull, 128ull, 38ull, 32ull, 1ull})
        for (uint32_t t : {1u, 3u, 26u, 32u})
            for (int form = 0; form < 9; ++form)
                for (uint32_t d = 4; d <= 2048; d += d < 160 ? 4 : d / 8 / 4 * 4)
                    for (double x = 0; x < 32; x += 0.1)
                        for (int o = -1; o < 2; ++o) {
                            const uint64_t batch = (uint64_t)(__builtin_exp2(x) / t) + 1 + o;
                            const int mode = form % 3;                             // plain, checked, in-tile dedup
                            const bool n_dev = form >= 6;
                            if (batch * t >= (1ull << 32) || (mode == 1 && d > 1024) || (n_dev && t > 1)) continue;
                            const QueryShape q = query_shape(t, batch, d, cus, mode == 1, mode == 2, form / 3 == 1 ? 32 : 8, n_dev);
                            const int id = (d == 128 ? 10000 : 0) + q.u * 100 + q.wpb;
                            if (q.kpw < 1 || q.kpw > 64) { std::printf("kpw %u\\n", q.kpw); return 1; }
                            if (mode == 2 ? (q.wpb != 4 && q.wpb != 8) : !kShapes[mode].count(id)) {
                                std::printf("mode %d d %u batch %llu tables %u cus %llu: shape %d\\n", mode, d, (unsigned long long)batch, t, (unsigned long long)cus, id);
                                return 1;
                            }
                            if (mode == 1 && (uint64_t)q.u * 64 < d / 4) { std::printf("a row of %u does not fit a group of %d\\n", d, q.u); return 1; }
                        }
    return 0;
}
"""


def test_every_shape_is_compiled_in(tmp_path):
    with open(SRC) as f:
        s = f.read()
    rule = s[s.index("struct QueryShape {"):s.index("template <int W, int U, int WPB, bool kCoherent, int kD>\nvoid launch_query_kernel")]
    dispatch = s[s.index("hps_status_t launch_query_w("):s.index("hps_status_t launch_query(uint32_t W")]
    shapes = {"false": set(), "true": set()}
    for label, u, wpb, checked, d in re.findall(r"case (\d+): launch_query_kernel<W, (\d+), (\d+), (true|false), (\d+)>", dispatch):
        assert int(label) == (10000 if d == "128" else 0) + int(u) * 100 + int(wpb)
        shapes[checked].add(int(label))
    assert shapes["false"] and shapes["true"]
    sets = ", ".join("{" + ", ".join(map(str, sorted(shapes[k]))) + "}" for k in ("false", "true"))
    src = tmp_path / "shapes.cpp"
    src.write_text("#include <cstdint>\n#include <cstdio>\n#include <set>\nconstexpr int kWave = 64;\nconstexpr uint32_t kMinKeysPerWave = 8;\n"
                   + "const std::set<int> kShapes[2] = {" + sets + "};\n" + rule + MAIN)
    exe = tmp_path / "shapes"
    subprocess.run(["g++", "-O2", "-std=c++17", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


LONG_ROWS = """
int main() {
    for (uint64_t cus : {256ull, 38ull})
        for (uint64_t d = 132; d < 1ull << 32; d += d / 64 * 4)
            for (double x = 0; x < 32; x += 0.25) {
                const uint64_t n = (uint64_t)__builtin_exp2(x);
                if (n * d >= 1ull << 38) continue;                         // a result of 1 TiB
                const QueryShape q = query_shape(1, n, (uint32_t)d, cus, false, false);
                const uint64_t rows = q.kpw < n ? q.kpw : n;
                if (q.kpw < 1 || rows * (d / 4) >= (1ull << 32) - 64 * 64) {
                    std::printf("d %llu batch %llu: %u keys per wave\\n", (unsigned long long)d, (unsigned long long)n, q.kpw);
                    return 1;
                }
            }
    return 0;
}
"""


def test_a_wave_can_count_the_chunks_of_its_rows(tmp_path):
    """The copy of a wave's rows numbers their 16-byte chunks in 32 bits, whatever the row's length."""
    with open(SRC) as f:
        s = f.read()
    rule = s[s.index("struct QueryShape {"):s.index("template <int W, int U, int WPB, bool kCoherent, int kD>\nvoid launch_query_kernel")]
    src = tmp_path / "long.cpp"
    src.write_text("#include <cstdint>\n#include <cstdio>\n#include <initializer_list>\nconstexpr int kWave = 64;\nconstexpr uint32_t kMinKeysPerWave = 8;\n"
                   + rule + LONG_ROWS)
    exe = tmp_path / "long"
    subprocess.run(["g++", "-O2", "-std=c++17", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_wide_sets_do_not_get_fifteen_workers(tmp_path):
    """Sixteen waves of one work-group have 128 registers each, too few for the probe of sets of 32 ways and more."""
    with open(SRC) as f:
        s = f.read()
    rule = s[s.index("struct QueryShape {"):s.index("template <int W, int U, int WPB, bool kCoherent, int kD>\nvoid launch_query_kernel")]
    src = tmp_path / "wide.cpp"
    src.write_text("#include <cstdint>\n#include <cstdio>\n#include <initializer_list>\nconstexpr int kWave = 64;\nconstexpr uint32_t kMinKeysPerWave = 8;\n"
                   + rule + """
int main() {
    int fifteen = 0;
    for (uint32_t ways : {1u, 2u, 4u, 8u, 16u, 32u, 64u})
        for (uint32_t d = 4; d < 256; d += 4)
            for (uint64_t n = 1; n < 1ull << 32; n += n / 7 + 1) {
                const int wpb = query_shape(1, n, d, 256, false, false, ways).wpb;
                fifteen += wpb == 15;
                if (wpb > 8 && ways > 16) { std::printf("ways %u d %u batch %llu: %d workers\\n", ways, d, (unsigned long long)n, wpb); return 1; }
            }
    return fifteen ? 0 : 2;
}
""")
    exe = tmp_path / "wide"
    subprocess.run(["g++", "-O2", "-std=c++17", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


DEALT = """
uint64_t with_keys;                                                   // the lanes of the wave that have any
#define __ballot(live) with_keys
uint32_t searched(uint32_t kpw, bool dealt) { return %(lanes)s; }
int main() {
    int partial = 0;
    for (uint32_t ways : {32u, 64u})
        for (bool checked : {false, true})
            for (uint32_t d = 4; d <= 1024; d += d < 160 ? 4 : d / 8 / 4 * 4)
                for (uint64_t batch = 1; batch < 1ull << 22; batch += batch / 37 + 1) {
                    const QueryShape q = query_shape(1, batch, d, 256, checked, false, ways, true);
                    const uint32_t kpw = q.kpw, WPB = (uint32_t)q.wpb, n_tiles = (uint32_t)((batch + kpw * WPB - 1) / (kpw * WPB));
                    const uint32_t deal = q.deal;
                    if (deal == 0) continue;
                    const uint32_t shift = 31u - (uint32_t)__builtin_clz(deal);
                    partial += kpw %% deal != 0;
                    uint64_t keys = 0;
                    for (uint64_t nd : {batch, batch / 3}) {
                        with_keys = 0;
                        keys = 0;
                        for (uint32_t lane = 0; lane < 64; ++lane) {
                            const uint32_t lt = 0, wave = 0, b = %(position)s;
                            with_keys |= (uint64_t)(b < nd) << lane;
                            keys += n_tiles * WPB;
                        }
                        const uint32_t last = with_keys ? 63 - (uint32_t)__builtin_clzll(with_keys) : 0, told = searched(kpw, true);
                        const uint32_t block = 8 * (64 / ways);           // lanes that probe_wave searches or leaves out together
                        if (last / block * block >= told || told > last + 1) {
                            std::printf("ways %%u d %%u %%llu of %%llu keys: %%u keys per wave, lane %%u is the last that has one, %%u are searched\\n", ways, d,
                                        (unsigned long long)nd, (unsigned long long)batch, kpw, last, told);
                            return 1;
                        }
                    }
                    if (keys < batch) { std::printf("batch %%llu: %%llu lanes\\n", (unsigned long long)batch, (unsigned long long)keys); return 1; }
                }
    return partial ? 0 : 2;
}
"""


def test_every_lane_that_is_dealt_a_key_is_searched(tmp_path):
    """A batch whose length is read on the device is dealt to the waves in sixteens (long rows: in fewer), up to more keys than kpw to a wave; in sets
    of 32 ways and more the probe leaves out the lanes behind those it is told of.  Deal and count are taken from the source."""
    with open(SRC) as f:
        s = f.read()
    rule = s[s.index("struct QueryShape {"):s.index("template <int W, int U, int WPB, bool kCoherent, int kD>\nvoid launch_query_kernel")]
    kernel = s[s.index("\nquery_kernel(const u64x4"):s.index("query_dedup_kernel(")]
    told = set(re.findall(r"probe_wave<W, KPW, \w+>\(K, key, set, [^;]*?(\w+)(?:, here)?\);", kernel))
    assert len(re.findall(r"probe_wave<", kernel)) == 3 and len(told) == 1, told
    told = told.pop()
    lanes = re.search(r"const uint32_t %s\s*= (.*?);" % told, kernel)
    src = tmp_path / "dealt.cpp"
    src.write_text("#include <cstdint>\n#include <cstdio>\n#include <initializer_list>\nconstexpr int kWave = 64;\nconstexpr uint32_t kMinKeysPerWave = 8;\n"
                   + rule + DEALT % {"lanes": lanes[1] if lanes else told,
                                     "position": re.search(r"if \(dealt\) b = (.*?);", kernel)[1]})
    exe = tmp_path / "dealt"
    subprocess.run(["g++", "-O2", "-std=c++17", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


WHOLE_DEALS = """
int main() {
    int dealt = 0;
    for (bool checked : {false, true})
        for (uint32_t d = 4; d <= 1024; d += 4)
            for (uint64_t batch = 1; batch <= 7 * 64 * 256; batch += batch / 37 + 1) {     // batches of one round
                const QueryShape q = query_shape(1, batch, d, 256, checked, false, 8, true);
                if (q.deal == 0) continue;
                ++dealt;
                const uint64_t row = (uint64_t)d * 4, rows = (q.kpw + q.deal - 1) / q.deal * q.deal;
                const bool power = (q.deal & (q.deal - 1)) == 0 && rows <= 64;
                if (!power || q.deal * row > 16384 || (q.kpw * row <= 30000 && rows * row > (uint64_t)q.u * 1024)) {
                    std::printf("d %u batch %llu: %u keys per wave in deals of %u, %d wave loads\\n", d, (unsigned long long)batch, q.kpw, q.deal, q.u);
                    return 1;
                }
            }
    return dealt ? 0 : 2;
}
"""


def test_dealt_rows_are_one_group(tmp_path):
    """Keys of a batch whose length is read on the device go to the waves in deals of up to 16 KiB of rows, and a wave's deals stay
    within one group of wave loads where its keys do with room for a deal that is not full."""
    with open(SRC) as f:
        s = f.read()
    rule = s[s.index("struct QueryShape {"):s.index("template <int W, int U, int WPB, bool kCoherent, int kD>\nvoid launch_query_kernel")]
    src = tmp_path / "whole.cpp"
    src.write_text("#include <cstdint>\n#include <cstdio>\n#include <initializer_list>\nconstexpr int kWave = 64;\nconstexpr uint32_t kMinKeysPerWave = 8;\n"
                   + rule + WHOLE_DEALS)
    exe = tmp_path / "whole"
    subprocess.run(["g++", "-O2", "-std=c++17", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def run_rule(tmp_path, body):
    """Compiles the rule of the launch shapes with a main of its own and runs it."""
    with open(SRC) as f:
        s = f.read()
    rule = s[s.index("struct QueryShape {"):s.index("template <int W, int U, int WPB, bool kCoherent, int kD>\nvoid launch_query_kernel")]
    src = tmp_path / "rule.cpp"
    src.write_text("#include <cstdint>\n#include <cstdio>\n#include <initializer_list>\nconstexpr int kWave = 64;\nconstexpr uint32_t kMinKeysPerWave = 8;\n"
                   + rule + body)
    exe = tmp_path / "rule"
    subprocess.run(["g++", "-O2", "-std=c++17", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_batches_of_4096_keys_and_more_have_16_to_a_wave(tmp_path):
    """Every work-group adds to one counter word: with fewer keys to a wave there are more of them."""
    run_rule(tmp_path, """
int main() {
    for (uint32_t ways : {1u, 8u, 64u})
        for (uint32_t d = 4; d <= 256; d += 4)
            for (uint64_t n = 4096; n < 30000; n += 97)
                for (bool checked : {false, true}) {
                    const uint32_t k = query_shape(1, n, d, 256, checked, false, ways).kpw;
                    if (k < 16) { std::printf("ways %u d %u batch %llu: %u keys per wave\\n", ways, d, (unsigned long long)n, k); return 1; }
                }
    return 0;
}
""")


def test_the_last_tiles_of_several_tables_do_not_start_a_round(tmp_path):
    """Rows of more than 256 bytes: full tiles of several tables, the last of each not full, do not leave a few work-groups
    to a round of their own."""
    run_rule(tmp_path, """
int main() {
    for (uint32_t tables = 2; tables <= 32; ++tables)
        for (uint32_t d : {68u, 128u, 320u, 512u})
            for (uint64_t batch = 512; batch < 60000; batch += batch / 50)
                for (bool checked : {false, true}) {
                    const QueryShape q = query_shape(tables, batch, d, 256, checked, false);
                    const uint64_t tiles = tables * ((batch + q.kpw * q.wpb - 1) / (q.kpw * q.wpb));
                    const uint64_t most = 32768 / (d * 4) > 64 ? 64 : 32768 / (d * 4);
                    if (tiles < 3 * 256 && tiles > 256 && tiles % 256 > 0 && tiles % 256 < 16 && q.kpw == most) {
                        std::printf("%u tables d %u batch %llu: %llu tiles\\n", tables, d, (unsigned long long)batch, (unsigned long long)tiles);
                        return 1;
                    }
                }
    return 0;
}
""")


def test_short_rows_are_not_spread_over_more_work_groups_than_they_fill(tmp_path):
    """Plain, rows of up to 128 bytes from where work-groups of 7 x 64 keys are more than the CUs: no more of them than full ones of 8
    workers would be; of up to 256 bytes: one round while 8 workers need no more."""
    run_rule(tmp_path, """
int main() {
    for (uint32_t ways : {1u, 8u, 16u})
        for (uint32_t tables : {1u, 2u, 13u, 26u})
            for (uint32_t d = 4; d <= 64; d += 4)
                for (bool n_dev : {false, true})
                    for (uint64_t batch = 114689 / tables + 1; batch * tables < (n_dev ? 1u << 18 : 1u << 19); batch += batch / 61 + 1) {
                        if (n_dev && tables > 1) continue;
                        const QueryShape q = query_shape(tables, batch, d, 256, false, false, ways, n_dev);
                        const uint64_t tiles = tables * ((batch + q.kpw * q.wpb - 1) / (q.kpw * q.wpb)), of8 = tables * ((batch + 511) / 512);
                        if (d <= 32 ? tiles > of8 : of8 <= 256 && tiles > 256) {
                            std::printf("ways %u tables %u d %u batch %llu: %llu work-groups\\n", ways, tables, d, (unsigned long long)batch, (unsigned long long)tiles);
                            return 1;
                        }
                    }
    return 0;
}
""")


def test_waves_do_not_search_wide_sets_for_nobody(tmp_path):
    """Sets of 32 and 64 ways are searched for 16 and 8 lanes at a time: while a batch fits the CUs that way, its waves have whole
    16s and whole 8s of keys, of 64 ways no more than 24."""
    run_rule(tmp_path, """
int main() {
    for (uint32_t ways : {32u, 64u})
        for (uint32_t d = 4; d <= 128; d += 4)
            for (uint64_t n = 4096; n <= (ways == 32 ? 16 * 7 * 256 : 24 * 7 * 256); n += 113)
                for (bool checked : {false, true}) {
                    const uint32_t k = query_shape(1, n, d, 256, checked, false, ways).kpw;
                    if (k % (ways == 32 ? 16 : 8) && !(checked && ways == 32 && n > 15 * 7 * 256)) { std::printf("ways %u d %u batch %llu: %u keys per wave\\n", ways, d, (unsigned long long)n, k); return 1; }
                    if (ways == 64 && k > (checked ? 32 : 24)) { std::printf("64 ways d %u batch %llu: %u keys per wave\\n", d, (unsigned long long)n, k); return 1; }
                }
    return 0;
}
""")


def test_a_wave_has_little_more_of_a_shorter_batch_than_another(tmp_path):
    """Rows of 2 KiB and more, length on the device, batches that take one round: of 70 % of the keys no wave gets
    more than 1.3 times the mean.  (1.44 for 32,768 rows of 2 KiB in deals of eight.)"""
    run_rule(tmp_path, """
int main() {
    for (uint32_t d : {512u, 640u, 768u, 1024u})
        for (bool checked : {false, true})
            for (uint64_t n = 23000 * 512 / d; n <= 32768 * 512 / d; n += 61) {
                const QueryShape q = query_shape(1, n, d, 256, checked, false, 8, true);
                if (!q.deal) { std::printf("d %u batch %llu is not dealt\\n", d, (unsigned long long)n); return 1; }
                const uint64_t waves = (n + q.kpw * q.wpb - 1) / (q.kpw * q.wpb) * q.wpb, m = n * 7 / 10;
                const uint64_t most = ((m + q.deal - 1) / q.deal + waves - 1) / waves * q.deal;
                if (most * waves * 10 > 13 * m) {
                    std::printf("d %u checked %d batch %llu: up to %llu keys to a wave, %g on average\\n", d, checked, (unsigned long long)n, (unsigned long long)most, (double)m / waves);
                    return 1;
                }
            }
    return 0;
}
""")


def test_short_rows_fill_their_last_round(tmp_path):
    """Plain, rows of up to 128 bytes, 11 or 15 workers: where full waves would leave the last of several rounds less than two thirds full, the waves
    are trimmed to fill three quarters of it."""
    run_rule(tmp_path, """
int main() {
    int trimmed = 0;
    for (uint32_t ways : {1u, 8u, 16u})
        for (uint32_t d = 4; d <= 32; d += 4)
            for (uint64_t n = 114689; n < 1u << 19; n += 997) {
                const QueryShape q = query_shape(1, n, d, 256, false, false, ways);
                const uint64_t full = (n + 64 * q.wpb - 1) / (64 * q.wpb), tiles = (n + q.kpw * q.wpb - 1) / (q.kpw * q.wpb);
                if (full <= 256 || full % 256 == 0 || full % 256 > 170) continue;
                ++trimmed;
                if (tiles % 256 && tiles % 256 < 192) {
                    std::printf("ways %u d %u batch %llu: %llu work-groups, %llu with full waves\\n", ways, d, (unsigned long long)n, (unsigned long long)tiles, (unsigned long long)full);
                    return 1;
                }
            }
    return trimmed ? 0 : 2;
}
""")


def test_wide_sets_do_not_make_waves_of_long_rows_longer(tmp_path):
    """Whole blocks of keys take a wave no further than 16 KiB of rows, and rows of more than 1 KiB are moved as in other sets."""
    run_rule(tmp_path, """
int main() {
    for (uint32_t ways : {32u, 64u})
        for (uint32_t d = 64; d <= 1024; d += 4)
            for (bool checked : {false, true})
                for (uint64_t n = 4096; n < 60000; n += 331) {
                    const uint32_t k = query_shape(1, n, d, 256, checked, false, ways).kpw, other = query_shape(1, n, d, 256, checked, false, 8).kpw;
                    const uint64_t some = 16384 / (d * 4);
                    if (d > 256 ? k != other : n < 2 * some * 256 && some >= 512 / ways && k > some) {
                        std::printf("%u ways d %u batch %llu: %u keys per wave, 8 ways %u\\n", ways, d, (unsigned long long)n, k, other);
                        return 1;
                    }
                }
    return 0;
}
""")
