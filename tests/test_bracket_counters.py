"""Where the hinted selection's counting pass counts (gd_bracket.h), gone through on the host: whatever
bits a column holds and whatever bracket its hints give, a value's counter is one of the workgroup's,
below, in or above the bracket as the value is.  The median of three is the one that the chip's
instruction takes: of the others the least where one is a NaN."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2605_17879_amd", "csrc")

HIP = """
#define __device__
#define __forceinline__ inline
"""

MAIN = r"""
#include "gd_bracket.h"
#include <math.h>
#include <stdio.h>
#include <random>
#include <vector>
#define CHECK(x) do { if (!(x)) { printf("line %d: %s (lo %08x hi %08x bits %08x lane %u)\n", __LINE__, #x, lo, hi, bits, lane); return false; } } while (0)

static float median(float x, float l, float h) {
    if (x != x || l != l || h != h) return fminf(fminf(x, l), h);
    return fmaxf(fminf(x, l), fminf(fmaxf(x, l), h));
}

template <int LOG_NB>
static uint32_t counter_of(uint32_t lo, uint32_t hi, uint32_t bits, uint32_t lane) {
    const int shift = shift_for<LOG_NB>(hi - lo);
    const BracketCounters<LOG_NB> c((lo & ~((1u << shift) - 1u)) >> shift, lane);
    return c.at(bits >> shift, c.base, median);
}

template <int LOG_NB>
static bool go_through() {
    constexpr uint32_t NB = 1u << LOG_NB;
    std::mt19937 rng(LOG_NB);
    std::vector<uint32_t> starts, spans;
    for (uint32_t i = 0; i < 70; ++i) starts.push_back(i);
    for (uint32_t at : {64u * 4u, 64u << 3, 64u << 10, 0x00800000u, 0x3F800000u, 0x42800000u, 0x5D000000u, 0x7C000000u, 0x7CFF0000u})
        for (uint32_t d = 0; d < 9; ++d) starts.push_back(at - 4 + d);
    for (uint32_t s : {2u * NB, 4u * NB, 64u * NB, 1u << 24, 0x20000000u})
        for (uint32_t d = 0; d < 3; ++d) spans.push_back(s - 1 + d);
    for (uint32_t s : {1u, 2u, 50u, NB / 2, NB - 1, NB, 3 * NB, 9 * NB}) spans.push_back(s);
    uint64_t counted = 0;
    for (uint32_t lo : starts)
        for (uint32_t span : spans) {
            const uint32_t hi = lo + span;
            uint32_t bits = 0, lane = 0;
            if (!bracket_counts<LOG_NB>(lo, hi)) continue;
            ++counted;
            const int shift = shift_for<LOG_NB>(span);
            const uint32_t first = lo >> shift << shift, end = first + (NB << shift);
            CHECK(shift >= 2 && end <= BRACKET_KEY_LIMIT);
            std::vector<uint32_t> values = {0u, 1u, 2u, 0x007FFFFFu, 0x00800000u, 0x3F800000u, 0x7F7FFFFFu, 0x7F800000u, 0x7F800001u,
                                            0x7FC00000u, 0x7FFFFFFFu, 0x80000000u, 0x80000001u, 0x80000100u, 0x807FFFFFu, 0xBF800000u,
                                            0xBFFFFFFFu, 0xC0000000u, 0xFF7FFFFFu, 0xFF800000u, 0xFF800001u, 0xFFC00000u, 0xFFFFFFFFu};
            for (uint32_t d = 0; d < 5; ++d)
                for (uint32_t at : {lo, hi, first, end}) values.push_back(at - 2 + d);
            for (uint32_t i = 0; i < 24; ++i) values.push_back(0xC0000000u + (rng() & 0xFFFFu));      // -2 and a little less
            for (uint32_t i = 0; i < 24; ++i) values.push_back((uint32_t)rng());
            for (uint32_t v : values)
                for (uint32_t l : {0u, 1u, 31u, 62u, 63u}) {
                    bits = v; lane = l;
                    const uint32_t at = counter_of<LOG_NB>(lo, hi, bits, lane), word = at / 4;
                    CHECK(at % 4 == 0 && word < 64 + NB + 64);
                    if (bits < first) CHECK(word < 64);
                    else if (bits < end) CHECK(word == 64 + ((bits - first) >> shift));
                    else CHECK(word >= 64 + NB && word <= 64 + NB + lane);
                }
        }
    uint32_t lo = 44, hi = 94, bits = 0xC0000000u + 20000u, lane = 63;
    CHECK(counted > 200);
    // (and why the bracket may not be a narrow one)
    CHECK(!bracket_counts<LOG_NB>(lo, hi) && counter_of<LOG_NB>(lo, hi, bits, lane) / 4 >= 64 + NB + 64);
    return true;
}

int main() {
    if (!go_through<11>() || !go_through<12>()) return 1;
    printf("ok\n");
    return 0;
}
"""


def test_every_value_is_counted_in_a_counter_of_its_own_side(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "go_through")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", f"-I{tmp_path}", f"-I{CSRC}", str(tmp_path / "main.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
