"""How many workgroups of a draft launch each segment gets, on the host: none walks through more chunks than the launch's mean (or one and
an eighth more, where the workgroups fit the device then), however uneven the segments are, and no other division is taken than the one by the
mean alone unless the busiest compute units have fewer chunks with it, or are an eighth as many."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "draft_shares.h"
#include <cstdio>
#include <random>
#include <vector>
using V = std::vector<uint32_t>;
static V many(int n, uint32_t c, V more = {}) { more.insert(more.end(), n, c); return more; }
static int check(const char* what, const V& chunks, uint32_t room, uint32_t cus, V* out = nullptr)
{
    V blocks(chunks.size(), 77), plain(chunks.size());
    pruner::share_workgroups(chunks.data(), (int32_t)chunks.size(), room, cus, blocks.data());
    int64_t total = 0, sum = 0, longest = 0, at_mean = 0;
    for (uint32_t c : chunks) total += c;
    const int64_t mean = total > (int64_t)room ? (total + room - 1) / room : 1;
    for (size_t i = 0; i < chunks.size(); ++i) {
        const int64_t c = chunks[i], b = blocks[i];
        if (b < (c > 0) || b > c) return std::printf("%s: %ld workgroups for %ld chunks\n", what, (long)b, (long)c), 1;
        sum += b;
        at_mean += plain[i] = (c + mean - 1) / mean;
        if (b > 0 && (c + b - 1) / b > longest) longest = (c + b - 1) / b;
    }
    if (longest > (at_mean > (int64_t)room ? mean + 1 + mean / 8 : mean)) return std::printf("%s: %ld chunks one after the other, mean %ld\n", what, (long)longest, (long)mean), 1;
    if (sum > (at_mean > (int64_t)room ? at_mean : room)) return std::printf("%s: %ld workgroups, room %ld\n", what, (long)sum, (long)room), 1;
    const pruner::Busiest now = pruner::busiest_units(chunks.data(), blocks.data(), (int32_t)chunks.size(), cus), before = pruner::busiest_units(chunks.data(), plain.data(), (int32_t)chunks.size(), cus);
    if (blocks != plain && chunks.size() > 1 && (now.chunks > before.chunks || (now.chunks == before.chunks && 8 * now.units >= before.units)))
        return std::printf("%s: %u units with %u chunks, %u with %u by the mean\n", what, now.units, now.chunks, before.units, before.chunks), 1;
    if (out) *out = blocks;
    return 0;
}
int main()
{
    int bad = 0;
    V got;
    bad += check("one large, nineteen small", many(19, 19, {10240}), 1024, 256);
    bad += check("one large, thirty small", many(30, 38, {19000}), 1024, 256);
    bad += check("one large, sixty small", many(60, 12, {6000}), 1024, 256);
    bad += check("400 small", many(400, 5), 768, 256);
    bad += check("600 small", many(600, 3), 1024, 256);
    bad += check("twenty of 59", many(20, 59), 1024, 256, &got) || got[0] != 30;     // (51 each would meet on the same units)
    bad += check("more segments than room", many(3000, 2), 1024, 256);
    bad += check("few", many(7, 3), 1024, 256, &got) || got[0] != 3;
    bad += check("empty ones", V{0, 5000, 0, 1}, 1024, 256);
    bad += check("nothing", V{0, 0}, 1024, 256);
    bad += check("one alone", V{3223}, 1024, 256, &got) || got[0] != 1024;           // the whole device
    bad += check("ten of 323", many(10, 323), 1024, 256, &got) || got[0] != 102;
    bad += check("twenty of 98", many(20, 98), 1024, 256, &got) || got[0] != 49;     // (51 each leave as many chunks to a unit)
    bad += check("eight of 306", many(8, 306), 1024, 256, &got) || got[0] != 102;    // (and so do 128 each)
    bad += check("three of 684", many(3, 684), 1024, 256, &got) || got[0] != 341;    // (as many on six units, on 172 by the mean)
    bad += check("fourteen of 235", many(14, 235), 1024, 256, &got) || got[0] != 73;
    bad += check("five of 352", many(5, 352), 768, 256, &got) || got[0] != 153;
    bad += check("ten of 326", many(10, 326), 1024, 256, &got) || got[0] != 102;
    bad += check("forty of 82", many(40, 82), 1024, 256, &got) || got[0] != 25;
    bad += check("twenty of 163", many(20, 163), 1024, 256, &got) || got[0] != 41;   // (51 each leave as many)
    bad += check("five of 2,149", many(5, 2149), 768, 256, &got) || got[0] != 153;   // 154 each do not fit
    for (int64_t chunks : {0, 690, 768, 1025, 1040, 1180, 1536, 2049, 2051, 2304}) bad += pruner::four_waves_pay(chunks, 256) ? std::printf("%ld chunks\n", (long)chunks) : 0;
    for (int64_t chunks : {769, 980, 1024, 1537, 1960, 2048, 2305, 2640, 3910, 21000}) bad += pruner::four_waves_pay(chunks, 256) ? 0 : std::printf("%ld chunks\n", (long)chunks);
    std::mt19937 rng(1);
    for (int t = 0; t < 20000 && !bad; ++t) {
        V c(1 + rng() % 60);
        for (uint32_t& x : c) x = rng() % (1u << (rng() % 16));
        const int cus = 1 + rng() % 300;
        bad += check("drawn", c, cus * (1 + rng() % 8), cus);
    }
    for (int t = 0; t < 2000 && !bad; ++t) {   // the busiest unit, counted one chunk after the other
        V c(1 + rng() % 9), b(c.size());
        for (size_t i = 0; i < c.size(); ++i) c[i] = rng() % 200, b[i] = c[i] ? 1 + rng() % c[i] : 0;
        const int cus = 1 + rng() % 40;
        V unit(cus, 0);
        uint32_t at = 0, most = 0;
        for (size_t i = 0; i < c.size(); at += b[i++])
            for (uint32_t k = 0; k < c[i]; ++k) ++unit[(at + k % b[i]) % cus];
        for (uint32_t u : unit) most = u > most ? u : most;
        uint32_t units = 0;
        for (uint32_t u : unit) units += u == most;
        const pruner::Busiest got = pruner::busiest_units(c.data(), b.data(), (int32_t)c.size(), cus);
        if (got.chunks != most || got.units != units) bad += std::printf("busiest unit\n");
    }
    return bad != 0;
}
"""


def test_no_workgroup_and_no_unit_has_more_than_by_the_mean(tmp_path):
    src, exe = tmp_path / "shares.cpp", tmp_path / "shares"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover", "-I", os.path.join(ROOT, "paper_2402_02361_amd", "csrc"), str(src), "-o", str(exe)])
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
