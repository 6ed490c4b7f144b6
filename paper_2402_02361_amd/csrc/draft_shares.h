// How many workgroups of a draft launch walk through each of its segments: plain C++, so that the rule can be checked on the host.
// It is asked for on every call, so it allocates nothing and divides in 32 bits.
#pragma once
#include <stdint.h>
#include <string.h>

namespace pruner {

constexpr int32_t kSharedSegments = 256, kMostUnits = 512;

struct Busiest {
    uint32_t chunks, units;   // of the compute units that have most; how many these are
};
// Where workgroups go to `cus` units in turn.  A segment's workgroups have as many chunks as each other, the first of them one more.
inline Busiest busiest_units(const uint32_t* chunks, const uint32_t* blocks, int32_t n, uint32_t cus)
{
    uint32_t step[kMostUnits + 1];   // from a unit to the next (modulo 2^32)
    memset(step, 0, (cus + 1) * sizeof(uint32_t));
    uint32_t all = 0, at = 0;
    auto add = [&](uint32_t whole, uint32_t left, uint32_t each) {   // to `whole` rounds of workgroups and `left` more, from `at` on
        all += whole * each;
        const uint32_t end = at + left;
        step[at] += each;
        step[end < cus ? end : cus] -= each;
        if (end > cus) step[0] += each, step[end - cus] -= each;
    };
    for (int32_t i = 0; i < n; ++i) {
        const uint32_t b = blocks[i];
        if (b < 1) continue;
        const uint32_t each = chunks[i] / b, longer = chunks[i] - each * b, rounds = b / cus, left = b - rounds * cus;
        const uint32_t longer_rounds = longer < cus ? 0u : longer / cus;
        add(longer_rounds, longer - longer_rounds * cus, 1);
        add(rounds, left, each);
        at += left;
        at -= at >= cus ? cus : 0u;
    }
    uint32_t most = 0, here = 0, units = 0;
    for (uint32_t u = 0; u < cus; ++u) {
        here += step[u];
        units = here > most ? 1 : units + (here == most);
        most = here > most ? here : most;
    }
    return Busiest{all + most, units};
}

// chunks[i]: pieces of segment i, one workgroup's at a time (fewer than 2^31 in all); room: workgroups that the device holds at once;
// blocks[i]: the workgroups that segment i gets.
// None has more chunks than the launch's mean.  What the device holds beyond that goes to the segments by their shares where the busiest
// compute units then have fewer chunks or are next to none (a filter's call: one GEMM of 3.2 M candidates, 782 workgroups of four 53.4 us,
// 1,024 of three or four 48.9; five convolutions of 960,001 75.5 and 70.4; 14 GEMMs and 6 batched ones of 240,000 51.0 and 46.6; 40 x 83,333 of
// four classes 56.6 and 53.9; three GEMMs of 700,001, nine chunks on 172 units or on six, 34.1 and 32.3).  Not where they have as many, longer
// workgroups of several segments on the same units (eight GEMMs of 312,501, 816 workgroups of three 37.1 us, 1,024 of two or three 38.2; 20 x 166,667
// of four classes 49.2 and 54.7), and not where there are so many segments that asking costs as much.  (Of several classes a count of chunks
// says less: 7 x 385,715 42.8 us by the mean and 45.8 by shares, which leave fewer to every unit.)  Where a
// workgroup for every mean is slightly more than fits, the shares rounded down are hardly longer (five convolutions of 2.2 M, 770 of 14 119 us,
// 765 of 14 or 15 106); shares alone would leave 19 chunks to one where all others have ten (10.5 M candidates of a GEMM and
// 19 x 19,456: 66 us, 52 so).
inline void share_workgroups(const uint32_t* chunks, int32_t n, uint32_t room, uint32_t cus, uint32_t* blocks)
{
    uint32_t total = 0, least = 0;
    for (int32_t i = 0; i < n; ++i) total += chunks[i];
    const uint32_t mean = total > room ? (total + room - 1) / room : 1;
    for (int32_t i = 0; i < n; ++i) least += blocks[i] = mean == 1 ? chunks[i] : (chunks[i] + mean - 1) / mean;
    if (mean == 1 || least == room || n > kSharedSegments || cus < 1 || cus > (uint32_t)kMostUnits) return;
    const double per_chunk = (double)room / total;
    auto share_of = [&](int32_t i) { return (uint32_t)(chunks[i] * per_chunk + 1e-6); };
    uint32_t fuller[kSharedSegments];
    if (least < room) {
        const uint32_t spare = room - least;
        uint32_t wanted = 0;
        for (int32_t i = 0; i < n; ++i) {
            const uint32_t share = share_of(i);
            wanted += fuller[i] = share > blocks[i] ? share - blocks[i] : 0;
        }
        const double handed_out = wanted > spare ? (double)spare / wanted : 1.0;
        for (int32_t i = 0; i < n; ++i) fuller[i] = blocks[i] + (wanted > spare ? (uint32_t)(fuller[i] * handed_out) : fuller[i]);
    } else {
        uint32_t sum = 0;
        for (int32_t i = 0; i < n; ++i) {
            fuller[i] = share_of(i);
            sum += fuller[i] = fuller[i] > 0 || chunks[i] == 0 ? fuller[i] : 1;
            if (chunks[i] > fuller[i] * (mean + 1 + mean / 8) || sum > least) return;
        }
    }
    const Busiest by_mean = busiest_units(chunks, blocks, n, cus), by_shares = busiest_units(chunks, fuller, n, cus);
    if (n == 1 || by_shares.chunks < by_mean.chunks || (by_shares.chunks == by_mean.chunks && 8 * by_shares.units < by_mean.units)) memcpy(blocks, fuller, n * sizeof(uint32_t));
}

// Whether the draft kernel for several closed forms is taken with four wavefronts per SIMD, two registers spilled, instead of three: where its
// workgroups then walk through fewer chunks one after the other (a filter's call, 176,000 candidates of ten segments 30.4 -> 27.5 us, 270,000 37.9 ->
// 36.5, 333,333 52.9 -> 49.3).  With as many either way the spilled registers are what is left of it (seven of 300,001, three chunks,
// 38.6 and 40.8; ten of 120,000, two, the kernel 14.3 and 15.7; of 70,000, one, 12.8 and 13.3).
constexpr int64_t rounds_of(int64_t chunks, int64_t at_once) { return (chunks + at_once - 1) / at_once; }
constexpr bool four_waves_pay(int64_t chunks, int64_t units) { return rounds_of(chunks, 4 * units) < rounds_of(chunks, 3 * units); }

}  // namespace pruner
