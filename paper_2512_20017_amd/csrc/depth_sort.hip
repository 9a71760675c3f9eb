// Depth order inside each tile's list. The binning kernels leave every tile's list of (depth bits, point index) pairs in no
// particular order, one that may differ from run to run; here the point indices of each list are put into the order of the depth bits,
// equal ones by point index. One launch of workgroups of eight wavefronts, every list on its own:
//   - short lists (long_list_from(): how short depends on how many lists there are; k_tile_lists lists the tiles longest first and
//     says how many are long): one WAVEFRONT per list, no workgroup barrier anywhere. Up to 64 entries by counting (every lane
//     compares its key with all others through the scalar unit), else stable least-significant-digit radix passes with 10-bit
//     digits. Keys and positions live in registers in list order; a pass scatters them into the wavefront's 6.5 KB of LDS and reads
//     them back in the new order;
//   - up to 5,632 entries: the same by a whole workgroup, each wavefront with its part of the list in registers;
//   - up to 8,192: what moves is the permutation (16-bit positions, two copies in LDS); the keys are fetched through it;
//   - longer lists: the pairs move between the global array and a second one, each wavefront sweeping its
//     part of the list once per pass (the first pass twice: count, then place; a placing sweep counts for the next pass).
// A pass ranks its entries per wavefront and round of 64 by ballots (lanes with the same digit find each other), the first lane of
// each group adds the group's size to the digit's counter in LDS (16 bits wide, two to a word) and gets back how many entries of
// that digit came before (earlier rounds of the wavefront: LDS executes a wavefront's operations in order), and hands that to its
// group through the LDS crossbar: equal digits keep their incoming order.
//
// Two passes, over the top 20 bits of the depths less the list's smallest (whose range is 25 or 26 bits: a few octaves. The bits as
// they are differ in 31 bits where a list has depths on both sides of 2.0, which every tile of a street has: 11 bits too coarse, and
// most lists were sorted three times over, 192 us -> 134 for 7.3 M pairs at 3840x2160). That orders a list but for
// neighbours, some per thousand entries, that agree in those bits, and for equal
// depths, which are in order only if they came in order. Where all such runs are of two entries and no depths are equal, as in nearly every
// list of a few hundred, the two change places on their way out. Else the runs are put right by counting: every entry of a run
// compares its depth and point index with the others' and goes to its rank. Where a run is longer than kCountRun entries (whole walls
// at one depth), the runs are numbered and the list is sorted again by number and point index in one key; where such a list also has
// depths that agree in the top bits and differ below, or where the key would not fit a word, by point index and then, which keeps
// that order, by all bits of the depths. All lists of 1M points at 1920x1080, binning included, with the depths rounded to 4, to 0.5 and to
// 0.03 (of 10 to 20 units), and each value four times, against sweeps that swapped neighbours, eight of them before all three sorts:
// 141 -> 106, 142 -> 109, 138 -> 104, 124 -> 90; as they are 80.
//
// The work is a chain of dependent LDS and cross-lane steps per list, and what hides it is other lists in flight: three workgroups
// per compute unit by LDS, 24 wavefronts, at most 80 registers. No scratch memory: a launch that has any is slower by tens of us.
// Against three 9-bit passes with a branch around every round of 64, four wavefronts to a workgroup, one list alone (us): 100
// entries 8.0 -> 3.7, 256 9.8 -> 4.4, 512 13.7 -> 4.6, 768 17.5 -> 5.9, 2,000 16.5 -> 11.5, 4,600 34.6 -> 22.6, 7,800 71.2 -> 35.6. All lists of
// 1M points at 1920x1080 (8,160 tiles, 1.9 M pairs, the longest list 4,835): 38 -> 28; 4,096 points at 128x128 20.4 -> 8.3.
// (Measured and dropped: each wavefront sorting its part and then finding every entry's place by binary search in the other parts:
// 2,000 entries 18 us, 4,600 37.)
#include "pbdr_internal.h"
#include "wave_ops.h"

#include <type_traits>

namespace pbdr {

constexpr int kSortWaves = 8, kSortThreads = 64 * kSortWaves;      // a workgroup
constexpr int kListBits = 10;                         // digit width of the list sorts
constexpr int kListBins = 1 << kListBits;
constexpr int kListWords = kListBins / 2;             // counters in LDS are 16 bits wide, two digits to a word (the LDS adds 32-bit words)
constexpr int kPerLane = kListWords / 64;             // a wavefront's counter words, per lane
constexpr int kFirstBits = 2 * kListBits;             // of the bits that differ, those the list is first sorted by
constexpr int kLongBits = 9;                          // digit width of the lists too long for LDS: their counters are 32 bits wide
constexpr int kLongBins = 1 << kLongBits;
static_assert(kWaveListMax % 64 == 0, "whole rounds");
constexpr int kWgKeyMax = 11 * kSortThreads;           // a workgroup's list with its keys in registers and LDS (11 rounds per wavefront)
constexpr int kWgListMax = 16 * kSortThreads;          // a workgroup's list with its permutation in LDS (16 rounds per wavefront)

// Runs of more entries with equal bits are not put right by counting, whose time grows with the run (64 instead of 32: depths rounded to
// 4 units 104 -> 109 us; 16: each value four times 90 -> 102).
constexpr uint32_t kCountRun = 32;
constexpr uint32_t kCountRunInMemory = 16;      // for the lists that do not fit the LDS, whose entries are fetched from memory each time

struct WaveSortLds {      // a wavefront's share of the LDS when it sorts a list of its own
    uint32_t key[kWaveListMax];
    union {
        struct { uint16_t idx[kWaveListMax]; uint32_t hist[kListWords]; };
        uint32_t val[kWaveListMax];      // (once the passes are done)
    };
};
struct WgSortLds {        // the workgroup's LDS when it sorts one list together
    union {
        struct { uint32_t key[kWgKeyMax]; uint16_t idx[kWgKeyMax]; };        // the list, keys and incoming positions
        struct { uint32_t key_[kWgKeyMax]; uint32_t val[kWgKeyMax]; };       // keys and point indices, once the passes are done
        uint16_t perm[2][kWgListMax];                                        // the permutation alone, twice
        uint32_t count[2][kSortWaves][kLongBins];                                     // two sets of full-width counters
        // per wavefront and digit: entries in the wavefront's part of the list, then where its first entry of that digit goes
        struct { uint32_t first_[kWgKeyMax + kWgKeyMax / 2]; uint32_t cnt[kSortWaves][kListWords]; };
    };
    uint32_t scan[kSortWaves];
    uint32_t any[2][kSortWaves];
    uint2 range[kSortWaves];
};
static_assert(sizeof(WgSortLds::perm) <= sizeof(WgSortLds::first_), "the permutation and the counters at the same time");
union ListSortLds { WgSortLds wg; WaveSortLds wave[kSortWaves]; };
static_assert(sizeof(ListSortLds) <= 53 * 1024, "three workgroups per compute unit");

// The passes by digits over the top `bits` bits of keys from 0 to `range`: their number and the shift of pass p (the topmost digit
// may reach past the highest of those bits, never past bit 31).
struct Passes { int lo, count; };
__device__ __forceinline__ Passes list_passes(uint32_t range, int bits, int digit)
{
    if (range == 0u) return Passes{0, 0};
    const int hi = 31 - __builtin_clz(range), lo = max(0, hi + 1 - bits);
    return Passes{lo, (hi - lo + digit) / digit};
}
__device__ __forceinline__ int list_shift(const Passes& p, int i, int digit) { return min(p.lo + digit * i, 32 - digit); }

// What a list in LDS is being sorted by: the top bits of the depths; the number of the run of equal depths, above the point index;
// where those two do not fit a word, the point index and then, which keeps that order, all bits of the depths.
enum class SortBy { kDepthTop, kRun, kIndex, kDepth };

// Entries of this wavefront with the same digit as this lane's that come before it: earlier rounds (through the
// digit's counter in `hist`, a row no other wavefront touches) plus lower lanes of this round. The lanes that share the
// digit are found bit by bit: a lane differs from this one if, for some bit, its bit (one ballot per bit) is not this
// lane's bit (sign-extended to a mask); both halves of the 64-lane sets are kept in 32-bit registers.
// kPacked: the counters are 16 bits wide, digit d in half d & 1 of word d >> 1 (for lists of fewer than 65,536 entries:
// no half ever carries into its neighbour); else one word per digit.
__device__ __forceinline__ uint32_t packed_half(uint32_t word, uint32_t digit) { return (word >> ((digit & 1u) << 4)) & 0xffffu; }

template <int kBits, bool kPacked>
__device__ __forceinline__ uint32_t digit_prefix(uint32_t* hist, uint32_t digit, bool valid)
{
    const int lane = threadIdx.x & 63;
    uint32_t dlo = 0u, dhi = 0u;
#pragma unroll
    for (int bit = 0; bit < kBits; ++bit) {
        const uint32_t ext = (uint32_t)__builtin_amdgcn_sbfe((int)digit, bit, 1);      // 0 or ~0
        const uint64_t m = __ballot(ext != 0u);
        dlo |= (uint32_t)m ^ ext;
        dhi |= (uint32_t)(m >> 32) ^ ext;
    }
    const uint64_t vm = __ballot(valid);
    const uint32_t plo = ~dlo & (uint32_t)vm, phi = ~dhi & (uint32_t)(vm >> 32);       // valid lanes with this lane's digit
    // lanes below this one among them
    const uint32_t below_lo = lane < 32 ? (1u << lane) - 1u : ~0u, below_hi = lane < 32 ? 0u : (1u << (lane - 32)) - 1u;
    const uint32_t rank = (uint32_t)__popc(plo & below_lo) + (uint32_t)__popc(phi & below_hi);
    uint32_t before = 0u;
    if (valid && rank == 0u) {
        const uint32_t group = (uint32_t)__popc(plo) + (uint32_t)__popc(phi);
        if (kPacked) before = packed_half(atomicAdd(&hist[digit >> 1], group << ((digit & 1u) << 4)), digit);
        else before = atomicAdd(&hist[digit], group);
    }
    const int leader = !valid ? lane : (plo ? __builtin_ctz(plo) : 32 + __builtin_ctz(phi));
    before = (uint32_t)__builtin_amdgcn_ds_bpermute(leader << 2, (int)before);
    return before + rank;
}

// exclusive scan over a wavefront's packed digit counters, 2 * kPerLane consecutive digits per lane, in place
__device__ __forceinline__ void wave_scan_digits(uint32_t* hist)
{
    const int lane = threadIdx.x & 63;
    uint32_t c[2 * kPerLane], tot = 0u;
#pragma unroll
    for (int q = 0; q < kPerLane; ++q) {
        const uint32_t w = hist[kPerLane * lane + q];
        c[2 * q] = w & 0xffffu; c[2 * q + 1] = w >> 16;
        tot += c[2 * q] + c[2 * q + 1];
    }
    uint32_t at = wave_inclusive_scan(tot, OpAdd{}) - tot;
#pragma unroll
    for (int q = 0; q < kPerLane; ++q) {
        const uint32_t a0 = at, a1 = at + c[2 * q];
        hist[kPerLane * lane + q] = a0 | (a1 << 16);
        at = a1 + c[2 * q + 1];
    }
}

__device__ __forceinline__ void wave_lds_sync()      // orders this wavefront's LDS writes before its later LDS reads
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// i < n - before, on the scalar side but for the comparison: "before + i < n" would keep a register for every before
__device__ __forceinline__ bool within(int i, uint32_t n, int before) { return i < (int)n - before; }

// how many lanes of the set lie below this one
__device__ __forceinline__ uint32_t lanes_below(uint64_t set) { return __builtin_amdgcn_mbcnt_hi((uint32_t)(set >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)set, 0u)); }

// The same value, as one that the compiler does not know: addresses and masks made of it are made where they stand. Else those of
// all of a list's rounds are worked out ahead of everything, and there are not enough registers to keep them.
__device__ __forceinline__ uint32_t anew_uniform(uint32_t v)
{
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ uint32_t anew(uint32_t v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// The list keys[0 .. L), values[0 .. L) in LDS is in order but for the runs of entries that agree in the bits from `shift` on. Puts the
// values of places `base` .. base + 63 where they belong: each entry of a run counts how many of the run come before it. One
// wavefront; the LDS holds whole rounds of 64 places.
__device__ __forceinline__ void rank_round(const uint32_t* keys, const uint32_t* values, uint32_t L, int shift, uint32_t base, uint32_t* out)
{
    const uint32_t lane = anew(threadIdx.x) & 63u, place = base + lane;
    // where runs start, a bit per place of a round (each place behind the end is a run of its own)
    const auto starts = [&](uint32_t b) {
        const uint32_t p = b + lane;
        return __ballot(p >= L || p == 0u || (keys[p] >> shift) != (keys[max(p, 1u) - 1u] >> shift));
    };
    const uint64_t here = starts(base), upto = ~0ull >> (63u - lane);
    uint32_t before = base, behind = base + 64u;      // the last start before the round's places, the first one behind them
    if ((here & 1ull) == 0ull) {
        uint64_t h;
        do { before -= 64u; h = starts(before); } while (h == 0ull);      // (place 0 is a start)
        before += 63u - (uint32_t)__builtin_clzll(h);
    }
    while (behind < L) {
        const uint64_t h = starts(behind);
        if (h) { behind += (uint32_t)__builtin_ctzll(h); break; }
        behind += 64u;
    }
    const uint64_t lo = here & upto, hi = here & ~upto;
    const uint32_t s = lo ? base + 63u - (uint32_t)__builtin_clzll(lo) : before;
    const uint32_t n = (hi ? base + (uint32_t)__builtin_ctzll(hi) : behind) - s;      // of the run: one or more
    const uint32_t value = values[place];
    const uint64_t mine = (uint64_t)keys[place] << 32 | value;
    uint32_t rank = 0u;
    if (__ballot(n > 1u) != 0ull) {
        for (uint32_t d = 0; __ballot(d < n) != 0ull; d += 4u) {
#pragma unroll
            for (uint32_t q = 0; q < 4u; ++q) {
                const uint32_t j = s + min(d + q, n - 1u);
                rank += (d + q < n && ((uint64_t)keys[j] << 32 | values[j]) < mine) ? 1u : 0u;
            }
        }
    }
    if (place < L) out[min(s + rank, L - 1u)] = value;      // (always below)
}

// Of a list in rounds of 64, a bit a round and lane: the bits of the entries before. first: that of the entry before the first.
__device__ __forceinline__ uint32_t of_entries_before(uint32_t bits, uint32_t first)
{
    const uint32_t wrapped = (uint32_t)__builtin_amdgcn_readlane((int)bits, 63) << 1 | first;      // lane 0's: the last lane's of the round before
    return (uint32_t)__builtin_amdgcn_update_dpp((int)wrapped, (int)bits, 0x138, 0xf, 0xf, false);      // wave_shr:1
}

// Which of the wavefront's R rounds hold an entry of a run of two or more? agree: a bit per round, this lane's entry agrees with the next place's.
__device__ __forceinline__ uint32_t rounds_of(uint32_t agree, int R)
{
    uint32_t rounds = 0u;
    for (int r = 0; r < R; ++r) {
        const uint64_t b = __ballot((agree >> r) & 1u);
        if (b) rounds |= (1u << r) | (uint32_t)(b >> 63) << (r + 1);
    }
    return rounds & ((1u << R) - 1u);
}

// Of a list in LDS in order of the bits from `shift` on, in the rounds of 64 places from `first` on that `rounds` names: does a run of entries
// that agree in those bits have more than kCountRun? One wavefront.
__device__ __forceinline__ bool long_runs(const uint32_t* keys, uint32_t L, int shift, uint32_t first, uint32_t rounds)
{
    bool any = false;
    for (; rounds != 0u; rounds &= rounds - 1u) {
        const uint32_t p = first + 64u * (uint32_t)__builtin_ctz(rounds) + (anew(threadIdx.x) & 63u);
        any |= p + kCountRun < L && keys[p + kCountRun] >> shift == keys[p] >> shift;
    }
    return __ballot(any) != 0ull;
}

// Do neighbours that agree in those bits differ below? Of the places from `place` on, `step` apart.
__device__ __forceinline__ bool mixed_runs(const uint32_t* keys, uint32_t L, int shift, uint32_t place, uint32_t step)
{
    bool any = false;
    for (uint32_t p = place; p + 1u < L; p += step) any |= keys[p] != keys[p + 1u] && keys[p] >> shift == keys[p + 1u] >> shift;
    return any;
}

// Keys of the number of an entry's run, 0 .. last_run, above its point index less the list's smallest, 0 .. values.
struct RunKey { bool fits; int bits; uint32_t mask, range; };
__device__ __forceinline__ RunKey run_key(uint32_t last_run, uint32_t values)
{
    const int bits = 32 - __builtin_clz(values | 1u), run_bits = last_run ? 32 - __builtin_clz(last_run) : 0;
    const uint32_t mask = (1u << (bits & 31)) - 1u;
    return RunKey{bits + run_bits <= 32 && bits < 32, bits & 31, mask, last_run << (bits & 31) | mask};
}

// One wavefront sorts a list of at most 64 entries by counting: how many entries have a smaller key.
__device__ __forceinline__ void wave_count_list(uint32_t L, const uint2* pairs, uint32_t* vals)
{
    const int lane = threadIdx.x & 63;
    uint32_t k = 0u, v = 0u, before = 0u;
    if ((uint32_t)lane < L) { const uint2 p = pairs[lane]; k = p.x; v = p.y; }
    for (uint32_t j = 0; j < L; ++j) before += (uint32_t)__builtin_amdgcn_readlane((int)k, (int)j) < k ? 1u : 0u;
    if ((uint32_t)lane >= L) before = 0u;
    if (wave_reduce(before, OpAdd{}) != L * (L - 1u) / 2u) {      // some are equal: then by value
        for (uint32_t j = 0; j < L; ++j)
            before += ((uint32_t)__builtin_amdgcn_readlane((int)k, (int)j) == k && (uint32_t)__builtin_amdgcn_readlane((int)v, (int)j) < v) ? 1u : 0u;
    }
    if ((uint32_t)lane < L) vals[min(before, L - 1u)] = v;
}

// One wavefront sorts the list pairs[0 .. L), 64 < L <= 64 R, into vals; the pairs are spent. The rounds of 64 are all
// walked, whatever the length: with a branch around every round none would overlap with the next, and each is a chain of LDS and
// cross-lane steps.
template <int R>
__device__ __forceinline__ void wave_sort_list(WaveSortLds& W, uint32_t L, uint2* pairs, uint32_t* vals)
{
    const int lane = threadIdx.x & 63;
    // the list in its current order: entry r * 64 + lane, with its incoming position. The places behind its end hold the largest
    // key: their digits are all ones, so they stay behind, and a pass needs no bounds.
    uint32_t key[R], id[R];      // id: the position, and during a pass its rank among equal digits above kIdBits
    constexpr int kIdBits = 16;
    const auto one_pass = [&](int shift) {
#pragma unroll
        for (int q = 0; q < kPerLane; ++q) W.hist[q * 64 + lane] = 0u;
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < R; ++r) id[r] |= digit_prefix<kListBits, true>(W.hist, (key[r] >> shift) & (kListBins - 1u), true) << kIdBits;
        wave_lds_sync();
        wave_scan_digits(W.hist);
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t digit = (anew(key[r]) >> shift) & (kListBins - 1u);
            const uint32_t pos = min(packed_half(W.hist[digit >> 1], digit) + (id[r] >> kIdBits), (uint32_t)kWaveListMax - 1u);      // (always below)
            W.key[pos] = key[r]; W.idx[pos] = (uint16_t)id[r];
        }
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < R; ++r) { key[r] = W.key[r * 64u + lane]; id[r] = W.idx[r * 64u + lane]; }
        wave_lds_sync();      // (the next pass, or the next list of this wavefront, writes the buffer again)
    };
    uint32_t* const words = reinterpret_cast<uint32_t*>(pairs);
    SortBy by = SortBy::kDepthTop;
    uint32_t range = 0u, value_base = 0u, value_mask = 0u;
#pragma unroll 1
    for (;;) {
        if (by != SortBy::kRun) {
            const uint32_t* const from = words + (by == SortBy::kIndex ? 1 : 0);      // (every other word)
            const uint32_t at = anew(lane);
            uint32_t lo = 0u, hi = 0u;      // (the smallest key, inverted)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                key[r] = 0xffffffffu;
                id[r] = r * 64u + at;
                if (within(lane, L, r * 64)) { key[r] = from[2u * (r * 64u + at)]; lo = max(lo, ~key[r]); hi = max(hi, key[r]); }
            }
            lo = ~wave_reduce(lo, OpMax{});
            range = wave_reduce(hi, OpMax{}) - lo;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, r * 64)) key[r] -= lo;
        }
        const Passes ps = list_passes(range, by == SortBy::kDepthTop ? kFirstBits : 32, kListBits);
        for (int p = 0; p < ps.count; ++p) one_pass(list_shift(ps, p, kListBits));
        if (by == SortBy::kRun) {      // (no two keys are equal; a key holds its point index)
            const uint32_t to = anew(lane);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, r * 64)) vals[r * 64u + to] = (key[r] & value_mask) + value_base;
            return;
        }
        if (by == SortBy::kDepthTop) {
            // a bit a round: the entry agrees with the next one, and is the larger of the two
            uint32_t agree = 0u, larger = 0u;
            bool more = range == 0u;      // are there equal ones, or more than two that agree?
            if (range != 0u) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane + 1, L, r * 64)) {
                        const uint32_t next = W.key[r * 64u + lane + 1u];
                        agree |= (next ^ key[r]) >> ps.lo == 0u ? 1u << r : 0u;
                        larger |= next < key[r] ? 1u << r : 0u;
                        more |= next == key[r];
                    }
                more |= (agree & of_entries_before(agree, 0u)) != 0u;
            }
            if (__ballot(more) == 0ull) {      // two that agree change places here if they have to
                const uint32_t smaller = of_entries_before(larger, 0u), to = anew(lane);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane, L, r * 64)) id[r] = words[2u * id[r] + 1u];
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane, L, r * 64)) vals[r * 64u + to + ((larger >> r) & 1u) - ((smaller >> r) & 1u)] = id[r];
                return;
            }
            uint32_t rounds = range != 0u ? rounds_of(agree, R) : 0u;      // with entries to be put right, a bit each
            if (range != 0u && !long_runs(W.key, L, ps.lo, 0u, rounds)) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane, L, r * 64)) id[r] = words[2u * id[r] + 1u];
                const uint32_t to = anew(lane);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (((rounds >> r) & 1u) == 0u && within(lane, L, r * 64)) vals[r * 64u + to] = id[r];
#pragma unroll
                for (int r = 0; r < R; ++r) W.val[r * 64u + lane] = id[r];
                wave_lds_sync();
                for (; rounds != 0u; rounds &= rounds - 1u) rank_round(W.key, W.val, L, ps.lo, 64u * (uint32_t)__builtin_ctz(rounds), vals);
                return;
            }
            // runs of equal depth, numbered, above the point indices less the list's smallest
            bool fits = false;
            if (range == 0u || __ballot(mixed_runs(W.key, L, ps.lo, lane, 64u)) == 0ull) {
                uint32_t lo = 0u, hi = 0u, count = 0u, last = 0u;
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane, L, r * 64)) { id[r] = words[2u * id[r] + 1u]; lo = max(lo, ~id[r]); hi = max(hi, id[r]); }
                if (range != 0u) {
                    for (uint32_t p = lane; p - lane < L; p += 64u) {      // (place 0 and those behind the end start no run)
                        const uint32_t k = W.key[p], up = (uint32_t)__shfl_up((int)k, 1, 64);
                        const bool starts = p < L && p != 0u && k != (lane == 0 ? last : up);
                        const uint64_t b = __ballot(starts);
                        last = (uint32_t)__builtin_amdgcn_readlane((int)k, 63);
                        W.key[p] = count + lanes_below(b) + (starts ? 1u : 0u);
                        count += (uint32_t)__popcll(b);
                    }
                }
                value_base = ~wave_reduce(lo, OpMax{});
                const RunKey rk = run_key(count, wave_reduce(hi, OpMax{}) - value_base);
                fits = rk.fits;
                value_mask = rk.mask;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    key[r] = within(lane, L, r * 64) ? (range != 0u ? W.key[r * 64u + lane] << rk.bits : 0u) | (id[r] - value_base) : 0xffffffffu;
                    id[r] = 0u;
                }
                range = rk.range;
                wave_lds_sync();
            }
            by = fits ? SortBy::kRun : SortBy::kIndex;
            continue;
        }
        // through the sorted positions
        const uint32_t to = anew(lane);
        if (by == SortBy::kDepth) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, r * 64)) key[r] = words[2u * id[r] + 1u];
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, r * 64)) vals[r * 64u + to] = key[r];
            return;
        }
#pragma unroll
        for (uint32_t half = 0; half < 2u; ++half) {      // (every entry is fetched before the first is stored)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, r * 64)) key[r] = words[2u * id[r] + half];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, r * 64)) words[2u * (r * 64u + to) + half] = key[r];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");      // (read back by other lanes)
            __builtin_amdgcn_wave_barrier();
        }
        by = SortBy::kDepth;
    }
}

// The wavefronts' digit counts, one row each, into where each wavefront's first entry of each digit goes: behind the smaller
// digits, and the wavefronts before it. A thread takes a word of the counters, all rows of it. (Every wavefront adding the rows up
// for itself reads all of them, eight words to a lane, eight lanes to a bank: 3 us a pass.) Starts and ends with a barrier.
__device__ __forceinline__ void wg_scan_digits(WgSortLds& S)
{
    static_assert(kListWords == kSortThreads, "a word per thread");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    __syncthreads();
    uint32_t c[kSortWaves], all = 0u;      // two digits to a word: a digit's count over the list is below 65,536
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) { c[w] = S.cnt[w][threadIdx.x]; all += c[w]; }
    const uint32_t tot = (all & 0xffffu) + (all >> 16), inc = wave_inclusive_scan(tot, OpAdd{});
    if (lane == 63) S.scan[wave] = inc;
    __syncthreads();
    uint32_t at = inc - tot;
#pragma unroll
    for (int w = 0; w + 1 < kSortWaves; ++w) at += w < wave ? S.scan[w] : 0u;
    uint32_t run = at | (at + (all & 0xffffu)) << 16;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) { S.cnt[w][threadIdx.x] = run; run += c[w]; }
    __syncthreads();
}

// Does any thread of the workgroup say so? A barrier; calls in a row take turns with `turn` (0, 1, 0, ...).
__device__ __forceinline__ bool wg_any(WgSortLds& S, int turn, bool v)
{
    const bool mine = __ballot(v) != 0ull;
    if ((threadIdx.x & 63u) == 0u) S.any[turn & 1][threadIdx.x >> 6] = mine ? 1u : 0u;
    __syncthreads();
    uint32_t any = 0u;
#pragma unroll
    for (int w = 0; w < kSortWaves; ++w) any |= S.any[turn & 1][w];
    return __builtin_amdgcn_readfirstlane(any) != 0u;
}

// The keys' range over the workgroup: the threads' largest and smallest (inverted) key in, the smallest out and the difference
// returned. One barrier; the next call is several barriers away.
__device__ __forceinline__ uint32_t wg_key_range(WgSortLds& S, uint32_t& lo, uint32_t hi)
{
    const uint32_t l = wave_reduce(lo, OpMax{}), h = wave_reduce(hi, OpMax{});
    if ((threadIdx.x & 63u) == 0u) S.range[threadIdx.x >> 6] = make_uint2(l, h);
    __syncthreads();
    uint2 all = S.range[0];
#pragma unroll
    for (int w = 1; w < kSortWaves; ++w) { const uint2 r = S.range[w]; all.x = max(all.x, r.x); all.y = max(all.y, r.y); }
    lo = ~(uint32_t)__builtin_amdgcn_readfirstlane((int)all.x);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)all.y) - lo;
}

// The list is in order but for the runs of entries that agree in the bits from `shift` on of the keys less lo: puts the point indices in
// order, each entry of a run by its rank. Returns false if a run is too long for that (vals is then written in part).
__device__ __forceinline__ bool rank_ties(WgSortLds& S, uint32_t L, uint32_t lo, int shift, const uint2* p, uint32_t* vals)
{
    bool fits = true;
    for (uint32_t i = threadIdx.x; i < L; i += kSortThreads) {
        const uint2 mine = p[i];
        const uint32_t top = (mine.x - lo) >> shift;
        uint32_t pos = i, d = 1u;
        for (; d <= kCountRunInMemory && d <= i; ++d) {
            const uint2 o = p[i - d];
            if ((o.x - lo) >> shift != top) break;
            if (mine.x < o.x || (mine.x == o.x && mine.y < o.y)) --pos;
        }
        fits &= d <= kCountRunInMemory;
        for (d = 1u; d <= kCountRunInMemory && i + d < L; ++d) {
            const uint2 o = p[i + d];
            if ((o.x - lo) >> shift != top) break;
            if (o.x < mine.x || (o.x == mine.x && o.y < mine.y)) ++pos;
        }
        fits &= d <= kCountRunInMemory;
        vals[pos] = mine.y;
    }
    return !wg_any(S, 0, !fits);
}

// A workgroup sorts the list pairs[0 .. L), L <= kWgListMax, into vals; the pairs are spent. The permutation perm[c][i] =
// incoming position of the entry now at i goes back and forth between its two copies in LDS; the keys are fetched through it.
__device__ __forceinline__ void wg_permute_list(WgSortLds& S, uint32_t L0, uint2* pairs, uint32_t* vals)
{
    uint32_t L = L0;
    constexpr int R = kWgListMax / kSortThreads;
    static_assert(R % 4 == 0, "rounds are taken four at a time");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // each wavefront takes a contiguous eighth of the list, in rounds of 64
    const uint32_t per_wave = ((L + kSortThreads - 1u) / kSortThreads) * 64u;
    const int nr0 = (int)(per_wave / 64u);
    const uint32_t wb = wave * per_wave, we0 = min(L, wb + per_wave);
    uint16_t* src = S.perm[0];
    uint16_t* dst = S.perm[1];
    auto one_pass = [&](int shift, const uint32_t* from, uint32_t lo) {
#pragma unroll
        for (int q = 0; q < kPerLane; ++q) S.cnt[wave][q * 64 + lane] = 0u;
        wave_lds_sync();
        uint32_t we = anew_uniform(we0);
        const int nr = nr0;
        uint32_t dp[R];      // per entry of this lane: digit | (entries of that digit before it in this wavefront's part) << kListBits
        const uint16_t* here = src + anew(wb + lane);
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += 4) {       // four rounds at a time, no branch between them
            if (r0 >= nr) break;
            uint32_t k[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                k[j] = 0u;
                if (within(lane, we, (int)wb + (r0 + j) * 64)) {
                    const uint32_t i = here[(r0 + j) * 64];
                    k[j] = from[2u * i];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t digit = ((k[j] - lo) >> shift) & (kListBins - 1u);
                dp[r0 + j] = digit | (digit_prefix<kListBits, true>(S.cnt[wave], digit, within(lane, we, (int)wb + (r0 + j) * 64)) << kListBits);
            }
        }
        wg_scan_digits(S);
        we = anew_uniform(we0); L = anew_uniform(L0);
        here = src + anew(wb + lane);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r % 8 == 0) asm volatile("" ::: "memory");      // (eight rounds in flight at a time)
            if (within(lane, we, (int)wb + r * 64)) {
                const uint32_t digit = dp[r] & (kListBins - 1u);
                const uint32_t pos = min(packed_half(S.cnt[wave][digit >> 1], digit) + (dp[r] >> kListBits), L - 1u);
                dst[pos] = here[r * 64];
            }
        }
        __syncthreads();      // the pass is written; the other copy of the permutation may be overwritten
        uint16_t* t = src; src = dst; dst = t;
    };
    // by depth bits; where that leaves equal ones out of order, by point index and then, which keeps that order, by depth bits again
#pragma unroll 1
    for (int stage = 0; stage < 3; ++stage) {
        uint32_t* const words = reinterpret_cast<uint32_t*>(pairs);
        const uint32_t* const from = words + (stage == 1 ? 1 : 0);      // (every other word)
        const uint32_t k0 = from[0];
        uint32_t lo = 0u, hi = 0u;      // (the smallest key, inverted)
        for (uint32_t i0 = 0; i0 < L; i0 += 8u * kSortThreads) {      // eight independent fetches in flight
            const uint32_t at = anew(threadIdx.x);
            uint32_t t[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint32_t i = i0 + r * (uint32_t)kSortThreads + at;
                t[r] = within((int)threadIdx.x, L, (int)i0 + r * kSortThreads) ? from[2u * i] : k0;
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const uint32_t i = i0 + r * (uint32_t)kSortThreads + at;
                lo = max(lo, ~t[r]); hi = max(hi, t[r]);
                if (within((int)threadIdx.x, L, (int)i0 + r * kSortThreads)) {
                    src[i] = (uint16_t)i;
                }
            }
        }
        const uint32_t diff = wg_key_range(S, lo, hi);      // (a barrier: keys and permutation are in place)
        const Passes ps = list_passes(diff, stage == 0 ? kFirstBits : 32, kListBits);
        for (int p = 0; p < ps.count; ++p) one_pass(list_shift(ps, p, kListBits), from, lo);
        // through the sorted positions; every entry is fetched before the first is stored
        uint2 out[R];
        const uint32_t to = anew(threadIdx.x);
        L = anew_uniform(L0);
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += 8) {      // (the addresses of eight rounds at a time)
#pragma unroll
            for (int r = r0; r < r0 + 8 && r < R; ++r) {
                out[r] = make_uint2(0u, 0u);
                if (within((int)threadIdx.x, L, r * kSortThreads)) out[r] = pairs[src[r * kSortThreads + threadIdx.x]];
            }
            asm volatile("" ::: "memory");
        }
        __syncthreads();
        L = anew_uniform(L0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (within((int)threadIdx.x, L, r * kSortThreads)) {
                if (stage == 2) vals[r * kSortThreads + to] = out[r].y;
                else pairs[r * kSortThreads + to] = out[r];
            }
        }
        if (stage == 2) return;
        __syncthreads();      // (also: the permutation may be written again)
        if (stage == 0 && rank_ties(S, L, lo, ps.lo, pairs, vals)) return;
    }
}

// A workgroup sorts the list pairs[0 .. L), L <= 8 * 64 R, into vals; the pairs are spent. As one wavefront does it, but for
// the counters: each wavefront holds an eighth of the places, R rounds of 64, and counts for itself; where its entries of a digit
// go then depends on the others' counts.
template <int R>
__device__ __forceinline__ void wg_sort_list(WgSortLds& S, uint32_t L, uint2* pairs, uint32_t* vals)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first = wave * 64 * R;
    uint32_t* const hist = S.cnt[wave];
    uint32_t key[R], id[R];      // id: the position, and during a pass its rank among the wavefront's equal digits above kIdBits
    constexpr int kIdBits = 16;
    const auto one_pass = [&](int shift) {
        // (this wavefront's counters were last read by itself)
#pragma unroll
        for (int q = 0; q < kPerLane; ++q) hist[q * 64 + lane] = 0u;
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < R; ++r) id[r] |= digit_prefix<kListBits, true>(hist, (key[r] >> shift) & (kListBins - 1u), true) << kIdBits;
        wg_scan_digits(S);      // (and every wavefront has fetched its entries of the pass before)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t digit = (anew(key[r]) >> shift) & (kListBins - 1u);
            const uint32_t pos = min(packed_half(hist[digit >> 1], digit) + (id[r] >> kIdBits), (uint32_t)kWgKeyMax - 1u);      // (always below)
            S.key[pos] = key[r]; S.idx[pos] = (uint16_t)id[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) { key[r] = S.key[first + r * 64 + lane]; id[r] = S.idx[first + r * 64 + lane]; }
    };
    uint32_t* const words = reinterpret_cast<uint32_t*>(pairs);
    SortBy by = SortBy::kDepthTop;
    uint32_t range = 0u, value_base = 0u, value_mask = 0u;
#pragma unroll 1
    for (;;) {
        if (by != SortBy::kRun) {
            const uint32_t* const from = words + (by == SortBy::kIndex ? 1 : 0);      // (every other word)
            const uint32_t at = anew(first + lane);
            uint32_t lo = 0u, hi = 0u;      // (the smallest key, inverted)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                key[r] = 0xffffffffu;
                id[r] = r * 64u + at;
                if (within(lane, L, first + r * 64)) { key[r] = from[2u * (r * 64u + at)]; lo = max(lo, ~key[r]); hi = max(hi, key[r]); }
            }
            range = wg_key_range(S, lo, hi);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, first + r * 64)) key[r] -= lo;
        }
        const Passes ps = list_passes(range, by == SortBy::kDepthTop ? kFirstBits : 32, kListBits);
        for (int p = 0; p < ps.count; ++p) one_pass(list_shift(ps, p, kListBits));
        if (by == SortBy::kRun) {      // (as in a wavefront's list, this and what follows)
            const uint32_t to = anew(first + lane);
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, first + r * 64)) vals[r * 64u + to] = (key[r] & value_mask) + value_base;
            return;
        }
        if (by == SortBy::kDepthTop) {
            uint32_t agree = 0u, larger = 0u;
            uint32_t agree0 = 0u, larger0 = 0u;      // the same of the entry before this wavefront's
            bool more = range == 0u;
            if (range != 0u) {
                const uint32_t at = anew(first + lane);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane + 1, L, first + r * 64)) {
                        const uint32_t next = S.key[at + r * 64 + 1];
                        agree |= (next ^ key[r]) >> ps.lo == 0u ? 1u << r : 0u;
                        larger |= next < key[r] ? 1u << r : 0u;
                        more |= next == key[r];
                    }
                if (first != 0 && first < (int)L) {
                    const uint32_t before = S.key[first - 1], own = S.key[first];
                    agree0 = (before ^ own) >> ps.lo == 0u ? 1u : 0u;
                    larger0 = own < before ? 1u : 0u;
                }
                more |= (agree & of_entries_before(agree, agree0)) != 0u;
            }
            if (!wg_any(S, 0, more)) {
                const uint32_t smaller = of_entries_before(larger, larger0), to = anew(first + lane);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane, L, first + r * 64)) id[r] = words[2u * id[r] + 1u];
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane, L, first + r * 64)) vals[r * 64u + to + ((larger >> r) & 1u) - ((smaller >> r) & 1u)] = id[r];
                return;
            }
            bool long_run = range == 0u;
            uint32_t rounds = 0u;      // of this wavefront's
            if (!long_run) {
                rounds = __builtin_amdgcn_readfirstlane(rounds_of(agree, R) | agree0);
                long_run = wg_any(S, 1, long_runs(S.key, L, ps.lo, first, rounds));
            }
            if (!long_run) {
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane, L, first + r * 64)) id[r] = words[2u * id[r] + 1u];
                const uint32_t to = anew(first + lane);
#pragma unroll
                for (int r = 0; r < R; ++r) S.val[to + r * 64] = id[r];
                __syncthreads();      // (before the stores to memory, which it would wait for)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (((rounds >> r) & 1u) == 0u && within(lane, L, first + r * 64)) vals[r * 64u + to] = id[r];
                for (; rounds != 0u; rounds &= rounds - 1u) rank_round(S.key, S.val, L, ps.lo, (uint32_t)first + 64u * (uint32_t)__builtin_ctz(rounds), vals);
                return;
            }
            bool fits = false;
            if (range == 0u || !wg_any(S, 0, mixed_runs(S.key, L, ps.lo, anew(threadIdx.x), kSortThreads))) {
                uint32_t lo = 0u, hi = 0u, count = 0u;
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (within(lane, L, first + r * 64)) { id[r] = words[2u * id[r] + 1u]; lo = max(lo, ~id[r]); hi = max(hi, id[r]); }
                if (range != 0u) {
                    const uint32_t ln = anew(threadIdx.x) & 63u;
                    uint32_t last = first != 0 ? S.key[first - 1] : 0u;
                    __syncthreads();      // (the runs' numbers take the keys' places)
                    for (uint32_t p = first + ln; p - ln < min(L, (uint32_t)first + 64u * R); p += 64u) {
                        const uint32_t k = S.key[p], up = (uint32_t)__shfl_up((int)k, 1, 64);
                        const bool starts = p < L && p != 0u && k != (ln == 0u ? last : up);
                        const uint64_t b = __ballot(starts);
                        last = (uint32_t)__builtin_amdgcn_readlane((int)k, 63);
                        S.key[p] = count + lanes_below(b) + (starts ? 1u : 0u);
                        count += (uint32_t)__popcll(b);
                    }
                }
                if ((anew(threadIdx.x) & 63u) == 0u) S.scan[wave] = count;
                hi = wg_key_range(S, lo, hi);      // (a barrier)
                value_base = lo;
                uint32_t before = 0u;
                count = 0u;
                for (int w = 0; w < kSortWaves; ++w) {
                    const uint32_t n = __builtin_amdgcn_readfirstlane(S.scan[w]);
                    before += w < wave ? n : 0u;
                    count += n;
                }
                const RunKey rk = run_key(count, hi);
                fits = rk.fits;
                value_mask = rk.mask;
                const uint32_t to = anew(first + lane);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    key[r] = within(lane, L, first + r * 64) ? (range != 0u ? (before + S.key[to + r * 64]) << rk.bits : 0u) | (id[r] - value_base) : 0xffffffffu;
                    id[r] = 0u;
                }
                range = rk.range;
                __syncthreads();      // (S.scan is written again by the passes)
            }
            by = fits ? SortBy::kRun : SortBy::kIndex;
            continue;
        }
        // through the sorted positions
        const uint32_t to = anew(first + lane);
        if (by == SortBy::kDepth) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, first + r * 64)) key[r] = words[2u * id[r] + 1u];
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, first + r * 64)) vals[r * 64u + to] = key[r];
            return;
        }
#pragma unroll
        for (uint32_t half = 0; half < 2u; ++half) {      // (every entry is fetched before the first is stored)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, first + r * 64)) key[r] = words[2u * id[r] + half];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (within(lane, L, first + r * 64)) words[2u * (r * 64u + to) + half] = key[r];
        }
        __syncthreads();
        by = SortBy::kDepth;
    }
}

// exclusive scan of one value per thread over the workgroup's threads
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* sScan)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t inc = wave_inclusive_scan(v, OpAdd{});
    if (lane == 63) sScan[wave] = inc;
    __syncthreads();
    uint32_t below = inc - v;
#pragma unroll
    for (int w = 0; w + 1 < kSortWaves; ++w) if (w < wave) below += sScan[w];
    __syncthreads();
    return below;
}

// Lists too long for LDS: one stable pass by the digit at `shift` of the depth bits, or of the point indices, from in to out, both of
// length L in global memory. Each wavefront takes a contiguous eighth of the list, in rounds of 64. `cur` holds, per wavefront
// and digit, how many of its entries have that digit: counted here in a sweep of its own if `count_first`, else by
// the previous pass, which knew where every entry went and so in whose eighth it would be (that is what `nxt` and
// `next_shift` are for: pass a negative shift when no pass follows). The counters are then turned into where the
// wavefront's first entry of each digit goes, and a sweep places the entries: digit_prefix() hands back the counter's
// value before the round's entries were added plus the lane's rank among them, which now is the entry's position.
// Nothing is kept per entry between the sweeps, so the list may be of any length.
__device__ __forceinline__ void long_list_pass(WgSortLds& S, uint32_t (*cur)[kLongBins], uint32_t (*nxt)[kLongBins], bool count_first, uint32_t L, uint32_t lo,
                                               int shift, int next_shift, bool by_index, const uint2* __restrict__ in, uint2* __restrict__ out)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t per_wave = ((L + kSortThreads - 1u) / kSortThreads) * 64u;
    const uint32_t wb = min(L, wave * per_wave), we = min(L, wb + per_wave);
    if (count_first) {
#pragma unroll
        for (int q = 0; q < kLongBins / 64; ++q) cur[wave][q * 64 + lane] = 0u;
        wave_lds_sync();
        for (uint32_t i0 = wb; i0 < we; i0 += 8u * 64u) {      // eight key fetches in flight at a time
            uint32_t k[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t i = i0 + j * 64u + lane;
                k[j] = i < we ? (by_index ? in[i].y : in[i].x) : 0u;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (i0 + j * 64u < we) digit_prefix<kLongBits, false>(cur[wave], ((k[j] - lo) >> shift) & (kLongBins - 1u), i0 + j * 64u + lane < we);
        }
    }
    __syncthreads();      // every wavefront's counts are in
    {   // a digit per thread: its run starts after all smaller digits; inside it the wavefronts follow each other
        static_assert(kLongBins == kSortThreads, "one digit per thread");
        uint32_t c[kSortWaves], tot = 0u;
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) { c[w] = cur[w][threadIdx.x]; tot += c[w]; }
        uint32_t at = block_exclusive_scan(tot, S.scan);
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) { cur[w][threadIdx.x] = at; at += c[w]; nxt[w][threadIdx.x] = 0u; }
    }
    __syncthreads();
    for (uint32_t i0 = wb; i0 < we; i0 += 8u * 64u) {
        uint2 p[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t i = i0 + j * 64u + lane;
            p[j] = i < we ? in[i] : make_uint2(0u, 0u);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (i0 + j * 64u < we) {
                const bool valid = i0 + j * 64u + lane < we;
                const uint32_t k = (by_index ? p[j].y : p[j].x) - lo;
                const uint32_t pos = min(digit_prefix<kLongBits, false>(cur[wave], (k >> shift) & (kLongBins - 1u), valid), L - 1u);      // < L for consistent counts
                if (valid) {
                    out[pos] = p[j];
                    if (next_shift >= 0) {      // the next pass finds this entry in the part of wavefront pos / per_wave
                        uint32_t w2 = 0u;
#pragma unroll
                        for (uint32_t w = 1u; w < (uint32_t)kSortWaves; ++w) w2 += pos >= w * per_wave ? 1u : 0u;
                        atomicAdd(&nxt[w2][(k >> next_shift) & (kLongBins - 1u)], 1u);
                    }
                }
            }
        }
    }
    __syncthreads();      // the pass is written and the next pass's counts are complete
}

// A workgroup sorts a list of any length, pairs[0 .. L), into vals, from one array to the other and back.
__device__ __forceinline__ void wg_sort_long(WgSortLds& S, uint32_t L, uint2* pairs, uint2* spare, uint32_t* vals)
{
    // the two sets of counters swap roles from pass to pass
    uint32_t (*c0)[kLongBins] = S.count[0];
    uint32_t (*c1)[kLongBins] = S.count[1];
    uint2 *here = pairs, *there = spare;      // the list, and where the next pass puts it
    // by depth bits; where that leaves equal ones out of order, by point index and then, which keeps that order, by depth bits again
#pragma unroll 1
    for (int stage = 0; stage < 3; ++stage) {
        uint32_t lo = 0u, hi = 0u;      // (the smallest key, inverted)
        for (uint32_t i = threadIdx.x; i < L; i += kSortThreads) {
            const uint32_t k = stage == 1 ? here[i].y : here[i].x;
            lo = max(lo, ~k); hi = max(hi, k);
        }
        const uint32_t diff = wg_key_range(S, lo, hi);
        const Passes ps = list_passes(diff, 32, kLongBits);
        for (int p = 0; p < ps.count; ++p) {
            const int next_shift = p + 1 < ps.count ? list_shift(ps, p + 1, kLongBits) : -1;
            long_list_pass(S, (p & 1) ? c1 : c0, (p & 1) ? c0 : c1, p == 0, L, lo, list_shift(ps, p, kLongBits), next_shift, stage == 1, here, there);
            uint2* t = here; here = there; there = t;
        }
        if (stage == 0 && rank_ties(S, L, 0u, 0, here, vals)) return;
    }
    for (uint32_t i = threadIdx.x; i < L; i += kSortThreads) vals[i] = here[i].y;
}

// Work items: tile_order lists the tiles longest first and its first `nbig` tiles are too long for one wavefront, so
// workgroups 0 .. nbig - 1 take one such list each, and every later workgroup takes eight shorter lists, one per
// wavefront.
__global__ __launch_bounds__(kSortThreads, 6) void k_tile_depth_sort(const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
                                                            uint32_t ntiles, const uint32_t* __restrict__ status,
                                                            uint32_t cap, uint2* __restrict__ pairs, uint32_t* __restrict__ vals,
                                                            uint2* __restrict__ spare)
{
    __shared__ ListSortLds U;
    const uint32_t nbig = min(status[kStNumBig], ntiles);
    if (blockIdx.x < nbig) {
        const uint32_t tile = tile_order[blockIdx.x];
        const uint32_t s = ranges[2 * tile], e = min(ranges[2 * tile + 1], cap), L = e > s ? e - s : 0u;
        uint2* const p = pairs + s;
        uint32_t* const v = vals + s;
        if (L > (uint32_t)kWgListMax) wg_sort_long(U.wg, L, p, spare + s, v);
        else if (L > (uint32_t)kWgKeyMax) wg_permute_list(U.wg, L, p, v);
        else if (L > 8u * kSortThreads) wg_sort_list<11>(U.wg, L, p, v);
        else if (L > 6u * kSortThreads) wg_sort_list<8>(U.wg, L, p, v);
        else if (L > 4u * kSortThreads) wg_sort_list<6>(U.wg, L, p, v);
        else if (L > 3u * kSortThreads) wg_sort_list<4>(U.wg, L, p, v);
        else if (L > 2u * kSortThreads) wg_sort_list<3>(U.wg, L, p, v);
        else if (L > (uint32_t)kSortThreads) wg_sort_list<2>(U.wg, L, p, v);
        else if (L > 0u) wg_sort_list<1>(U.wg, L, p, v);
        return;
    }
    // (uniform per wavefront, which the compiler has to be told: then the rounds of a list are scalar branches)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t idx = nbig + (blockIdx.x - nbig) * (uint32_t)kSortWaves + (uint32_t)wave;
    if (idx >= ntiles) return;
    const uint32_t tile = tile_order[idx];
    const uint32_t s = ranges[2 * tile], e = min(ranges[2 * tile + 1], cap);
    if (e <= s) return;
    // (a list of long_list_from() entries or more cannot come here: k_tile_lists counted it among the first nbig)
    WaveSortLds& W = U.wave[wave];
    const uint32_t L = e - s;
    uint2* const p = pairs + s;
    uint32_t* const v = vals + s;
    if (L <= 64u) wave_count_list(L, p, v);
    else if (L <= 128u) wave_sort_list<2>(W, L, p, v);
    else if (L <= 192u) wave_sort_list<3>(W, L, p, v);
    else if (L <= 256u) wave_sort_list<4>(W, L, p, v);
    else if (L <= 384u) wave_sort_list<6>(W, L, p, v);
    else if (L <= 512u) wave_sort_list<8>(W, L, p, v);
    else if (L <= (uint32_t)kWaveListMax) wave_sort_list<kWaveListMax / 64>(W, L, p, v);
}

hipError_t launch_tile_depth_sort(const CamDev& cam, const Layout& L, char* ws, hipStream_t s)
{
    const auto u32 = [&](size_t off) { return reinterpret_cast<uint32_t*>(ws + off); };
    const uint32_t ntiles = (uint32_t)(cam.TX * cam.TY);
    ProfScope prof(kKTileDepthSort, s);
    // a list of the workgroup kind has at least long_list_from() entries, which bounds how many of them `cap` pairs can
    // hold, and so how many workgroups can have work: the rest would only start and leave, which is not free on an
    // image of 32,400 tiles
    const uint32_t big_max = min(ntiles, L.cap / long_list_from(ntiles) + 1u);
    const uint32_t items_max = min(ntiles, big_max + (ntiles + kSortWaves - 1u) / kSortWaves);
    hipLaunchKernelGGL(k_tile_depth_sort, dim3(items_max), dim3(kSortThreads), 0, s, u32(L.off_ranges), u32(L.off_tile_order), ntiles, u32(L.off_status),
                       L.cap, reinterpret_cast<uint2*>(ws + L.off_pairs), u32(L.off_vals), reinterpret_cast<uint2*>(ws + L.off_spare));
    return hipGetLastError();
}

}  // namespace pbdr
