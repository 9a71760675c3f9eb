// Per-tile compositing, forward and backward (image_render and image_render.backward: paper Sec. 2.1 "computes the
// color of each pixel front to back, blending the overlapping splats until full opacity is reached"; Alg. 1
// lines 12 and 18).
//
// One workgroup (4 wavefronts of 64) per 16x16 tile; each wavefront owns one 8x8 pixel quadrant, each row of 16 lanes one
// 4x4 cell of it. The forward kernel works out once per (tile, splat) which of the tile's sixteen cells the splat can reach
// with alpha >= 1/255 (conservatively) and leaves them, 16 bits per list position, for the backward pass. A wavefront then
// takes the splats that reach its quadrant 64 at a time and makes a list for each of its four cells, and a visit is one
// entry of each: four splats at once, on 16 pixels each. Against one splat per visit on the whole quadrant that is 24 % fewer
// visits at 1M points, 1920x1080 (2.91 -> 2.22 M; a third fewer on small splats). The cull never changes a result: every
// visited (pixel, splat) pair still takes the full per-pixel tests.
//
// The per-pair arithmetic is branch-free and in the log2 domain: alpha = min(0.99, 2^e) with e = log2 o - q(d) and
// q = log2(e) * sigma folded into the conic of the raster record. Plain VALU work: no dense contraction, so no MFMA.
#include "composite_common.h"
#include "pair_reduce.h"

#include <type_traits>

namespace pbdr {

// e = log2(o) - q(dx, dy), the same roundings wherever it is evaluated: the backward pass has to find the same pairs blended
// that the forward pass blended, whichever variant of a walk either takes.
__device__ __forceinline__ float log2_alpha(float A, float B, float C, float L, float dx, float dy)
{
    return fmaf(-(C * dy), dy, fmaf(-fmaf(B, dy, A * dx), dx, L));
}

// q(dx, dy) >= 0, the rule's "sigma < 0: skip", for splats whose conic is not safely definite. On q itself: e <= L would let
// a form below zero by less than half a last place of L through, and stop a splat whose opacity is NaN, which blends with
// the alpha of the clamp.
__device__ __forceinline__ bool form_not_negative(float A, float B, float C, float dx, float dy)
{
    return fmaf(C * dy, dy, fmaf(B, dy, A * dx) * dx) >= 0.f;
}

// A staged splat of the forward kernel: 48 bytes, so that one LDS address register serves the three reads of a visit.
struct StageRec {
    float4 a, b;                           // mx, my, A, B; C, L, red, green
    float c;                               // blue
    uint32_t pos;                          // place in the tile's list, from one
    uint32_t kind;                         // kSplatPlain, kSplatDefinite or 0
    uint32_t pad;
};

// Which of the eight 4x4-pixel cells, two rows of four, whose first pixel centre lies at (lx, ly) from the splat's centre can
// the splat reach with alpha >= 1/255? Bit 4 r + c for row r and column c. e: the ellipse of splat_ellipse(). Per row of
// cells the ellipse's extent in x over the row's pixel rows: its right end x(y) = sqrt(K - D y^2) - B y (in units of four
// pixels) is concave in y, so the largest x lies at the y of the ellipse's rightmost point, moved to the nearest y of the
// row; the left end likewise. A row outside the ellipse is not reached: the square root of a negative number is NaN,
// which ends as an empty set of columns.
__device__ __forceinline__ uint32_t reached_cells(const float4& e, float lx, float ly)
{
    const float u0 = 1.f - 0.25f * lx, v0 = 4.75f + 0.25f * lx;
    uint32_t cells = 0u;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const float lo = ly + (float)(4 * r), hi = lo + 3.f;
        const float yr = __builtin_amdgcn_fmed3f(-e.z, lo, hi), yl = __builtin_amdgcn_fmed3f(e.z, lo, hi);
        const float u = __builtin_amdgcn_sqrtf(e.x - e.y * yr * yr) + (u0 - e.w * yr);       // columns c with 4 c <= xr - lx:  c < u
        const float v = __builtin_amdgcn_sqrtf(e.x - e.y * yl * yl) + (v0 + e.w * yl);       // columns c with 4 c + 3 >= xl - lx:  c >= 4 - v
        const int below = 1 << (int)__builtin_amdgcn_fmed3f(u, 0.f, 4.f), from = 16 >> (int)__builtin_amdgcn_fmed3f(v, 0.f, 4.f);
        cells |= (uint32_t)max(below - from, 0) << (4 * r);
    }
    return cells;
}

// The walks of both kernels come in three kinds, chosen per window or batch (uniform): without the clamp and the sign test,
// neither of which can fire where every conic is safely definite and every opacity at most 0.98; with the clamp alone; and with
// both, for the other states a caller may hand in. All are unrolled and ask for records ahead alike: one splat above 0.98 is
// in a quarter of the batches of an untrained scene and in nearly all of a fitted one. Forward / backward call in us, 1M
// points (clusters), 1920x1080, by share of points with opacity 0.9975, this against two kinds of which the second had all
// tests, one visit at a time: none 183.4 / 247.1 against 183.0 / 245.8, 5 % 184.6 / 251.6 (187.0 / 266.4), 50 % 181.7 / 241.5
// (185.5 / 257.2); 200k points, 1280x720, 5 %: 123.1 / 120.7 (127.4 / 141.8). The clamp in every definite walk instead of a
// kind without it: 185.1 / 250.3 where no opacity is above 0.98.
constexpr int kWalkPlain = 0, kWalkClamped = 1, kWalkGeneral = 2;
template <int kKind>
using WalkKind = std::integral_constant<int, kKind>;

// Forward. The workgroup stages the records of 256 list positions at a time, one per thread, and finds their cells; most lists are
// not much longer. Then the wavefronts go on by themselves: each compacts the positions that reach its quadrant, takes them 64 at
// a time and writes the lists of its cells, LDS offsets of 16 bits; the entries behind a list's end name a record that reaches
// nothing. (Each wavefront fetching the records of its own windows, twice as many in all and a round trip to memory per window:
// 1M points 75.4 us instead of 71.5, 200k 42.3 instead of 40.3, 4,096 20.0 instead of 18.4.) A walk reads two entries per cell and trip: their alphas do not
// depend on each other, which gives the vector ALU two independent chains; the blends stay in list order.
// Against one splat a visit on the whole quadrant: the benchmark's view (1M points, 1920x1080, bench.py) 103.8 -> 88.9 us,
// 77 -> 64 M vector instructions, its 4K street view (8M points) 326 -> 235; clusters and boxes as perf/cases.py draws them,
// 1M points at 1920x1080 88.6 -> 74.7, 200k at 1280x720 51.0 -> 39.9, 30k at 1031x517 21.9 -> 19.0, 4096 at 128x128
// 28.1 -> 20.0 (the launch lasts as long as its longest list).
// (Measured and dropped, where this one took 87 us at 1M points and 25 at 30k: a wavefront per 8x8 quadrant or per 16x8 half
// tile with two pixels a lane, each finding its own cells: 102 and 91, and 27.6 and 39 at 30k points, where the chip is not
// full; 512 positions at a time: 90, five workgroups fit instead of eight.)
constexpr int kFwdChunk = 256;                   // list positions whose cells are worked out at a time

__global__ __launch_bounds__(256) void k_composite_fwd(CamDev cam, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
                                                       const uint32_t* __restrict__ vals, const Packed* __restrict__ packed,
                                                       uint16_t* __restrict__ cells, float bg0, float bg1, float bg2,
                                                       float* __restrict__ image, float* __restrict__ final_T,
                                                       uint32_t* __restrict__ last_idx)
{
    constexpr int kGroups = 4, kPosBits = 12;
    static_assert(kFwdChunk <= 1 << kPosBits && kFwdChunk % 256 == 0, "a position and four cells in 16 bits");
    __shared__ StageRec sRec[kFwdChunk + 1];                   // the last one reaches nothing
    __shared__ uint16_t sHits[4][kFwdChunk];                   // position in the chunk | the quadrant's cells << kPosBits
    __shared__ __align__(8) uint16_t sList[4][kGroups * 64 + 4];
    __shared__ uint16_t sCells[kFwdChunk];
    const int tile = (int)tile_order[blockIdx.x];
    const int tiy = tile / cam.TX, tix = tile - tiy * cam.TX;
    const int tx0 = (cam.otx + tix) * kTile, ty0 = (cam.oty + tiy) * kTile;
    const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = lane >> 4;
    const int px = tx0 + (wave & 1) * 8 + (group & 1) * 4 + (lane & 3), py = ty0 + (wave >> 1) * 8 + (group >> 1) * 4 + ((lane >> 2) & 3);
    const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
    const bool inside = px >= cam.rx0 && px < cam.rx1 && py >= cam.ry0 && py < cam.ry1;
    uint16_t* const list_w = sList[wave];
    uint16_t* const hits_w = sHits[wave];
    constexpr uint32_t kNoRec = (uint32_t)(kFwdChunk * sizeof(StageRec));
    static_assert(kNoRec < 65536u, "offsets of 16 bits");
    if (threadIdx.x == 0) {
        sRec[kFwdChunk].a = make_float4(0.f, 0.f, 0.f, 0.f);
        sRec[kFwdChunk].b = make_float4(0.f, -1e30f, 0.f, 0.f);
        sRec[kFwdChunk].c = 0.f;
    }
    static_assert(kFwdChunk == 256, "a position per thread");
    uint32_t id = start + threadIdx.x < end ? vals[start + threadIdx.x] : 0u;      // of this thread's position in the next chunk
    const auto rec_at = [&](uint32_t off) { return reinterpret_cast<const StageRec*>(reinterpret_cast<const char*>(sRec) + off); };
    float T = 1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
    uint32_t last = 0u;
    unsigned long long live = __ballot(inside);
    for (uint32_t base = start; base < end; base += kFwdChunk) {
        if (base != start && __syncthreads_or(live != 0ull) == 0) break;
        const int cnt = (int)min((uint32_t)kFwdChunk, end - base);
        const int j = threadIdx.x;
        uint32_t word = 0u;
        if (j < cnt) {
            const float4* rec = reinterpret_cast<const float4*>(packed + id);
            const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2], ellipse = rec[3];
            id = base + kFwdChunk + j < end ? vals[base + kFwdChunk + j] : 0u;
            sRec[j].a = r0; sRec[j].b = r1;
            *reinterpret_cast<float4*>(&sRec[j].c) = make_float4(r2.x, __uint_as_float(base - start + j + 1u), r2.w, 0.f);
            const float lx = (float)tx0 + 0.5f - r0.x, ly = (float)ty0 + 0.5f - r0.y;
            word = by_quadrant(reached_cells(ellipse, lx, ly)) | (by_quadrant(reached_cells(ellipse, lx, ly + 8.f)) << 8);
            cells[base + j] = (uint16_t)word;
        }
        sCells[j] = (uint16_t)word;
        __syncthreads();
        int nhit = 0;
#pragma unroll
        for (int r = 0; r < kFwdChunk; r += 64) {      // (positions past the end have no cells)
            const uint32_t m = ((uint32_t)sCells[r + lane] >> (4 * wave)) & 15u;
            const unsigned long long b = __ballot(m != 0u);
            if (m) hits_w[nhit + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = (uint16_t)((uint32_t)(r + lane) | (m << kPosBits));
            nhit += __builtin_popcountll(b);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        for (int w0 = 0; w0 < nhit; w0 += 64) {
            if (live == 0ull) break;
            uint32_t m = 0u, kind = kSplatPlain, mine = 0u;
            constexpr uint32_t kNone = kNoRec * 0x10001u;
            *reinterpret_cast<uint2*>(list_w + 4 * lane) = make_uint2(kNone, kNone);
            if (w0 + lane < nhit) {
                const uint32_t h = hits_w[w0 + lane];
                m = h >> kPosBits;
                mine = (h & ((1u << kPosBits) - 1u)) * (uint32_t)sizeof(StageRec);
                kind = rec_at(mine)->kind;
            }
            const bool all_definite = __ballot((kind & kSplatDefinite) == 0u) == 0ull, all_plain = __ballot(kind != kSplatPlain) == 0ull;
            int n = 0;
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                const bool on = (m & (1u << g)) != 0u && ((live >> (16 * g)) & 0xffffull) != 0ull;
                const unsigned long long b = __ballot(on);
                if (on) list_w[g * 64 + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = (uint16_t)mine;
                n = max(n, (int)__builtin_popcountll(b));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            uint32_t last_off = ~0u;
            const uint16_t* const my_list = list_w + group * 64;
            auto walk = [&](auto kind) {
                constexpr bool kClamp = decltype(kind)::value >= kWalkClamped, kSign = decltype(kind)::value >= kWalkGeneral;
                struct Visit { float alpha, r, g, b; bool ok; };
                auto eval = [&](uint32_t off, Visit& v) {
                    const StageRec* rec = rec_at(off);
                    const float4 a = rec->a, b = rec->b;
                    v.b = rec->c; v.r = b.z; v.g = b.w;
                    const float dx = fx - a.x, dy = fy - a.y;
                    const float e = log2_alpha(a.z, a.w, b.x, b.y, dx, dy);
                    const float raw = __builtin_amdgcn_exp2f(e);
                    v.alpha = kClamp ? fminf(kAlphaMax, raw) : raw;
                    v.ok = (!kSign || form_not_negative(a.z, a.w, b.x, dx, dy)) && v.alpha >= kAlphaMin;
                };
                auto blend = [&](uint32_t off, const Visit& v) {
                    const float aT = v.alpha * T;
                    const float Tn = T - aT;            // T (1 - alpha), with the product the weight needs anyway
                    const bool bl = blend_decision(live, v.ok, Tn);
                    const float w = bl ? aT : 0.f;
                    C0 += v.r * w; C1 += v.g * w; C2 += v.b * w;
                    T = bl ? Tn : T;
                    last_off = bl ? off : last_off;
                };
                uint32_t next = *reinterpret_cast<const uint32_t*>(my_list);
                for (int i = 0; i < n; i += 2) {
                    const uint32_t o0 = next & 0xffffu, o1 = next >> 16;
                    next = *reinterpret_cast<const uint32_t*>(my_list + i + 2);      // (behind the last one: padding or the next list, not used)
                    asm volatile("" ::: "memory");                                   // asked for here, a trip ahead
                    Visit v0, v1;
                    eval(o0, v0);
                    eval(o1, v1);
                    blend(o0, v0);
                    blend(o1, v1);
                }
            };
            if (all_plain) walk(WalkKind<kWalkPlain>{});
            else if (all_definite) walk(WalkKind<kWalkClamped>{});
            else walk(WalkKind<kWalkGeneral>{});
            if (last_off != ~0u) last = rec_at(last_off)->pos;
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            __builtin_amdgcn_wave_barrier();             // the next window overwrites the lists
        }
    }
    if (inside) {
        const size_t HW = (size_t)cam.W * cam.H;
        const size_t pix = (size_t)(py - cam.ry0) * (size_t)cam.W + (size_t)(px - cam.rx0);
        image[pix] = C0 + T * bg0;
        image[HW + pix] = C1 + T * bg1;
        image[2 * HW + pix] = C2 + T * bg2;
        final_T[pix] = T;
        last_idx[pix] = last;
    }
}

// Backward. Per pixel, back to front from its last blended splat: T_k = T_{k+1} / (1 - alpha_k),
//   dL/dalpha_k = T_k (c_k . g) - S_k / (1 - alpha_k),  S_k = sum_{i>k} w_i (c_i . g) + T_final (bg . g).
// With ds = dL/dsigma = -alpha dL/dalpha (zero where alpha was clamped), every splat gradient is a sum over pixels of
//   w g_c (3 colours)  and the six moments  ds (1, dx, dy, dx^2, dx dy, dy^2):
//   d conic = (S3/2, S4, S5/2), d mean2d = -(qa S1 + qb S2, qc S2 + qb S1), d opacity = -S0 / o.
//
// The list is searched 256 positions at a time for the splats that reach the tile (a third of them do not); these are
// taken in batches of 64, last splats first, whose records go straight from memory into LDS: a wavefront asks for the next
// batch's before it walks the current one, so the trip hides behind the walk and takes no registers. Each wavefront makes
// the lists of its quadrant's four cells and visits one entry of each at a time, as in the forward kernel.
//
// The sums over pixels are taken four visits at a time. A visit only stores its ds and w as two rows of 64 floats in
// LDS (a transpose: the values of one visit sit across the lanes, the sums want the pixels of one visit inside a lane).
// After four visits a row of 16 lanes takes each visit and a quad of lanes each cell: a lane reads ds and w of four
// neighbouring pixels, a row of the cell, and forms their nine weighted sums with weights it holds for the whole tile (the
// pixels' dL/dcolour and their coordinates X, Y about the tile's middle: with dx = X0 + X, dy = Y0 + Y for a per-(tile, splat)
// offset (X0, Y0), the six moments follow from the moments of ds against 1, X, Y, X^2, XY, Y^2, whatever the splat); two
// exchanges inside the quad finish the sums of sixteen (splat, cell) pairs at once.
// The four cells of a visit hold different splats, and two of them may come to the same splat at any distance, so their
// sums cannot be added into a splat's accumulator right away (taking turns cell by cell, read, add, write: 24 LDS
// instructions per four visits, 221 us). They are kept by visit and cell, 24 visits long; then lane j, which stands for
// splat j of the batch and knows its places in the four lists, fetches and adds its up to four entries.
// Batches whose conics are all safely definite, on pixels whose gradients are finite, take a walk in which a lane that does not
// blend has alpha = 0 and needs no other select: 1 / (1 - alpha) = 1, and all of its products are zero.
//
// No atomics, global or LDS: each wavefront leaves its quadrant's sums by splat in LDS, and the lanes of one of them (in
// turn from batch to batch) add the four quadrants' nine sums, turn them into gradients and write them
// to partial[u] (12 floats per pair), where u is the pair's position in the unsorted duplicate list (slot_base[id] +
// rank of this tile in the splat's rectangle). A splat's pairs are contiguous there, so a per-splat kernel adds them
// up afterwards (k_gather_splat_grads).
//
// Against one splat a visit on the whole quadrant: the benchmark's view (1M points, 1920x1080, bench.py) 213 -> 182 us,
// 143 -> 112 M vector instructions, its 4K street view 597 -> 427; clusters and boxes as perf/cases.py draws them, 1M points at
// 1920x1080 182 -> 156, 200k at 1280x720 106 -> 72, 30k at 1031x517 48 -> 33, 4096 at 128x128 65 -> 38. What is left is bound
// by latency as much as by issue (five workgroups per compute unit by registers and LDS). Records asked for two visits ahead
// are 2 to 6 % of that. States that no preprocessing makes lost by it: with a tenth of all conics indefinite (a list then holds
// the splat for every cell, and a visit that no lane blends is reduced like any other) 289 against 276 us at 1M points for the
// whole backward call, with all of them 449 against 321; at 200k points and below up to a third they are faster too.
// (Measured and dropped, where this one took 185 us at 1M points: four workgroups with runs of 32 visits: 203; six with 16: 212, the
// registers spill; one wavefront per tile that takes the four quadrants in turn: the few tiles with thousands of splats then
// run four times longer. The contraction on fp32 matrix instructions: these hold the SIMD for their 32 cycles, plain vector
// instructions of other wavefronts do not overlap with them, and most of their output columns are of no use here.)
constexpr int kVisitSlots = 4;     // visits staged per reduction: one per row of 16 lanes
constexpr int kBwdBatch = 64;      // splats taken at a time: one per lane
constexpr int kBwdVisits = 24;     // visits whose sums a wavefront keeps before it adds them up by splat (a multiple of kVisitSlots)
constexpr int kVisitFloats = 36;   // a visit's sums: eight of each cell, then the ninth of each cell
constexpr int kBwdChunk = 256;     // list positions that are searched for splats that reach the tile at a time

// 5 workgroups per compute unit: 96 registers, 32 KB of LDS
__global__ __launch_bounds__(256, 5) void k_composite_bwd(CamDev cam, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
                                                       const uint32_t* __restrict__ vals, const Packed* __restrict__ packed,
                                                       const uint16_t* __restrict__ cells, const uint32_t* __restrict__ slot_base,
                                                       float bg0, float bg1, float bg2, const float* __restrict__ final_T,
                                                       const uint32_t* __restrict__ last_idx,
                                                       const float* __restrict__ dL_dimage, uint32_t cap,
                                                       const uint32_t* __restrict__ status, float4* __restrict__ partial)
{
    constexpr int kStride = kBwdBatch + 1;                         // the last record of each part reaches nothing
    __shared__ float4 sRec[2][3 * kStride];                        // two batches of raster records, in three parts of 16 bytes
    // per wavefront: the nine sums of every visit and cell of the current run of visits, [visit][cell][value]; then, at the end
    // of a batch, the wavefront's sums by splat, [splat][value]
    __shared__ __align__(16) float sSum[4][kBwdVisits * kVisitFloats];
    __shared__ __align__(16) float sV[4][2 * kVisitSlots * 64];   // per wavefront: rows 2s (ds) and 2s + 1 (w) of visit slot s
    __shared__ __align__(8) uint16_t sList[4][4 * kBwdBatch];
    __shared__ uint32_t sId[kBwdChunk];
    __shared__ uint16_t sCell[kBwdChunk];
    __shared__ unsigned long long sReach[kBwdChunk / 64];
    __shared__ uint32_t sMax[4];
    static_assert(kBwdVisits * kVisitFloats >= 9 * kBwdBatch && kBwdVisits % kVisitSlots == 0, "the sums by splat fit where the sums by visit were");
    const int tile = (int)tile_order[blockIdx.x];
    const int tile_y = tile / cam.TX, tile_x = tile - tile_y * cam.TX;
    const int tx0 = (cam.otx + tile_x) * kTile, ty0 = (cam.oty + tile_y) * kTile;
    const uint32_t start = ranges[2 * tile], end = ranges[2 * tile + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = lane >> 4;
    const int px = tx0 + (wave & 1) * 8 + (group & 1) * 4 + (lane & 3), py = ty0 + (wave >> 1) * 8 + (group >> 1) * 4 + ((lane >> 2) & 3);
    const bool inside = px >= cam.rx0 && px < cam.rx1 && py >= cam.ry0 && py < cam.ry1;
    const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
    const size_t HW = (size_t)cam.W * cam.H;
    // this call, counted from one (uniform values, kept on the scalar side)
    const uint32_t epoch_lo = __builtin_amdgcn_readfirstlane(status[kStEpoch]) + 1u;
    const uint32_t epoch_hi = __builtin_amdgcn_readfirstlane(status[kStEpoch + 1]) + (epoch_lo == 0u ? 1u : 0u);
    float T = 1.f, g0 = 0.f, g1 = 0.f, g2c = 0.f;
    uint32_t last = 0;
    if (inside) {
        const uint32_t pix = (uint32_t)(py - cam.ry0) * (uint32_t)cam.W + (uint32_t)(px - cam.rx0);
        T = final_T[pix];
        last = min(last_idx[pix], end - start);   // never walk past the tile's list, whatever the caller passed
        g0 = dL_dimage[pix]; g1 = dL_dimage[HW + pix]; g2c = dL_dimage[2 * HW + pix];
    }
    float Sfx = T * (bg0 * g0 + bg1 * g1 + bg2 * g2c);
    uint32_t wmax = last;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) wmax = max(wmax, (uint32_t)__shfl_xor((int)wmax, d, 64));
    wmax = __builtin_amdgcn_readfirstlane(wmax);
    if (lane == 0) sMax[wave] = wmax;
    if (threadIdx.x < 2) {
        sRec[threadIdx.x][kBwdBatch] = make_float4(0.f, 0.f, 0.f, 0.f);
        sRec[threadIdx.x][kStride + kBwdBatch] = make_float4(0.f, -1e30f, 0.f, 0.f);
        sRec[threadIdx.x][2 * kStride + kBwdBatch] = make_float4(0.f, 0.f, 0.f, __uint_as_float(kSplatPlain));
    }
    __syncthreads();
    const uint32_t tile_last = __builtin_amdgcn_readfirstlane(max(max(sMax[0], sMax[1]), max(sMax[2], sMax[3])));
    if (tile_last == 0) return;
    float* const sVw = sV[wave];
    float* const sSumW = sSum[wave];
    uint16_t* const list_w = sList[wave];
    // In a reduction lane l takes visit slot l / 16 and the four pixels held by the wavefront's lanes 4 pg .. 4 pg + 3,
    // pg = l % 16: a row of a 4x4 cell. Their dL/dcolour come from those lanes, through LDS.
    const int pg = lane & 15, cell = pg >> 2, quad_lane = lane & 3;
    float4 G0, G1, G2;
    {
        sVw[lane] = g0; sVw[64 + lane] = g1; sVw[128 + lane] = g2c;
        __builtin_amdgcn_wave_barrier();
        G0 = *reinterpret_cast<const float4*>(sVw + 4 * pg);
        G1 = *reinterpret_cast<const float4*>(sVw + 64 + 4 * pg);
        G2 = *reinterpret_cast<const float4*>(sVw + 128 + 4 * pg);
        __builtin_amdgcn_wave_barrier();
    }
    // coordinates of the first of the four pixels about the tile's pixel (8, 8), which keeps the moments and so their rounding
    // small; the others are X + 1, X + 2, X + 3 on the same row
    const float PX = (float)((wave & 1) * 8 + (cell & 1) * 4 - 8), PY = (float)((wave >> 1) * 8 + (cell >> 1) * 4 + quad_lane - 8);
    const float* const rd_row = sVw + 128 * (lane >> 4) + 4 * pg;
    float* const wr_row = sVw + lane;
    float* const wr_sum = sSumW + kVisitFloats * (lane >> 4) + 8 * cell + 2 * quad_lane;
    float* const wr_ninth = sSumW + kVisitFloats * (lane >> 4) + 32 + cell;
    // the gradient of every pixel finite: then the products of a lane that a visit does not blend are zero without a select
    const bool finite_pixels = __ballot(!(fabsf(g0) + fabsf(g1) + fabsf(g2c) + fabsf(Sfx) < 1e15f)) == 0ull;
    // Reduces the staged rows: the sums of slot s go to place i + s of the run. finite: the gradient of every pixel is; else a
    // pixel that did not blend the splat (w = 0) is left out of the colour sums, so that a NaN or an infinity at one pixel
    // reaches the splats which that pixel blended and no other (a cell's list holds every splat that comes near).
    auto reduce_slots = [&](auto finite, int i) {
        const auto term = [](float wk, float g) { return !decltype(finite)::value && wk == 0.f ? 0.f : wk * g; };
        __builtin_amdgcn_wave_barrier();
        const float4 d = *reinterpret_cast<const float4*>(rd_row);
        const float4 w = *reinterpret_cast<const float4*>(rd_row + 64);
        __builtin_amdgcn_wave_barrier();
        const float m0 = (d.x + d.y) + (d.z + d.w);
        const float s1 = d.y + 2.f * d.z + 3.f * d.w;             // sum of ds i and of ds i^2 over the pixels X + i
        const float s2 = d.y + 4.f * d.z + 9.f * d.w;
        const float mx = PX * m0 + s1;
        const float mxx = PX * (mx + s1) + s2;                    // sum of ds (PX + i)^2 = PX (PX m0 + 2 s1) + s2
        const float my = PY * m0;
        const float v8[8] = {term(w.x, G0.x) + term(w.y, G0.y) + term(w.z, G0.z) + term(w.w, G0.w),
                             term(w.x, G1.x) + term(w.y, G1.y) + term(w.z, G1.z) + term(w.w, G1.w),
                             term(w.x, G2.x) + term(w.y, G2.y) + term(w.z, G2.z) + term(w.w, G2.w),
                             m0, mx, my, mxx, PY * mx};
        float2 part;
        quad_sum8(v8, quad_lane, part);
        const float ninth = quad_sum(PY * my);
        *reinterpret_cast<float2*>(wr_sum + kVisitFloats * i) = part;
        wr_ninth[kVisitFloats * i] = ninth;
    };
    for (int chunk = (int)((tile_last - 1u) / kBwdChunk); chunk >= 0; --chunk) {
        const uint32_t coff = (uint32_t)chunk * kBwdChunk;         // 0-based list position of the chunk's first splat
        // the chunk's splats that reach the tile, in list order
        uint32_t word[kBwdChunk / 256], id[kBwdChunk / 256];
#pragma unroll
        for (int k = 0; k < kBwdChunk / 256; ++k) {
            const uint32_t p = coff + k * 256u + threadIdx.x;
            word[k] = p < tile_last ? (uint32_t)cells[start + p] : 0u;
            id[k] = p < tile_last ? vals[start + p] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kBwdChunk / 256; ++k) {
            const unsigned long long b = __ballot(word[k] != 0u);
            if (lane == 0) sReach[4 * k + wave] = b;
        }
        __syncthreads();
        int total = 0, rank_last = 0;
        {
            const int lc = (int)min(last, coff + kBwdChunk) - (int)coff;     // positions of the chunk the pixel went through
            int before[kBwdChunk / 256];
#pragma unroll
            for (int j = 0; j < kBwdChunk / 64; ++j) {
                const unsigned long long b = sReach[j];
#pragma unroll
                for (int k = 0; k < kBwdChunk / 256; ++k) if (j == 4 * k + wave) before[k] = total;
                const int in = lc - 64 * j;                        // how many of these 64
                const unsigned long long upto = in >= 64 ? ~0ull : in <= 0 ? 0ull : (1ull << in) - 1ull;
                rank_last += __builtin_popcountll(b & upto);
                total += __builtin_popcountll(b);
            }
#pragma unroll
            for (int k = 0; k < kBwdChunk / 256; ++k) {
                const unsigned long long b = sReach[4 * k + wave];
                if (word[k] != 0u) {
                    const int at = before[k] + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                    sId[at] = id[k];
                    sCell[at] = (uint16_t)word[k];
                }
            }
            total = __builtin_amdgcn_readfirstlane(total);
        }
        __syncthreads();
        const int nbatch = (total + kBwdBatch - 1) / kBwdBatch;
        // asks for a batch's records, straight into LDS
        auto fetch = [&](int bi) {
            if (lane < min(kBwdBatch, total - bi * kBwdBatch)) {
                const float4* rec = reinterpret_cast<const float4*>(packed + sId[bi * kBwdBatch + lane]);
                float4* dst = sRec[bi & 1];
#pragma unroll
                for (int k = 0; k < 3; ++k) load_to_lds16(rec + k, dst + k * kStride);
            }
        };
        if (nbatch > 0 && wave == ((nbatch - 1) & 3)) fetch(nbatch - 1);
        for (int bi = nbatch - 1; bi >= 0; --bi) {
            const int boff = bi * kBwdBatch;
            const int cnt = min(kBwdBatch, total - boff);
            wait_loads();       // the records this wavefront asked for are there
            __syncthreads();                                       // (and the last batch's sums have been read)
            const bool writer = wave == (bi & 3);
            uint32_t pair_base = 0u;
            if (writer && lane < cnt) pair_base = slot_base[sId[boff + lane]];      // asked for now, used when the batch's records are written
            asm volatile("" ::: "memory");
            if (bi > 0 && wave == ((bi - 1) & 3)) fetch(bi - 1);
            const float4* const rec_b = sRec[bi & 1];
            float4 acc0 = make_float4(0.f, 0.f, 0.f, 0.f), acc1 = acc0;
            float acc8 = 0.f;
            const uint32_t m = lane < cnt ? ((uint32_t)sCell[boff + lane] >> (4 * wave)) & 15u : 0u;
            if (__ballot(rank_last > boff) != 0ull) {              // else nothing of this batch was blended by this wavefront
                constexpr uint32_t kNone = (uint32_t)kBwdBatch * 16u * 0x10001u;
                *reinterpret_cast<uint2*>(list_w + 4 * lane) = make_uint2(kNone, kNone);
                const float4 kind = rec_b[2 * kStride + min(lane, cnt - 1)];
                const float4 col = rec_b[kStride + min(lane, cnt - 1)];
                const uint32_t kind_bits = __float_as_uint(kind.w);
                const bool all_plain = __ballot(kind_bits != kSplatPlain) == 0ull;
                const bool all_sound = __ballot(!((kind_bits & kSplatDefinite) != 0u && fabsf(kind.x) + fabsf(col.z) + fabsf(col.w) < 1e15f)) == 0ull && finite_pixels;
                int n = 0;
                int place[4];             // of this lane's splat in the lists, the last splat first
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const unsigned long long b = __ballot((m & (1u << g)) != 0u);
                    const int c = __builtin_popcountll(b);
                    place[g] = c - 1 - (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                    if (m & (1u << g)) list_w[g * kBwdBatch + place[g]] = (uint16_t)(lane * 16);
                    else place[g] = 255;
                    n = max(n, c);
                }
                const uint32_t places = (uint32_t)place[0] | ((uint32_t)place[1] << 8) | ((uint32_t)place[2] << 16) | ((uint32_t)place[3] << 24);
                const int last_off = (rank_last - boff - 1) * 16;     // of the last splat of the batch that the pixel came to
                const uint16_t* const my_list = list_w + group * kBwdBatch;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                for (int first = 0; first < n; first += kBwdVisits) {
                    const int count = min(kBwdVisits, n - first);
                    struct Rec { uint32_t off; float4 a, b; float blue; };
                    auto read = [&](uint32_t off) {
                        const char* rec = reinterpret_cast<const char*>(rec_b) + off;
                        return Rec{off, *reinterpret_cast<const float4*>(rec), *reinterpret_cast<const float4*>(rec + 16 * kStride),
                                   *reinterpret_cast<const float*>(rec + 32 * kStride)};
                    };
                    auto visit = [&](auto kind, const Rec& r, float* rows) {
                        constexpr bool kClamp = decltype(kind)::value >= kWalkClamped, kGeneral = decltype(kind)::value >= kWalkGeneral;
                        const float4 a = r.a, b = r.b;
                        const float cb = r.blue;
                        const uint32_t off = r.off;
                        const float dx = fx - a.x, dy = fy - a.y;
                        const float e = log2_alpha(a.z, a.w, b.x, b.y, dx, dy);
                        const float raw = __builtin_amdgcn_exp2f(e);
                        const float al = kClamp ? fminf(kAlphaMax, raw) : raw;
                        const bool hit = ((int)off <= last_off) && (!kGeneral || form_not_negative(a.z, a.w, b.x, dx, dy)) && (al >= kAlphaMin);
                        const float alpha = hit ? al : 0.f;
                        const float ioma = __builtin_amdgcn_rcpf(1.f - alpha);
                        const float Tk = T * ioma;                              // transmittance in front of this splat
                        const float w = !kGeneral || hit ? alpha * Tk : 0.f;
                        const float cg = b.z * g0 + b.w * g1 + cb * g2c;
                        const float dL_dalpha = Tk * cg - Sfx * ioma;
                        float ds = -alpha * dL_dalpha;
                        if (kClamp) ds = ((!kGeneral || hit) && raw < kAlphaMax) ? ds : 0.f;      // zero where alpha was clamped
                        T = !kGeneral || hit ? Tk : T;
                        if (!kGeneral || hit) Sfx += w * cg;
                        rows[0] = ds;
                        rows[64] = w;
                    };
                    const uint16_t* const run = my_list + first;
                    auto walk = [&](auto kind) {
                        auto reduce = [&](int i) {
                            if (decltype(kind)::value < kWalkGeneral || finite_pixels) reduce_slots(std::true_type{}, i);
                            else reduce_slots(std::false_type{}, i);
                        };
                        int i = 0;
                        for (; i + kVisitSlots <= count; i += kVisitSlots) {
                            // a record is asked for two visits ahead (the empty statements keep the reads from sinking to their use)
                            const uint2 o = *reinterpret_cast<const uint2*>(run + i);
                            const Rec r0 = read(o.x & 0xffffu), r1 = read(o.x >> 16);
                            asm volatile("" ::: "memory");
                            visit(kind, r0, wr_row);
                            const Rec r2 = read(o.y & 0xffffu);
                            asm volatile("" ::: "memory");
                            visit(kind, r1, wr_row + 128);
                            const Rec r3 = read(o.y >> 16);
                            asm volatile("" ::: "memory");
                            visit(kind, r2, wr_row + 256);
                            visit(kind, r3, wr_row + 384);
                            reduce(i);
                        }
                        if (i < count) {      // (what the rows of the other slots hold goes to places that no splat has)
                            float* rows = wr_row;
                            if ((count - i) & 2) {
                                visit(kind, read(run[i]), rows);
                                visit(kind, read(run[i + 1]), rows + 128);
                                rows += 256;
                            }
                            if (count & 1) visit(kind, read(run[count - 1]), rows);
                            reduce(i);
                        }
                    };
                    if (all_plain && all_sound) walk(WalkKind<kWalkPlain>{});
                    else if (all_sound) walk(WalkKind<kWalkClamped>{});
                    else walk(WalkKind<kWalkGeneral>{});
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const uint32_t at = ((places >> (8 * g)) & 255u) - (uint32_t)first;
                        if (at < (uint32_t)kBwdVisits) {
                            const float* v = sSumW + kVisitFloats * at;
                            const float4 v0 = *reinterpret_cast<const float4*>(v + 8 * g), v1 = *reinterpret_cast<const float4*>(v + 8 * g + 4);
                            acc0.x += v0.x; acc0.y += v0.y; acc0.z += v0.z; acc0.w += v0.w;
                            acc1.x += v1.x; acc1.y += v1.y; acc1.z += v1.z; acc1.w += v1.w;
                            acc8 += v[32 + g];
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
            reinterpret_cast<float4*>(sSumW)[lane] = acc0;
            reinterpret_cast<float4*>(sSumW)[kBwdBatch + lane] = acc1;
            sSumW[8 * kBwdBatch + lane] = acc8;
            __syncthreads();
            if (writer && lane < cnt) {
                // where this (tile, splat) pair sits in the unsorted duplicate list
                const float4 ra = rec_b[lane], rb = rec_b[kStride + lane], rc = rec_b[2 * kStride + lane];
                int x0, y0, x1, y1;
                tile_rect(cam, ra.x, ra.y, __float_as_int(rc.y), x0, y0, x1, y1);
                const uint32_t u = pair_base + (uint32_t)((tile_y - y0) * (x1 - x0) + (tile_x - x0));
                if (u < cap && tile_x >= x0 && tile_x < x1 && tile_y >= y0 && tile_y < y1) {
                    float acc[9];
                    const auto over_quadrants = [&](int k) { return (sSum[0][k] + sSum[1][k]) + (sSum[2][k] + sSum[3][k]); };
#pragma unroll
                    for (int k = 0; k < 8; ++k) acc[k] = over_quadrants(4 * ((k & 4) * (kBwdBatch / 4) + lane) + (k & 3));
                    acc[8] = over_quadrants(8 * kBwdBatch + lane);
                    const float qa = 2.f * kLn2 * ra.z, qb = kLn2 * ra.w, qc = 2.f * kLn2 * rb.x, o = rc.z;
                    // from the tile's frame to offsets from the splat centre: dx = X0 + X, dy = Y0 + Y
                    const float X0 = (float)tx0 + 8.5f - ra.x, Y0 = (float)ty0 + 8.5f - ra.y;
                    const float m0 = acc[3], mx = acc[4], my = acc[5];
                    const float s0 = m0, s1 = X0 * m0 + mx, s2 = Y0 * m0 + my;
                    const float s3 = X0 * (X0 * m0 + 2.f * mx) + acc[6];
                    const float s4 = X0 * (Y0 * m0 + my) + Y0 * mx + acc[7];
                    const float s5 = Y0 * (Y0 * m0 + 2.f * my) + acc[8];
                    float4* dst = partial + (size_t)3 * u;
                    dst[0] = make_float4(-(qa * s1 + qb * s2), -(qc * s2 + qb * s1),                      // d mean2d
                                         0.5f * s3, s4);                                                  // d conic a, b
                    dst[1] = make_float4(0.5f * s5, o > 0.f ? -s0 / o : 0.f,                               // d conic c, d opacity
                                         acc[0], acc[1]);                                                 // d red, d green
                    // d blue, then the stamp that tells the gather this record belongs to this backward call
                    dst[2] = make_float4(acc[2], 0.f, __uint_as_float(epoch_lo), __uint_as_float(epoch_hi));
                }
            }
        }
        __syncthreads();   // the chunk's lists and sums are rewritten by the next chunk
    }
}

// Adds up, per point, the per-tile partial sums of its pairs (contiguous in the unsorted duplicate list, 48 bytes
// each) into dL/d(splat state) of the visible points; culled points are not written. Balanced by pairs: see
// pair_reduce.h.
// The sums are first stored as one 48-byte record per point, by point index (nine 4-byte stores per point into nine
// planes touch nine cache lines where this touches one),
// then a streaming kernel over all points copies the records of listed points into the planes of the splat-state
// gradient.
struct StoreSplatGrad {
    float4* rec;
    const uint32_t* order;
    __device__ __forceinline__ void operator()(uint32_t rank, const float (&v)[9]) const
    {
        float4* dst = rec + (size_t)3 * order[rank];
        dst[0] = make_float4(v[0], v[1], v[2], v[3]);
        dst[1] = make_float4(v[4], v[5], v[6], v[7]);
        dst[2] = make_float4(v[8], 0.f, 0.f, 0.f);
    }
};

__global__ __launch_bounds__(256) void k_gather_splat_grads(int n, const uint32_t* __restrict__ status,
                                                            const uint32_t* __restrict__ order,
                                                            const uint32_t* __restrict__ offsets,
                                                            const uint32_t* __restrict__ chunk_rank,
                                                            const float4* __restrict__ partial, uint32_t cap,
                                                            float* __restrict__ carry, float4* __restrict__ rec)
{
    __shared__ uint32_t sEnd[4][64];
    const uint32_t w = blockIdx.x * 4u + (threadIdx.x >> 6);
    gather_wave<3, 9, true>(w, n, status, offsets, chunk_rank, partial, cap, carry, sEnd[threadIdx.x >> 6], StoreSplatGrad{rec, order});
}

// records -> planes, for the points binning listed (tiles_touched > 0). A point whose pairs are cut by a boundary of the gather's
// chunks is put together here (record_from_carries), and the call's epoch is closed: a launch of its own for that took 5 us.
__global__ __launch_bounds__(256) void k_grad_records_to_planes(int n, const uint32_t* __restrict__ tiles_touched,
                                                                const float4* __restrict__ rec, CarryFold cf, SplatGradDev g2)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i == 0) close_backward_epoch(cf.status);
    if (i >= n) return;
    const uint32_t pairs = tiles_touched[i];
    if (pairs == 0) return;
    const size_t N = (size_t)n;
    const float4 a = rec[(size_t)3 * i], b = rec[(size_t)3 * i + 1], c = rec[(size_t)3 * i + 2];
    float v[9] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x};
    (void)record_from_carries<9>(cf, cf.slot_base[i], pairs, v);
    g2.mean2d[i] = v[0]; g2.mean2d[N + i] = v[1];
    g2.conic[i] = v[2]; g2.conic[N + i] = v[3]; g2.conic[2 * N + i] = v[4];
    g2.opacity[i] = v[5];
    g2.color[i] = v[6]; g2.color[N + i] = v[7]; g2.color[2 * N + i] = v[8];
}

// Measurement aid: the forward walk with counters instead of colours. counters[0] += list entries examined per pixel
// (up to and including the one that ends the pixel), counters[1] += pairs blended.
__global__ __launch_bounds__(256) void k_render_stats(CamDev cam, const uint32_t* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
                                                      const uint32_t* __restrict__ vals, const Packed* __restrict__ packed,
                                                      unsigned long long* __restrict__ counters)
{
    __shared__ float4 sA[kBatch];
    __shared__ float4 sB[kBatch];
    __shared__ unsigned long long sCnt[2];
    const TileCtx c = tile_ctx(cam, ranges, tile_order);
    const float fx = (float)c.px + 0.5f, fy = (float)c.py + 0.5f;
    float T = 1.f;
    uint32_t examined = 0, blended = 0;
    bool done = !c.inside;
    if (threadIdx.x < 2) sCnt[threadIdx.x] = 0ull;
    for (uint32_t base = c.start; base < c.end; base += kBatch) {
        if (__syncthreads_count(!done) == 0) break;
        const uint32_t idx = base + threadIdx.x;
        if (idx < c.end) {
            const float4* rec = reinterpret_cast<const float4*>(packed + vals[idx]);
            sA[threadIdx.x] = rec[0]; sB[threadIdx.x] = rec[1];
        }
        __syncthreads();
        const int cnt = (int)min((uint32_t)kBatch, c.end - base);
        if (!done) {
            for (int j = 0; j < cnt; ++j) {
                const float4 a = sA[j];
                const float4 b = sB[j];
                const float dx = fx - a.x, dy = fy - a.y;
                const float e = log2_alpha(a.z, a.w, b.x, b.y, dx, dy);
                ++examined;
                if (!form_not_negative(a.z, a.w, b.x, dx, dy)) continue;
                const float alpha = fminf(kAlphaMax, __builtin_amdgcn_exp2f(e));
                if (alpha < kAlphaMin) continue;
                const float Tn = T - alpha * T;     // as the forward kernel forms it
                if (Tn < kTStop) { done = true; break; }
                T = Tn;
                ++blended;
            }
        }
    }
    __syncthreads();
    atomicAdd(&sCnt[0], (unsigned long long)examined);
    atomicAdd(&sCnt[1], (unsigned long long)blended);
    __syncthreads();
    if (threadIdx.x < 2 && sCnt[threadIdx.x]) atomicAdd(&counters[threadIdx.x], sCnt[threadIdx.x]);
}

__global__ __launch_bounds__(256) void k_fill_f32(float* __restrict__ p, float v, size_t count)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < count) p[i] = v;
}

hipError_t launch_composite_fwd(const CamDev& cam, const Layout& L, char* ws, const float bg[3], float* image,
                                float* final_T, uint32_t* last_idx, hipStream_t s)
{
    const uint32_t* ranges = reinterpret_cast<const uint32_t*>(ws + L.off_ranges);
    const uint32_t* tile_order = reinterpret_cast<const uint32_t*>(ws + L.off_tile_order);
    const uint32_t* vals = reinterpret_cast<const uint32_t*>(ws + L.off_vals);
    const Packed* packed = reinterpret_cast<const Packed*>(ws + L.off_packed);
    ProfScope prof(kKCompositeFwd, s);
    hipLaunchKernelGGL(k_composite_fwd, dim3((unsigned)(cam.TX * cam.TY)), dim3(256), 0, s, cam, ranges, tile_order, vals, packed,
                       reinterpret_cast<uint16_t*>(ws + L.off_reach), bg[0], bg[1], bg[2], image, final_T, last_idx);
    return hipGetLastError();
}

CarryFold carry_fold(const Layout& L, char* ws)
{
    return CarryFold{reinterpret_cast<const float*>(ws + L.off_carry), reinterpret_cast<const uint32_t*>(ws + L.off_slot_base),
                     reinterpret_cast<uint32_t*>(ws + L.off_status), L.cap};
}

hipError_t launch_composite_bwd(const CamDev& cam, const Layout& L, char* ws, int n, const float bg[3], const float* final_T, const uint32_t* last_idx, const float* dL_dimage,
                                const SplatGradDev& g2, hipStream_t s)
{
    const uint32_t* ranges = reinterpret_cast<const uint32_t*>(ws + L.off_ranges);
    const uint32_t* tile_order = reinterpret_cast<const uint32_t*>(ws + L.off_tile_order);
    const uint32_t* vals = reinterpret_cast<const uint32_t*>(ws + L.off_vals);
    const Packed* packed = reinterpret_cast<const Packed*>(ws + L.off_packed);
    const uint32_t* offsets = reinterpret_cast<const uint32_t*>(ws + L.off_offsets);
    const uint32_t* slot_base = reinterpret_cast<const uint32_t*>(ws + L.off_slot_base);
    const uint32_t* order = reinterpret_cast<const uint32_t*>(ws + L.off_order);
    uint32_t* status = reinterpret_cast<uint32_t*>(ws + L.off_status);
    float4* partial = reinterpret_cast<float4*>(ws + L.off_partial);
    {
        ProfScope prof(kKCompositeBwd, s);
        hipLaunchKernelGGL(k_composite_bwd, dim3((unsigned)(cam.TX * cam.TY)), dim3(256), 0, s, cam, ranges, tile_order, vals, packed,
                           reinterpret_cast<const uint16_t*>(ws + L.off_reach), slot_base, bg[0], bg[1], bg[2], final_T, last_idx, dL_dimage,
                           L.cap, status, partial);
    }
    if (n > 0) {
        ProfScope prof(kKGather, s);
        const uint32_t* chunk_rank = reinterpret_cast<const uint32_t*>(ws + L.off_chunk_rank);
        float* carry = reinterpret_cast<float*>(ws + L.off_carry);
        const unsigned nwave = (unsigned)gather_chunks_max(L.cap);
        float4* rec = reinterpret_cast<float4*>(ws + L.off_grad_rec);
        hipLaunchKernelGGL(k_gather_splat_grads, dim3((nwave + 3) / 4), dim3(256), 0, s, n, status, order, offsets, chunk_rank, partial,
                           L.cap, carry, rec);
        if (g2.mean2d != nullptr)
            hipLaunchKernelGGL(k_grad_records_to_planes, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n,
                               reinterpret_cast<const uint32_t*>(ws + L.off_touched), rec, carry_fold(L, ws), g2);
        // else the caller goes on from the records with launch_preprocess_bwd_records, whose kernel puts the records cut
        // by wavefront boundaries together itself and closes the epoch (carry_fold below): one launch fewer
    }
    return hipGetLastError();
}

hipError_t launch_render_stats(const CamDev& cam, const Layout& L, char* ws, uint64_t* counters, hipStream_t s)
{
    const uint32_t* ranges = reinterpret_cast<const uint32_t*>(ws + L.off_ranges);
    const uint32_t* tile_order = reinterpret_cast<const uint32_t*>(ws + L.off_tile_order);
    const uint32_t* vals = reinterpret_cast<const uint32_t*>(ws + L.off_vals);
    const Packed* packed = reinterpret_cast<const Packed*>(ws + L.off_packed);
    ProfScope prof(kKStats, s);
    hipLaunchKernelGGL(k_fill_f32, dim3(1), dim3(256), 0, s, reinterpret_cast<float*>(counters), 0.f, (size_t)4);
    hipLaunchKernelGGL(k_render_stats, dim3((unsigned)(cam.TX * cam.TY)), dim3(256), 0, s, cam, ranges, tile_order, vals, packed,
                       reinterpret_cast<unsigned long long*>(counters));
    return hipGetLastError();
}

}  // namespace pbdr
