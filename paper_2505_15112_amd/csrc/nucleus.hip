// nucleus.hip -- sorting as much of every row as the top-p sampler reads
// (Section 5 "Top-p or Nucleus Sampling").
//
// The cutoff and the draw look at a row's largest probabilities only, down to
// where their running sum reaches p, and at values only: the one source index
// they need is found afterwards.  So instead of sorting whole rows with their
// indices (four radix passes, 16 bytes per element and pass), the elements
// that can matter are gathered bin by bin and sorted in LDS:
//  * k_nuc_hist, per tile of a row: a sample of the row gives a monotone map
//    from keys to at most 4096 bins, fine where the row's keys are dense; the
//    tile's elements are counted per bin;
//  * k_nuc_pick, one workgroup per row: the bins in descending order, the
//    first at which a lower bound of the running sum (each element counted as
//    its bin's least key) passes p, hence how many elements the draw needs, and
//    the groups that they form;
//  * k_nuc_gather: those elements, keys and source indices, to the row's list,
//    group by group (some thousand elements: the bins that start in one window of
//    the sorted row);
//  * k_nuc_sort, one workgroup per group: sorts its keys in LDS, in descending
//    order.
// Workgroups are numbered tile by tile (or group by group) of all rows, so that
// with a multiple of 8 rows everything of one row runs on one XCD and finds the
// row's list in its L2.  Rows of up to kNucGroupMax elements are one group, sorted
// whole by k_nuc_sort_row alone.  The draw (rows.hip) then runs on the sorted keys
// with the same additions as on a whole sorted row, so its results are the same.
//
// Bound: two reads of the rows from HBM (22 us for 128 x 131072) and the LDS
// work of the sort.  Kernel times at 128 x 131072, p = 0.9 (about 38000
// elements of each row gathered): histogram 20 us, pick 9, gather 27 (105 MB
// moved), sort 24, and the draw 5 + 9; the call 272 us by the row sort, 92 us
// this way.  4 x 200003: 93 -> 43 us, each of the six kernels a few us of
// latency.  Rows whose elements crowd at few values cost more, but no more than
// the row sort, within a few per cent, up to 2^18 elements: 128 x 131072 equal
// 367 -> 161 us, flat with a tenth of zeros 345 -> 222, 4 x 200003 147 -> 154.  At
// 2^20 one workgroup counts such a crowd: 1 x 2^20 equal 275 -> 364, flat with zeros
// 244 -> 557, 16 of them 610 -> 776; rows of 2^20 sorted to their end take up to 1.15
// times the row sort, ordinary ones at p = 0.9 87 -> 57 (1) and 296 -> 175 (16).
// Only rows in which a structure that follows the 512 places of the sample hides
// most elements from it take 3 to 50 times as long (windows, see nuc_window).
// Measured on the way: the elements scattered to their bins by LDS counters
// instead of gathered (one 8-byte store per lane and line): 62 us for the
// scatter; a workgroup for every group a row could have, most of them without
// work: 9 ns each, 26 us.
#include <limits.h>

#include <type_traits>

#include "launch.hpp"
#include "nucleus.hpp"

namespace ls {

constexpr int kNucThreads = 1024;
constexpr int kNucWaves = kNucThreads / kWave;
constexpr int kNucSample = 2048;  // elements of a row that shape its map
constexpr int kNucPer = 12;              // keys per thread in a group's sort
constexpr uint32_t kNucGroupMax = kNucPer * kNucThreads;  // 12288
constexpr uint32_t kNucSlots = 14336;    // two sorts' LDS fits a CU
static_assert(kNucSlots % (2 * kNucThreads) == 0, "whole words per thread");
constexpr int64_t kNucMaxLen = int64_t(1) << 20;
constexpr uint32_t kNucMinGroup = 4096;
constexpr uint32_t kNucMaxGroups = 1024;  // table room in LDS
static_assert(kNucMaxLen / kNucMinGroup * 2 <= kNucMaxGroups, "a row's groups fit the tables");
constexpr uint16_t kNucNoGroup = 0xFFFF;
constexpr uint32_t kNucMaxSegs = 40;  // 2^20 + 3 positions of 32768, 2^18 + 3 of 8192: 33
// The last two bins are in no map (see k_nuc_hist): the elements above the
// sampled range, and the flag of a row that holds a NaN.
constexpr int kNucAbove = kNucBins - 2, kNucNan = kNucBins - 1;

// Exclusive scan over the workgroup; s_w: one word per wave.  One barrier
// inside; s_w may be rewritten after the next one.
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* s_w, uint32_t* total) {
    const int w = threadIdx.x / kWave;
    const uint32_t inc = wave_incl_scan(v);
    if (lane_id() == kWave - 1) s_w[w] = inc;
    __syncthreads();
    const uint32_t t = lane_id() < kNucWaves ? s_w[lane_id()] : 0u;
    const uint32_t sc = wave_incl_scan(t);
    const int wu = __builtin_amdgcn_readfirstlane(w);
    *total = lane_read(sc, kNucWaves - 1);
    return (wu > 0 ? lane_read(sc, wu - 1) : 0u) + inc - v;
}

// One more in LDS counter c[i], for the active lanes: those with the first one's
// i by one addition.  (Crowds again: 64 lanes on one counter take their turns.)
__device__ __forceinline__ void nuc_count(uint32_t* c, uint32_t i) {
    const bool with = i == uni(i);
    const uint64_t same = __ballot(with);
    if (!with || lanes_below(same) == 0)
        atomicAdd(&c[i], with ? (uint32_t)__builtin_popcountll(same) : 1u);
}

// ---------------------------------------------------------------- the row's elements

// A workgroup's 4096 J positions of a row in groups of four, thread t's
// group j at position (j kNucThreads + t) 4 - shift of the tile: `shift` (0 to
// 3) places the groups on 16-byte boundaries whatever the row's alignment, and
// a group that crosses either end of the row is loaded element by element
// (in[j], bit e: element e lies in the row).
template <int J>
struct NucTile {
    uint32_t v[J][4];
    int32_t pos0;   // row position of v[0][0]
    uint32_t in;    // bit 4 j + e, when not `full`
    bool full;      // uniform: every position lies in the row
    __device__ __forceinline__ uint32_t pos(int j, int e) const {
        return (uint32_t)(pos0 + j * (kNucThreads * 4) + e);
    }
    __device__ __forceinline__ void load(const uint32_t* xr, int32_t len, uint32_t seg) {
        static_assert(J * 4 <= 32, "one bit per element");
        const int32_t shift = (int32_t)((uintptr_t)xr / 4 % 4);
        const int32_t base = (int32_t)(seg * (4096u * J)) - shift;
        pos0 = base + (int32_t)threadIdx.x * 4;
        full = base >= 0 && base + 4096 * J <= len;
        in = ~0u;
        if (full) {
            const uint32_t* p = xr + base;
#pragma unroll
            for (int j = 0; j < J; ++j)
                load_vec<uint32_t, uint32_t, 4, true>(p + (j * kNucThreads + threadIdx.x) * 4, v[j]);
        } else {
            in = 0u;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int32_t q = pos0 + j * (kNucThreads * 4);
                if (q >= 0 && q + 4 <= len) {
                    load_vec<uint32_t, uint32_t, 4, true>(xr + q, v[j]);
                    in |= 15u << (4 * j);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool ok = q + e >= 0 && q + e < len;
                        v[j][e] = ok ? xr[q + e] : 0u;
                        in |= (ok ? 1u : 0u) << (4 * j + e);
                    }
                }
            }
        }
    }
    // f(bits of four elements, position of the first, which of them lie in the
    // row), in uniform control flow
    template <class F>
    __device__ __forceinline__ void each4(F f) const {
        uint32_t q0 = (uint32_t)pos0;
        asm volatile("" : "+v"(q0));
#pragma unroll
        for (int j = 0; j < J; ++j)
            f(v[j], q0 + (uint32_t)(j * kNucThreads * 4), full ? 15u : (in >> (4 * j)) & 15u);
    }
    // f(bits, position, in the row) for every position, in uniform control flow
    template <class F>
    __device__ __forceinline__ void each(F f) const {
        uint32_t q0 = (uint32_t)pos0;
        asm volatile("" : "+v"(q0));  // no per-group positions kept live from the loads
        if (full) {
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    f(v[j][e], q0 + (uint32_t)(j * kNucThreads * 4 + e), true);
        } else {
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    f(v[j][e], q0 + (uint32_t)(j * kNucThreads * 4 + e),
                      ((in >> (4 * j + e)) & 1u) != 0);
        }
    }
};

// ---------------------------------------------------------------- histogram

// Tile counts per bin (16-bit: a tile has at most 32768 elements), and, from
// the row's first tile, the row's map.  Every tile of a row derives the same
// map from the same sample: 512 groups of 4 consecutive elements spread over
// the row.  The sampled range is cut into at most 2048 cells; a cell with s
// samples is cut into the least power of two >= s / 2 bins: at most s - 1 of
// them for s > 2, so at most 4094 in all.  Where no cell has more samples than
// stand for `fine` elements the cells are the bins, and the map is not looked up
// (one LDS read less per element).
//
// Elements above the sampled range are counted in bin kNucAbove, and their sum
// kept (above[tile]): the largest probabilities, few and mostly not in the
// sample, carry much of the mass.  Bin kNucNan is 1 if the tile has a NaN with
// its sign bit clear: it sorts before everything, and no running sum of its row
// reaches p.
template <int J>
__global__ __launch_bounds__(kNucThreads) LS_OCCUPANCY8 void k_nuc_hist(
    const uint32_t* x, int32_t len, uint32_t nrows, uint32_t segs, uint16_t* hist, NucRow* rows,
    uint32_t* maps, double* above, uint32_t fine) {
    __shared__ uint32_t s_map[kNucCells];
    __shared__ uint32_t s_h[kNucBins];
    __shared__ uint32_t s_w[kNucWaves], s_w2[kNucWaves];
    __shared__ uint32_t s_dense;
    __shared__ double s_above;
    const uint32_t seg = blockIdx.x / nrows, row = blockIdx.x - seg * nrows;
    const uint32_t tile_id = row * segs + seg;
    const uint32_t* xr = x + (int64_t)row * len;
    const uint32_t t = threadIdx.x;
    // the sample (len > kNucGroupMax > kNucSample), loaded before the tile: it
    // is waited for first
    uint32_t smp[4];
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    if (t < kNucSample / 4) {
        const uint32_t q = (uint32_t)((uint64_t)t * (uint32_t)(len - 4) / (kNucSample / 4 - 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) smp[e] = xr[q + e];
    }
    __builtin_amdgcn_sched_barrier(0);
    NucTile<J> tile;
    tile.load(xr, len, seg);
    __builtin_amdgcn_sched_barrier(0);
    if (t < kNucSample / 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) smp[e] = nuc_key(smp[e]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            mn = smp[e] < mn ? smp[e] : mn;
            mx = smp[e] > mx ? smp[e] : mx;
        }
    }
    mn = wave_reduce_min(mn);
    mx = ~wave_reduce_min(~mx);
    if (lane_id() == 0) {
        s_w[t / kWave] = mn;
        s_w2[t / kWave] = mx;
    }
    for (int i = t; i < kNucCells; i += kNucThreads) s_map[i] = 0;
    for (int i = t; i < kNucBins; i += kNucThreads) s_h[i] = 0;
    if (t == 0) {
        s_dense = 0;
        s_above = 0.0;
    }
    __syncthreads();
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int q = 0; q < kNucSample / 4 / kWave; ++q) {
        lo = s_w[q] < lo ? s_w[q] : lo;
        hi = s_w2[q] > hi ? s_w2[q] : hi;
    }
    lo = uni(lo);
    hi = uni(hi);
    const uint32_t range = hi - lo;
    const int bits = range ? 32 - __builtin_clz(range) : 0;
    const uint32_t shift = bits > 11 ? (uint32_t)(bits - 11) : 0u;  // range >> shift < 2048
    if (t < kNucSample / 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) atomicAdd(&s_map[(smp[e] - lo) >> shift], 1u);
    }
    __syncthreads();
    // cells 2 t and 2 t + 1: their bins
    uint32_t sub[2], n[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t s = s_map[2 * t + i];
        if ((uint64_t)s * (uint32_t)len > (uint64_t)kNucSample * fine) atomicMax(&s_dense, 1u);
        if (s > kNucSample / 4) atomicMax(&s_dense, 2u);
        const uint32_t b = s > 2 ? 32u - (uint32_t)__builtin_clz((s + 1) / 2 - 1) : 0u;
        sub[i] = b < shift ? b : shift;
    }
    __syncthreads();
    const bool direct = s_dense == 0;  // uniform over the row's tiles
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        sub[i] = direct ? 0u : sub[i];
        n[i] = 1u << sub[i];
    }
    uint32_t total;
    const uint32_t first = block_excl_scan(n[0] + n[1], s_w, &total);
    s_map[2 * t] = first | sub[0] << 16;
    s_map[2 * t + 1] = (first + n[0]) | sub[1] << 16;
    __syncthreads();
    int32_t top = 0;
    auto count = [&](auto bin_of, auto add) {
        tile.each([&](uint32_t b, uint32_t, bool ok) {
            if (!ok) return;
            top = top > (int32_t)b ? top : (int32_t)b;
            const uint32_t k = nuc_key(b);
            const bool over = k > hi;
            if (over) atomicAdd(&s_above, (double)Bits<float>::from(b));
            const uint32_t bin = bin_of(k > lo ? k - lo : 0u);
            add(over ? kNucAbove : bin);
        });
    };
    auto one = [&](uint32_t bin) { atomicAdd(&s_h[bin], 1u); };
    // keys above hi index no cell: the bin they would get is not used
    auto cell = [&](uint32_t d) { return d >> shift; };
    auto mapped = [&](uint32_t d) {
        const uint32_t c = d >> shift;
        const uint32_t e = s_map[c < kNucCells ? c : kNucCells - 1];
        return (e & 0xFFFFu) + ((d & ((1u << shift) - 1u)) >> (shift - (e >> 16)));
    };
    if (direct)
        count(cell, one);
    else if (s_dense == 1)
        count(mapped, one);
    else  // much of the row in one cell
        count(mapped, [&](uint32_t bin) { nuc_count(s_h, bin); });
    if (top > 0x7F800000) s_h[kNucNan] = 1;  // every such thread stores the same
    if (seg == 0) {
        uint32_t* m = maps + (int64_t)row * kNucCells;
        m[2 * t] = s_map[2 * t];
        m[2 * t + 1] = s_map[2 * t + 1];
        if (t == 0) {
            rows[row].lo = lo;
            rows[row].hi = hi;
            rows[row].shift = shift;
            rows[row].direct = direct;
        }
    }
    __syncthreads();
    // bins 4 t .. 4 t + 3 (as 8 bytes)
    ushort4 c;
    c.x = (uint16_t)s_h[4 * t];
    c.y = (uint16_t)s_h[4 * t + 1];
    c.z = (uint16_t)s_h[4 * t + 2];
    c.w = (uint16_t)s_h[4 * t + 3];
    reinterpret_cast<ushort4*>(hist + (int64_t)tile_id * kNucBins)[t] = c;
    if (t == 0) above[tile_id] = s_above;
}

// ---------------------------------------------------------------- how far to sort

// One workgroup per row.  Thread t takes the four bins at descending places
// 4 t .. 4 t + 3 (bin kNucBins - 1 - place).
__global__ __launch_bounds__(kNucThreads) void k_nuc_pick(const uint16_t* hist, uint32_t segs,
                                                          const uint32_t* maps, float p,
                                                          int32_t len,
                                                          NucRow* rows, const double* above,
                                                          uint32_t window, uint32_t slots,
                                                          uint2* groups, uint32_t* cursors,
                                                          uint16_t* bin_groups) {
    __shared__ uint32_t s_cell[kNucBins], s_map[kNucCells];
    __shared__ uint32_t s_w[kNucWaves];
    __shared__ double s_d[kNucWaves];
    __shared__ uint32_t s_need, s_sorted, s_key, s_nan;
    __shared__ uint32_t s_g[kNucMaxGroups], s_low[kNucMaxGroups], s_id[kNucMaxGroups];
    const int64_t row = blockIdx.x;
    const uint32_t t = threadIdx.x;
    const int w = t / kWave;
    const uint16_t* rh = hist + row * segs * kNucBins;
    // counts: the bins at places 4 t .. 4 t + 3 are bins b0 + 3 .. b0
    const uint32_t b0 = kNucBins - 4 - 4 * t;
    uint32_t cnt[4] = {0u, 0u, 0u, 0u};
#pragma unroll 16
    for (uint32_t s = 0; s < segs; ++s) {
        const ushort4 c = *reinterpret_cast<const ushort4*>(rh + (int64_t)s * kNucBins + b0);
        cnt[0] += c.w;
        cnt[1] += c.z;
        cnt[2] += c.y;
        cnt[3] += c.x;
    }
    double over = 0.0;  // thread 0: the sum of the elements above the range
    if (t < kWave) {
        static_assert(kNucMaxSegs <= kWave, "one lane per tile");
        over = t < segs ? above[row * segs + t] : 0.0;
        for (int d = kWave / 2; d >= 1; d /= 2) over += __shfl_xor(over, d);
    }
    if (t == 0) {
        s_nan = cnt[0];  // bin kNucNan: a flag, not a count
        cnt[0] = 0;
    }
    const NucRow r = rows[row];
    if (t == 0) {
        s_need = (uint32_t)len;
        s_sorted = (uint32_t)len;
        s_key = 0u;
    }
    if (t < slots) s_g[t] = s_low[t] = UINT_MAX;
    // every bin's least key
    uint32_t low[4];
    if (r.direct) {  // uniform: bin b is cell b
#pragma unroll
        for (int i = 0; i < 4; ++i) low[i] = r.lo + ((b0 + 3 - i) << r.shift);
    } else {
        // the cell a bin belongs to is the last one whose first bin is not
        // after it: a running maximum over the bins of the cells' marks
        const uint2 e2 = reinterpret_cast<const uint2*>(maps + row * kNucCells)[t];
        for (int i = t; i < kNucBins; i += kNucThreads) s_cell[i] = 0;
        s_map[2 * t] = e2.x;
        s_map[2 * t + 1] = e2.y;
        __syncthreads();
        s_cell[e2.x & 0xFFFFu] = 2 * t;  // distinct bins
        s_cell[e2.y & 0xFFFFu] = 2 * t + 1;
        __syncthreads();
        uint32_t run = 0, cell[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // bins 4 t + i
            const uint32_t c = s_cell[4 * t + i];
            run = c > run ? c : run;
            cell[i] = run;
        }
        // wave maximum scan (maxima of ~v by the minimum's moves)
        uint32_t inc = ~run;
        inc = dpp_umin<0x111, 0xf>(inc);
        inc = dpp_umin<0x112, 0xf>(inc);
        inc = dpp_umin<0x114, 0xf>(inc);
        inc = dpp_umin<0x118, 0xf>(inc);
        inc = dpp_umin<0x142, 0xa>(inc);
        inc = dpp_umin<0x143, 0xc>(inc);
        inc = ~inc;
        if (lane_id() == kWave - 1) s_w[w] = inc;
        uint32_t before = wave_shr1(inc);
        __syncthreads();
        for (int q = 0; q < w; ++q) before = s_w[q] > before ? s_w[q] : before;
#pragma unroll
        for (int i = 0; i < 4; ++i) s_cell[4 * t + i] = cell[i] > before ? cell[i] : before;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t b = b0 + 3 - i, c = s_cell[b];
            const uint32_t e = s_map[c];
            low[i] = r.lo + (c << r.shift) + ((b - (e & 0xFFFFu)) << (r.shift - (e >> 16)));
        }
    }
    double mass = 0.0, m[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t b = b0 + 3 - i;
        if (b == 0) low[i] = 0u;  // the first bin takes every key below lo
        if (b == kNucAbove) low[i] = r.hi + 1u;  // not empty: hi is not the last key
        // the least value; a bin that reaches below the finite ones bounds nothing
        const float v = Bits<float>::from(nuc_bits(low[i]));
        m[i] = cnt[i] ? (v >= -3.4028235e38f ? (double)cnt[i] * (double)v : -__builtin_inf()) : 0.0;
        if (b == kNucAbove) m[i] = over;
        mass += m[i];
    }
    __syncthreads();  // s_w free
    uint32_t total;
    const uint32_t own = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    uint32_t start[4];
    start[0] = block_excl_scan(own, s_w, &total);
#pragma unroll
    for (int i = 1; i < 4; ++i) start[i] = start[i - 1] + cnt[i - 1];
    // running lower bound before this thread's bins
    auto add = [](double a, uint64_t o) { return a + __builtin_bit_cast(double, o); };
    auto moved = [](double v, auto c, auto m) {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        return ((uint64_t)dpp0<c(), m()>((uint32_t)(u >> 32)) << 32) | dpp0<c(), m()>((uint32_t)u);
    };
    double inc = mass;
#define LS_STEP(C, M) \
    inc = add(inc, moved(inc, std::integral_constant<int, C>{}, std::integral_constant<int, M>{}))
    LS_STEP(0x111, 0xf);
    LS_STEP(0x112, 0xf);
    LS_STEP(0x114, 0xf);
    LS_STEP(0x118, 0xf);
    LS_STEP(0x142, 0xa);
    LS_STEP(0x143, 0xc);
#undef LS_STEP
    if (lane_id() == kWave - 1) s_d[w] = inc;
    double before = __builtin_bit_cast(
        double, moved(inc, std::integral_constant<int, 0x138>{}, std::integral_constant<int, 0xf>{}));
    __syncthreads();
    for (int q = 0; q < w; ++q) before += s_d[q];
    // The draw adds in 32 bits, each addition off by at most 2^-24 of a sum whose
    // terms up to the crossing have one sign: fewer than 48 additions deep inside a
    // tile and over the head tiles, one more for every step of 8192 behind them.
    // Whatever these lose, its running sum has reached p where the bound is past
    // p by as much (and as much again: 64 instead of 48, the steps of the whole row).
    const double lost = (64 + len / 8192) * 0x1p-24;  // 1.1e-5 at 2^20 elements
    const double goal = (double)p + lost * (p < 0.f ? -(double)p : (double)p);
    if (!s_nan) {
        double s = before;
        uint32_t n = UINT_MAX;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s += m[i];
            if (n == UINT_MAX && cnt[i] && s >= goal) n = start[i] + cnt[i];
        }
        if (n != UINT_MAX) atomicMin(&s_need, n);
    }
    __syncthreads();
    const uint32_t need = s_need;
    // The bins that start before `need` are sorted; those that start in one window
    // of the sorted row are a group, but one of more elements than a window is a
    // group of its own (the next bin then starts in a later window): mostly it is a
    // crowd of few values, which k_nuc_sort handles best alone.  Behind `need`
    // the sorted row is not written; the draw reads whole tiles, but what
    // follows the crossing changes nothing in what it finds.
    auto group_of = [&](uint32_t first, uint32_t count) {
        return first / window * 2 + (count > window ? 1u : 0u);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (cnt[i] && start[i] < need) {
            const uint32_t g = group_of(start[i], cnt[i]);
            atomicMin(&s_g[g], start[i]);
            atomicMin(&s_low[g], low[i]);
            if (start[i] + cnt[i] >= need) {  // the last one
                s_sorted = start[i] + cnt[i];
                s_key = low[i];
            }
        }
    }
    __syncthreads();
    // groups are numbered without the empty windows: {first position, least key},
    // where its list slots start, and the end
    static_assert(kNucMaxGroups <= kNucThreads, "a thread per group");
    const uint32_t gs = t < slots ? s_g[t] : UINT_MAX;
    uint32_t ng;
    const uint32_t id = block_excl_scan(gs != UINT_MAX ? 1u : 0u, s_w, &ng);
    uint2* gr = groups + row * (slots + 1);
    if (gs != UINT_MAX) {
        gr[id] = make_uint2(gs, s_low[t]);
        cursors[row * slots + id] = gs;
        s_id[t] = id;
    }
    if (t == 0) {
        gr[ng] = make_uint2(s_sorted, 0u);
        rows[row].key_min = s_key;
        rows[row].groups = ng;
    }
    __syncthreads();
    // every bin's group (bins b0 .. b0 + 3, places 3 .. 0)
    uint16_t bg[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        bg[3 - i] = cnt[i] && start[i] < need ? (uint16_t)s_id[group_of(start[i], cnt[i])] : kNucNoGroup;
    reinterpret_cast<ushort4*>(bin_groups + row * kNucBins)[b0 / 4] =
        make_ushort4(bg[0], bg[1], bg[2], bg[3]);
}

// ---------------------------------------------------------------- gather

// The tile's elements with keys from key_min up, keys and source indices, to
// the row's list, group by group (in any order within a group), so that the sort
// of a group reads its own keys only: group g has the list's slots [groups[g].x,
// groups[g + 1].x).  The tile's share of each group is known from its bins'
// counts, and reserved by one atomic per group; its elements take their slots by
// LDS counters.  With one run of slots per tile instead, the sort picking its
// group's keys out of the whole list, the gather takes 22 instead of 27 us at 128
// x 131072 and p = 0.9, the sort 33 instead of 25 and the draw's lookup in the list
// 15 instead of 9; and long rows read groups x list: 1 x 2^20, softmax of N(0,
// 4), 117 us a call at p = 0.9 and 817 at p = 1, now 59 and 270.  Without the ring
// (the search and the slot for every element of the tile) 36 us.
template <int J>
__global__ __launch_bounds__(kNucThreads) LS_OCCUPANCY8 void k_nuc_gather(
    const uint32_t* x, int32_t len, uint32_t nrows, uint32_t segs, const NucRow* rows,
    const uint16_t* hist, const uint16_t* bin_groups, const uint2* groups, uint32_t* cursors,
    uint32_t slots, uint32_t* keys, uint32_t* idx, uint32_t stride) {
    __shared__ uint32_t s_low[kNucMaxGroups], s_to[kNucMaxGroups];
    const uint32_t seg = blockIdx.x / nrows, row = blockIdx.x - seg * nrows;
    const uint32_t t = threadIdx.x;
    NucTile<J> tile;
    tile.load(x + (int64_t)row * len, len, seg);
    const uint32_t key_min = rows[row].key_min, ng = uni(rows[row].groups);
    const ushort4 c = reinterpret_cast<const ushort4*>(
        hist + (int64_t)(row * segs + seg) * kNucBins)[t];
    const ushort4 g = reinterpret_cast<const ushort4*>(bin_groups + (int64_t)row * kNucBins)[t];
    // past the last group least keys of 0: the search below stays before them
    s_low[t] = t < ng ? groups[(int64_t)row * (slots + 1) + t].y : 0u;
    s_to[t] = 0;
    __syncthreads();
    auto add = [&](uint32_t n, uint32_t group) {
        if (n != 0 && group != kNucNoGroup) atomicAdd(&s_to[group], n);
    };
    if (g.x == g.y && g.x == g.z && g.x == g.w) {
        add((uint32_t)c.x + c.y + c.z + c.w, g.x);
    } else {
        add(c.x, g.x);
        add(c.y, g.y);
        add(c.z, g.z);
        add(c.w, g.w);
    }
    __syncthreads();
    if (t < ng && s_to[t] != 0)
        s_to[t] = __hip_atomic_fetch_add(&cursors[(int64_t)row * slots + t], s_to[t],
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    uint32_t* kr = keys + (int64_t)row * stride;
    uint32_t* ir = idx + (int64_t)row * stride;
    // The wave's kept elements go through a ring in LDS, so that what follows is
    // done 64 kept ones at a time, not for every element of the row: the group
    // of a key (how many groups' least keys are above it), and its slot (the
    // group of the first lane takes its lanes' slots by one atomic, lanes of other
    // groups one each).
    constexpr uint32_t kRing = 512;  // fewer than 64 left, and 256 more
    __shared__ uint2 s_ring[kNucWaves][kRing];
    uint2* ring = s_ring[uni(t / kWave)];
    const uint32_t lane = lane_id();
    const uint32_t step0 = ng > 1 ? 1u << (31 - __builtin_clz(ng - 1)) : 0u;
    uint32_t head = 0, tail = 0;  // uniform
    auto flush = [&](uint32_t n) {
        wave_lds_sync();
        const uint2 kp = ring[(head + lane) % kRing];
        head += n;
        if (lane >= n) return;
        uint32_t grp = 0;
        for (uint32_t d = step0; d != 0; d >>= 1) grp += s_low[grp + d - 1] > kp.x ? d : 0u;
        const bool with = grp == uni(grp);  // lane 0 is among them
        const uint64_t same = __ballot(with);
        uint32_t to = 0;
        if (!with || lane == 0)
            to = atomicAdd(&s_to[grp], with ? (uint32_t)__builtin_popcountll(same) : 1u);
        if (with) to = uni(to) + lanes_below(same);
        if (to < (uint32_t)len) {  // always; checked all the same
            kr[to] = kp.x;
            ir[to] = kp.y;
        }
    };
    tile.each4([&](const uint32_t(&b)[4], uint32_t pos, uint32_t in) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t key = nuc_key(b[e]);
            const bool q = ((in >> e) & 1u) && key >= key_min;
            const uint64_t m = __ballot(q);
            if (q) ring[(tail + lanes_below(m)) % kRing] = make_uint2(key, pos + e);
            tail += (uint32_t)__builtin_popcountll(m);
        }
#pragma unroll 1
        while (tail - head >= kWave) flush(kWave);
    });
    if (tail != head) flush(tail - head);
}

// ---------------------------------------------------------------- a group's sort

// The thread's number, as a value that nothing is hoisted out of loops for
// (addresses derived from it would stay live through the whole kernel).
__device__ __forceinline__ uint32_t nuc_thread() {
    uint32_t t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}
constexpr uint32_t kNucFew = 64;
struct NucSortLds {
    uint32_t key[kNucGroupMax];
    uint32_t slot[kNucSlots / 2];  // two 16-bit counters a word
    uint32_t w[kNucWaves];
    uint32_t mixed;
};

// The keys L.key[0, n), all in [hi - range, hi], to out[0, n) in descending
// order (as float bits), by stable 8-bit digit passes over their distance below
// hi, as many as the range has bytes; ranking as in k_radix8_scatter.  The time
// does not depend on the keys: for crowded slots of nuc_sort.
__device__ __forceinline__ void nuc_digits(uint32_t n, uint32_t hi, uint32_t range, uint32_t* out,
                                        NucSortLds& L) {
    static_assert(kNucWaves * 256 <= kNucSlots / 2, "digit counts of every wave fit the slots");
#pragma unroll 1
    for (int shift = 0; shift < 32 && (range >> shift) != 0; shift += 8) {
        const uint32_t t = nuc_thread(), lane = t % kWave, w = uni(t / kWave);
        const uint32_t place = w * kNucPer * kWave + lane;  // the lane's key of chunk e: + e kWave
        uint32_t* wh = L.slot + w * 256;
        // places from n on hold the largest distance: they stay last in every pass
        uint32_t d[kNucPer], rank[kNucPer / 2];  // ranks in the wave, two a register
        __syncthreads();  // L.key written, L.slot free
#pragma unroll
        for (int e = 0; e < kNucPer; ++e)
            d[e] = place + e * kWave < n ? hi - L.key[place + e * kWave] : 0xFFFFFFFFu;
#pragma unroll
        for (int i = 0; i < 4; ++i) wh[i * kWave + lane] = 0;
        wave_lds_sync();
#pragma unroll
        for (int e = 0; e < kNucPer; ++e) {
            const uint32_t q = (d[e] >> shift) & 255u;
            const uint64_t peers = peers8_all(q);
            const uint32_t below = lanes_below(peers);
            const uint32_t size = (uint32_t)__builtin_popcountll(peers);
            if (below == 0) atomicAdd(&wh[q], size);
            const uint32_t r = wh[q] - size + below;
            rank[e / 2] = e % 2 ? rank[e / 2] | r << 16 : r;
            asm volatile("" : "+v"(rank[e / 2]));
            __builtin_amdgcn_sched_barrier(0);  // one key's ballots at a time: registers
        }
        __syncthreads();
        // digit t: every wave's first place
        uint32_t tot = 0, total;
        if (t < 256)
#pragma unroll 4
            for (int k = 0; k < kNucWaves; ++k) tot += L.slot[k * 256 + t];
        uint32_t first = block_excl_scan(tot, L.w, &total);
        if (t < 256)
#pragma unroll 4
            for (int k = 0; k < kNucWaves; ++k) {
                const uint32_t c = L.slot[k * 256 + t];
                L.slot[k * 256 + t] = first;
                first += c;
            }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < kNucPer; ++e) {
            const uint32_t to = (e % 2 ? rank[e / 2] >> 16 : rank[e / 2] & 0xFFFFu) + wh[(d[e] >> shift) & 255u];
            if (to < n) L.key[to] = hi - d[e];
            if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();
    for (uint32_t i = nuc_thread(); i < n; i += kNucThreads) out[i] = nuc_bits(L.key[i]);
}

// Sorts n <= kNucGroupMax keys, key[e] being number threadIdx.x + e kNucThreads,
// in descending order to out[0, n) (as float bits).  The key range [lo, hi] is
// spread over kNucSlots slots (linearly: keys that are about evenly dense in it
// are about one a slot); the keys are counted per slot, moved to their slots'
// places in LDS, and each finds its rank among the keys of its slot by looking
// at them all.  A slot of more than kNucFew keys that are all equal needs no
// look; with any other such slot (keys far from evenly dense: one outlier is
// enough) the group goes by digit passes, since the looks would be quadratic
// (the call on 64 x 12288, softmax of N(0, 10^-6) with a tenth of every row zero:
// 4700 us by looks, 73 so; softmax of N(0, 4): 37).
__device__ void nuc_sort(const uint32_t (&key)[kNucPer], uint32_t n, uint32_t lo, uint32_t hi,
                         uint32_t* out, NucSortLds& L) {
    const uint32_t t = nuc_thread();
    const uint32_t range = hi - lo;
    const bool direct = range < kNucSlots;
    const uint32_t mult = uni((uint32_t)((double)kNucSlots * 4294967296.0 / ((double)range + 1.0)));
    auto slot_of = [&](uint32_t k) {
        const uint32_t d = hi - k;
        const uint32_t s = direct ? d : __umulhi(d, mult);
        return s < kNucSlots ? s : kNucSlots - 1;
    };
    __syncthreads();  // L free
    for (uint32_t i = t; i < kNucSlots / 2; i += kNucThreads) L.slot[i] = 0;
    if (t == 0) L.mixed = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kNucPer; ++e)
        if (t + e * kNucThreads < n) {
            const uint32_t s = slot_of(key[e]);
            atomicAdd(&L.slot[s / 2], 1u << (16 * (s & 1)));
        }
    __syncthreads();
    // thread t: kWords words of two slots, counts to first places
    constexpr int kWords = kNucSlots / 2 / kNucThreads;
    uint32_t c[kWords], sum = 0;
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
        c[i] = L.slot[kWords * t + i];
        sum += (c[i] & 0xFFFFu) + (c[i] >> 16);
    }
    uint32_t total;
    uint32_t at = block_excl_scan(sum, L.w, &total);
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
        const uint32_t a = c[i] & 0xFFFFu, b = c[i] >> 16;
        if ((a > b ? a : b) > kNucFew) L.mixed = 1;
        L.slot[kWords * t + i] = at | (at + a) << 16;
        at += a + b;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kNucPer; ++e)
        if (t + e * kNucThreads < n) {
            const uint32_t s = slot_of(key[e]);
            const uint32_t old = atomicAdd(&L.slot[s / 2], 1u << (16 * (s & 1)));
            const uint32_t i = (old >> (16 * (s & 1))) & 0xFFFFu;
            if (i < kNucGroupMax) L.key[i] = key[e];  // always; checked all the same
        }
    __syncthreads();
    // a slot's counter is now its end, the one before it its first place
    auto end_of = [&](uint32_t s) { return (L.slot[s / 2] >> (16 * (s & 1))) & 0xFFFFu; };
    if (L.mixed) {  // uniform: some slot has many keys; are they equal?
        __syncthreads();
        for (uint32_t i = t; i < n; i += kNucThreads) {
            const uint32_t k = L.key[i], s = slot_of(k);
            const uint32_t first = s ? end_of(s - 1) : 0u;
            if (end_of(s) - first > kNucFew && L.key[first] != k) L.mixed = 2;
        }
        __syncthreads();
    }
    if (L.mixed == 2) {  // uniform
        nuc_digits(n, hi, range, out, L);
        return;
    }
#pragma unroll 4
    for (uint32_t i = t; i < n; i += kNucThreads) {
        const uint32_t k = L.key[i], s = slot_of(k);
        const uint32_t first = s ? end_of(s - 1) : 0u, last = end_of(s);
        uint32_t r = i;
        if (last - first > 1u && last - first <= kNucFew) {
            r = first;
            for (uint32_t j = first; j < last; ++j) {
                const uint32_t o = L.key[j];
                r += (o > k || (o == k && j < i)) ? 1u : 0u;
            }
        }
        out[r] = nuc_bits(k);
    }
}

// Least and largest of the workgroup's keys.
__device__ __forceinline__ void nuc_range(const uint32_t (&key)[kNucPer], uint32_t n, uint32_t* lo,
                                          uint32_t* hi, NucSortLds& L) {
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    const uint32_t t = nuc_thread();
#pragma unroll
    for (int e = 0; e < kNucPer; ++e)
        if (t + e * kNucThreads < n) {
            mn = key[e] < mn ? key[e] : mn;
            mx = key[e] > mx ? key[e] : mx;
        }
    mn = wave_reduce_min(mn);
    mx = ~wave_reduce_min(~mx);
    __syncthreads();
    if (lane_id() == 0) {
        L.key[threadIdx.x / kWave] = mn;
        L.key[kNucWaves + threadIdx.x / kWave] = mx;
    }
    __syncthreads();
    for (int q = 0; q < kNucWaves; ++q) {
        mn = L.key[q] < mn ? L.key[q] : mn;
        mx = L.key[kNucWaves + q] > mx ? L.key[kNucWaves + q] : mx;
    }
    *lo = uni(mn);
    *hi = uni(mx);
}

// f(key) for the m keys at `keys` (4-byte aligned; up to 3 words after them may be
// read): 16-byte loads, three in flight a thread.
template <class F>
__device__ __forceinline__ void nuc_each(const uint32_t* keys, uint32_t m, F f) {
    const uint32_t t4 = nuc_thread() * 4;
    constexpr uint32_t kLoads = 3, kStep = 4 * kNucThreads;
    uint32_t b = 0;
#pragma unroll 1
    for (; b + kLoads * kStep <= m; b += kLoads * kStep) {
        const uint32_t* kb = keys + b;  // uniform
        u32x4_a4 v[kLoads];
#pragma unroll
        for (uint32_t q = 0; q < kLoads; ++q)
            v[q] = *reinterpret_cast<const u32x4_a4*>(kb + (q * kStep + t4));
#pragma unroll
        for (uint32_t q = 0; q < kLoads; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) f(v[q][e]);
    }
#pragma unroll 1
    for (uint32_t i = b + t4; i < m; i += kStep) {
        const u32x4_a4 v = *reinterpret_cast<const u32x4_a4*>(keys + i);
#pragma unroll
        for (uint32_t e = 0; e < 4; ++e)
            if (i + e < m) f(v[e]);
    }
}

// A group too large for LDS (a bin of many elements: most of them equal, or so
// close together that the sample's map did not part them) is sorted in windows
// of at most kNucGroupMax keys from the top down, until those left are few
// values.  nuc_limits: the least and the largest of the m keys at lk that are at
// most cap (least > largest: none).
__device__ void nuc_limits(const uint32_t* lk, uint32_t m, uint32_t cap, uint32_t* lo,
                           uint32_t* hi, uint32_t* s_v) {
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    nuc_each(lk, m, [&](uint32_t k) {
        if (k <= cap) {
            mn = k < mn ? k : mn;
            mx = k > mx ? k : mx;
        }
    });
    const uint32_t t = nuc_thread();
    __syncthreads();
    if (t < 2) s_v[t] = t - 1u;  // the largest value, 0
    __syncthreads();
    mn = wave_reduce_min(mn);
    mx = ~wave_reduce_min(~mx);
    if (lane_id() == 0) {
        atomicMin(&s_v[0], mn);
        atomicMax(&s_v[1], mx);
    }
    __syncthreads();
    *lo = uni(s_v[0]);
    *hi = uni(s_v[1]);
}

constexpr uint32_t kNucParts = 4096;
static_assert(kNucParts <= kNucSlots / 2 && kNucParts == 4 * kNucThreads, "four parts a thread");

// Keys of fewer than kNucParts values, [lo, hi], in descending order to out[0,
// room): each value is counted and written as often as it is there.  The other
// keys of lk[0, m) are above hi; `room` are not.  (Crowds are what makes large
// groups: equal elements, masked zeros, flat rows.  In windows, three reads of the
// list each, the call on softmax of N(0, 10^-5) with a tenth of the row zero took
// 31.4 ms at 1 x 2^20 and 1.37 ms at 128 x 131072; so 0.43 to 0.6 and 0.23.)
__device__ void nuc_emit(const uint32_t* lk, uint32_t m, uint32_t lo, uint32_t hi, uint32_t* out,
                         uint32_t room, NucSortLds& L) {
    const uint32_t range = hi - lo;
    if (range == 0) {
        for (uint32_t i = nuc_thread(); i < room; i += kNucThreads) out[i] = nuc_bits(hi);
        return;
    }
    uint32_t* own = L.slot + 4 * nuc_thread();
    __syncthreads();  // L free
#pragma unroll
    for (int i = 0; i < 4; ++i) own[i] = 0;
    __syncthreads();
    nuc_each(lk, m, [&](uint32_t k) {
        const uint32_t d = hi - k;
        if (d <= range) nuc_count(L.slot, d);
    });
    __syncthreads();
    own = L.slot + 4 * nuc_thread();
    uint32_t total;
    uint32_t at = block_excl_scan(own[0] + own[1] + own[2] + own[3], L.w, &total);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t c = own[i];
        own[i] = at;
        at += c;
    }
    __syncthreads();
    total = uni(total);
    if (total > room) return;  // uniform; only when the row was rewritten while the call ran
    // short runs one wave each, 64 values a round; long ones the workgroup
    constexpr uint32_t kLong = 1024;
    const uint32_t w = uni(nuc_thread() / kWave);
#pragma unroll 1
    for (uint32_t b = 0; b <= range; b += kWave) {
        const uint32_t p = b + lane_id();
        const uint32_t first = L.slot[p], last = p + 1 < kNucParts ? L.slot[p + 1] : total;
        const uint64_t longer = __ballot(last - first > kLong), some = __ballot(last > first);
        const bool mine = b / kWave % kNucWaves == w;
#pragma unroll 1
        for (uint64_t runs = mine ? some : longer; runs != 0; runs &= runs - 1) {
            const int l = __builtin_ctzll(runs);
            const bool all = (longer >> l) & 1;
            const uint32_t n = lane_read(last, l) - lane_read(first, l), step = all ? kNucThreads : kWave;
            uint32_t* o = out + lane_read(first, l);
            const uint32_t v = nuc_bits(hi - (b + l));
#pragma unroll 1
            for (uint32_t i = all ? nuc_thread() : lane_id(); i < n; i += step) o[i] = v;
        }
    }
}

// The next window of the m keys at lk, those in [lo, top] left (kNucParts values
// or more): keys in [*from, *hi]; *fits 0: the key *hi alone, more often than
// that.  The keys left are counted in at most kNucParts equal parts of their range;
// the parts from the top that fit together are the window, and a first part that
// does not fit is cut up again.
__device__ void nuc_window(const uint32_t* lk, uint32_t m, uint32_t lo, uint32_t top,
                           uint32_t* from, uint32_t* hi, uint32_t* fits, uint32_t* s_v,
                           NucSortLds& L) {
    const uint32_t t = nuc_thread();
    while (true) {  // the range [lo, top] gets 4096 times smaller each time
        const uint32_t range = top - lo;
        const int bits = range ? 32 - __builtin_clz(range) : 0;
        const uint32_t sh = bits > 12 ? (uint32_t)(bits - 12) : 0u;
        __syncthreads();
        for (uint32_t i = t; i < kNucParts; i += kNucThreads) L.slot[i] = 0;
        if (t < 2) s_v[2 + t] = 0;
        __syncthreads();
        nuc_each(lk, m, [&](uint32_t k) {
            if (k >= lo && k <= top) nuc_count(L.slot, (top - k) >> sh);
        });
        __syncthreads();
        uint32_t total;
        uint32_t inc = block_excl_scan(L.slot[4 * t] + L.slot[4 * t + 1] + L.slot[4 * t + 2] +
                                           L.slot[4 * t + 3], L.w, &total);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            inc += L.slot[4 * t + i];
            if (inc <= kNucGroupMax) {
                atomicMax(&s_v[2], inc);
                atomicMax(&s_v[3], 4 * t + i + 1);  // parts that fit
            }
        }
        __syncthreads();
        *fits = uni(s_v[2]);
        *hi = top;
        if (*fits > 0) {
            const uint64_t span = (uint64_t)uni(s_v[3]) << sh;
            *from = span > range ? lo : top + 1u - (uint32_t)span;
            return;
        }
        if (sh == 0) {  // the largest key alone does not fit
            *from = top;
            return;
        }
        const uint32_t part = 1u << sh;  // the largest key's part
        lo = range >= part ? top - part + 1u : lo;
    }
}

// Of the m keys at `keys` (4-byte aligned; up to 3 words after them may be read)
// those in [lo, hi] (at most kNucGroupMax; of more only the number is right) to
// L.key, in any order; returns their number.  16-byte loads; per element of a
// lane the wave's kept ones go to consecutive LDS slots.
__device__ __forceinline__ uint32_t nuc_select(const uint32_t* keys, uint32_t m, uint32_t lo,
                                               uint32_t hi, uint32_t* s_n, NucSortLds& L) {
    const uint32_t t = nuc_thread();
    const u32x4_a4* k4 = reinterpret_cast<const u32x4_a4*>(keys);
    __syncthreads();
    if (t == 0) *s_n = 0;
    __syncthreads();
    const uint32_t range = hi - lo;
    constexpr int kLoads = 2, kEach = kLoads * 4;
    for (uint32_t b = 0; b < m; b += kEach * kNucThreads) {
        u32x4_a4 v[kLoads];
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const uint32_t i = b + (q * kNucThreads + t) * 4;  // what lies past m is masked
            v[q] = i < m ? k4[i / 4] : u32x4_a4{0u, 0u, 0u, 0u};
        }
        uint64_t mk[kEach];  // the wave's kept lanes, per element
        uint32_t cnt = 0;
        if (b + kEach * kNucThreads <= m) {  // uniform
#pragma unroll
            for (int q = 0; q < kEach; ++q) mk[q] = __ballot(v[q / 4][q % 4] - lo <= range);
        } else {
#pragma unroll
            for (int q = 0; q < kEach; ++q)
                mk[q] = __ballot(b + (q / 4 * kNucThreads + t) * 4 + q % 4 < m &&
                                 v[q / 4][q % 4] - lo <= range);
        }
#pragma unroll
        for (int q = 0; q < kEach; ++q) cnt += (uint32_t)__builtin_popcountll(mk[q]);
        if (cnt == 0) continue;  // uniform in the wave
        uint32_t at = 0;
        if (lane_id() == 0) at = atomicAdd(s_n, cnt);
        at = uni(at);
        if (at + cnt > kNucGroupMax) continue;  // only their number is wanted
#pragma unroll
        for (int q = 0; q < kEach; ++q) {
            const uint32_t to = at + lanes_below(mk[q]);
            if ((mk[q] >> lane_id()) & 1u) L.key[to] = v[q / 4][q % 4];
            at += (uint32_t)__builtin_popcountll(mk[q]);
        }
    }
    __syncthreads();
    return uni(*s_n);
}

// Workgroup blockIdx.x / rows of row blockIdx.x % rows takes every parts-th
// group of the row: its list slots, sorted; a group too large for LDS window by
// window.
__global__ __launch_bounds__(kNucThreads) LS_OCCUPANCY8 void k_nuc_sort(
    const uint32_t* keys, uint32_t stride, int32_t len, uint32_t rows, uint32_t parts,
    const NucRow* info, const uint2* groups, uint32_t slots, float* sorted) {
    __shared__ NucSortLds L;
    __shared__ uint32_t s_v[4];
    const uint32_t part = blockIdx.x / rows, row = blockIdx.x - part * rows;
    const uint2* gr = groups + (int64_t)row * (slots + 1);
    const uint32_t ng = uni(info[row].groups);
    for (uint32_t g = part; g < ng; g += parts) {
        const uint32_t first = uni(gr[g].x), m = uni(gr[g + 1].x) - first;
        const uint32_t* lk = keys + (int64_t)row * stride + first;
        uint32_t* out = reinterpret_cast<uint32_t*>(sorted) + (int64_t)row * len + first;
        uint32_t cap = UINT_MAX;
        for (uint32_t a = 0; a < m;) {  // once, unless m is too large; every step writes a key
            const bool big = m > kNucGroupMax;
            uint32_t from, hi, fits = 1, n = m;
            if (big) {
                uint32_t least, largest;
                nuc_limits(lk, m, cap, &least, &largest, s_v);
                if (least > largest) return;  // uniform; as below
                if (largest - least < kNucParts) {
                    nuc_emit(lk, m, least, largest, out + a, m - a, L);
                    break;
                }
                nuc_window(lk, m, least, largest, &from, &hi, &fits, s_v, L);
                n = nuc_select(lk, m, from, hi, s_v, L);
                // only when the row was rewritten while the call ran, so that the
                // list and the histogram disagree; the loop ends all the same
                if (n == 0 || a + n > m) return;  // uniform
                cap = from - 1u;
            }
            uint32_t* o = out + a;
            a += n;
            if (fits == 0) {  // one key, more often than fits
                for (uint32_t i = nuc_thread(); i < n; i += kNucThreads) o[i] = nuc_bits(hi);
                continue;
            }
            if (n > kNucGroupMax) return;  // never
            uint32_t key[kNucPer];
            const uint32_t t0 = nuc_thread();
#pragma unroll
            for (int e = 0; e < kNucPer; ++e) {
                const uint32_t i = t0 + e * kNucThreads;
                key[e] = i < n ? (big ? L.key[i] : lk[i]) : 0u;
            }
            nuc_range(key, n, &from, &hi, L);
            nuc_sort(key, n, from, hi, o, L);
        }
    }
}

// Rows of up to kNucGroupMax elements, whole.
__global__ __launch_bounds__(kNucThreads) void k_nuc_sort_row(const uint32_t* x, int32_t len,
                                                              float* sorted) {
    __shared__ NucSortLds L;
    const int64_t row = blockIdx.x;
    const uint32_t* xr = x + row * len;
    uint32_t key[kNucPer];
#pragma unroll
    for (int e = 0; e < kNucPer; ++e) {
        const uint32_t i = threadIdx.x + e * kNucThreads;
        key[e] = i < (uint32_t)len ? nuc_key(xr[i]) : 0u;
    }
    uint32_t lo, hi;
    nuc_range(key, (uint32_t)len, &lo, &hi, L);
    nuc_sort(key, (uint32_t)len, lo, hi, reinterpret_cast<uint32_t*>(sorted) + row * len, L);
}

// ---------------------------------------------------------------- launch

static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

// Tiles of 32768 positions when they occupy the chip, of 8192 otherwise (us a call
// at tiles of 32768 / 8192: 1 x 20000 44.6 / 36.9, 4 x 32000 47.1 / 37.4, 64 x 32000
// 52.8 / 40.7, 150 x 40000 70.0 / 67.5); rows beyond 2^18 have too many small ones
// for the tables (kNucMaxSegs).
static uint32_t nucleus_tile(int64_t rows, int64_t len) {
    return rows * len >= int64_t(256) * 32768 || len > (1 << 18) ? 32768u : 8192u;
}
// Elements per group: large groups read the list fewer times (four a row at
// p = 0.9 over softmax rows, so that the two workgroups of every CU sort the
// 512 of 128 rows in one round), small ones occupy the chip when there are few
// rows.  The rest up to kNucGroupMax is room for the group's last bin.
static uint32_t nucleus_window(int64_t rows, int64_t len) {
    return rows * len >= int64_t(256) * 32768 ? 11264u : kNucMinGroup;
}

struct NucLayout {
    uint32_t segs, window, slots, stride;
    size_t keys, idx, hist, above, maps, rows, groups, cursors, end;  // after the sorted keys
};
static NucLayout nucleus_layout(int64_t rows, int64_t len) {
    NucLayout l{};
    const size_t n = (size_t)rows * (size_t)len;
    l.keys = align256(n * 4);
    if (len <= (int64_t)kNucGroupMax) {
        l.end = l.keys;
        return l;
    }
    const uint32_t tile = nucleus_tile(rows, len);
    // rows that start off 16-byte boundaries: up to 3 positions before them
    l.segs = (uint32_t)((len + 3 + tile - 1) / tile);
    l.window = nucleus_window(rows, len);
    l.slots = (uint32_t)((len + l.window - 1) / l.window) * 2;  // the most groups a row can have
    l.stride = (uint32_t)((len + 3) / 4 * 4);
    const size_t tiles = (size_t)rows * l.segs;
    l.idx = l.keys + align256((size_t)rows * l.stride * 4);
    l.hist = l.idx + align256((size_t)rows * l.stride * 4);
    l.above = l.hist + tiles * kNucBins * sizeof(uint16_t);
    l.maps = l.above + align256(tiles * sizeof(double));
    l.rows = l.maps + (size_t)rows * kNucCells * sizeof(uint32_t);
    l.groups = l.rows + (size_t)rows * sizeof(NucRow);
    l.cursors = l.groups + (size_t)rows * (l.slots + 1) * sizeof(uint2);
    l.end = l.cursors + (size_t)rows * l.slots * sizeof(uint32_t);
    return l;
}

template <int J>
static void nucleus_bins(const uint32_t* x, int64_t rows, int64_t len, float p, uint32_t heads,
                         const NucLayout& l, char* s, hipStream_t stream) {
    uint16_t* hist = reinterpret_cast<uint16_t*>(s + l.hist);
    double* above = reinterpret_cast<double*>(s + l.above);
    uint32_t* maps = reinterpret_cast<uint32_t*>(s + l.maps);
    NucRow* info = reinterpret_cast<NucRow*>(s + l.rows);
    uint2* groups = reinterpret_cast<uint2*>(s + l.groups);
    uint32_t* cursors = reinterpret_cast<uint32_t*>(s + l.cursors);
    uint16_t* bin_groups = reinterpret_cast<uint16_t*>(maps);  // in the maps' place
    uint32_t* keys = reinterpret_cast<uint32_t*>(s + l.keys);
    uint32_t* idx = reinterpret_cast<uint32_t*>(s + l.idx);
    float* sorted = reinterpret_cast<float*>(s);
    const int32_t n = (int32_t)len;
    // 16-byte aligned rows need no room before their start
    const bool vec = len % 4 == 0 && (uintptr_t)x % 16 == 0;
    const uint32_t segs = vec ? (uint32_t)((len + 4096 * J - 1) / (4096 * J)) : l.segs;
    const unsigned tiles = (unsigned)(rows * segs);
    hipLaunchKernelGGL(k_nuc_hist<J>, dim3(tiles), dim3(kNucThreads), 0, stream, x, n,
                       (uint32_t)rows, segs, hist, info, maps, above,
                       kNucGroupMax - l.window < 4096u ? kNucGroupMax - l.window : 4096u);
    hipLaunchKernelGGL(k_nuc_pick, dim3((unsigned)rows), dim3(kNucThreads), 0, stream,
                       (const uint16_t*)hist, segs, (const uint32_t*)maps, p, n, info,
                       (const double*)above, l.window, l.slots, groups, cursors, bin_groups);
    hipLaunchKernelGGL(k_nuc_gather<J>, dim3(tiles), dim3(kNucThreads), 0, stream, x, n,
                       (uint32_t)rows, segs, (const NucRow*)info, (const uint16_t*)hist,
                       (const uint16_t*)bin_groups, (const uint2*)groups, cursors, l.slots, keys,
                       idx, l.stride);
    // as many workgroups a row as groups are usual, or as fit the chip at once
    // (two a CU), should that be more; those without a group cost 9 ns each
    const uint32_t want = (heads * 4096u * 5 / 4 + l.window - 1) / l.window;
    const uint32_t fit = (uint32_t)(512 / rows);
    const uint32_t most = want > fit ? want : fit;
    const uint32_t parts = most < l.slots ? most : l.slots;
    hipLaunchKernelGGL(k_nuc_sort, dim3((unsigned)rows * parts), dim3(kNucThreads), 0, stream,
                       (const uint32_t*)keys, l.stride, n, (uint32_t)rows, parts,
                       (const NucRow*)info, (const uint2*)groups, l.slots, sorted);
}

// The sorted rows (stride len) at the start of scratch (16-byte aligned; 16
// bytes per element hold everything): in every row as many elements as a draw
// at p with `heads` head tiles reads; *src: where their source indices are
// found.  Rows of up to kNucMaxLen elements.
hipError_t launch_nucleus_sort(const float* probs, float p, uint32_t heads, int64_t rows,
                               int64_t len, void* scratch, size_t scratch_bytes, NucSource* src,
                               hipStream_t stream) {
    const uint32_t* x = reinterpret_cast<const uint32_t*>(probs);
    char* s = reinterpret_cast<char*>(scratch);
    const NucLayout l = nucleus_layout(rows, len);
    if (len > kNucMaxLen || l.end > scratch_bytes) return hipErrorInvalidValue;  // not its rows
    *src = NucSource{};
    src->x = x;
    if (len <= (int64_t)kNucGroupMax) {
        hipLaunchKernelGGL(k_nuc_sort_row, dim3((unsigned)rows), dim3(kNucThreads), 0, stream, x,
                           (int32_t)len, reinterpret_cast<float*>(s));
        return hipGetLastError();
    }
    if (nucleus_tile(rows, len) == 32768u)
        nucleus_bins<8>(x, rows, len, p, heads, l, s, stream);
    else
        nucleus_bins<2>(x, rows, len, p, heads, l, s, stream);
    src->keys = reinterpret_cast<const uint32_t*>(s + l.keys);
    src->idx = reinterpret_cast<const uint32_t*>(s + l.idx);
    src->rows = reinterpret_cast<const NucRow*>(s + l.rows);
    src->groups = reinterpret_cast<const uint2*>(s + l.groups);
    src->slots = l.slots;
    src->stride = l.stride;
    return hipGetLastError();
}

}  // namespace ls
