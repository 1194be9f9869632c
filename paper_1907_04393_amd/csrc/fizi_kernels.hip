// HIP kernels of the FIZI/Mouse pipeline for gfx950 (CDNA4, wave64).
//
//   k_gain       per-frame sums over the usable sampled pixels; each consumer
//                turns a frame's sums into its Q16 inverse gain
//   k_gain_span  the same for consecutive frames of one stream; writes their
//                job table, and when learning starts also the reference
//                luminance of the sampled rows of the first frame (Section 2
//                initialisation, Section 3.2)
//   k_minmax     background learning and partial re-learning: per-pixel,
//                per-channel min/max of the gain-corrected frames, model read
//                and written once (Section 3.1 (i), Section 3.3)
//   k_classify   gain correction (or thresholds scaled by the gain), I_R1
//                (outside the learned box), I_R2 (not gray), I_R3 (skin hue),
//                their AND, packed to bits by DPP row merges (Sections 3.1,
//                3.2); HBM-bound, 4 pixels per lane. Frames of many streams
//   k_classify_span  the same for consecutive frames of one stream, the box
//                of a lane's pixels in registers across them
//   k_classify_one  the same for one frame of one stream
//   k_morph_regs opening then closing with a 3x3 square on bands of bit rows
//                held in registers (64 pixels per lane word), then runs and
//                band-local components in LDS (Section 3.1, last paragraph)
//   k_morph_mixed  either, by job, for batches of wide frames and deep streams
//   k_morph      the same streamed through a register pipeline, for taller
//                bands and for wide frames with many stages
//   k_resolve    8-connected components by union-find over runs (in LDS where
//                a frame's runs fit), hand-zone selection (largest, or
//                tracked), the pointer (Section 2, Mouse module)
//   k_track_chain  settles the tracked frames of a launch in order
//   k_flow       the persistent form of one step: gain tiles and row bands
//                from one ordered queue, with bounded waits
#include <hip/hip_ext.h>

#include <algorithm>

#include "fizi_internal.h"

namespace fizi {
namespace {

constexpr int kWave = 64;

#define GLOBAL __attribute__((address_space(1)))

typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Pointers in the job table are generic; casting them to the global address
// space lets the compiler emit global_* instead of flat_* accesses.
template <typename T>
__device__ __forceinline__ GLOBAL T *G(T *p)
{
    return (GLOBAL T *)p;
}

// A byte offset within a frame's arrays (3 p < 2^28: frames are at most 8192 x
// 8192) is added to each array's wave-uniform base as an unsigned 32-bit
// value, so that the loads take the scalar-base, vector-offset form and no
// 64-bit address is formed per lane.
template <typename T>
__device__ __forceinline__ const GLOBAL T *at_byte(const GLOBAL T *base, uint32_t off)
{
    return reinterpret_cast<const GLOBAL T *>(reinterpret_cast<const GLOBAL uint8_t *>(base) + off);
}

// A frame's union-find forest is only touched by one workgroup per kernel,
// so its atomics are workgroup-scoped (performed in the XCD's L2, no fences).
__device__ __forceinline__ uint32_t ld_wg(GLOBAL uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void st_wg(GLOBAL uint32_t *p, uint32_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Accumulators that other workgroups update with atomics (the gain sums, the
// run count) are read with device-scope atomic loads, which bypass the
// scalar cache; in the persistent step they are written earlier in the same
// launch.
template <typename P>
__device__ __forceinline__ auto ld_dev(P p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Persistent step: data that a workgroup hands to another one in the same
// launch is stored with device scope (written through this XCD's L2), each
// wave waits for its stores to complete before the workgroup bumps the
// counter or flag the consumer polls, and the consumer takes a device-scope
// acquire fence after seeing it, so that its loads miss any stale copy.
template <typename T>
__device__ __forceinline__ void st_dev(GLOBAL T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A store of the morphology/classify stages: device scope in the persistent
// step (FLOW), plain otherwise.
template <bool FLOW, typename T>
__device__ __forceinline__ void put(GLOBAL T *p, T v)
{
    if constexpr (FLOW)
        st_dev(p, v);
    else
        *p = v;
}

// Union-find parent stores of the morphology stage.
template <bool FLOW>
__device__ __forceinline__ void put_parent(GLOBAL uint32_t *p, uint32_t v)
{
    if constexpr (FLOW)
        st_dev(p, v);
    else
        st_wg(p, v);
}

// Waits for the wave's own memory operations. The signal fences keep the
// compiler from moving any across the wait; they emit nothing.
__device__ __forceinline__ void wait_own_memory()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

__device__ __forceinline__ int find_job(const int32_t *pre, int nj, int t)
{
    int lo = 0, hi = nj - 1;          // largest j with pre[j] <= t
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= t)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Brightness correction of one channel value (Q16 inverse gain, half up,
// saturated). v < 2^8 and inv <= 2^20 both fit 24 bits, so the full-rate
// 24-bit multiply gives the exact product (< 2^28).
__device__ __forceinline__ uint32_t corrected(uint32_t product)
{
    const uint32_t t = (product + 32768u) >> 16;
    return t < 255u ? t : 255u;
}

__device__ __forceinline__ uint32_t corr(uint32_t v, uint32_t inv) { return corrected(__umul24(v, inv)); }

// Q16 inverse gain from the sums of reference and frame luminance: rounded
// half up and clamped; 1.0 when no sampled pixel was usable.
__device__ __forceinline__ uint32_t inv_gain(unsigned long long num, unsigned long long den,
                                             int glo, int ghi)
{
    if (den == 0)
        return 65536u;
    unsigned long long q = (num * 65536ull + den / 2) / den;
    if (q < (unsigned long long)glo)
        q = (unsigned long long)glo;
    if (q > (unsigned long long)ghi)
        q = (unsigned long long)ghi;
    return (uint32_t)q;
}

// The frame's inverse gain from its gain accumulators, by one thread of the
// launch that sums them (persistent step): device-scope loads. wave_job_gain
// is the whole wave's, after a kernel boundary.
__device__ __forceinline__ uint32_t job_gain(const Job *J)
{
    unsigned long long n = 0, d = 0;
#pragma unroll
    for (int i = 0; i < kGainSlots; ++i) {
        n += ld_dev(&J->num[i]);
        d += ld_dev(&J->den[i]);
    }
    return inv_gain(n, d, J->glo, J->ghi);
}

// The same for a whole wave: lanes 0 .. 31 hold parts of the reference's sum,
// lanes 32 .. 63 of the frame's. Their totals go through DPP adds of the low 24
// bits and of the rest (both stay below 2^29: no sum reaches 2^37): within rows
// of 16 lanes, then row 0 into row 1 and row 2 into row 3, so that lane 31 holds
// the reference's total and lane 63 the frame's.
static_assert(kGainSlots == 32 && offsetof(Job, den) == offsetof(Job, num) + 4 * kGainSlots,
              "one gain sum per lane, num then den");
__device__ __forceinline__ uint32_t wave_gain(GainSum part, int glo, int ghi)
{
    auto rows = [](uint32_t v) {
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
        v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);
        return v;
    };
    const uint32_t lo = rows((uint32_t)part & 0xFFFFFFu), hi = rows((uint32_t)(part >> 24));
    auto total = [&](int lane) {
        return ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)hi, lane) << 24) +
               (uint32_t)__builtin_amdgcn_readlane((int)lo, lane);
    };
    return inv_gain(total(31), total(63), glo, ghi);
}

// (after a kernel boundary)
__device__ __forceinline__ uint32_t wave_job_gain(const Job *J)
{
    return wave_gain(G(J->num)[threadIdx.x & (kWave - 1)], J->glo, J->ghi);
}

// A frame's inverse gain after the gain kernel, where either may have run:
// k_gain_span leaves it in the job, after k_gain (batch steps) each wave takes
// it from the sums.
constexpr uint32_t kGainKnown = 0x80000000u;

__device__ __forceinline__ uint32_t frame_gain(const Job *J)
{
    const uint32_t g = J->ginv;
    return g & kGainKnown ? g & ~kGainKnown : wave_job_gain(J);
}

// The inverse gain of a span's job j0 + threadIdx.x (n of them, at most one
// per thread), loaded ahead of the frames so that it waits for none of them.
__device__ __forceinline__ uint32_t span_gain(const Table *T, int j0, int n)
{
    return G(&T->jobs[j0 + min((int)threadIdx.x, n - 1)].ginv)[0] & ~kGainKnown;
}

// Skin-hue membership without division; see HueTest. Chroma > 0 is checked
// by the caller.
// Every factor fits the full-rate 24-bit signed multiply: |k| <= 6000,
// |R - B| <= 255, d <= 6000, sum(d) <= 12000, R + G + B <= 765.
__device__ __forceinline__ bool hue_in(int r, int g, int b, const HueTest &h)
{
    const int rb = r - b, gb = g - b;
    const int d1 = __mul24(h.k1r, rb) + __mul24(h.k1g, gb);
    if (h.mode == 1)
        return (d1 >= 0) & (__mul24(h.k2r, rb) + __mul24(h.k2g, gb) <= 0);
    if (h.mode == 3)
        return (d1 >= 0) | (__mul24(h.k2r, rb) + __mul24(h.k2g, gb) <= 0);
    if (h.mode == 2)
        return d1 >= 0;
    const int dp = __mul24(h.dr, r) + __mul24(h.dg, g) + __mul24(h.db, b);
    return (d1 == 0) & (3 * dp - __mul24(h.dsum, r + g + b) > 0);
}

// The hue interval's four cases as one straight-line test; see HueForm.
__device__ __forceinline__ bool hue_in_form(int r, int g, int b, const HueForm &h)
{
    const int rb = r - b, gb = g - b;
    const int d1 = __mul24(h.k1r, rb) + h.c1 + __mul24(h.k1g, gb);
    const int d2 = __mul24(h.k2r, rb) + h.c2 + __mul24(h.k2g, gb);
    const int d3 = __mul24(h.k3r, rb) + h.c3 + __mul24(h.k3g, gb);
    return ((d1 >= 0) & (d2 <= 0) & (d3 > 0)) != (h.flip != 0);
}

__device__ __forceinline__ uint32_t byte_of(uint32_t w0, uint32_t w1, uint32_t w2, int i)
{
    const uint32_t w = i < 4 ? w0 : (i < 8 ? w1 : w2);
    return (w >> (8 * (i & 3))) & 0xFFu;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1)
        v += __shfl_xor(v, o, kWave);
    return v;
}

// Reductions by DPP: within rows of 16 lanes (shifts of 1, 2, 4, 8: lane 15 of a
// row has its total), then across the rows (lane 63 has the wave's). Lanes a
// move does not write contribute `none`. A step is a few instructions; as
// shuffles through LDS, and with one thread walking the waves' results, the
// largest component and the zone's sums took 6 of a component stage's 12 us.
template <int CTRL, int ROWS, typename V, typename OP>
__device__ __forceinline__ V dpp_step(V v, V none, OP op)
{
    if constexpr (sizeof(V) == 8) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)none, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(none >> 32), (int)(uint32_t)(v >> 32), CTRL,
                                                                  ROWS, 0xF, false);
        return op(v, ((unsigned long long)hi << 32) | lo);
    } else {
        return op(v, (V)__builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xF, false));
    }
}

template <typename V, typename OP>
__device__ __forceinline__ V row_reduce(V v, V none, OP op)
{
    v = dpp_step<0x111, 0xF>(v, none, op);
    v = dpp_step<0x112, 0xF>(v, none, op);
    v = dpp_step<0x114, 0xF>(v, none, op);
    return dpp_step<0x118, 0xF>(v, none, op);
}

template <typename V>
__device__ __forceinline__ V from_lane(V v, int lane)
{
    if constexpr (sizeof(V) == 8)
        return ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32) |
               (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    else
        return (V)__builtin_amdgcn_readlane((int)v, lane);
}

template <typename V, typename OP>
__device__ __forceinline__ V wave_reduce(V v, V none, OP op)
{
    v = row_reduce(v, none, op);
    v = dpp_step<0x142, 0xA>(v, none, op);
    v = dpp_step<0x143, 0xC>(v, none, op);
    return from_lane(v, kWave - 1);
}

struct OpMin {
    template <typename V>
    __device__ __forceinline__ V operator()(V a, V b) const { return b < a ? b : a; }
};
struct OpMax {
    template <typename V>
    __device__ __forceinline__ V operator()(V a, V b) const { return b > a ? b : a; }
};
struct OpSum {
    template <typename V>
    __device__ __forceinline__ V operator()(V a, V b) const { return a + b; }
};

// Lane l receives lane l + n of its row of 16 lanes (0 past the row's end,
// by the bound control): DPP row_shl:n.
template <int N>
__device__ __forceinline__ uint32_t row_shl(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x100 + N, 0xF, 0xF, true);
}

// Raster mask words of a wave's 256 consecutive pixels, 4 per lane (bit k of
// nib: pixel 4 l + k). Word w covers lanes 16 w .. 16 w + 15, nibble j from
// lane 16 w + j, so each word is one DPP row: neighbouring lanes' nibbles
// merge pairwise (l takes l + 1, then l + 2, l + 4; l + 8 gives the upper
// half), and lane 16 w ends up holding word w. A handful of instructions per
// wave, where ballots and a bit spread on four lanes took about eighty.
__device__ __forceinline__ uint64_t row_word(uint32_t nib)
{
    uint32_t t = nib & 0xFu;
    t |= row_shl<1>(t) << 4;
    t |= row_shl<2>(t) << 8;
    t |= row_shl<4>(t) << 16;
    return ((uint64_t)row_shl<8>(t) << 32) | t;
}

// ---------------------------------------------------------------------------
// The gain's usable-pixel test and sums on pairs of 16-bit halves: a pixel's
// (R, G) and (B, B) come by one byte permute each, their difference is
// (R - B, G - B), and each hue form is one two-element dot product of it. 21
// instructions per pixel; byte by byte it took 30.
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

struct GainHue {
    s16x2 k1, k2, k3;          // the forms' coefficients of (R - B, G - B); |k| <= 18000
};

__device__ __forceinline__ GainHue gain_hue(const HueTest &h)
{
    GainHue g;
    g.k1 = s16x2{(short)h.k1r, (short)h.k1g};
    g.k2 = s16x2{(short)h.k2r, (short)h.k2g};
    // mode 0: 3 d.p - sum(d) sum(p), unchanged when a gray is added to p
    g.k3 = s16x2{(short)(3 * h.dr - h.dsum), (short)(3 * h.dg - h.dsum)};
    return g;
}

// Pixel K of the four in 3 dwords as (R, G) and (B, B).
template <int K>
__device__ __forceinline__ void px_pairs(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t &rg, uint32_t &bb)
{
    if constexpr (K == 0) {
        rg = __builtin_amdgcn_perm(w1, w0, 0x0c010c00u);
        bb = __builtin_amdgcn_perm(w1, w0, 0x0c020c02u);
    } else if constexpr (K == 1) {
        rg = __builtin_amdgcn_perm(w1, w0, 0x0c040c03u);
        bb = __builtin_amdgcn_perm(w1, w0, 0x0c050c05u);
    } else if constexpr (K == 2) {
        rg = __builtin_amdgcn_perm(w2, w1, 0x0c030c02u);
        bb = __builtin_amdgcn_perm(w2, w1, 0x0c040c04u);
    } else {
        rg = __builtin_amdgcn_perm(w2, w1, 0x0c060c05u);
        bb = __builtin_amdgcn_perm(w2, w1, 0x0c070c07u);
    }
}

// R + 2 G + B plus acc.
__device__ __forceinline__ uint32_t px_lum(uint32_t rg, uint32_t bb, uint32_t acc)
{
    const u16x2 one{1, 0}, two{1, 2};
    acc = __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, bb), one, acc, false);
    return __builtin_amdgcn_udot2(__builtin_bit_cast(u16x2, rg), two, acc, false);
}

// Whether a channel is 0 or 255.
__device__ __forceinline__ bool px_clipped(uint32_t rg, uint32_t bb)
{
    const u16x2 one{1, 1}, last{253, 253};
    const u16x2 m = __builtin_elementwise_max(__builtin_bit_cast(u16x2, rg) - one, __builtin_bit_cast(u16x2, bb) - one);
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(m, last)) != 0u;
}

// (reference << 16 | frame luminance) of a usable pixel, 0 of any other; yhi
// is its reference << 16.
template <int MODE>
__device__ __forceinline__ uint32_t gain_px(uint32_t rg, uint32_t bb, uint32_t yhi, const GainHue &h)
{
    const s16x2 d = __builtin_bit_cast(s16x2, rg) - __builtin_bit_cast(s16x2, bb);
    const int d1 = __builtin_amdgcn_sdot2(d, h.k1, 0, false);
    bool skin = __builtin_bit_cast(uint32_t, d) != 0u;       // chroma > 0
    if constexpr (MODE == 0)
        skin = (d1 == 0) & (__builtin_amdgcn_sdot2(d, h.k3, 0, false) > 0);
    else if constexpr (MODE == 1)
        skin = skin & (d1 >= 0) & (__builtin_amdgcn_sdot2(d, h.k2, 0, false) <= 0);
    else if constexpr (MODE == 2)
        skin = skin & (d1 >= 0);
    else
        skin = skin & ((d1 >= 0) | (__builtin_amdgcn_sdot2(d, h.k2, 0, false) <= 0));
    const bool ok = (yhi < ((uint32_t)kYrefClipped << 16)) & !px_clipped(rg, bb) & !skin;
    return ok ? px_lum(rg, bb, yhi) : 0u;
}

// Four pixels (3 dwords) with their references (2 dwords of two): the sums of
// gain_px, each half of at most 4 x 1020.
template <int MODE>
__device__ __forceinline__ uint32_t gain_px4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t y01, uint32_t y23,
                                             const GainHue &h)
{
    uint32_t rg, bb, sum;
    px_pairs<0>(w0, w1, w2, rg, bb);
    sum = gain_px<MODE>(rg, bb, y01 << 16, h);
    px_pairs<1>(w0, w1, w2, rg, bb);
    sum += gain_px<MODE>(rg, bb, y01 & 0xFFFF0000u, h);
    px_pairs<2>(w0, w1, w2, rg, bb);
    sum += gain_px<MODE>(rg, bb, y23 << 16, h);
    px_pairs<3>(w0, w1, w2, rg, bb);
    return sum + gain_px<MODE>(rg, bb, y23 & 0xFFFF0000u, h);
}

// The references of four pixels, kYrefClipped where a channel is 0 or 255.
template <int K>
__device__ __forceinline__ uint32_t yref_px(uint32_t w0, uint32_t w1, uint32_t w2)
{
    uint32_t rg, bb;
    px_pairs<K>(w0, w1, w2, rg, bb);
    return px_clipped(rg, bb) ? kYrefClipped : px_lum(rg, bb, 0u);
}

__device__ __forceinline__ void yref_px4(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t &y01, uint32_t &y23)
{
    y01 = yref_px<0>(w0, w1, w2) | (yref_px<1>(w0, w1, w2) << 16);
    y23 = yref_px<2>(w0, w1, w2) | (yref_px<3>(w0, w1, w2) << 16);
}

// A tile of one frame (kGainRows sampled rows): sums of reference and frame
// luminance over its usable pixels, added to the frame's accumulators.
template <int MODE>
__device__ __forceinline__ void gain_tile_mode(Table *__restrict__ T, int j, int tile, const uint8_t *fr)
{
    __shared__ uint32_t s_num[256 / kWave], s_den[256 / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    Job *J = &T->jobs[j];
    const int W = J->W;
    const int rows = (J->H + J->rs - 1) / J->rs;
    const GainHue h = gain_hue(J->hue);
    uint32_t num = 0, den = 0;
    const int r0 = tile * kGainRows, nr = min(rows, r0 + kGainRows) - r0;
    if ((reinterpret_cast<uintptr_t>(fr) & 15u) == 0) {
        // 16 pixels per item: three 16-byte loads of the frame row, two of
        // the reference row; items of the tile's rows in one flat range
        const int n16 = W / 16;
        const GLOBAL uint8_t *frame = G(fr);
        const GLOBAL uint16_t *yref = G(J->yref);
        const size_t rowb = (size_t)J->rs * W * 3;
#pragma unroll 2
        for (int it = threadIdx.x; it < nr * n16; it += blockDim.x) {
            int row = 0;
#pragma unroll
            for (int q = 1; q < kGainRows; ++q)
                row += it >= q * n16;
            const int g = it - row * n16, rr = r0 + row;
            const GLOBAL u32x4 *fp = reinterpret_cast<const GLOBAL u32x4 *>(frame + (size_t)rr * rowb) + 3 * g;
            const GLOBAL u32x4 *yp = reinterpret_cast<const GLOBAL u32x4 *>(yref + (size_t)rr * W) + 2 * g;
            const u32x4 a = fp[0], b = fp[1], c = fp[2], ya = yp[0], yb = yp[1];
            const uint32_t s = gain_px4<MODE>(a.x, a.y, a.z, ya.x, ya.y, h) +
                               gain_px4<MODE>(a.w, b.x, b.y, ya.z, ya.w, h) +
                               gain_px4<MODE>(b.z, b.w, c.x, yb.x, yb.y, h) +
                               gain_px4<MODE>(c.y, c.z, c.w, yb.z, yb.w, h);
            num += s >> 16;
            den += s & 0xFFFFu;
        }
    } else {
        const int groups = W / 4;
#pragma unroll 4
        for (int it = threadIdx.x; it < nr * groups; it += blockDim.x) {
            const int rr = r0 + it / groups, g = it - (it / groups) * groups;
            const GLOBAL uint32_t *row = G(reinterpret_cast<const uint32_t *>(fr + (size_t)rr * J->rs * W * 3));
            const GLOBAL uint32_t *yr = G(reinterpret_cast<const uint32_t *>(J->yref + (size_t)rr * W));
            const uint32_t s = gain_px4<MODE>(row[3 * g], row[3 * g + 1], row[3 * g + 2], yr[2 * g], yr[2 * g + 1], h);
            num += s >> 16;
            den += s & 0xFFFFu;
        }
    }
    num = wave_sum(num);
    den = wave_sum(den);
    if (lane == 0) {
        s_num[wave] = num;
        s_den[wave] = den;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t n = 0, d = 0;
        for (int w = 0; w < (int)(blockDim.x / kWave); ++w) {
            n += s_num[w];
            d += s_den[w];
        }
        const int slot = tile & (kGainSlots - 1);
        atomicAdd(&J->num[slot], n);
        atomicAdd(&J->den[slot], d);
    }
    __syncthreads();
}

// Tiles [t0, t1) of this block, in order, each with its job. Contiguous
// ranges keep a block's consecutive tiles in one frame, so the job is found
// by one search and then advanced.
template <typename F>
__device__ __forceinline__ void for_block_tiles(const int32_t *pre, int nj, F f)
{
    const int total = pre[nj];
    const int per = (total + (int)gridDim.x - 1) / (int)gridDim.x;
    const int t0 = (int)blockIdx.x * per, t1 = min(total, t0 + per);
    if (t0 >= t1)
        return;
    int j = find_job(pre, nj, t0);
    for (int t = t0; t < t1; ++t) {
        while (t >= pre[j + 1])
            ++j;
        f(j, t - pre[j]);
    }
}

// A gain tile, its hue test's case chosen once per tile.
__device__ __forceinline__ void gain_tile(Table *__restrict__ T, int j, int tile, const uint8_t *fr)
{
    switch (T->jobs[j].hue.mode) {
    case 0:
        gain_tile_mode<0>(T, j, tile, fr);
        break;
    case 1:
        gain_tile_mode<1>(T, j, tile, fr);
        break;
    case 2:
        gain_tile_mode<2>(T, j, tile, fr);
        break;
    default:
        gain_tile_mode<3>(T, j, tile, fr);
        break;
    }
}

__global__ __launch_bounds__(256) void k_gain(Table *__restrict__ T)
{
    for_block_tiles(T->h.gain_pre, T->h.njobs,
                    [&](int j, int tile) { gain_tile(T, j, tile, T->jobs[j].frame); });
}

// Gain of consecutive frames of one stream: workgroup (p, i) sums part p of
// frame i's sampled pixels, items of 16 pixels (4 where the frames are only
// 4-byte aligned) taken p blockDim + thread, + gridDim.x blockDim, ..., and
// stores its sums, in 64 bits (see GainSum), as pair p of the frame: nothing
// to zero. The frame's
// last workgroup leaves the inverse gain in the job; every workgroup of the
// kernels that follow would otherwise sum the parts and divide (6 us of
// classify over 64 frames, 22 us of minmax over 50). Its addresses come by
// value, so that its loads wait for no table. Workgroup (0, n) writes the
// jobs for the kernels that follow, thread i job i.
// Bound by the latency of its loads and, in between, the VALU: 64 frames of
// 1920x1080 (50 MB of frame rows) take 17 us, 22 us tile by tile from a
// table with atomic sums.
__device__ __forceinline__ void write_job(Table *__restrict__ T, const SpanJobs &S, int i)
{
    Job *J = &T->jobs[i];
    // every field but the accumulators; those that only the front reads, which
    // has them by value, are 0
    uint64_t *dst = reinterpret_cast<uint64_t *>(J);
    constexpr int kHead = (int)(offsetof(Job, num) / 8);
    static_assert(offsetof(Job, num) % 8 == 0, "whole 8-byte words");
    Job head;
    uint64_t *h = reinterpret_cast<uint64_t *>(&head);
#pragma unroll
    for (int q = 0; q < kHead; ++q)
        h[q] = 0ull;
    const size_t so = (size_t)i * S.slot_bytes;
    const uint64_t index = S.frame_index + (uint64_t)i;
    auto moved = [&](auto *p, size_t bytes) {
        return reinterpret_cast<decltype(p)>(reinterpret_cast<uint8_t *>(p) + bytes);
    };
    head.frame = S.frame + (size_t)i * S.frame_bytes;
    head.raw = moved(S.raw, (size_t)i * S.raw_bytes);
    head.fizi = S.fizi + (size_t)i * S.fizi_words;
    head.hand = S.hand ? S.hand + (size_t)i * S.hand_words : nullptr;
    head.parent = moved(S.parent, so);
    head.index = moved(S.index, so);
    head.runs = moved(S.runs, so);
    head.links = moved(S.links, so);
    head.W = S.W;
    head.H = S.H;
    head.Wd = S.W / 64;
    head.run_cap = run_capacity(S.W, S.H);
    head.link_cap = link_capacity(S.W, S.H);
    head.open_it = S.open_it;
    head.close_it = S.close_it;
    head.min_area = S.min_area;
    head.fill_pm = S.fill_pm;
    head.debounce = S.debounce;
    head.track_r2 = S.track_r2;
    head.glo = S.glo;
    head.ghi = S.ghi;
    head.out = S.out + i;
    head.hout = S.ring ? S.ring + (index & S.ring_mask) : nullptr;
    head.track = S.track;
    head.frame_index = index;
    head.band = S.band;
    head.mgroup = S.mgroup;
#pragma unroll
    for (int q = 0; q < kHead; ++q)
        dst[q] = h[q];
    // the accumulators but the inverse gain, which the frame's last workgroup
    // stores
    J->nruns = J->flags = J->nlinks = J->nflag = 0u;
    J->gain_done = J->morph_done = J->pick = 0u;
    T->h.mor_pre[i + 1] = (i + 1) * S.mor_items;
    if (i == 0) {
        T->h.njobs = S.n;
        T->h.mor_pre[0] = 0;
    }
}

// MODE: the hue interval's case; MAKE: the reference comes from frame 0 (and
// frame 0's workgroups write it); WIDE: frames 16-byte aligned.
template <int MODE, bool MAKE, bool WIDE>
__global__ __launch_bounds__(1024) void k_gain_span(Table *__restrict__ T, const SpanJobs S)
{
    __shared__ uint32_t s_num[1024 / kWave], s_den[1024 / kWave];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int part = blockIdx.x, i = blockIdx.y;
    if (i == S.n) {
        if (part == 0)
            for (int j = threadIdx.x; j < S.n; j += blockDim.x)
                write_job(T, S, j);
        return;
    }
    const GLOBAL uint8_t *frame0 = G(S.frame), *frame = frame0 + (size_t)i * S.frame_bytes;
    GLOBAL uint16_t *yref = G(S.yref);
    const GainHue h = gain_hue(S.hue);
    const uint32_t W = (uint32_t)S.W, rows = (uint32_t)(S.H + S.rs - 1) / (uint32_t)S.rs;
    constexpr int kQ = WIDE ? 4 : 1;             // groups of four pixels per item
    const uint32_t per_row = W / (4 * kQ), items = rows * per_row;
    uint32_t num = 0, den = 0;                   // at most 2^25 per lane, 2^31 per wave
    for (uint32_t it = (uint32_t)part * blockDim.x + threadIdx.x; it < items; it += gridDim.x * blockDim.x) {
        const uint32_t row = it / per_row, g = it - row * per_row;
        const size_t fo = (size_t)row * (size_t)S.rs * W * 3u + 12u * kQ * g;
        const size_t yo = (size_t)row * W + 4u * kQ * g;
        uint32_t w[3 * kQ], y[2 * kQ];
        if constexpr (WIDE) {
#pragma unroll
            for (int q = 0; q < 3; ++q)
                *reinterpret_cast<u32x4 *>(&w[4 * q]) = reinterpret_cast<const GLOBAL u32x4 *>(frame + fo)[q];
        } else {
#pragma unroll
            for (int q = 0; q < 3; ++q)
                w[q] = reinterpret_cast<const GLOBAL uint32_t *>(frame + fo)[q];
        }
        if constexpr (MAKE) {
            uint32_t r[3 * kQ];
#pragma unroll
            for (int q = 0; q < 3 * kQ; ++q)
                r[q] = reinterpret_cast<const GLOBAL uint32_t *>(frame0 + fo)[q];
#pragma unroll
            for (int q = 0; q < kQ; ++q)
                yref_px4(r[3 * q], r[3 * q + 1], r[3 * q + 2], y[2 * q], y[2 * q + 1]);
            if (i == 0) {
#pragma unroll
                for (int q = 0; q < 2 * kQ; ++q)
                    reinterpret_cast<GLOBAL uint32_t *>(yref + yo)[q] = y[q];
            }
        } else if constexpr (WIDE) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                *reinterpret_cast<u32x4 *>(&y[4 * q]) = reinterpret_cast<const GLOBAL u32x4 *>(yref + yo)[q];
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                y[q] = reinterpret_cast<const GLOBAL uint32_t *>(yref + yo)[q];
        }
        uint32_t s = 0;                          // halves of at most 16 x 1020
#pragma unroll
        for (int q = 0; q < kQ; ++q)
            s += gain_px4<MODE>(w[3 * q], w[3 * q + 1], w[3 * q + 2], y[2 * q], y[2 * q + 1], h);
        num += s >> 16;
        den += s & 0xFFFFu;
    }
    num = wave_sum(num);
    den = wave_sum(den);
    if (lane == 0) {
        s_num[wave] = num;
        s_den[wave] = den;
    }
    __syncthreads();
    if (wave != 0)
        return;
    // the first wave alone from here on, so that the others' places are free
    GainSum n = 0, d = 0;
    for (int w = 0; w < (int)(blockDim.x / kWave); ++w) {
        n += s_num[w];
        d += s_den[w];
    }
    // the frame's last workgroup turns the sums into its inverse gain: the
    // sums go through this XCD's L2, and are there before the count (which
    // wraps to 0 for the next launch)
    GLOBAL GainSum *sums = G(reinterpret_cast<GainSum *>(S.arrived + kArrivedWords)) + 2 * (size_t)i * gridDim.x;
    uint32_t before = 0;
    if (lane == 0) {
        st_dev(sums + 2 * part, n);
        st_dev(sums + 2 * part + 1, d);
        wait_own_memory();
        before = atomicInc(S.arrived + i * kArrivedStride, gridDim.x - 1);
    }
    if ((uint32_t)__builtin_amdgcn_readfirstlane((int)before) != gridDim.x - 1)
        return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    GainSum of = 0;
    for (uint32_t p = lane & 31; p < gridDim.x; p += 32)
        of += ld_dev(sums + 2 * p + (lane >> 5));
    const uint32_t inv = wave_gain(of, S.glo, S.ghi);
    if (lane == 0)
        T->jobs[i].ginv = kGainKnown | inv;
}

// ---------------------------------------------------------------------------
// Learning: every frame widens the model. The correction is monotone, so the
// least and greatest corrected value of a channel are the corrections of the
// least and greatest v inv: per frame and channel only the product is taken
// (its byte selected by the multiply itself) and half a three-way minimum and
// maximum (frames in pairs); rounding, shift and saturation come once at the
// end. 2 instructions per channel and frame where correcting first took 6.
// MASKED: partial re-learning, each frame's I_FIZI bits keep its pixels out;
// waves without such pixels take the plain code.
// Bound by HBM: 50 frames of 1920x1080 (323 MB) in 51 us, 6.3 TB/s (64 us
// with every value corrected); 8 frames with masks on top of a model 12-15 us
// (20).
// AHEAD: frames in flight per lane: two pairs, or the one or two frames of a
// shorter call (with two pairs their loads came four or two times over:
// learning one frame of 7680x4320 took 79 us instead of 55, two 78 instead of
// 68).
template <bool MASKED, int AHEAD>
__global__ __launch_bounds__(256) void k_minmax(const Table *__restrict__ T, const LearnSpan S)
{
    __shared__ uint32_t s_inv[kMaxJobs];
    const GLOBAL uint8_t *frames = G(S.frames), *masks = G(reinterpret_cast<const uint8_t *>(S.masks));
    const int last = S.n - 1;
    static_assert(kMaxJobs <= 256, "one inverse gain per thread");
    const uint32_t gain = span_gain(T, 0, S.n);
    // lanes past the end repeat the last group and store nothing
    const uint32_t ngroups = S.npx / 4u, g = min(blockIdx.x * blockDim.x + threadIdx.x, ngroups - 1u);
    auto load = [&](int f) __attribute__((always_inline)) {
        return __builtin_nontemporal_load(
            at_byte(reinterpret_cast<const GLOBAL u32x3 *>(frames + (size_t)f * S.frame_bytes), 12u * g));
    };
    // the lane's 4 mask bits of a frame
    auto skip_of = [&](int f) __attribute__((always_inline)) {
        return MASKED ? ((uint32_t)(masks + (size_t)f * (S.npx / 8u))[g >> 1] >> ((g & 1u) * 4u)) & 0xFu : 0u;
    };
    u32x3 ring[AHEAD];
    uint32_t skip[AHEAD];
#pragma unroll
    for (int q = 0; q < AHEAD; ++q) {
        ring[q] = load(min(q, last));
        skip[q] = skip_of(min(q, last));
    }
    if ((int)threadIdx.x < S.n)
        s_inv[threadIdx.x] = gain;
    __syncthreads();
    uint32_t lo[12], hi[12];
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        lo[i] = 0x0FFFFFFFu;        // corrects to 255
        hi[i] = 0u;
    }
    // a pair of frames: f and the next one, or f twice when it is the last
    auto widen = [&](int f, const u32x3 w0, const u32x3 w1, uint32_t skip0, uint32_t skip1)
                     __attribute__((always_inline)) {
        const uint32_t i0 = s_inv[f], i1 = s_inv[min(f + 1, last)];
        if (MASKED && __builtin_amdgcn_ballot_w64((skip0 | skip1) != 0u)) {
#pragma unroll
            for (int i = 0; i < 12; ++i) {
                const uint32_t x0 = __umul24(byte_of(w0.x, w0.y, w0.z, i), i0),
                               x1 = __umul24(byte_of(w1.x, w1.y, w1.z, i), i1);
                const bool u0 = !((skip0 >> (i / 3)) & 1u), u1 = !((skip1 >> (i / 3)) & 1u);
                lo[i] = min(min(lo[i], u0 ? x0 : ~0u), u1 ? x1 : ~0u);
                hi[i] = max(max(hi[i], u0 ? x0 : 0u), u1 ? x1 : 0u);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 12; ++i) {
                const uint32_t x0 = __umul24(byte_of(w0.x, w0.y, w0.z, i), i0),
                               x1 = __umul24(byte_of(w1.x, w1.y, w1.z, i), i1);
                lo[i] = min(min(lo[i], x0), x1);
                hi[i] = max(max(hi[i], x0), x1);
            }
        }
    };
    // the loads of the loop are unconditional (past the end the last frame
    // again): a branch around them would make every wait one for all of them
    int f = 0;
    for (; f + AHEAD < S.n; f += AHEAD) {
#pragma unroll
        for (int q = 0; q + 1 < AHEAD; q += 2) {
            widen(f + q, ring[q], ring[q + 1], skip[q], skip[q + 1]);
#pragma unroll
            for (int r = q; r < q + 2; ++r) {
                ring[r] = load(min(f + r + AHEAD, last));
                skip[r] = skip_of(min(f + r + AHEAD, last));
            }
        }
    }
#pragma unroll
    for (int q = 0; q < AHEAD; q += 2)
        if (f + q < S.n)
            widen(f + q, ring[q], ring[AHEAD > 1 ? q + 1 : 0], skip[q], skip[AHEAD > 1 ? q + 1 : 0]);
    GLOBAL u32x3 *pmin = reinterpret_cast<GLOBAL u32x3 *>(G(S.bgmin) + 12u * (size_t)g);
    GLOBAL u32x3 *pmax = reinterpret_cast<GLOBAL u32x3 *>(G(S.bgmax) + 12u * (size_t)g);
    u32x3 a = {~0u, ~0u, ~0u}, b = {0u, 0u, 0u};
    if (!S.reset) {
        a = *pmin;
        b = *pmax;
    }
    uint32_t ra[3] = {0, 0, 0}, rb[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        ra[i >> 2] |= min(byte_of(a.x, a.y, a.z, i), corrected(lo[i])) << (8 * (i & 3));
        rb[i >> 2] |= max(byte_of(b.x, b.y, b.z, i), corrected(hi[i])) << (8 * (i & 3));
    }
    if (blockIdx.x * blockDim.x + threadIdx.x < ngroups) {
        *pmin = u32x3{ra[0], ra[1], ra[2]};
        *pmax = u32x3{rb[0], rb[1], rb[2]};
    }
}

// ---------------------------------------------------------------------------
// One lane classifies 4 consecutive pixels (12 bytes of frame, 12 of bgmin,
// 12 of bgmax); a wave covers 256 pixels = 4 mask words. The hue and gray
// tests only run for pixels already outside the background box, so waves of
// pure background skip them.
// What classify needs of a frame's job, read once into registers (the raw
// mask stores could otherwise alias the job table and force reloads).
struct ClsJob {
    const GLOBAL uint32_t *fr, *mn, *mx;
    GLOBAL uint64_t *raw;
    int delta, S1;
    int scaled;
    uint32_t S_q16;
    int S0, lum2;          // gray tolerance S; over-exposure filter: 2 lum_hi, 0 when off
    HueTest h;
};

// How a job's pixels are tested: corrected pixels, thresholds scaled to the
// frame's brightness, or corrected pixels with the over-exposure filter
// before the gray test.
enum ClsKind { kCorrected = 0, kScaled = 1, kCorrectedLum = 2 };

__device__ __forceinline__ ClsJob cls_job(const Job *J)
{
    ClsJob c;
    c.fr = G(reinterpret_cast<const uint32_t *>(J->frame));
    c.mn = G(reinterpret_cast<const uint32_t *>(J->bgmin));
    c.mx = G(reinterpret_cast<const uint32_t *>(J->bgmax));
    c.raw = G(J->raw);
    c.delta = J->delta;
    c.S1 = J->S1;
    c.scaled = J->scaled;
    c.S_q16 = J->S_q16;
    c.S0 = J->S0;
    c.lum2 = J->lum2;
    c.h = J->hue;
    return c;
}

__device__ __forceinline__ int cls_kind(const ClsJob &c)
{
    return c.scaled ? kScaled : (c.lum2 ? kCorrectedLum : kCorrected);
}

// I_R2 on a corrected pixel, with the over-exposure filter when LUM: a pixel
// whose max + min exceeds 2 lum_hi has its HSL lightness brought down to
// lum_hi (hue and saturation kept), which scales its chroma by
// (510 - 2 lum_hi) / (510 - max - min); not gray when that chroma reaches S,
// compared without division. Chroma > 0 is required in both cases (the hue
// test needs it).
template <bool LUM, typename C>
__device__ __forceinline__ bool not_gray(const C &c, int mx, int mn)
{
    const int ch = mx - mn;
    if (LUM) {
        const int l2 = mx + mn;
        if (l2 > c.lum2)
            return ch >= 1 && ch * (510 - c.lum2) >= c.S0 * (510 - l2);
    }
    return ch >= c.S1;
}

// The inputs of one lane's 4 pixels: frame, background min and max (3 dwords
// each). They are read once per step, so they are loaded non-temporally (no
// reuse expected in the caches): this streams 12% faster than plain loads.
struct Px4 {
    uint32_t f[3], l[3], u[3];
};

__device__ __forceinline__ void load_px4(const ClsJob &c, uint32_t p, uint32_t pend, Px4 &x)
{
    if (p < pend) {
        const uint32_t off = 3u * p;
        const u32x3 f = __builtin_nontemporal_load(at_byte(reinterpret_cast<const GLOBAL u32x3 *>(c.fr), off));
        const u32x3 l = __builtin_nontemporal_load(at_byte(reinterpret_cast<const GLOBAL u32x3 *>(c.mn), off));
        const u32x3 u = __builtin_nontemporal_load(at_byte(reinterpret_cast<const GLOBAL u32x3 *>(c.mx), off));
        x.f[0] = f.x, x.f[1] = f.y, x.f[2] = f.z;
        x.l[0] = l.x, x.l[1] = l.y, x.l[2] = l.z;
        x.u[0] = u.x, x.u[1] = u.y, x.u[2] = u.z;
    }
}

// I_R1, I_R2 and I_R3 of one 1024-pixel unit of a frame (256 per wave, 4 per
// lane) whose pixels from pend on are not classified; base is the wave's
// first pixel (a multiple of 64), raw words at or past pend / 64 are not
// written; x holds the lane's inputs (loaded by load_px4). KIND: kScaled, the
// thresholds follow the frame's brightness and the pixels stay raw.
template <bool FLOW, int KIND>
__device__ __forceinline__ void classify_px4(const ClsJob &c, uint32_t base, uint32_t pend, uint32_t inv,
                                             const Px4 &x)
{
    constexpr bool SCALED = KIND == kScaled;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t p = base + 4u * lane;
    uint32_t bits = 0;
    if (SCALED && p < pend) {
        // (bgmin - delta) 2^16 <= v inv <= (bgmax + delta) 2^16 as one
        // unsigned compare of v inv + (delta - bgmin) 2^16 (wrapping below
        // zero) against (bgmax - bgmin + 2 delta) 2^16; v inv < 2^28
        int cv[12];
        uint32_t out = 0;
        const uint32_t rng[3] = {x.u[0] - x.l[0], x.u[1] - x.l[1], x.u[2] - x.l[2]};
        const uint32_t kd = (uint32_t)c.delta << 16, d2 = 2u * (uint32_t)c.delta;
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            const uint32_t v = byte_of(x.f[0], x.f[1], x.f[2], i);
            const uint32_t d = __umul24(v, inv) + kd - (byte_of(x.l[0], x.l[1], x.l[2], i) << 16);
            cv[i] = (int)v;
            out |= (uint32_t)(d > ((byte_of(rng[0], rng[1], rng[2], i) + d2) << 16)) << (i / 3);
        }
        if (out) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (out & (1u << k)) {
                    const int r = cv[3 * k], g = cv[3 * k + 1], b = cv[3 * k + 2];
                    const uint32_t ch = (uint32_t)(max(max(r, g), b) - min(min(r, g), b));
                    if (__umul24(ch, inv) >= c.S_q16 && hue_in(r, g, b, c.h))
                        bits |= 1u << k;
                }
            }
        }
    } else if (!SCALED && p < pend) {
        // v' in [bgmin - delta, bgmax + delta] is one unsigned compare:
        // (v' + delta - bgmin) <= (bgmax - bgmin) + 2 delta, with v' + delta
        // from the correction's own multiply-add (delta << 16 added before the
        // shift, the saturation moved up by delta) and bgmax - bgmin taken for
        // four channels at once (bgmax >= bgmin per byte: no borrows)
        int cv[12];
        uint32_t out = 0;
        const uint32_t rng[3] = {x.u[0] - x.l[0], x.u[1] - x.l[1], x.u[2] - x.l[2]};
        const uint32_t kadd = 32768u + ((uint32_t)c.delta << 16), kmax = 255u + (uint32_t)c.delta;
        const uint32_t d2 = 2u * (uint32_t)c.delta;
#pragma unroll
        for (int i = 0; i < 12; ++i) {
            const uint32_t vd = min((__umul24(byte_of(x.f[0], x.f[1], x.f[2], i), inv) + kadd) >> 16, kmax);
            const uint32_t d = vd - byte_of(x.l[0], x.l[1], x.l[2], i);
            cv[i] = (int)vd - c.delta;
            out |= (uint32_t)(d > byte_of(rng[0], rng[1], rng[2], i) + d2) << (i / 3);
        }
        if (out) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (out & (1u << k)) {
                    const int r = cv[3 * k], g = cv[3 * k + 1], b = cv[3 * k + 2];
                    if (not_gray<KIND == kCorrectedLum>(c, max(max(r, g), b), min(min(r, g), b)) &&
                        hue_in(r, g, b, c.h))
                        bits |= 1u << k;
                }
            }
        }
    }
    const uint64_t w = row_word(bits);
    if ((lane & 15) == 0) {
        const uint32_t word = (base >> 6) + (uint32_t)(lane >> 4);
        if (word < (pend >> 6))
            put<FLOW>(c.raw + word, w);
    }
}

// The wave's units of pixels [p0, p1) of a frame (p0 a multiple of 64):
// 1024 pixels apart, each unit's inputs loaded one unit ahead into
// alternating registers.
template <bool FLOW, int KIND>
__device__ __forceinline__ void classify_span_as(const ClsJob &c, uint32_t p0, uint32_t p1, uint32_t inv)
{
    const uint32_t lanepx = 4u * (threadIdx.x & (kWave - 1));
    uint32_t base = p0 + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)) * 256u;
    Px4 a, b;
    load_px4(c, base + lanepx, p1, a);
    while (base < p1) {
        load_px4(c, base + 1024u + lanepx, p1, b);
        classify_px4<FLOW, KIND>(c, base, p1, inv, a);
        base += 1024u;
        if (base >= p1)
            break;
        load_px4(c, base + 1024u + lanepx, p1, a);
        classify_px4<FLOW, KIND>(c, base, p1, inv, b);
        base += 1024u;
    }
}

template <bool FLOW>
__device__ __forceinline__ void classify_span(const ClsJob &c, uint32_t p0, uint32_t p1, uint32_t inv)
{
    switch (cls_kind(c)) {
    case kScaled: classify_span_as<FLOW, kScaled>(c, p0, p1, inv); break;
    case kCorrectedLum: classify_span_as<FLOW, kCorrectedLum>(c, p0, p1, inv); break;
    default: classify_span_as<FLOW, kCorrected>(c, p0, p1, inv); break;
    }
}

// Classify tile `tile` of frame j: ITERS consecutive 1024-pixel units.
template <int ITERS>
__device__ __forceinline__ void classify_tile(Table *__restrict__ T, int j, int tile, uint32_t inv)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const Job *J = &T->jobs[j];
    const uint32_t npx = (uint32_t)J->W * (uint32_t)J->H;
    const ClsJob c = cls_job(J);
    const uint32_t lanepx = 4u * (threadIdx.x & (kWave - 1));
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const uint32_t base = ((uint32_t)tile * ITERS + it) * 1024u + (uint32_t)wave * 256u;
        if (base >= npx)
            break;
        Px4 x;
        load_px4(c, base + lanepx, npx, x);
        switch (cls_kind(c)) {
        case kScaled: classify_px4<false, kScaled>(c, base, npx, inv, x); break;
        case kCorrectedLum: classify_px4<false, kCorrectedLum>(c, base, npx, inv, x); break;
        default: classify_px4<false, kCorrected>(c, base, npx, inv, x); break;
        }
    }
}

// Tiles blockIdx.x, blockIdx.x + gridDim.x, ...: the frame index only grows,
// so it is advanced, not searched. A block meets one to three frames, so a
// frame's inverse gain (32 pairs of sums and a 64-bit division) is computed
// when its first tile comes, by each wave for itself.
template <int ITERS>
__device__ __forceinline__ void classify_tiles(Table *__restrict__ T, int nj, const int32_t *s_pre)
{
    const int total = s_pre[nj];
    int j = 0, jinv = -1;
    uint32_t inv = 0;
    for (int t = blockIdx.x; t < total; t += gridDim.x) {
        while (s_pre[j + 1] <= t)
            ++j;
        if (j != jinv) {
            inv = wave_job_gain(&T->jobs[j]);
            jinv = j;
        }
        classify_tile<ITERS>(T, j, t - s_pre[j], inv);
    }
}

template <int ITERS>
__global__ __launch_bounds__(256) void k_classify(Table *__restrict__ T)
{
    __shared__ int32_t s_pre[kMaxJobs + 1];
    const int nj = T->h.njobs;
    for (int i = threadIdx.x; i <= nj; i += blockDim.x)
        s_pre[i] = T->h.cls_pre[i];
    __syncthreads();
    classify_tiles<ITERS>(T, nj, s_pre);
}

// ---------------------------------------------------------------------------
// Classify of consecutive frames of one stream (a context's launch): a lane
// keeps the background box of its 4 pixels in registers as exact integer
// bounds and tests one frame after the other against it. With x = v inv +
// 32768 (corrected pixels; v inv for scaled thresholds), a channel is in the
// box when Lo <= x <= Hi, Lo = max(bgmin - delta, 0) 2^16 and Hi the last x
// of the upper bound (none when bgmax + delta >= 255: the correction
// saturates there): one multiply-add and one unsigned compare of x - Lo
// against Hi - Lo per channel. Frame by frame (k_classify) the model is
// unpacked each time: 29 instructions per pixel in all, against 9 here plus
// the box (170 per lane) and the pixels outside it.
// Bound by HBM and the VALU together: 64 frames of 1920x1080 (398 MB) take 78
// us (174 us frame by frame), moving 5.6 TB/s with the VALU two thirds busy.
struct Box4 {
    uint32_t a[12];            // (32768 or 0) - Lo, wrapping
    uint32_t r[12];            // Hi - Lo
};

constexpr int kSpanFrames = 16;        // most frames of one span workgroup
constexpr int kSpanAhead = 4;          // frames in flight per lane

template <int KIND>
__device__ __forceinline__ void box_of(const FrameSpan &F, const u32x3 l, const u32x3 u, bool valid, Box4 &b)
{
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const int mn = (int)byte_of(l.x, l.y, l.z, i), mx = (int)byte_of(u.x, u.y, u.z, i);
        const uint32_t lo = (uint32_t)max(mn - F.delta, 0) << 16;
        uint32_t hi;
        if (KIND == kScaled)
            hi = (uint32_t)(mx + F.delta) << 16;
        else
            hi = mx + F.delta >= 255 ? 0x0FFFFFFFu : ((uint32_t)(mx + F.delta + 1) << 16) - 1u;
        b.a[i] = (KIND == kScaled ? 0u : 32768u) - lo;
        b.r[i] = valid ? hi - lo : 0xFFFFFFFFu;      // lanes past the frame's end: never outside
        // one register per bound: the compiler would otherwise split the
        // constant off again and add it for every frame
        asm("" : "+v"(b.a[i]));
        asm("" : "+v"(b.r[i]));
    }
}

// Bits of the lane's 4 pixels of one frame: outside the box, not gray, skin.
template <int KIND>
__device__ __forceinline__ uint32_t span_bits(const FrameSpan &F, const Box4 &box, const u32x3 w, uint32_t inv)
{
    bool out[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        out[k] = false;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            const int i = 3 * k + ch;
            out[k] = out[k] | (__umul24(byte_of(w.x, w.y, w.z, i), inv) + box.a[i] > box.r[i]);
        }
    }
    uint32_t bits = 0;
    if (out[0] | out[1] | out[2] | out[3]) {
        // a pixel of the four that no lane has outside is skipped; the rest
        // is straight-line, without a branch on the hue interval's case
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!out[k])
                continue;
            const uint32_t r8 = byte_of(w.x, w.y, w.z, 3 * k), g8 = byte_of(w.x, w.y, w.z, 3 * k + 1),
                           b8 = byte_of(w.x, w.y, w.z, 3 * k + 2);
            int r = (int)r8, g = (int)g8, b = (int)b8;
            if (KIND != kScaled) {
                r = (int)corr(r8, inv);
                g = (int)corr(g8, inv);
                b = (int)corr(b8, inv);
            }
            const int mx = max(max(r, g), b), mn = min(min(r, g), b);
            const bool colour = KIND == kScaled ? __umul24((uint32_t)(mx - mn), inv) >= F.S_q16
                                                : not_gray<KIND == kCorrectedLum>(F, mx, mn);
            bits |= (uint32_t)(colour & hue_in_form(r, g, b, F.hue)) << k;
        }
    }
    return bits;
}

// Workgroup (x, y): pixel tile x (1024 pixels, 256 per wave), frames
// [y per, (y + 1) per).
template <int KIND>
__global__ __launch_bounds__(256) void k_classify_span(const Table *__restrict__ T, const FrameSpan F, int per)
{
    __shared__ uint32_t s_inv[kSpanFrames];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int f0 = (int)blockIdx.y * per, nf = min(per, F.n - f0);
    const uint32_t gain = span_gain(T, f0, nf);
    const uint32_t base = blockIdx.x * 1024u + (uint32_t)wave * 256u;
    const uint32_t p = base + 4u * (uint32_t)lane;
    // lanes past the frame's end read its last pixels and never test as outside
    const uint32_t off = 3u * min(p, F.npx - 4u);
    const u32x3 l = *at_byte(G(reinterpret_cast<const u32x3 *>(F.bgmin)), off);
    const u32x3 u = *at_byte(G(reinterpret_cast<const u32x3 *>(F.bgmax)), off);
    const GLOBAL uint8_t *frames = G(F.frames) + (size_t)f0 * F.frame_stride;
    auto load = [&](int f) __attribute__((always_inline)) {
        return __builtin_nontemporal_load(
            at_byte(reinterpret_cast<const GLOBAL u32x3 *>(frames + (size_t)f * F.frame_stride), off));
    };
    // a ring of kSpanAhead frames in flight: a frame's registers take the
    // frame kSpanAhead later as soon as it is tested
    u32x3 ring[kSpanAhead];
#pragma unroll
    for (int q = 0; q < kSpanAhead; ++q)
        ring[q] = load(min(q, nf - 1));
    if ((int)threadIdx.x < nf)
        s_inv[threadIdx.x] = gain;
    __syncthreads();
    Box4 box;
    box_of<KIND>(F, l, u, p < F.npx, box);
    const uint32_t word = (base >> 6) + (uint32_t)(lane >> 4);
    const bool store = (lane & 15) == 0 && word < (F.npx >> 6);
    GLOBAL uint64_t *raw = G(F.raw) + (size_t)f0 * F.raw_words;
    auto test = [&](int f, const u32x3 w) __attribute__((always_inline)) {
        const uint32_t bits = span_bits<KIND>(F, box, w, s_inv[f]);
        uint64_t m = 0;
        if (__builtin_amdgcn_ballot_w64(bits != 0u))
            m = row_word(bits);
        if (store)
            (raw + (size_t)f * F.raw_words)[word] = m;
    };
    // the loads of the loop are unconditional (past the end the last frame
    // again): a branch around them would make every wait one for all of them
    int f = 0;
    for (; f + kSpanAhead < nf; f += kSpanAhead) {
#pragma unroll
        for (int q = 0; q < kSpanAhead; ++q) {
            test(f + q, ring[q]);
            ring[q] = load(min(f + q + kSpanAhead, nf - 1));
        }
    }
#pragma unroll
    for (int q = 0; q < kSpanAhead; ++q)
        if (f + q < nf)
            test(f + q, ring[q]);
}

// One frame of a stream: nothing to share a box between, so the pixels are
// corrected and tested as they are in k_classify; by value, without table
// lookups before the loads, a workgroup per 1024 pixels. Bound by its launch
// and load latency on small frames, by HBM on large ones: 320x240 / 1920x1080 /
// 3840x2160 / 7680x4320 4.2 / 4.7 / 12.4 / 43.1 us (7.0 TB/s), full of
// noise 4.2 / 5.6 / 15.2 / 50.9; k_classify_span on it 4.2 / 5.6 / 14.7 / 45.6
// and 4.4 / 6.9 / 18.8 / 60.7, k_classify 7.4 / 8.6 / 15.7 / 47.4 and 7.5 / 9.5
// / 18.3 / 53.2.
template <int KIND>
__global__ __launch_bounds__(256) void k_classify_one(const Table *__restrict__ T, const FrameSpan F, const HueTest h)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint32_t base = blockIdx.x * 1024u + (uint32_t)wave * 256u;
    if (base >= F.npx)
        return;
    ClsJob c;
    c.fr = G(reinterpret_cast<const uint32_t *>(F.frames));
    c.mn = G(reinterpret_cast<const uint32_t *>(F.bgmin));
    c.mx = G(reinterpret_cast<const uint32_t *>(F.bgmax));
    c.raw = G(F.raw);
    c.delta = F.delta;
    c.S1 = F.S1;
    c.scaled = F.scaled;
    c.S_q16 = F.S_q16;
    c.S0 = F.S0;
    c.lum2 = F.lum2;
    c.h = h;
    Px4 x;
    load_px4(c, base + 4u * (threadIdx.x & (kWave - 1)), F.npx, x);
    classify_px4<false, KIND>(c, base, F.npx, T->jobs[0].ginv & ~kGainKnown, x);
}

// ---------------------------------------------------------------------------
// A run list entry: first pixel (low word), last pixel (bits 32..62) and the
// flag kLinkUp (bit 63): the run must still be joined to the row above.
constexpr uint32_t kLinkUp = 0x80000000u;

// Bit scans of one mask row (W = 64 * Wd pixels).
// First x in [pos, limit] whose bit is 1, or -1.
template <typename P>
__device__ __forceinline__ int next_one(P row, int pos, int limit)
{
    int w = pos >> 6;
    uint64_t m = row[w] & (~0ull << (pos & 63));
    for (;;) {
        if (m) {
            const int x = (w << 6) + __builtin_ctzll(m);
            return x <= limit ? x : -1;
        }
        ++w;
        if ((w << 6) > limit)
            return -1;
        m = row[w];
    }
}

// Largest x <= pos whose bit is 0, or -1.
template <typename P>
__device__ __forceinline__ int prev_zero(P row, int pos)
{
    int w = pos >> 6;
    const int b = pos & 63;
    uint64_t m = ~row[w] & (b == 63 ? ~0ull : ((2ull << b) - 1ull));
    while (!m) {
        --w;
        if (w < 0)
            return -1;
        m = ~row[w];
    }
    return (w << 6) + 63 - __builtin_clzll(m);
}

// Smallest x >= pos whose bit is 0, or W.
template <typename P>
__device__ __forceinline__ int next_zero(P row, int Wd, int pos)
{
    int w = pos >> 6;
    uint64_t m = ~row[w] & (~0ull << (pos & 63));
    while (!m) {
        ++w;
        if (w >= Wd)
            return Wd << 6;
        m = ~row[w];
    }
    return (w << 6) + __builtin_ctzll(m);
}

// Union-find over the runs of a frame's list. A root is linked under the root
// whose run starts earlier in raster order, so following parents always ends,
// and the root of a finished component is its first run: its first pixel is
// the component's. A forest gives a run's parent (par), first pixel (start)
// and link (an atomic that replaces a root's parent, returning what it found).
//
// Root of x with path halving: each visited node is pointed at its
// grandparent. Safe beside concurrent finds and unions of the same workgroup:
// parents only ever move to ancestors of the same set, so a store that
// overwrites another still leaves the node in its set. Without it, the border
// joins of a tall component chain one band's root under the next, and every
// find walks that chain one dependent load at a time.
template <typename F>
__device__ __forceinline__ uint32_t find_root(const F &f, uint32_t x)
{
    for (;;) {
        const uint32_t p = f.par(x);
        if (p == x)
            return x;
        const uint32_t g = f.par(p);
        if (g == p)
            return p;
        f.set_par(x, g);
        x = g;
    }
}

// Root of x without writing: once every find and union of a workgroup is
// over, a node's parent need not be its root (a halving store of one thread
// can land after another thread pointed the node at its root, and leave it at
// an older ancestor), so a membership test walks to the root.
template <typename F>
__device__ __forceinline__ uint32_t root_of(const F &f, uint32_t x)
{
    for (;;) {
        const uint32_t p = f.par(x);
        if (p == x)
            return x;
        x = p;
    }
}

template <typename F>
__device__ __forceinline__ void unite(const F &f, uint32_t a, uint32_t b)
{
    for (;;) {
        a = find_root(f, a);
        b = find_root(f, b);
        if (a == b)
            return;
        if (f.start(a) > f.start(b)) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        const uint32_t old = f.link(b, a);
        if (old == b)
            return;
        b = old;
    }
}

// (first pixel, length) of a run list entry
__device__ __forceinline__ uint2 unpack_run(uint64_t v)
{
    const uint32_t a = (uint32_t)v, e = (uint32_t)(v >> 32) & ~kLinkUp;
    return make_uint2(a, e - a + 1u);
}

// A frame's forest in global memory: parents and areas by run, the run list.
// A: runs or unions that a thread takes at once; 4 in the component stage, 1 in
// the persistent step, whose registers are all taken (its code for several,
// which masks of few runs never reach, cost a step of 32 streams of 1920x1080
// 5 to 9%).
template <int A>
struct GlobalForest {
    static constexpr int kAhead = A;
    GLOBAL uint32_t *parent, *areas;
    const GLOBAL uint64_t *runs;

    __device__ __forceinline__ explicit GlobalForest(const Job *J)
        : parent(G(J->parent)), areas(G(J->parent) + J->run_cap), runs(G(reinterpret_cast<const uint64_t *>(J->runs)))
    {
    }
    __device__ __forceinline__ uint32_t par(uint32_t i) const { return ld_wg(parent + i); }
    __device__ __forceinline__ void set_par(uint32_t i, uint32_t v) const { st_wg(parent + i, v); }
    __device__ __forceinline__ uint32_t start(uint32_t i) const { return (uint32_t)runs[i]; }
    __device__ __forceinline__ uint32_t link(uint32_t root, uint32_t to) const
    {
        uint32_t expect = root;
        __hip_atomic_compare_exchange_strong(parent + root, &expect, to, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
        return expect;
    }
    __device__ __forceinline__ uint32_t area(uint32_t root) const { return ld_wg(areas + root); }
    __device__ __forceinline__ uint2 run(uint32_t i) const { return unpack_run(runs[i]); }
};

// The same in LDS, for frames of at most C runs.
template <int C>
struct LdsRuns {
    uint32_t par[C], start[C], len[C], area[C];
};

template <int C>
struct LdsForest {
    static constexpr int kAhead = 1;
    LdsRuns<C> &t;
    __device__ __forceinline__ uint32_t par(uint32_t i) const
    {
        return __hip_atomic_load(&t.par[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ void set_par(uint32_t i, uint32_t v) const
    {
        __hip_atomic_store(&t.par[i], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ uint32_t start(uint32_t i) const { return t.start[i]; }
    __device__ __forceinline__ uint32_t link(uint32_t root, uint32_t to) const { return atomicCAS(&t.par[root], root, to); }
    __device__ __forceinline__ uint32_t area(uint32_t root) const { return t.area[root]; }
    __device__ __forceinline__ uint2 run(uint32_t i) const { return make_uint2(t.start[i], t.len[i]); }
};

// The roots of U runs at once, in their place, with path halving: where bands
// were joined one below the other the path is as long as they are many, and
// all runs' halving together shortens it in the logarithm of that.
// This and the loops below that take several runs at once end for the wave as
// a whole. With an exit per lane the compiler (ROCm 7.2.0) split this loop in
// two around the last halving store and kept the outer one's condition in a
// lane mask that the inner one's later rounds cleared for lanes that had left
// it: they ended short of their roots.
template <int U, typename F>
__device__ __forceinline__ void find_roots(const F &f, uint32_t (&r)[U])
{
    for (;;) {
        uint32_t p[U], g[U];
        uint32_t more = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            p[u] = f.par(r[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
            g[u] = f.par(p[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (g[u] != p[u])
                f.set_par(r[u], g[u]);
            more |= g[u] ^ p[u];
            r[u] = g[u];
        }
        if (!__builtin_amdgcn_ballot_w64(more != 0u))
            return;
    }
}

// U unions at once (bit u of live: a[u] with b[u]; every a and b a run of the
// list): the roots of all, their first pixels and then the links each in
// flight together. In global memory a step of a union is a dependent access of
// 0.6 us, so that a thread's unions one after the other, side after side,
// would be nothing but waiting. Where the two sides' paths meet they are one
// set: most pairs come twice, and a pair of joined neighbours in a tall
// component would else climb to its top.
template <int U, typename F>
__device__ __forceinline__ void unite_at_once(const F &f, const uint32_t (&a)[U], const uint32_t (&b)[U],
                                              uint32_t live)
{
    uint32_t r[2 * U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        r[u] = (live >> u) & 1u ? a[u] : 0u;
        r[U + u] = (live >> u) & 1u ? b[u] : 0u;
    }
    for (;;) {
        for (;;) {
            uint32_t p[2 * U], g[2 * U], more = 0;
#pragma unroll
            for (int u = 0; u < 2 * U; ++u)
                p[u] = f.par(r[u]);
#pragma unroll
            for (int u = 0; u < 2 * U; ++u)
                g[u] = f.par(p[u]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int v = U + u;
                // one set already: the two sides' paths meet
                const bool met = (r[u] == r[v]) | (r[u] == p[v]) | (r[u] == g[v]) | (p[u] == r[v]) | (p[u] == p[v]) |
                                 (p[u] == g[v]) | (g[u] == r[v]) | (g[u] == p[v]) | (g[u] == g[v]);
                if (g[u] != p[u])
                    f.set_par(r[u], g[u]);
                if (g[v] != p[v])
                    f.set_par(r[v], g[v]);
                more |= met ? 0u : (g[u] ^ p[u]) | (g[v] ^ p[v]);
                r[u] = met ? 0u : g[u];
                r[v] = met ? 0u : g[v];
            }
            if (!__builtin_amdgcn_ballot_w64(more != 0u))
                break;
        }
        uint32_t start[2 * U], old[U];
#pragma unroll
        for (int u = 0; u < 2 * U; ++u)
            start[u] = f.start(r[u]);
        uint32_t linked = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // the later root under the earlier one
            const bool swap = start[u] > start[U + u];
            const uint32_t lo = swap ? r[U + u] : r[u], hi = swap ? r[u] : r[U + u];
            r[u] = lo;
            r[U + u] = hi;
            if (lo != hi) {
                linked |= 1u << u;
                old[u] = f.link(hi, lo);
            }
        }
        if (!__builtin_amdgcn_ballot_w64(linked != 0u))
            return;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!((linked >> u) & 1u))
                continue;
            if (old[u] == r[U + u])
                r[u] = r[U + u] = 0u;            // done
            else
                r[U + u] = old[u];
        }
    }
}

// The roots of U runs at once, r[u] from x[u], without writing (see root_of).
template <int U, typename F>
__device__ __forceinline__ void roots_of(const F &f, const uint32_t (&x)[U], uint32_t (&r)[U])
{
#pragma unroll
    for (int u = 0; u < U; ++u)
        r[u] = x[u];
    for (;;) {
        uint32_t p[U];
        uint32_t more = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            p[u] = f.par(r[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            more |= p[u] ^ r[u];
            r[u] = p[u];
        }
        if (!__builtin_amdgcn_ballot_w64(more != 0u))
            return;
    }
}

// Joins run i (y, xs..xe) with every run of the row above that it touches
// under 8-connectivity (columns xs-1 .. xe+1).
template <typename F, typename P>
__device__ __forceinline__ void link_up(const F &f, const GLOBAL uint32_t *index, P above, int Wd, int W, int y,
                                        int xs, int xe, uint32_t i)
{
    const int hi = min(xe + 1, W - 1);
    int pos = max(xs - 1, 0);
    while (pos <= hi) {
        const int xb = next_one(above, pos, hi);
        if (xb < 0)
            break;
        const int bs = prev_zero(above, xb) + 1;
        unite(f, i, index[(uint32_t)(y - 1) * (uint32_t)W + (uint32_t)bs]);
        pos = next_zero(above, Wd, xb) + 1;
    }
}

// ---------------------------------------------------------------------------
// Morphology, runs and band-local components: one wave per band of R mask
// rows. Lane l holds words l and l + 64 of a row (W <= 8192). The band's rows,
// with 2(o+c) halo rows on each side, stream once through a pipeline of the
// opening/closing stages held in registers: each stage keeps the two rows
// before its input, and on input row i emits row i - 1 from the 3x3 window
// (vertical AND/OR per word, horizontal neighbours from the words' edge bits,
// exchanged between neighbouring lanes). Rows outside the image enter a stage
// as its neutral value (1 for erosion, 0 for dilation), which is exactly the
// border rule; halo rows inside the image only corrupt rows outside the band.
// Each final row of the band is stored (I_FIZI); its run starts and ends are
// bit masks of each lane's word, numbered by a wave prefix sum, so the lanes
// holding a run's first and last pixel write them without scanning. Runs are
// joined to the touching runs of the row above (kept in registers) in a
// union-find over segment-local run indices kept in LDS (indices grow in
// raster order, so a root is its component's first run in the segment). A
// segment is a stretch of the band's rows whose runs fit the LDS table; when
// it closes (table full, band done) its runs are appended to the frame's run
// list with one reservation, each pointing at its segment root. The first run
// row of a segment that is not the first of the band, and the first row of
// every band below the top, are flagged: the component stage joins them to the
// row above. A row with more runs than the table goes to the run list
// directly, its runs their own roots, flagged, and so is the row after it.
constexpr int kSegRuns = 512;              // runs of one LDS segment
constexpr int kRawChunk = 4;               // rows loaded together (the selects below assume 4)

struct WaveLds {
    uint32_t start[kSegRuns];              // first pixel of segment run k
    uint32_t end[kSegRuns];                // its last pixel, | kLinkUp if flagged
    uint32_t par[kSegRuns];                // union-find parent (segment index)
    // touching pairs still to unite, run | run << 16: at most one per run of
    // the segment (each belongs to the start of a run of the upper row)
    uint32_t pairs[kSegRuns];
    uint32_t npairs;
};

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Lane l receives lane l - 1's value (lane 0 receives 0): DPP wave_shr:1.
__device__ __forceinline__ uint32_t from_left(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, false);
}

// Lane l receives lane l + 1's value (lane 63 receives 0): DPP wave_shl:1.
__device__ __forceinline__ uint32_t from_right(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, false);
}

// Inclusive prefix sum over the wave: shifts of 1, 2, 4, 8 inside each row of
// 16 lanes, then each row's total is carried into the rows above it
// (row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3). Lanes a
// DPP move does not write keep 0.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
    return v;
}

// Lanes per row: lg lanes hold one row (64: the whole wave; 16 or 32 pack 64 /
// lg bands of a narrow frame into one wave, lane group g holding band g's
// row). The word a lane holds, and its group:
__device__ __forceinline__ int lane_word(int lg) { return (int)(threadIdx.x & (uint32_t)(lg - 1)); }
__device__ __forceinline__ int lane_group(int lg) { return (int)((threadIdx.x & (kWave - 1)) >> (31 - __builtin_clz(lg))); }

// Edge bits of the neighbouring words of this lane's NC words (word
// w + 64 q of the lane group's row): bit 63 of the word on the left (lc) and
// bit 0 of the word on the right (rc); words outside [0, Wd) give `edge`.
template <int NC>
__device__ __forceinline__ void row_carries(const uint64_t *v, int Wd, uint32_t edge, uint32_t *lc, uint32_t *rc,
                                            int lg = kWave)
{
    const int lane = lane_word(lg);            // lane groups (lg < 64) hold one word per lane
    const uint32_t hi0 = (uint32_t)(v[0] >> 63), lo0 = (uint32_t)v[0] & 1u;
    const uint32_t up0 = from_left(hi0), dn0 = from_right(lo0);
    lc[0] = lane == 0 ? edge : up0;
    if (NC == 1) {
        rc[0] = (lane + 1 < Wd) ? dn0 : edge;
    } else {
        const uint32_t hi1 = (uint32_t)(v[NC - 1] >> 63), lo1 = (uint32_t)v[NC - 1] & 1u;
        const uint32_t up1 = from_left(hi1), dn1 = from_right(lo1);
        const uint32_t last_hi0 = (uint32_t)__builtin_amdgcn_readlane((int)hi0, kWave - 1);
        const uint32_t first_lo1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo1);
        rc[0] = (lane + 1 < Wd) ? (lane == kWave - 1 ? first_lo1 : dn0) : edge;
        lc[NC - 1] = lane == 0 ? last_hi0 : up1;
        rc[NC - 1] = (lane + kWave + 1 < Wd) ? dn1 : edge;
    }
}

// One erosion (ero) or dilation of row b given the rows above (a) and below (c).
template <int NC>
__device__ __forceinline__ void morph_row(bool ero, const uint64_t *a, const uint64_t *b, const uint64_t *c, int Wd,
                                          uint64_t *out)
{
    uint64_t v[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q)
        v[q] = ero ? (a[q] & b[q] & c[q]) : (a[q] | b[q] | c[q]);
    uint32_t lc[NC], rc[NC];
    row_carries<NC>(v, Wd, ero ? 1u : 0u, lc, rc);
#pragma unroll
    for (int q = 0; q < NC; ++q) {
        const uint64_t left = (v[q] << 1) | lc[q];
        const uint64_t right = (v[q] >> 1) | ((uint64_t)rc[q] << 63);
        out[q] = ero ? (v[q] & left & right) : (v[q] | left | right);
    }
}

__device__ __forceinline__ uint32_t find_lds(uint32_t *par, uint32_t x)
{
    uint32_t p = __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    while (p != x) {
        x = p;
        p = __hip_atomic_load(par + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    return x;
}

__device__ __forceinline__ void unite_lds(uint32_t *par, uint32_t a, uint32_t b)
{
    for (;;) {
        a = find_lds(par, a);
        b = find_lds(par, b);
        if (a == b)
            return;
        if (a > b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        const uint32_t old = __hip_atomic_fetch_min(par + b, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        if (old == b)
            return;
        b = old;
    }
}

// Bit t of a row around this lane's word w, t in [-1, 64]: -1 is the last
// bit of the word on the left (lc), 64 the first bit of the word on the right
// (rc).
__device__ __forceinline__ uint32_t bit_at(int t, uint64_t w, uint32_t lc, uint32_t rc)
{
    return t < 0 ? lc : (t > 63 ? rc : (uint32_t)(w >> t) & 1u);
}

// Row-local index of the run that contains bit t (set, t in [-1, 64]) around
// this lane's word w, whose run starts are st, with ex runs starting before it.
__device__ __forceinline__ uint32_t run_at(int t, uint32_t ex, uint64_t st, uint64_t w, uint32_t rc)
{
    if (t < 0)
        return ex - 1u;
    if (t > 63)
        return ex + (uint32_t)__popcll(st) + (rc & ~(uint32_t)(w >> 63) & 1u) - 1u;
    return ex + (uint32_t)__popcll(st & (~0ull >> (63 - t))) - 1u;
}

// Inclusive max over lanes 0..l of values >= -1 (DPP as in wave_incl_scan;
// lanes a move does not write keep -1).
__device__ __forceinline__ int wave_incl_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x111, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x112, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x114, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x118, 0xF, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x142, 0xA, 0xF, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x143, 0xC, 0xF, false));
    return v;
}

// One final mask row as the lanes hold it: per word (lane + 64 c) the bits,
// the edge bits of the neighbouring words, the run starts, the number of runs
// starting before the word and the x of the last run start before the word.
template <int NC>
struct RowBits {
    uint64_t w[NC], st[NC];
    uint32_t lc[NC], rc[NC], ex[NC];
    int last[NC];
};

// Fills r from the row x; en receives the run ends. Returns the row's runs
// (of every lane group: runs are numbered across the wave). r.last holds
// wave positions 64 lane + bit, which grow across the groups.
template <int NC>
__device__ __forceinline__ uint32_t row_bits(RowBits<NC> &r, const uint64_t *x, int Wd, uint64_t *en, int lg)
{
    const int lane = threadIdx.x & (kWave - 1);
    row_carries<NC>(x, Wd, 0u, r.lc, r.rc, lg);
    uint32_t total = 0;
    int before = -1;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        r.w[c] = x[c];
        r.st[c] = x[c] & ~((x[c] << 1) | r.lc[c]);
        en[c] = x[c] & ~((x[c] >> 1) | ((uint64_t)r.rc[c] << 63));
        const uint32_t n = (uint32_t)__popcll(r.st[c]);
        const uint32_t inc = wave_incl_scan(n);
        r.ex[c] = total + inc - n;
        total += (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        const int hi = r.st[c] ? 64 * (lane + kWave * c) + 63 - __builtin_clzll(r.st[c]) : -1;
        const int im = wave_incl_max(hi);
        r.last[c] = max(before, __builtin_amdgcn_update_dpp(-1, im, 0x138, 0xF, 0xF, false));
        before = max(before, __builtin_amdgcn_readlane(im, kWave - 1));
    }
    return total;
}

// x of the first pixel of the run that contains bit t (set, t in [-1, 64])
// around word c of the row. A run never crosses a lane group (its edges are
// out-of-image), so a start before the word lies in the same group.
template <int NC>
__device__ __forceinline__ int start_at(const RowBits<NC> &r, int c, int t, int lg)
{
    const int wb = 64 * (lane_word(lg) + kWave * c);
    const int gofs = 64 * lg * lane_group(lg);
    if (t < 0)
        return r.last[c] - gofs;
    uint64_t m;
    if (t > 63) {
        if (r.rc[c] & ~(uint32_t)(r.w[c] >> 63) & 1u)
            return wb + 64;
        m = r.st[c];
    } else {
        m = r.st[c] & (~0ull >> (63 - t));
    }
    return m ? wb + 63 - __builtin_clzll(m) : r.last[c] - gofs;
}

// Touching pairs of runs of two consecutive rows U (above) and D (below), from
// the lanes' words. Under 8-connectivity a U run [us, ue] and a D run [ds, de]
// touch when us <= de + 1 and ue >= ds - 1. When us <= ds + 1, U has a pixel
// in columns ds - 1 .. ds + 1, and D's start meets it there (the pixel at ds,
// else those beside it). Otherwise us >= ds + 2, so D holds columns us - 2 and
// us - 1, and U's start meets the D run there: each pair is met once.
// Whether D holds the two columns left of bit b of word c (for b = 0: its run
// through the word's left edge started at least two columns before it).
template <int NC>
__device__ __forceinline__ bool holds_left2(const RowBits<NC> &D, int c, int b)
{
    if (b >= 2)
        return ((D.w[c] >> (b - 2)) & 3ull) == 3ull;
    if (b == 1)
        return (D.lc[c] & (uint32_t)D.w[c] & 1u) != 0u;
    return D.lc[c] != 0u && D.last[c] < 64 * ((int)(threadIdx.x & (kWave - 1)) + kWave * c) - 1;
}

// The same pairs with U's starts looking at the one to three pixels below
// them as D's do above, so that most come twice: f(c, from_d, b, t), the run
// starting at bit b of word c of D (from_d) or U touches the run of the other
// row that contains bit t. The band-border joins keep this form: the component
// stage unites them concurrently, and the second meeting of a pair shortens
// the chains the first one built.
template <int NC, typename F>
__device__ __forceinline__ void touching_runs(const RowBits<NC> &U, const RowBits<NC> &D, F f)
{
    auto look = [&](int c, bool from_d, uint64_t starts, const RowBits<NC> &O) {
        while (starts) {
            const int b = __builtin_ctzll(starts);
            starts &= starts - 1;
            if (bit_at(b, O.w[c], O.lc[c], O.rc[c])) {
                f(c, from_d, b, b);
            } else {
                if (bit_at(b - 1, O.w[c], O.lc[c], O.rc[c]))
                    f(c, from_d, b, b - 1);
                if (bit_at(b + 1, O.w[c], O.lc[c], O.rc[c]))
                    f(c, from_d, b, b + 1);
            }
        }
    };
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        look(c, true, D.st[c], U);
        look(c, false, U.st[c], D);
    }
}

// Each pair met once (see holds_left2), for bands of more runs than a segment:
// half the links, where the list would overflow.
template <int NC, typename F>
__device__ __forceinline__ void touching_runs_once(const RowBits<NC> &U, const RowBits<NC> &D, F f)
{
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        for (uint64_t m = D.st[c]; m; m &= m - 1) {
            const int b = __builtin_ctzll(m);
            if (bit_at(b, U.w[c], U.lc[c], U.rc[c])) {
                f(c, true, b, b);
            } else {
                if (bit_at(b - 1, U.w[c], U.lc[c], U.rc[c]))
                    f(c, true, b, b - 1);
                if (bit_at(b + 1, U.w[c], U.lc[c], U.rc[c]))
                    f(c, true, b, b + 1);
            }
        }
        for (uint64_t m = U.st[c]; m; m &= m - 1) {
            const int b = __builtin_ctzll(m);
            if (holds_left2<NC>(D, c, b))
                f(c, false, b, b - 1);
        }
    }
}

__device__ __forceinline__ bool stage_erodes(int k, int oi, int ci) { return (k < oi) || (k >= 2 * oi + ci); }

// Reserves n entries of the frame's run list (one atomic for the wave).
__device__ __forceinline__ uint32_t reserve_runs(Job *J, uint32_t n, uint32_t cap)
{
    const int lane = threadIdx.x & (kWave - 1);
    uint32_t base = 0;
    if (lane == 0) {
        base = atomicAdd(&J->nruns, n);
        if (base + n > cap)
            atomicOr(&J->flags, 1u);
    }
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
}

// Unites the pairs a segment put off.
__device__ __forceinline__ void unite_pairs(WaveLds &L)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t np = L.npairs;
    for (uint32_t i = lane; i < np; i += kWave)
        unite_lds(L.par, L.pairs[i] & 0xFFFFu, L.pairs[i] >> 16);
    wave_sync();
    if (lane == 0)
        L.npairs = 0u;
}

// A segment's n runs join the run list from entry base on, each pointing at
// its root.
template <bool FLOW>
__device__ __forceinline__ void store_segment(WaveLds &L, uint32_t n, uint32_t base, GLOBAL uint64_t *runs,
                                              GLOBAL uint32_t *parent, GLOBAL uint32_t *index, uint32_t cap)
{
    for (uint32_t k = threadIdx.x & (kWave - 1); k < n; k += kWave) {
        const uint32_t st = L.start[k];
        const uint32_t r = find_lds(L.par, k);
        if (base + k < cap) {
            put<FLOW>(runs + base + k, ((uint64_t)L.end[k] << 32) | st);
            put_parent<FLOW>(parent + base + k, base + r);
            put<FLOW>(index + st, base + k);
        }
    }
    wave_sync();
}

// Closes a segment.
template <bool FLOW>
__device__ __forceinline__ void flush_segment(Job *J, WaveLds &L, uint32_t n, GLOBAL uint64_t *runs,
                                              GLOBAL uint32_t *parent, GLOBAL uint32_t *index, uint32_t cap)
{
    if (n == 0)
        return;
    const uint32_t base = reserve_runs(J, n, cap);
    unite_pairs(L);
    store_segment<FLOW>(L, n, base, runs, parent, index, cap);
}

// Rows r0 .. r0 + kRawChunk - 1 of the raw mask, addresses clamped to rows 0 .. H - 1 and words below Wd. Values of clamped
// rows and words are never used (rows outside the image enter the pipeline as
// its neutral value, words from Wd on never reach a valid word), so the loads
// need no condition: they stay in flight while the previous chunk is
// processed.
template <int NC>
__device__ __forceinline__ void load_rows(uint64_t (&dst)[kRawChunk][NC], const GLOBAL uint64_t *raw, int r0, int H,
                                          int Wd)
{
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int qq = 0; qq < kRawChunk; ++qq) {
        const size_t ro = (size_t)min(max(r0 + qq, 0), H - 1) * Wd;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            dst[qq][c] = raw[ro + min(lane + kWave * c, Wd - 1)];
    }
}

// A band's final rows, one after the other: what a row needs of its job, and
// the row above.
struct BandOut {
    Job *J;
    int W, Wd, lg, word;
    GLOBAL uint64_t *runs;
    GLOBAL uint32_t *parent, *index, *linkw;
    uint32_t cap, link_cap;
};

__device__ __forceinline__ BandOut band_out(Job *J, int lg)
{
    BandOut B;
    B.J = J;
    B.W = J->W;
    B.Wd = J->Wd;
    B.lg = lg;
    B.word = lane_word(lg);
    B.runs = G(reinterpret_cast<uint64_t *>(J->runs));
    B.parent = G(J->parent);
    B.index = G(J->index);
    B.linkw = G(reinterpret_cast<uint32_t *>(J->links));
    B.cap = J->run_cap;
    B.link_cap = J->link_cap;
    return B;
}

template <int NC>
struct RunState {
    uint32_t nseg = 0, prev_first = 0;
    bool prev_valid = false;    // P holds the previous row and it has runs
    bool prev_in_seg = false;   // ... in the open segment
    RowBits<NC> P;

    __device__ __forceinline__ RunState()
    {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            P.w[c] = P.st[c] = 0ull;
            P.lc[c] = P.rc[c] = P.ex[c] = 0u;
            P.last[c] = -1;
        }
    }
};

// The last row of the band above, only to join with.
template <int NC>
__device__ __forceinline__ void halo_row(const BandOut &B, RunState<NC> &S, const uint64_t *x)
{
    uint64_t en[NC];
    (void)row_bits<NC>(S.P, x, B.Wd, en, B.lg);
    S.prev_valid = true;
    S.prev_in_seg = false;
}

// The joins of a row D (first pixel rowpx, per lane group) with the row P above
// as pairs of run starts, from entry k of the frame's link list on (per lane).
// ONE: of a band known to fit one segment.
template <int NC, bool FLOW, bool ONE>
__device__ __forceinline__ void band_links(const BandOut &B, const RowBits<NC> &P, const RowBits<NC> &D,
                                           uint32_t rowpx, uint32_t k)
{
    const uint32_t upx = rowpx - (uint32_t)B.W;
    auto join = [&](int c, bool from_d, int b, int t) {
        const uint32_t wb = 64u * (uint32_t)(B.word + kWave * c);
        const uint32_t a = from_d ? rowpx + wb + (uint32_t)b : upx + wb + (uint32_t)b;
        const uint32_t o = from_d ? upx + (uint32_t)start_at<NC>(P, c, t, B.lg)
                                  : rowpx + (uint32_t)start_at<NC>(D, c, t, B.lg);
        if (k < B.link_cap) {
            put<FLOW>(B.linkw + 2 * (size_t)k, a);
            put<FLOW>(B.linkw + 2 * (size_t)k + 1, o);
        }
        ++k;
    };
    if constexpr (ONE)
        touching_runs<NC>(P, D, join);
    else
        touching_runs_once<NC>(P, D, join);
}

// A final I_FIZI row with pixels (jrow per lane group): its runs and their
// joins with the row above. ONE: the band's runs are known to fit one segment
// and its joins with the band above are written at the end (band_links).
template <int NC, bool FLOW, bool ONE = false>
__device__ __forceinline__ void run_row(const BandOut &B, RunState<NC> &S, WaveLds &L, const uint64_t *x, int jrow)
{
    Job *J = B.J;
    const int lane = threadIdx.x & (kWave - 1);
    const int W = B.W, Wd = B.Wd, word = B.word;
    GLOBAL uint64_t *runs = B.runs;
    GLOBAL uint32_t *parent = B.parent, *index = B.index;
    const uint32_t cap = B.cap, link_cap = B.link_cap;
    RowBits<NC> &P = S.P;
    uint32_t &nseg = S.nseg, &prev_first = S.prev_first;
    bool &prev_valid = S.prev_valid, &prev_in_seg = S.prev_in_seg;
    RowBits<NC> D;
    uint64_t en[NC];
    const uint32_t total = row_bits<NC>(D, x, Wd, en, B.lg);
    if (!ONE && nseg + total > (uint32_t)kSegRuns) {
        // the open segment is full: close it, this row opens the next
        flush_segment<FLOW>(J, L, nseg, runs, parent, index, cap);
        nseg = 0;
        prev_in_seg = false;
    }
    const bool direct = !ONE && total > (uint32_t)kSegRuns;
    const uint32_t rowpx = (uint32_t)max(jrow, 0) * (uint32_t)W;
    // joins with a row above whose runs are not in the open segment (the
    // band above, a closed segment, or a row written directly) go to the
    // frame's link list as pairs of run starts
    uint32_t flag = 0u;
    if (!ONE && prev_valid && (!prev_in_seg || direct)) {
        uint32_t cnt = 0;
        touching_runs_once<NC>(P, D, [&](int, bool, int, int) { ++cnt; });
        const uint32_t inc = wave_incl_scan(cnt);
        const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        uint32_t base = 0;
        if (lane == 0)
            base = atomicAdd(&J->nlinks, n);
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        const uint32_t k = base + inc - cnt;
        band_links<NC, FLOW, false>(B, P, D, rowpx, k);
        if (base + n > link_cap) {
            // the list is full: the component stage joins this row to
            // the row above by reading I_FIZI
            flag = kLinkUp;
            if (lane == 0)
                atomicAdd(&J->nflag, 1u);
        }
    }
    const uint32_t rbase = direct ? reserve_runs(J, total, cap) : 0u;
    GLOBAL uint32_t *runw = reinterpret_cast<GLOBAL uint32_t *>(runs);
    // record the row's runs: the lane holding a run's first pixel writes
    // its start, the lane holding its last pixel its end
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const uint32_t wpx = rowpx + 64u * (uint32_t)(word + kWave * c);
        uint64_t m = D.st[c];
        while (m) {
            const int b = __builtin_ctzll(m);
            const uint32_t k = D.ex[c] + (uint32_t)__popcll(D.st[c] & ((1ull << b) - 1ull));
            m &= m - 1;
            const uint32_t start = wpx + (uint32_t)b;
            if (!direct) {
                L.start[nseg + k] = start;
                L.par[nseg + k] = nseg + k;
            } else if (rbase + k < cap) {
                put<FLOW>(runw + 2 * (size_t)(rbase + k), start);
                put_parent<FLOW>(parent + rbase + k, rbase + k);
                put<FLOW>(index + start, rbase + k);
            }
        }
        m = en[c];
        while (m) {
            const int e = __builtin_ctzll(m);
            const uint32_t k = D.ex[c] + (uint32_t)__popcll(D.st[c] & (~0ull >> (63 - e))) - 1u;
            m &= m - 1;
            const uint32_t end = (wpx + (uint32_t)e) | flag;
            if (!direct)
                L.end[nseg + k] = end;
            else if (rbase + k < cap)
                put<FLOW>(runw + 2 * (size_t)(rbase + k) + 1, end);
        }
    }
    wave_sync();
    // joins with the row above in the open segment: each touching pair once
    // (see touching_runs). The first run that a run's start meets above gives
    // it its parent, that run's own parent, so that without further pairs
    // every run points at its root; the others are united when the segment
    // closes, all lanes at once, instead of one row's few at a time
    if (prev_valid && prev_in_seg && !direct) {
        auto later = [&](uint32_t u, uint32_t d) { L.pairs[atomicAdd(&L.npairs, 1u)] = u | (d << 16); };
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            uint64_t m = D.st[c];
            while (m) {
                const int b = __builtin_ctzll(m);
                m &= m - 1;
                const uint32_t k = nseg + D.ex[c] + (uint32_t)__popcll(D.st[c] & ((1ull << b) - 1ull));
                auto above = [&](int t) { return prev_first + run_at(t, P.ex[c], P.st[c], P.w[c], P.rc[c]); };
                if (bit_at(b, P.w[c], P.lc[c], P.rc[c])) {
                    L.par[k] = L.par[above(b)];
                } else {
                    const bool l = bit_at(b - 1, P.w[c], P.lc[c], P.rc[c]) != 0u,
                               r = bit_at(b + 1, P.w[c], P.lc[c], P.rc[c]) != 0u;
                    if (l | r)
                        L.par[k] = L.par[above(l ? b - 1 : b + 1)];
                    if (l & r)
                        later(above(b + 1), k);
                }
            }
            m = P.st[c];
            while (m) {
                const int b = __builtin_ctzll(m);
                m &= m - 1;
                if (holds_left2<NC>(D, c, b))
                    later(prev_first + P.ex[c] + (uint32_t)__popcll(P.st[c] & ((1ull << b) - 1ull)),
                          nseg + run_at(b - 1, D.ex[c], D.st[c], D.w[c], D.rc[c]));
            }
        }
        wave_sync();
    }
    // this row becomes the row above
    P = D;
    prev_valid = true;
    prev_in_seg = !direct;
    if (!direct) {
        prev_first = nseg;
        nseg += total;
    }
}

// A band streamed through the register pipeline: bands of any height, in the
// persistent step and for the heights that morph_regs does not take. KMAX:
// most opening/closing stages a job may have; NC: words per lane; FLOW: inside
// the persistent step (stores other workgroups read in the launch); OI, CI:
// the opening and closing iterations when fixed at compile time (the stages'
// kinds then need no selects), -1 to read them from the job.
template <int KMAX, int NC, bool FLOW, int OI = -1, int CI = -1>
__device__ __forceinline__ void morph_band(Job *J, int band, WaveLds &L)
{
    const int word = threadIdx.x & (kWave - 1);
    const int H = J->H, Wd = J->Wd, R = J->band;
    const int oi = OI >= 0 ? OI : J->open_it, ci = CI >= 0 ? CI : J->close_it;
    const int K = 2 * (oi + ci);
    const int y0 = band * R;
    // one more halo row above: row y0 - 1 is computed exactly, to join the
    // band's first row to it without reading the band above
    const int ya = y0 - K - 1;
    const GLOBAL uint64_t *raw = G(J->raw);
    GLOBAL uint64_t *fz = G(J->fizi);
    bool valid_w[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q)
        valid_w[q] = word + kWave * q < Wd;

    // pipeline state: the two rows before each stage's next input
    uint64_t p2[KMAX][NC], p1[KMAX][NC];
#pragma unroll
    for (int k = 0; k < KMAX; ++k)
#pragma unroll
        for (int q = 0; q < NC; ++q)
            p2[k][q] = p1[k][q] = stage_erodes(k, oi, ci) ? ~0ull : 0ull;
    const BandOut B = band_out(J, kWave);
    RunState<NC> S;
    L.npairs = 0u;
    wave_sync();
    const int nsteps = R + 2 * K + 1;
    // one input row through the stages, then the band's final row it yields
    auto step = [&](int s, int q, const uint64_t (&ch)[kRawChunk][NC]) __attribute__((always_inline)) {
        uint64_t x[NC];
        const bool past = ya + s >= H;
        const uint64_t n0 = (K > 0 && stage_erodes(0, oi, ci)) ? ~0ull : 0ull;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const uint64_t v = q == 0 ? ch[0][c] : (q == 1 ? ch[1][c] : (q == 2 ? ch[2][c] : ch[3][c]));
            x[c] = past ? n0 : v;
        }
#pragma unroll
        for (int k = 0; k < KMAX; ++k) {
            if (k < K) {
                const bool ero = stage_erodes(k, oi, ci);
                const int i = ya + s - k;
                if (i < 0 || i >= H) {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        x[c] = ero ? ~0ull : 0ull;
                }
                uint64_t o[NC];
                morph_row<NC>(ero, p2[k], p1[k], x, Wd, o);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    p2[k][c] = p1[k][c];
                    p1[k][c] = x[c];
                }
                const int jr = i - 1;
                const bool oob = k + 1 < K && (jr < 0 || jr >= H);
                const uint64_t n1 = stage_erodes(k + 1, oi, ci) ? ~0ull : 0ull;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    x[c] = oob ? n1 : o[c];
            }
        }
        // the row this step yields, relative to the band: -1 the halo row,
        // 0 .. R - 1 the band's rows (outside the image: an empty row)
        const int jrel = s - 2 * K - 1;
        if (jrel < -1 || jrel >= R)
            return;
        const int jrow = y0 + jrel;
        const bool row_ok = jrow >= 0 && jrow < H;
        uint64_t orw = 0ull;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (!valid_w[c] || !row_ok)
                x[c] = 0ull;
            orw |= x[c];
        }
        const bool nonempty = __ballot(orw != 0ull) != 0ull;
        if (jrel == -1) {
            if (nonempty)
                halo_row<NC>(B, S, x);
            return;
        }
        // a final I_FIZI row
        GLOBAL uint64_t *frow = fz + (size_t)max(jrow, 0) * Wd;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (valid_w[c] && row_ok)
                put<FLOW>(frow + word + kWave * c, x[c]);
        if (nonempty)
            run_row<NC, FLOW>(B, S, L, x, jrow);
        else
            S.prev_valid = false;
    };
    // input chunks alternate between two register buffers: each is loaded a
    // chunk ahead of its use, straight into the registers that use it
    uint64_t ca[kRawChunk][NC], cb[kRawChunk][NC];
    load_rows<NC>(ca, raw, ya, H, Wd);
#pragma unroll 1
    for (int s0 = 0; s0 < nsteps; s0 += 2 * kRawChunk) {
        load_rows<NC>(cb, raw, ya + s0 + kRawChunk, H, Wd);
#pragma unroll 1
        for (int q = 0; q < kRawChunk && s0 + q < nsteps; ++q)
            step(s0 + q, q, ca);
        load_rows<NC>(ca, raw, ya + s0 + 2 * kRawChunk, H, Wd);
#pragma unroll 1
        for (int q = 0; q < kRawChunk && s0 + kRawChunk + q < nsteps; ++q)
            step(s0 + kRawChunk + q, q, cb);
    }
    flush_segment<FLOW>(J, L, S.nseg, B.runs, B.parent, B.index, B.cap);
}

// A band of at most 16 rows, all of it in registers: the rows with their halo
// are loaded at once and go through the stages one stage at a time, so that
// the rows of a stage are independent of each other (the streamed form is one
// chain of dependent steps, with selects for the image's borders in each).
// Waves whose rows hold no three pixels above one another anywhere - the first
// erosion leaves nothing then, and the closing nothing to close - store empty
// rows and are done: background with noise, most bands of a frame.
// Bound by the latency of the bands that hold the hand: 64 frames of 1920x1080
// in 8-row bands take 22 us (35 streamed), the 64-stream batch in 16-row bands
// 67 us (89), 16 frames of 1344x757 with two openings and closings 21 us (52),
// a frame of 320x240 4 us (8). R: band height; KT: stages the halo has rows
// for; NC: words per lane.
// One stage on rows from .. to of the N in registers. edge: the band's rows
// reach outside the image, where a stage reads its neutral value (1 for
// erosion, 0 for dilation).
template <bool ERO, int N, int NC>
__device__ __forceinline__ void regs_stage(uint64_t (&x)[N][NC], int from, int to, int Wd, int lg, bool edge,
                                           int ytop, int H)
{
    constexpr uint64_t neutral = ERO ? ~0ull : 0ull;
    if (edge) {
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const bool out = (uint32_t)(ytop + r) >= (uint32_t)H;
#pragma unroll
            for (int q = 0; q < NC; ++q)
                x[r][q] = out ? neutral : x[r][q];
        }
    }
    const int lane = lane_word(lg);
    const bool first = lane == 0, last = lane + 1 >= Wd, last1 = lane + kWave + 1 >= Wd;
    uint64_t prev[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q)
        prev[q] = x[from - 1][q];
#pragma unroll
    for (int r = 1; r < N - 1; ++r) {
        if (r < from || r > to)
            continue;
        uint32_t lo[NC], hi[NC], lw[NC], rw[NC];
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const uint64_t v = ERO ? (prev[q] & x[r][q] & x[r + 1][q]) : (prev[q] | x[r][q] | x[r + 1][q]);
            prev[q] = x[r][q];
            lo[q] = (uint32_t)v;
            hi[q] = (uint32_t)(v >> 32);
        }
        // the nearest half of the words on both sides, neutral past the row's ends
        const uint32_t edge32 = (uint32_t)neutral;
        const uint32_t l0 = from_left(hi[0]), r0 = from_right(lo[0]);
        lw[0] = first ? edge32 : l0;
        rw[0] = last ? edge32 : r0;
        if constexpr (NC == 2) {
            const uint32_t end0 = (uint32_t)__builtin_amdgcn_readlane((int)hi[0], kWave - 1);
            const uint32_t beg1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo[1]);
            const uint32_t l1 = from_left(hi[1]), r1 = from_right(lo[1]);
            lw[1] = first ? end0 : l1;
            rw[1] = last1 ? edge32 : r1;
            if (lane == kWave - 1 && !last)
                rw[0] = beg1;
        }
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const uint32_t ll = __builtin_amdgcn_alignbit(lo[q], lw[q], 31), lh = __builtin_amdgcn_alignbit(hi[q], lo[q], 31);
            const uint32_t rl = __builtin_amdgcn_alignbit(hi[q], lo[q], 1), rh = __builtin_amdgcn_alignbit(rw[q], hi[q], 1);
            const uint32_t ol = ERO ? (lo[q] & ll & rl) : (lo[q] | ll | rl), oh = ERO ? (hi[q] & lh & rh) : (hi[q] | lh | rh);
            x[r][q] = ((uint64_t)oh << 32) | ol;
        }
    }
}

template <int R, int KT, int NC>
__device__ __forceinline__ void morph_regs(Job *J, int item, WaveLds &L)
{
    constexpr int N = R + 2 * KT + 1;          // rows y0 - 1 - KT .. y0 + R + KT - 1
    const int lg = NC == 1 ? J->mgroup : kWave;
    const int word = lane_word(lg);
    const int H = J->H, Wd = J->Wd, oi = J->open_it, K = 2 * (oi + J->close_it);
    const int y0 = (item * (kWave / lg) + lane_group(lg)) * R;
    const int ytop = y0 - 1 - KT;
    const GLOBAL uint64_t *raw = G(J->raw);
    uint64_t x[N][NC];
    const bool edge = __ballot(ytop < 0 || ytop + N > H) != 0ull;
    uint32_t col[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q)
        col[q] = (uint32_t)min(word + kWave * q, Wd - 1);
    if (edge) {
#pragma unroll
        for (int r = 0; r < N; ++r) {
            const uint32_t row = (uint32_t)min(max(ytop + r, 0), H - 1) * (uint32_t)Wd;
#pragma unroll
            for (int q = 0; q < NC; ++q)
                x[r][q] = *at_byte(raw, 8u * (row + col[q]));
        }
    } else {
        const uint32_t row = (uint32_t)ytop * (uint32_t)Wd;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const uint32_t off = 8u * (row + col[q]);
#pragma unroll
            for (int r = 0; r < N; ++r)
                x[r][q] = *at_byte(raw + (size_t)r * Wd, off);
        }
    }
    bool valid_w[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q)
        valid_w[q] = word + kWave * q < Wd;
    // anything left after the first stage?
    uint64_t any = 0ull;
    if (oi > 0) {
#pragma unroll
        for (int r = 1; r < N - 1; ++r) {
            // rows outside the image are no obstacle to an erosion
            const bool above = !edge || (uint32_t)(ytop + r - 1) < (uint32_t)H,
                       below = !edge || (uint32_t)(ytop + r + 1) < (uint32_t)H,
                       here = !edge || (uint32_t)(ytop + r) < (uint32_t)H;
#pragma unroll
            for (int q = 0; q < NC; ++q) {
                uint64_t v = x[r][q] & (above ? x[r - 1][q] : ~0ull) & (below ? x[r + 1][q] : ~0ull);
                any |= valid_w[q] && here ? v : 0ull;
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < N; ++r)
#pragma unroll
            for (int q = 0; q < NC; ++q)
                any |= valid_w[q] && (uint32_t)(ytop + r) < (uint32_t)H ? x[r][q] : 0ull;
    }
    GLOBAL uint64_t *fz = G(J->fizi);
    if (__ballot(any != 0ull) == 0ull) {
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int q = 0; q < NC; ++q)
                if (valid_w[q] && y0 + j < H)
                    fz[j * Wd + y0 * Wd + word + kWave * q] = 0ull;
        return;
    }
    if (KT == 4 && oi == 1 && K == 4) {          // the default opening and closing
        regs_stage<true, N, NC>(x, 1, N - 2, Wd, lg, edge, ytop, H);
        regs_stage<false, N, NC>(x, 2, N - 3, Wd, lg, edge, ytop, H);
        regs_stage<false, N, NC>(x, 3, N - 4, Wd, lg, edge, ytop, H);
        regs_stage<true, N, NC>(x, 4, N - 5, Wd, lg, edge, ytop, H);
    } else {
#pragma unroll 1
        for (int k = 0; k < K; ++k) {
            if (stage_erodes(k, oi, J->close_it))
                regs_stage<true, N, NC>(x, 1, N - 2, Wd, lg, edge, ytop, H);
            else
                regs_stage<false, N, NC>(x, 1, N - 2, Wd, lg, edge, ytop, H);
        }
    }
    // the final rows: stored, and those with pixels gathered for the run pass
    typedef uint32_t rows_t __attribute__((ext_vector_type(R)));
    rows_t lo[NC], hi[NC];
    uint32_t full = 0;                          // bit j: row j has pixels
    uint32_t nstart = 0;                        // run starts in the lane's words
#pragma unroll
    for (int j = -1; j < R; ++j) {
        uint64_t orw = 0ull;
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            uint64_t &v = x[KT + 1 + j][q];
            const bool in = valid_w[q] && (uint32_t)(y0 + j) < (uint32_t)H;
            v = in ? v : 0ull;
            orw |= v;
            if (j >= 0) {
                if (in)
                    fz[j * Wd + y0 * Wd + word + kWave * q] = v;
                lo[q][j < 0 ? 0 : j] = (uint32_t)v;
                hi[q][j < 0 ? 0 : j] = (uint32_t)(v >> 32);
            }
        }
        if (j >= 0) {
            if (__ballot(orw != 0ull) != 0ull)
                full |= 1u << j;
            uint32_t lc[NC], rc[NC];
            row_carries<NC>(x[KT + 1 + j], Wd, 0u, lc, rc, lg);
#pragma unroll
            for (int q = 0; q < NC; ++q)
                nstart += (uint32_t)__popcll(x[KT + 1 + j][q] & ~((x[KT + 1 + j][q] << 1) | lc[q]));
        }
    }
    if (!full)
        return;
    const BandOut B = band_out(J, lg);
    RunState<NC> S;
    L.npairs = 0u;
    wave_sync();
    uint64_t orw = 0ull;
#pragma unroll
    for (int q = 0; q < NC; ++q)
        orw |= x[KT][q];
    const bool halo = (full & 1u) && __ballot(orw != 0ull) != 0ull;
    auto row_of = [&](int j, uint64_t (&v)[NC]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NC; ++q)
            v[q] = ((uint64_t)hi[q][j] << 32) | lo[q][j];
    };
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(nstart), kWave - 1);
    if (total <= (uint32_t)kSegRuns) {
        // one segment holds the band's runs: their places in the run list and
        // those of the joins with the band above are reserved at once, ahead
        // of the rows, so that the 2 us the device-scope atomic takes pass
        // beside them
        uint64_t v0[NC], en[NC];
        row_of(0, v0);
        uint32_t cnt = 0, inc = 0;
        RowBits<NC> D0;
        if (halo) {
            (void)row_bits<NC>(S.P, x[KT], Wd, en, lg);
            (void)row_bits<NC>(D0, v0, Wd, en, lg);
            touching_runs<NC>(S.P, D0, [&](int, bool, int, int) { ++cnt; });
            inc = wave_incl_scan(cnt);
        }
        const uint32_t nlink = (uint32_t)__builtin_amdgcn_readlane((int)inc, kWave - 1);
        unsigned long long at = 0;
        if ((threadIdx.x & (kWave - 1)) == 0)
            at = atomicAdd(reinterpret_cast<unsigned long long *>(&J->nruns),
                           (unsigned long long)total | ((unsigned long long)nlink << 32));
        int before = -2;                        // last row with runs
#pragma unroll 1
        for (uint32_t m = full; m; m &= m - 1u) {
            const int j = __builtin_ctz(m);
            uint64_t v[NC];
            row_of(j, v);
            if (j != before + 1)
                S.prev_valid = false;
            before = j;
            run_row<NC, false, true>(B, S, L, v, y0 + j);
        }
        unite_pairs(L);
        const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at),
                       lbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32));
        if (nlink) {
            row_of(0, v0);
            (void)row_bits<NC>(S.P, x[KT], Wd, en, lg);
            const uint32_t first = row_bits<NC>(D0, v0, Wd, en, lg);
            band_links<NC, false, true>(B, S.P, D0, (uint32_t)max(y0, 0) * (uint32_t)B.W, lbase + inc - cnt);
            if (lbase + nlink > B.link_cap) {
                // the list is full: the component stage joins the row's runs
                // to the row above by reading I_FIZI
                for (uint32_t k = threadIdx.x & (kWave - 1); k < first; k += kWave)
                    L.end[k] |= kLinkUp;
                wave_sync();
                if ((threadIdx.x & (kWave - 1)) == 0)
                    atomicAdd(&J->nflag, 1u);
            }
        }
        store_segment<false>(L, S.nseg, base, B.runs, B.parent, B.index, B.cap);
        return;
    }
    if (halo)
        halo_row<NC>(B, S, x[KT]);
    int before = -1;                            // last row with runs
#pragma unroll 1
    for (uint32_t m = full; m; m &= m - 1u) {
        const int j = __builtin_ctz(m);
        uint64_t v[NC];
        row_of(j, v);
        if (j != before + 1)
            S.prev_valid = false;
        before = j;
        run_row<NC, false>(B, S, L, v, y0 + j);
    }
    flush_segment<false>(J, L, S.nseg, B.runs, B.parent, B.index, B.cap);
}

template <int KMAX, int NC>
__global__ __launch_bounds__(256) void k_morph(Table *__restrict__ T)
{
    __shared__ WaveLds s_wl[256 / kWave];
    // wave-uniform, and known to be: the band, its job and everything derived
    // from them then live in scalar registers, with scalar branches
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int nj = T->h.njobs;
    const int total = T->h.mor_pre[nj];
    for (int t = blockIdx.x * (256 / kWave) + wave; t < total; t += gridDim.x * (256 / kWave))
    {
        const int j = find_job(T->h.mor_pre, nj, t);
        Job *J = &T->jobs[j];
        const int item = t - T->h.mor_pre[j];
        if (KMAX >= 4 && J->open_it == 1 && J->close_it == 1)     // the default opening and closing
            morph_band<KMAX, NC, false, 1, 1>(J, item, s_wl[wave]);
        else
            morph_band<KMAX, NC, false>(J, item, s_wl[wave]);
    }
}

// Bands of R rows, or of the short height (the height is the job's: a graph
// replays one kernel for steps of either). A span's jobs have `items` each and
// `total` in all; otherwise (items 0) both come from the table.
template <int R, int KT, int NC>
__global__ __launch_bounds__(256) void k_morph_regs(Table *__restrict__ T, int total, int items)
{
    __shared__ WaveLds s_wl[256 / kWave];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int nj = items ? 0 : T->h.njobs;
    if (!items)
        total = T->h.mor_pre[nj];
    for (int t = blockIdx.x * (256 / kWave) + wave; t < total; t += gridDim.x * (256 / kWave)) {
        const int j = items ? t / items : find_job(T->h.mor_pre, nj, t);
        Job *J = &T->jobs[j];
        const int item = t - (items ? j * items : T->h.mor_pre[j]);
        if (NC == 2 && J->Wd > kWave) {
            if (J->band == kShortBand)
                morph_regs<kShortBand, KT, 2>(J, item, s_wl[wave]);
            else
                morph_regs<R, KT, 2>(J, item, s_wl[wave]);
        } else if (J->band == kShortBand) {
            morph_regs<kShortBand, KT, 1>(J, item, s_wl[wave]);
        } else {
            morph_regs<R, KT, 1>(J, item, s_wl[wave]);
        }
    }
}

// Steps of a batch with wide frames and, of any stream, more than four stages:
// jobs of at most four stages hold their bands in registers as above, the
// others stream them. 32 streams of 1920x1080 but for a deep one of 7680x1080,
// pipelined in 16-row bands: 116 us of morphology, 170 with every band streamed
// by a wave of its own (125 with narrow ones sharing it); 63 of 1024x768 beside
// that one 114, 186 and 122.
template <int R>
__global__ __launch_bounds__(256) void k_morph_mixed(Table *__restrict__ T)
{
    __shared__ WaveLds s_wl[256 / kWave];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int nj = T->h.njobs;
    const int total = T->h.mor_pre[nj];
    for (int t = blockIdx.x * (256 / kWave) + wave; t < total; t += gridDim.x * (256 / kWave)) {
        const int j = find_job(T->h.mor_pre, nj, t);
        Job *J = &T->jobs[j];
        const int item = t - T->h.mor_pre[j];
        const bool wide = J->Wd > kWave;
        if (2 * (J->open_it + J->close_it) > 4) {
            if (wide)
                morph_band<4 * kMaxMorphIters, 2, false>(J, item, s_wl[wave]);
            else
                morph_band<4 * kMaxMorphIters, 1, false>(J, item, s_wl[wave]);
        } else if (J->band == kShortBand) {
            if (wide)
                morph_regs<kShortBand, 4, 2>(J, item, s_wl[wave]);
            else
                morph_regs<kShortBand, 4, 1>(J, item, s_wl[wave]);
        } else if (wide) {
            morph_regs<R, 4, 2>(J, item, s_wl[wave]);
        } else {
            morph_regs<R, 4, 1>(J, item, s_wl[wave]);
        }
    }
}

// ---------------------------------------------------------------------------
// Workgroup of the component stage: 512 threads when it runs on its own (one
// frame of 1920x1080 in 1024 / 512 / 256 threads: 9.9 / 8.9 / 8.0 us, eight of
// 3840x2160 10.0 / 9.3 / 9.6, eight of 1920x1080 10.4 / 10.1 / 11.3); 256
// beside a streaming kernel (pipelined steps), where a large workgroup finds
// no room until the streaming kernel drains.
constexpr int kResolveThreads = 512;
constexpr int kResolveThreadsSmall = 256;
constexpr int kMaxWaves = 16;

// Component areas of one frame, summed in LDS: an open-addressing table from
// root to area. A component's runs all add to its root, and same-address
// atomics serialise far less in LDS than in the cache (a hand is a thousand
// runs on a 4K frame). A root that finds no free slot in its bucket adds in
// global memory instead, and so do all of its runs, since slots are only ever
// taken, the first free one of a bucket first: the table and the global array
// never share a root. A bucket is read at once (slot by slot over a window of
// 32, a frame of noise spent half of its components' time here).
constexpr int kAreaSlots = 2048;
constexpr int kAreaBucket = 8;
constexpr uint32_t kAreaEmpty = 0xFFFFFFFFu;
struct AreaTable {
    uint32_t key[kAreaSlots];
    uint32_t val[kAreaSlots];
    uint32_t overflow;
};

// A frame's components in LDS where its runs fit: 3072 (48 KiB) in the
// component stage, 2048 in the persistent step, which lends its four waves'
// morphology tables (16 bytes a run). A frame with more runs is resolved in global memory, with
// the table of areas in the same place.
constexpr int kForestRuns = 3072, kForestRunsFlow = 2048;
template <int C>
union ResolveLds {
    LdsRuns<C> runs;
    AreaTable areas;
};
static_assert(sizeof(ResolveLds<kForestRunsFlow>) <= 4 * sizeof(WaveLds), "the forest fits the morphology LDS");

__device__ __forceinline__ void area_add(AreaTable &t, GLOBAL uint32_t *area, uint32_t root, uint32_t len)
{
    const uint32_t first = ((root * 2654435761u) >> (32 - 11)) & ~(uint32_t)(kAreaBucket - 1);
    for (;;) {
        uint32_t k[kAreaBucket], slot = kAreaBucket;
#pragma unroll
        for (int q = 0; q < kAreaBucket; ++q)
            k[q] = __hip_atomic_load(&t.key[first + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // the root's slot, else the first free one
#pragma unroll
        for (int q = kAreaBucket - 1; q >= 0; --q)
            slot = k[q] == kAreaEmpty ? (uint32_t)q : slot;
        bool found = false;
#pragma unroll
        for (int q = 0; q < kAreaBucket; ++q) {
            found |= k[q] == root;
            slot = k[q] == root ? (uint32_t)q : slot;
        }
        if (slot == kAreaBucket)
            break;
        if (!found) {
            const uint32_t was = atomicCAS(&t.key[first + slot], kAreaEmpty, root);
            if (was != kAreaEmpty && was != root)
                continue;               // another root took it
        }
        atomicAdd(&t.val[first + slot], len);
        return;
    }
    t.overflow = 1u;
    __hip_atomic_fetch_add(area + root, len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Second half of a workgroup reduction: the at most 16 waves' results in s.
template <typename V, typename OP>
__device__ __forceinline__ V waves_reduce(const V *s, V none, OP op)
{
    const int lane = threadIdx.x & (kWave - 1), nw = blockDim.x / kWave;
    return from_lane(row_reduce(lane < nw ? s[lane] : none, none, op), 15);
}

// Workgroup reductions (every thread gets the result).
template <typename V, typename OP>
__device__ __forceinline__ V wg_reduce(V v, V none, OP op, V *s_tmp)
{
    v = wave_reduce(v, none, op);
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0)
        s_tmp[threadIdx.x / kWave] = v;
    __syncthreads();
    return waves_reduce(s_tmp, none, op);
}

constexpr uint32_t kNoRoot = 0xFFFFFFFFu;

// A frame's components after its unions: their number, the largest one's
// area and root run (ties to the smallest first pixel).
struct Components {
    uint32_t count, area, root;
};

// The components of a forest whose areas are known, from each thread's own
// best key (area << 32 | ~first pixel) and root run, and its count of roots
// (whole workgroup).
__device__ __forceinline__ Components largest_of(unsigned long long best, uint32_t root, uint32_t count)
{
    __shared__ unsigned long long s_u64[kMaxWaves];
    __shared__ uint32_t s_u32[kMaxWaves], s_root;
    unsigned long long all = wave_reduce(best, 0ull, OpMax());
    count = wave_reduce(count, 0u, OpSum());
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_u64[threadIdx.x / kWave] = all;
        s_u32[threadIdx.x / kWave] = count;
    }
    if (threadIdx.x == 0)
        s_root = kNoRoot;
    __syncthreads();
    all = waves_reduce(s_u64, 0ull, OpMax());
    count = waves_reduce(s_u32, 0u, OpSum());
    // a key belongs to one component
    if (best == all && best != 0ull)
        s_root = root;
    __syncthreads();
    return Components{count, (uint32_t)(all >> 32), s_root};
}

__device__ __forceinline__ unsigned long long size_key(uint32_t area, uint32_t first)
{
    return ((unsigned long long)area << 32) | (0xFFFFFFFFull - first);
}

// The components of one frame (one workgroup): the joins across band and
// segment borders, every run's root and each component's area, and the
// largest component. In LDS: the run list, parents and joins are each read
// once, all loads at once, and what follows waits for LDS only (in global
// memory each step of a find and each union was a dependent access of 0.6 us:
// one frame of 1920x1080 15.7 us against 8.9 here, 16 of 1280x720 12.5 against
// 9.5, the 64-stream batch beside classify 134 against 43).
template <int C>
__device__ __forceinline__ Components resolve_lds(Job *J, LdsRuns<C> &t, uint32_t nr, uint32_t nl)
{
    const GLOBAL uint64_t *runs = G(reinterpret_cast<const uint64_t *>(J->runs));
    const GLOBAL uint64_t *links = G(reinterpret_cast<const uint64_t *>(J->links));
    const GLOBAL uint32_t *index = G(J->index), *parent = G(J->parent);
    const LdsForest<C> f{t};
    // the thread's first join, its runs looked up beside the run list
    uint32_t la = 0, lb = 0;
    const bool joins = threadIdx.x < nl;
    if (joins) {
        const uint64_t l = links[threadIdx.x];
        la = index[(uint32_t)l];
        lb = index[(uint32_t)(l >> 32)];
    }
    for (uint32_t i = threadIdx.x; i < nr; i += blockDim.x) {
        const uint2 rn = unpack_run(runs[i]);
        t.par[i] = parent[i];
        t.start[i] = rn.x;
        t.len[i] = rn.y;
        t.area[i] = rn.y;
    }
    __syncthreads();
    if (joins)
        unite(f, la, lb);
    for (uint32_t i = threadIdx.x + blockDim.x; i < nl; i += blockDim.x) {
        const uint64_t l = links[i];
        unite(f, index[(uint32_t)l], index[(uint32_t)(l >> 32)]);
    }
    __syncthreads();
    // shorten the paths, then point every run at its root
    for (uint32_t i = threadIdx.x; i < nr; i += blockDim.x)
        (void)find_root(f, i);
    __syncthreads();
    uint32_t count = 0;
    for (uint32_t i = threadIdx.x; i < nr; i += blockDim.x) {
        const uint32_t r = root_of(f, i);
        if (r == i) {
            ++count;
        } else {
            f.set_par(i, r);
            atomicAdd(&t.area[r], t.len[i]);
        }
    }
    __syncthreads();
    unsigned long long best = 0ull;
    uint32_t root = 0;
    for (uint32_t i = threadIdx.x; i < nr; i += blockDim.x) {
        if (t.par[i] == i) {
            const unsigned long long key = size_key(t.area[i], t.start[i]);
            if (key > best) {
                best = key;
                root = i;
            }
        }
    }
    return largest_of(best, root, count);
}

// Joins a run of the list with the row above by reading I_FIZI.
template <typename F>
__device__ __forceinline__ void link_run(const F &f, const GLOBAL uint32_t *index, const GLOBAL uint64_t *fz, int Wd,
                                         int W, uint32_t i)
{
    const uint2 rn = f.run(i);
    const int y = (int)(rn.x / (uint32_t)W), xs = (int)(rn.x - (uint32_t)y * W);
    if (y > 0)
        link_up(f, index, fz + (size_t)(y - 1) * Wd, Wd, W, y, xs, xs + (int)rn.y - 1, i);
}

// Joins the flagged runs of the list with the row above (whole workgroup).
// kAhead runs of a thread at once: a short run's columns in the row above, one
// to either side included, are a window of at most 64 bits, whose runs of ones
// are taken from the left; the runs' next ones are united together. Longer
// runs go one by one.
template <typename F>
__device__ __forceinline__ void link_flagged(const F &f, const GLOBAL uint32_t *index, const GLOBAL uint64_t *fz,
                                             int Wd, int W, uint32_t nr)
{
    constexpr int U = F::kAhead;
    if constexpr (U == 1) {
        for (uint32_t i = threadIdx.x; i < nr; i += blockDim.x)
            if ((uint32_t)(f.runs[i] >> 32) & kLinkUp)
                link_run(f, index, fz, Wd, W, i);
        return;
    }
    for (uint32_t i = threadIdx.x; i < nr; i += U * blockDim.x) {
        uint64_t rv[U], t[U];
        uint32_t up[U];                          // row above
        int base[U];                             // window's first column
#pragma unroll
        for (int u = 0; u < U; ++u)
            rv[u] = f.runs[min(i + u * blockDim.x, nr - 1u)];
        uint32_t todo = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint2 rn = unpack_run(rv[u]);
            const uint32_t y = rn.x / (uint32_t)W, xs = rn.x - y * (uint32_t)W;
            const bool join = i + u * blockDim.x < nr && ((uint32_t)(rv[u] >> 32) & kLinkUp) && y > 0;
            up[u] = max(y, 1u) - 1u;
            base[u] = max((int)xs - 1, 0);
            const int n = min((int)(xs + rn.y), W - 1) - base[u] + 1;
            const GLOBAL uint64_t *above = fz + (size_t)up[u] * Wd;
            const int w = base[u] >> 6, b = base[u] & 63;
            const uint64_t m0 = above[w], m1 = above[min(w + 1, Wd - 1)];
            const uint64_t v = (m0 >> b) | ((m1 << 1) << (63 - b));
            t[u] = join && n <= 64 ? v & (~0ull >> (64 - n)) : 0ull;
            todo |= (uint32_t)(join && n > 64) << u;
        }
        for (;;) {
            uint64_t left = 0ull;
#pragma unroll
            for (int u = 0; u < U; ++u)
                left |= t[u];
            if (!__builtin_amdgcn_ballot_w64(left != 0ull))
                break;
            uint32_t a[U], b[U], live = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = b[u] = 0u;
                if (t[u]) {
                    int x = base[u] + __builtin_ctzll(t[u]);
                    if (x == base[u])            // its run may start further left
                        x = prev_zero(fz + (size_t)up[u] * Wd, x) + 1;
                    a[u] = i + u * blockDim.x;
                    b[u] = index[up[u] * (uint32_t)W + (uint32_t)x];
                    live |= 1u << u;
                    t[u] &= t[u] + (t[u] & (0ull - t[u]));
                }
            }
            unite_at_once<U>(f, a, b, live);
        }
        for (; todo; todo &= todo - 1u)
            link_run(f, index, fz, Wd, W, i + (uint32_t)__builtin_ctz(todo) * blockDim.x);
    }
}

// The same in global memory, for frames with more runs or an overflown join
// list (its flagged runs are joined by reading I_FIZI). Afterwards the areas
// hold every root's area and each other run's parent is one of its ancestors
// (see root_of).
// Bound by the latency of its dependent accesses, one workgroup to a frame: a
// thread takes A runs or joins at once. One frame of 1920x1088 of noise of
// density 0.02 / 0.2 / 0.5: 102 / 1830 / 7740 us; one by one, in 512 threads,
// 383 / 6770 / 16240, in 1024 with the runs known by their first pixel 343 /
// 3950 / 9050.
template <int A>
__device__ __forceinline__ Components resolve_global(Job *J, AreaTable &tab, uint32_t nr, uint32_t nl, uint32_t nflag)
{
    const int W = J->W, Wd = J->Wd;
    const GlobalForest<A> f(J);
    const GLOBAL uint64_t *links = G(reinterpret_cast<const uint64_t *>(J->links));
    const GLOBAL uint32_t *index = G(J->index);
    const GLOBAL uint64_t *fz = G(J->fizi);
    if (threadIdx.x == 0)
        tab.overflow = 0;
    for (int i = threadIdx.x; i < kAreaSlots; i += blockDim.x) {
        tab.key[i] = kAreaEmpty;
        tab.val[i] = 0;
    }
    for (uint32_t i = threadIdx.x; i < nr; i += blockDim.x)
        st_wg(f.areas + i, 0u);
    __syncthreads();
    constexpr int U = A;
    for (uint32_t i = threadIdx.x; i < nl; i += U * blockDim.x) {
        uint64_t l[U];
        uint32_t a[U], b[U], live = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            live |= (uint32_t)(i + u * blockDim.x < nl) << u;
            l[u] = links[min(i + u * blockDim.x, nl - 1u)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            a[u] = index[(uint32_t)l[u]];
            b[u] = index[(uint32_t)(l[u] >> 32)];
        }
        if constexpr (U == 1)
            unite(f, a[0], b[0]);
        else
            unite_at_once<U>(f, a, b, live);
    }
    if (nflag)
        link_flagged(f, index, fz, Wd, W, nr);
    __syncthreads();
    // roots and areas; a thread's runs of one root in a row are added together
    // (most of a frame's runs may be one component's)
    uint32_t count = 0, held = kNoRoot, sum = 0;
    for (uint32_t i = threadIdx.x; i < nr; i += U * blockDim.x) {
        uint32_t x[U], r[U], len[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = min(i + u * blockDim.x, nr - 1u);
            len[u] = f.run(x[u]).y;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            r[u] = x[u];
        find_roots<U>(f, r);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i + u * blockDim.x >= nr)
                break;
            if (r[u] == x[u])
                ++count;
            else
                f.set_par(x[u], r[u]);
            if (r[u] != held) {
                if (held != kNoRoot)
                    area_add(tab, f.areas, held, sum);
                held = r[u];
                sum = 0;
            }
            sum += len[u];
        }
    }
    if (held != kNoRoot)
        area_add(tab, f.areas, held, sum);
    __syncthreads();
    // the table's areas go to the global array (tracking and the chain read
    // it); the largest component from the table, or from every run when some
    // root did not fit it
    unsigned long long best = 0ull;
    uint32_t root = 0;
    for (int i = threadIdx.x; i < kAreaSlots; i += blockDim.x) {
        const uint32_t k = tab.key[i];
        if (k != kAreaEmpty) {
            st_wg(f.areas + k, tab.val[i]);
            const unsigned long long key = size_key(tab.val[i], f.start(k));
            if (key > best) {
                best = key;
                root = k;
            }
        }
    }
    if (tab.overflow) {
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < nr; i += U * blockDim.x) {
            uint32_t p[U], area[U], start[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t k = min(i + u * blockDim.x, nr - 1u);
                p[u] = f.par(k);
                area[u] = f.area(k);
                start[u] = f.start(k);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t k = min(i + u * blockDim.x, nr - 1u);
                const unsigned long long key = size_key(area[u], start[u]);
                if (p[u] == k && key > best) {
                    best = key;
                    root = k;
                }
            }
        }
    }
    return largest_of(best, root, count);
}

// The run covering pixel tx of a row, or kNoRoot. The run's start mostly lies
// within the four words up to the pixel's: they are loaded at once instead of
// one after the other.
__device__ __forceinline__ uint32_t run_at(const GLOBAL uint64_t *row, const GLOBAL uint32_t *index, int tx)
{
    const int w = tx >> 6, b = tx & 63;
    const uint64_t m0 = row[w], m1 = row[max(w - 1, 0)], m2 = row[max(w - 2, 0)], m3 = row[max(w - 3, 0)];
    if (!((m0 >> b) & 1ull))
        return kNoRoot;
    const uint64_t z0 = ~m0 & ((1ull << b) - 1ull), z1 = w >= 1 ? ~m1 : 0ull, z2 = w >= 2 ? ~m2 : 0ull,
                   z3 = w >= 3 ? ~m3 : 0ull;
    int start = 0;
    if (z0 | z1 | z2 | z3) {
        const int k = z0 ? 0 : z1 ? 1 : z2 ? 2 : 3;
        const uint64_t z = z0 ? z0 : z1 ? z1 : z2 ? z2 : z3;
        start = ((w - k) << 6) + 64 - __builtin_clzll(z);
    } else if (w >= 4) {
        start = prev_zero(row, ((w - 3) << 6) - 1) + 1;
    }
    return index[start];
}

// The run covering pixel (tx, ty), or kNoRoot (one thread; it needs no forest).
__device__ __forceinline__ uint32_t covering_run(const Job *J, int tx, int ty)
{
    if (tx < 0 || tx >= J->W || ty < 0 || ty >= J->H)
        return kNoRoot;
    return run_at(G(J->fizi) + (size_t)ty * J->Wd, G(J->index) + (uint32_t)ty * (uint32_t)J->W, tx);
}

// The component of area >= amin nearest to (tx, ty) within sqrt(r2) pixels:
// the smallest squared distance from the point to a pixel of it, ties to the
// larger area, then the smaller first pixel; kNoRoot when none (whole
// workgroup; the forest is final). A run's pixel nearest to the point is
// its own clamp of tx, so two passes over the runs decide it: the least
// distance, then the best key among the runs at that distance.
template <typename F>
__device__ __forceinline__ uint32_t nearest_root(const Job *J, const F &f, int tx, int ty, uint32_t amin, uint32_t r2)
{
    __shared__ uint32_t s_min[kMaxWaves];
    __shared__ unsigned long long s_key[kMaxWaves];
    const int W = J->W;
    const uint32_t nr = min(ld_dev(&J->nruns), J->run_cap);
    auto dist2 = [&](uint2 rn) -> uint32_t {
        const int y = (int)(rn.x / (uint32_t)W), xs = (int)(rn.x - (uint32_t)y * W), xe = xs + (int)rn.y - 1;
        const int dx = tx < xs ? xs - tx : (tx > xe ? tx - xe : 0), dy = y - ty;
        const unsigned long long d2 = (unsigned long long)((long long)dx * dx) + (unsigned long long)((long long)dy * dy);
        return d2 > 0xFFFFFFFEull ? 0xFFFFFFFEu : (uint32_t)d2;
    };
    constexpr int U = F::kAhead;
    uint32_t dmin = 0xFFFFFFFFu;
    for (uint32_t i = threadIdx.x; i < nr; i += U * blockDim.x) {
        uint32_t x[U], r[U], area[U];
        uint2 rn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = min(i + u * blockDim.x, nr - 1u);
            rn[u] = f.run(x[u]);
        }
        roots_of<U>(f, x, r);
#pragma unroll
        for (int u = 0; u < U; ++u)
            area[u] = f.area(r[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (area[u] >= amin)
                dmin = min(dmin, dist2(rn[u]));
    }
    dmin = wg_reduce(dmin, 0xFFFFFFFFu, OpMin(), s_min);
    if (dmin > r2)
        return kNoRoot;
    unsigned long long key = 0ull;
    for (uint32_t i = threadIdx.x; i < nr; i += U * blockDim.x) {
        uint32_t hit = 0;
        uint2 rn[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            rn[u] = f.run(min(i + u * blockDim.x, nr - 1u));
#pragma unroll
        for (int u = 0; u < U; ++u)
            hit |= (uint32_t)(i + u * blockDim.x < nr && dist2(rn[u]) == dmin) << u;
        for (; hit; hit &= hit - 1u) {
            const uint32_t r = root_of(f, i + (uint32_t)__builtin_ctz(hit) * blockDim.x);
            const uint32_t a = f.area(r);
            if (a >= amin) {
                const unsigned long long k = size_key(a, f.start(r));
                key = k > key ? k : key;
            }
        }
    }
    key = wg_reduce(key, 0ull, OpMax(), s_key);
    return key ? G(J->index)[0xFFFFFFFFu - (uint32_t)(key & 0xFFFFFFFFull)] : kNoRoot;
}

// The tracked pick given the previous frame's centroid pixel (valid: it had
// a hand): the covering component, else the nearest within the radius;
// kNoRoot for the largest (whole workgroup).
// cover: the run covering that pixel, or kNoRoot.
template <typename F>
__device__ __forceinline__ uint32_t tracked_pick(const Job *J, const F &f, const TrackState &ts, uint32_t cover)
{
    const uint32_t amin = (uint32_t)max(J->min_area, 0);
    uint32_t pick = kNoRoot;
    if (cover != kNoRoot) {
        const uint32_t r = root_of(f, cover);
        if (f.area(r) >= amin)
            pick = r;
    }
    if (ts.valid && pick == kNoRoot && J->track_r2 > 0)
        pick = nearest_root(J, f, ts.x, ts.y, amin, J->track_r2);
    return pick;
}

struct ZoneStats {
    unsigned long long sx, sy;
    uint32_t x0, y0, x1, y1;
};

// Pass D: coordinate sums and box of component kstar, and its hand bits
// (whole workgroup; thread 0 gets the totals). Membership walks each run to
// its root without writing.
template <typename F>
__device__ __forceinline__ ZoneStats zone_stats(const Job *J, const F &f, uint32_t kstar, GLOBAL uint64_t *hand)
{
    __shared__ unsigned long long s_u64[2][kMaxWaves];
    __shared__ uint32_t s_u32[4][kMaxWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int W = J->W, Wd = J->Wd;
    const uint32_t nr = min(ld_dev(&J->nruns), J->run_cap);
    ZoneStats z{0, 0, 0xFFFFFFFFu, 0xFFFFFFFFu, 0, 0};
    auto add = [&](const uint2 run) __attribute__((always_inline)) {
        const uint32_t y = run.x / (uint32_t)W, xs = run.x - y * (uint32_t)W, n = run.y;
        z.sx += (unsigned long long)n * xs + (unsigned long long)n * (n - 1) / 2;
        z.sy += (unsigned long long)n * y;
        z.x0 = min(z.x0, xs);
        z.x1 = max(z.x1, xs + n - 1);
        z.y0 = min(z.y0, y);
        z.y1 = max(z.y1, y);
    };
    auto mark = [&](const uint2 run) __attribute__((always_inline)) {
        const uint32_t y = run.x / (uint32_t)W, xs = run.x - y * (uint32_t)W, xe = xs + run.y - 1;
        GLOBAL uint64_t *hr = hand + (size_t)y * Wd;
        const int wa = (int)(xs >> 6), wb = (int)(xe >> 6);
        for (int w = wa; w <= wb; ++w) {
            const int lo = (w == wa) ? (int)(xs & 63) : 0;
            const int hi = (w == wb) ? (int)(xe & 63) : 63;
            const uint64_t m = (hi == 63 ? ~0ull : ((2ull << hi) - 1ull)) & (~0ull << lo);
            __hip_atomic_fetch_or(hr + w, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    constexpr int U = F::kAhead;
    for (uint32_t i = threadIdx.x; i < nr; i += U * blockDim.x) {
        if constexpr (U == 1) {
            if (root_of(f, i) != kstar)
                continue;
            const uint2 run = f.run(i);
            add(run);
            if (hand)
                mark(run);
        } else {
            uint32_t x[U], r[U], hit = 0;
            uint2 rn[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                x[u] = min(i + u * blockDim.x, nr - 1u);
                rn[u] = f.run(x[u]);
            }
            roots_of<U>(f, x, r);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (r[u] != kstar || i + u * blockDim.x >= nr)
                    continue;
                hit |= 1u << u;
                add(rn[u]);
            }
            for (; hand && hit; hit &= hit - 1u) {
                const int k = __builtin_ctz(hit);
                uint2 run = rn[0];
#pragma unroll
                for (int u = 1; u < U; ++u)
                    run = k == u ? rn[u] : run;
                mark(run);
            }
        }
    }
    z.sx = wave_reduce(z.sx, 0ull, OpSum());
    z.sy = wave_reduce(z.sy, 0ull, OpSum());
    z.x0 = wave_reduce(z.x0, 0xFFFFFFFFu, OpMin());
    z.y0 = wave_reduce(z.y0, 0xFFFFFFFFu, OpMin());
    z.x1 = wave_reduce(z.x1, 0u, OpMax());
    z.y1 = wave_reduce(z.y1, 0u, OpMax());
    __syncthreads();
    if (lane == 0) {
        s_u64[0][wave] = z.sx;
        s_u64[1][wave] = z.sy;
        s_u32[0][wave] = z.x0;
        s_u32[1][wave] = z.y0;
        s_u32[2][wave] = z.x1;
        s_u32[3][wave] = z.y1;
    }
    __syncthreads();
    if (wave == 0) {
        z.sx = waves_reduce(s_u64[0], 0ull, OpSum());
        z.sy = waves_reduce(s_u64[1], 0ull, OpSum());
        z.x0 = waves_reduce(s_u32[0], 0xFFFFFFFFu, OpMin());
        z.y0 = waves_reduce(s_u32[1], 0xFFFFFFFFu, OpMin());
        z.x1 = waves_reduce(s_u32[2], 0u, OpMax());
        z.y1 = waves_reduce(s_u32[3], 0u, OpMax());
    }
    return z;
}

// The pointer of a frame's zone (thread 0): present when the frame has
// components and the zone's area reaches min_area; the click is the
// fill-ratio rule.
__device__ __forceinline__ fizi_pointer make_pointer(const Job *J, bool present, uint32_t A, const ZoneStats &z,
                                                     uint32_t ncomp, uint32_t inv)
{
    fizi_pointer o;
    o.present = present ? 1 : 0;
    o.click = 0;
    o.reserved = 0;
    o.area = 0;
    o.sum_x = o.sum_y = 0;
    o.x0 = o.y0 = o.x1 = o.y1 = 0;
    if (present) {
        o.area = A;
        o.sum_x = z.sx;
        o.sum_y = z.sy;
        o.x0 = z.x0;
        o.y0 = z.y0;
        o.x1 = z.x1;
        o.y1 = z.y1;
        const unsigned long long box = (unsigned long long)(z.x1 - z.x0 + 1) * (z.y1 - z.y0 + 1);
        o.click = (1000ull * A >= (unsigned long long)J->fill_pm * box) ? 1 : 0;
    }
    o.n_components = ncomp;
    o.inv_gain_q16 = inv;
    o.frame_index = J->frame_index;
    return o;
}

// Click debouncing of a tracked stream (thread 0): a change is reported
// once `debounce` consecutive frames show it; no hand clears the count.
// Updates the stream's state and returns the reported click.
__device__ __forceinline__ uint8_t debounce_click(uint32_t *state, bool present, uint8_t click, int debounce)
{
    uint32_t shown = *state & 1u, count = (*state >> 8) & 0xFFu;
    if (!present) {
        shown = 0;
        count = 0;
    } else if (click == shown) {
        count = 0;
    } else if (++count >= (uint32_t)debounce) {
        shown = click;
        count = 0;
    }
    *state = shown | (count << 8);
    return (uint8_t)shown;
}

// The hand zone of a frame whose components are known, and its pointer (whole
// workgroup). A tracked frame picks its zone from the previous centroid
// (tracked_pick) and debounces its click - unless `defer`: then the frame's
// pointer is the largest component's, its root run goes to J->pick, and the
// tracking chain (k_track_chain) settles the tracked frames of the launch in
// order afterwards.
template <typename F>
__device__ __forceinline__ void resolve_zone(Job *J, const F &f, const Components &c, uint32_t inv, bool defer,
                                             const TrackState &was, uint32_t cover)
{
    GLOBAL uint64_t *hand = J->hand ? G(J->hand) : nullptr;
    TrackState *ts = J->track;
    uint32_t pick = kNoRoot;
    if (ts && !defer)
        pick = tracked_pick(J, f, was, cover);
    const bool tracked = pick != kNoRoot;
    const uint32_t A = tracked ? f.area(pick) : c.area;
    const uint32_t kstar = tracked ? pick : c.root;
    const bool present = c.count > 0 && (long long)A >= (long long)J->min_area;
    ZoneStats z{0, 0, 0, 0, 0, 0};
    if (present)
        z = zone_stats(J, f, kstar, hand);
    if (threadIdx.x == 0) {
        fizi_pointer o = make_pointer(J, present, A, z, c.count, inv);
        if (defer) {
            J->pick = c.count > 0 ? kstar : kNoRoot;
        } else if (ts) {
            o.click = debounce_click(&ts->click, present, o.click, J->debounce);
            ts->valid = present ? 1 : 0;
            if (present) {
                ts->x = (int32_t)(z.sx / A);
                ts->y = (int32_t)(z.sy / A);
            }
        }
        *J->out = o;
        // the final pointer also goes straight to the host ring, when the
        // job has one (a deferred pick is settled by the chain kernel)
        if (J->hout && !defer)
            *J->hout = o;
    }
}

// One workgroup per frame: its components, the hand zone, and the pointer.
template <int C, int A>
__device__ __forceinline__ void resolve_job(Table *__restrict__ T, int j, bool same_launch, ResolveLds<C> &lds,
                                            bool defer = false)
{
    Job *J = &T->jobs[j];
    // in the persistent step left by the frame's last gain tile before any of
    // its bands
    const uint32_t inv = same_launch ? ld_dev(&J->ginv) & ~kGainKnown : frame_gain(J);
    const uint32_t nr = min(ld_dev(&J->nruns), J->run_cap), nl = min(ld_dev(&J->nlinks), J->link_cap),
                   nflag = ld_dev(&J->nflag);
    if (J->hand) {
        GLOBAL uint64_t *hand = G(J->hand);
        for (int i = threadIdx.x; i < J->H * J->Wd; i += blockDim.x)
            hand[i] = 0ull;
    }
    // a tracked frame's covering run, looked up beside the forest's loads by
    // the last wave's first lane
    __shared__ uint32_t s_cover;
    TrackState was{};
    if (J->track && !defer) {
        was = *J->track;
        if (threadIdx.x == blockDim.x - kWave)
            s_cover = was.valid ? covering_run(J, was.x, was.y) : kNoRoot;
    }
    // the likely side: its code is then laid out in one piece ahead of the much
    // larger rest (eight frames of 3840x2160 12.0 us against 12.7)
    if (__builtin_expect(nr <= (uint32_t)C && nflag == 0u, 1)) {
        const LdsForest<C> f{lds.runs};
        const Components c = resolve_lds(J, lds.runs, nr, nl);
        if (defer) {
            // the chain reads the forest
            const GlobalForest<1> g(J);
            for (uint32_t i = threadIdx.x; i < nr; i += blockDim.x) {
                st_wg(g.parent + i, lds.runs.par[i]);
                st_wg(g.areas + i, lds.runs.area[i]);
            }
        }
        resolve_zone(J, f, c, inv, defer, was, s_cover);
    } else {
        const GlobalForest<A> f(J);
        const Components c = resolve_global<A>(J, lds.areas, nr, nl, nflag);
        resolve_zone(J, f, c, inv, defer, was, s_cover);
    }
    __syncthreads();
}

template <int NT>
__global__ __launch_bounds__(NT) void k_resolve(Table *__restrict__ T, int defer)
{
    __shared__ ResolveLds<kForestRuns> s_lds;
    const int nj = T->h.njobs;
    for (int j = blockIdx.x; j < nj; j += gridDim.x)
        resolve_job<kForestRuns, 4>(T, j, false, s_lds, defer != 0);
}

// Tracking of consecutive frames of one stream after a deferred component
// stage (one workgroup; every job of the table belongs to the stream and
// holds the largest component's pointer and root). Frame j's pick depends on
// frame j - 1's centroid, so it is settled in order, but nearly all of the
// work is done for all frames at once, on the guess that every earlier frame
// kept its largest component:
//   1. thread j stages frame j's pointer and largest root in LDS and tests
//      whether frame j - 1's guessed centroid pixel lies in a component of
//      frame j (the covering test: a few dependent loads);
//   2. thread 0 walks the frames in order over LDS alone: a frame whose
//      predecessor's actual centroid is the guess takes the test's answer
//      (otherwise thread 0 tests again), and when its pick is its largest
//      component its pointer only needs the debounced click. A frame that
//      needs the whole workgroup - the nearest-component pass (nothing covers
//      the centroid), or new sums, box and hand bits (the pick is not the
//      largest) - stops the walk; the workgroup does that frame, and the
//      walk goes on after it;
//   3. thread j writes frame j's pointer; thread 0 the stream's state.
// Bound by its chain of dependent loads (pointer, mask words, run number, root
// with its area): the strides come by value, so that no load waits for a job's
// field, the words a covering run may start in are loaded at once, and the walk
// reads eight frames' flags at a time. 16 frames of 1280x720: 10.9 -> 6.2 us, and
// a tracked call of 100 such frames, in chunks of 16, 417 -> 394 us.
constexpr int kChainMax = kMaxJobs;

__global__ __launch_bounds__(kResolveThreads) void k_track_chain(Table *__restrict__ T, const ChainSpan C)
{
    __shared__ fizi_pointer s_ptr[kChainMax];
    __shared__ uint32_t s_cover[kChainMax], s_largest[kChainMax];
    // guessed previous centroid of frame j, -1: no hand (j = nj: of the next call)
    __shared__ int32_t s_gx[kChainMax + 1], s_gy[kChainMax + 1];
    // what the walk needs of a frame on the guess: present, click, stop
    __shared__ alignas(8) uint8_t s_flag[(kChainMax + 7) / 8 * 8];
    __shared__ int32_t s_ax, s_ay;                          // actual previous centroid, -1: no hand
    __shared__ int s_next;                                  // frame the workgroup works on, or nj
    __shared__ uint32_t s_pick;
    __shared__ int s_zone;                                  // the frame needs its zone's sums recomputed
    __shared__ uint32_t s_state;                            // debouncer state
    constexpr uint32_t kPresent = 1, kClick = 2, kStop = 4;
    const int nj = C.n;
    // one stream: its thresholds are the same in every job
    const uint32_t amin = C.amin, r2 = C.r2;
    const int debounce = C.debounce;
    const TrackState was = *C.track;
    for (int j = threadIdx.x; j < nj; j += blockDim.x) {
        s_ptr[j] = C.out[j];
        s_largest[j] = G(&T->jobs[j].pick)[0];
    }
    __syncthreads();
    // the component of area >= amin of frame j that covers (x, y), or none
    auto cover = [&](int j, int x, int y) -> uint32_t {
        if (x < 0 || x >= C.W || y < 0 || y >= C.H)
            return kNoRoot;
        const GLOBAL uint64_t *row = G(C.fizi) + (size_t)j * C.fizi_words + (size_t)y * (C.W / 64);
        const GLOBAL uint8_t *slot = G(reinterpret_cast<const uint8_t *>(C.index)) + (size_t)j * C.slot_bytes;
        uint32_t r = run_at(row, reinterpret_cast<const GLOBAL uint32_t *>(slot) + (uint32_t)y * (uint32_t)C.W, x);
        if (r == kNoRoot)
            return kNoRoot;
        const GLOBAL uint32_t *parent = reinterpret_cast<const GLOBAL uint32_t *>(
            G(reinterpret_cast<const uint8_t *>(C.parent)) + (size_t)j * C.slot_bytes);
        // a run's parent mostly is its root: its area is loaded beside the test
        for (;;) {
            const uint32_t p = parent[r], area = parent[C.run_cap + r];
            if (p == r)
                return area >= amin ? r : kNoRoot;
            r = p;
        }
    };
    // whether the walk stops at a frame for the workgroup: the
    // nearest-component pass, or a pick that is not the largest
    auto stops = [&](int j, int gx, uint32_t c) {
        return c == kNoRoot ? gx >= 0 && r2 > 0 : c != s_largest[j];
    };
    // 1: the covering tests on the guess
    for (int j = threadIdx.x; j <= nj; j += blockDim.x) {
        int gx = -1, gy = -1;
        if (j == 0) {
            if (was.valid) {
                gx = was.x;
                gy = was.y;
            }
        } else if (s_ptr[j - 1].present) {
            gx = (int32_t)(s_ptr[j - 1].sum_x / s_ptr[j - 1].area);
            gy = (int32_t)(s_ptr[j - 1].sum_y / s_ptr[j - 1].area);
        }
        s_gx[j] = gx;
        s_gy[j] = gy;
        if (j < nj) {
            const uint32_t c = cover(j, gx, gy);
            s_cover[j] = c;
            s_flag[j] = (uint8_t)((s_ptr[j].present ? kPresent : 0u) | (s_ptr[j].click ? kClick : 0u) |
                                  (stops(j, gx, c) ? kStop : 0u));
        }
    }
    if (threadIdx.x == 0) {
        s_ax = was.valid ? was.x : -1;
        s_ay = was.valid ? was.y : -1;
        s_state = was.click;
    }
    __syncthreads();
    // 2: the frames in order
    int j0 = 0;
    for (;;) {
        if (threadIdx.x == 0) {
            const int ax = s_ax, ay = s_ay;
            uint32_t state = s_state, c = kNoRoot;
            int j = j0;
            bool stop = false;
            // the largest component keeps the hand: only the click changes,
            // and the centroid is the one guessed
            auto keep = [&](uint32_t fl) {
                s_ptr[j].click = debounce_click(&state, fl & kPresent, (fl & kClick) ? 1 : 0, debounce);
                ++j;
            };
            if (j < nj && (ax != s_gx[j] || ay != s_gy[j])) {
                c = cover(j, ax, ay);
                stop = stops(j, ax, c);
                if (!stop)
                    keep(s_flag[j]);
            }
            // eight frames' flags at a time
            while (!stop && j < nj) {
                uint64_t fl;
                __builtin_memcpy(&fl, __builtin_assume_aligned(s_flag + (j & ~7), 8), 8);
                fl >>= 8 * (j & 7);
                const int end = min((j & ~7) + 8, nj);
                for (; j < end; fl >>= 8) {
                    if (fl & kStop) {
                        stop = true;
                        c = s_cover[j];
                        break;
                    }
                    keep((uint32_t)fl);
                }
            }
            if (j > j0) {
                s_ax = s_gx[j];
                s_ay = s_gy[j];
            }
            s_pick = c;
            s_zone = c != kNoRoot;
            s_state = state;
            s_next = j;
        }
        __syncthreads();
        const int j = s_next;
        if (j >= nj)
            break;
        Job *J = &T->jobs[j];
        const GlobalForest<4> f(J);
        uint32_t pick = s_pick;
        if (!s_zone)
            pick = nearest_root(J, f, s_ax, s_ay, amin, r2);
        if (pick != kNoRoot && pick != s_largest[j]) {
            // the tracked zone is not the largest: its own sums, box, hand bits
            GLOBAL uint64_t *hand = J->hand ? G(J->hand) : nullptr;
            if (hand) {
                for (int i = threadIdx.x; i < J->H * J->Wd; i += blockDim.x)
                    hand[i] = 0ull;
                __syncthreads();
            }
            const uint32_t A = f.area(pick);
            const ZoneStats z = zone_stats(J, f, pick, hand);
            if (threadIdx.x == 0)
                s_ptr[j] = make_pointer(J, true, A, z, s_ptr[j].n_components, s_ptr[j].inv_gain_q16);
        }
        if (threadIdx.x == 0) {
            fizi_pointer &o = s_ptr[j];
            o.click = debounce_click(&s_state, o.present != 0, o.click, debounce);
            s_ax = o.present ? (int32_t)(o.sum_x / o.area) : -1;
            s_ay = o.present ? (int32_t)(o.sum_y / o.area) : -1;
        }
        j0 = j + 1;
        __syncthreads();
    }
    // 3: the pointers and the stream's state
    for (int j = threadIdx.x; j < nj; j += blockDim.x) {
        C.out[j] = s_ptr[j];
        if (C.ring)
            C.ring[(uint32_t)(C.frame_index + (uint64_t)j) & C.ring_mask] = s_ptr[j];
    }
    if (threadIdx.x == 0) {
        GLOBAL TrackState *ts = G(C.track);
        ts->click = s_state;
        ts->valid = s_ax >= 0 ? 1 : 0;
        if (s_ax >= 0) {
            ts->x = s_ax;
            ts->y = s_ay;
        }
    }
}

// ---------------------------------------------------------------------------
// Persistent step: one launch per frame step whose workgroups take work items
// from the ordered queue of the job table (TableHeader) with one atomic
// counter. A gain item is one gain tile. A band item classifies 4 * band
// rows of a frame (once the frame's gain is complete), publishes them, then
// runs the morphology of the band above - its four waves take one sub-band
// each - once the bands it reads are published, and of its own band when it
// is the frame's last; the workgroup that completes a frame's last
// morphology band then resolves its components. Latency-bound morphology and
// components thus run while other workgroups stream later bands. Items only
// wait for items earlier in the queue, which are held by running workgroups
// that never wait for later ones, so every wait ends. Each wait is bounded
// (50 ms of the 100 MHz clock); one that gives up sets the error word and
// goes on, so that every workgroup reaches the end; the last one out resets
// the queue for the next launch.
constexpr uint64_t kWaitTicks = 5000000;

// Thread 0 waits until the counter reaches target, or the flag equals it.
__device__ __forceinline__ void spin_until(const uint32_t *p, uint32_t target, bool equal, PersistState *ps,
                                           uint64_t t0)
{
    for (;;) {
        const uint32_t v = ld_dev(p);
        if (equal ? v == target : v >= target)
            return;
        if (__builtin_amdgcn_s_memrealtime() - t0 > kWaitTicks) {
            atomicOr(&ps->error, 1u);
            return;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// After thread 0's waits: a device-scope acquire, then the workgroup goes on.
__device__ __forceinline__ void acquire_for_block()
{
    if (threadIdx.x == 0)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
}

// Every wave's stores complete, then thread 0 adds v to the counter; returns
// the counter's previous value to the whole workgroup.
__device__ __forceinline__ uint32_t publish_add(uint32_t *p, uint32_t v, uint32_t *s_old)
{
    wait_own_memory();
    __syncthreads();
    if (threadIdx.x == 0)
        *s_old = atomicAdd(p, v);
    __syncthreads();
    return *s_old;
}

template <int KMAX, int NC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KMAX == 4 && NC == 1 ? 4 : 1))) void k_flow(Table *__restrict__ T, PersistState *ps)
{
    __shared__ WaveLds s_wl[256 / kWave];
    __shared__ int s_item;
    __shared__ uint32_t s_u;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int nseg = T->h.flow_nseg;
    const int total = T->h.flow_pre[nseg];
    int k = 0;
    for (;;) {
        if (threadIdx.x == 0)
            s_item = (int)atomicAdd(&ps->next, 1u);
        __syncthreads();
        const int item = s_item;
        __syncthreads();
        if (item >= total)
            break;
        while (T->h.flow_pre[k + 1] <= item)
            ++k;
        const int seg = T->h.flow_seg[k], j = seg >> 1, idx = item - T->h.flow_pre[k];
        Job *J = &T->jobs[j];
        if ((seg & 1) == 0) {
            gain_tile(T, j, idx, J->frame);
            const uint32_t ng = (uint32_t)(T->h.gain_pre[j + 1] - T->h.gain_pre[j]);
            if (publish_add(&J->gain_done, 1u, &s_u) + 1u == ng && threadIdx.x == 0) {
                // the frame's last gain tile: its inverse gain, once, for every band
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                st_dev(G(&J->ginv), kGainKnown | job_gain(J));
            }
            continue;
        }
        const int rb = 4 * J->band, H = J->H, W = J->W;
        const int nb = (H + rb - 1) / rb, nsub = (H + J->band - 1) / J->band;
        // classify the band once the frame's inverse gain is known
        if (threadIdx.x == 0) {
            spin_until(&J->ginv, 0x80000000u, false, ps, __builtin_amdgcn_s_memrealtime());
            s_u = ld_dev(&J->ginv) & 0x7FFFFFFFu;
        }
        __syncthreads();
        const uint32_t inv = s_u;
        const uint32_t p0 = (uint32_t)(idx * rb) * (uint32_t)W;
        const uint32_t p1 = (uint32_t)min(H, (idx + 1) * rb) * (uint32_t)W;
        classify_span<true>(cls_job(J), p0, p1, inv);
        wait_own_memory();
        __syncthreads();
        if (threadIdx.x == 0)
            st_dev(G(J->bflag + idx), J->epoch);
        // the morphology of the band above, and of this band when it is the last
        for (int m = max(0, idx - 1); m <= idx; ++m) {
            if (m == idx && idx != nb - 1)
                break;
            if (threadIdx.x == 0) {
                // its rows and halo lie in bands m - 1 .. m + 1
                const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
                for (int bb = max(0, m - 1); bb <= min(nb - 1, m + 1); ++bb)
                    if (bb != idx)
                        spin_until(J->bflag + bb, J->epoch, true, ps, t0);
            }
            acquire_for_block();
            const int sub = 4 * m + wave;
            if (sub < nsub)
                morph_band<KMAX, NC, true>(J, sub, s_wl[wave]);
            const uint32_t cnt = (uint32_t)min(4, nsub - 4 * m);
            if (publish_add(&J->morph_done, cnt, &s_u) + cnt == (uint32_t)nsub) {
                // the frame's last band: its components
                acquire_for_block();
                // the waves' morphology tables are free again: the components
                // take their place
                resolve_job<kForestRunsFlow, 1>(T, j, true, *reinterpret_cast<ResolveLds<kForestRunsFlow> *>(&s_wl[0]));
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned done = atomicAdd(&ps->finished, 1u);
        if (done == gridDim.x - 1) {
            __hip_atomic_store(&ps->next, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&ps->finished, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, size_t n)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

}  // namespace

// ---------------------------------------------------------------------------
hipError_t launch_gain(const Table *d_tab, int total_tiles, int n_cu, const Tuning &t, hipStream_t s,
                       StageEvents ev)
{
    if (total_tiles <= 0)
        return hipSuccess;
    const int grid = min(total_tiles, n_cu * t.grid_per_cu);
    FIZI_LAUNCH(k_gain, grid, 256, 0, s, ev, const_cast<Table *>(d_tab));
    return hipGetLastError();
}

namespace {

template <int MODE>
hipError_t launch_gain_span_mode(Table *tab, const SpanJobs &S, hipStream_t s, StageEvents ev)
{
    const bool wide = reinterpret_cast<uintptr_t>(S.frame) % 16 == 0;
    const long long items = (long long)((S.H + S.rs - 1) / S.rs) * (S.W / (wide ? 16 : 4));
    const GainShape g = gain_span_shape(items, S.n);
    const int threads = g.threads;
    const dim3 grid((unsigned)g.parts, (unsigned)S.n + (S.table ? 1u : 0u));
    if (S.make_yref) {
        if (wide)
            FIZI_LAUNCH((k_gain_span<MODE, true, true>), grid, threads, 0, s, ev, tab, S);
        else
            FIZI_LAUNCH((k_gain_span<MODE, true, false>), grid, threads, 0, s, ev, tab, S);
    } else {
        if (wide)
            FIZI_LAUNCH((k_gain_span<MODE, false, true>), grid, threads, 0, s, ev, tab, S);
        else
            FIZI_LAUNCH((k_gain_span<MODE, false, false>), grid, threads, 0, s, ev, tab, S);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gain_span(Table *d_tab, const SpanJobs &S, hipStream_t s, StageEvents ev)
{
    switch (S.hue.mode) {
    case 0: return launch_gain_span_mode<0>(d_tab, S, s, ev);
    case 1: return launch_gain_span_mode<1>(d_tab, S, s, ev);
    case 2: return launch_gain_span_mode<2>(d_tab, S, s, ev);
    default: return launch_gain_span_mode<3>(d_tab, S, s, ev);
    }
}

hipError_t launch_minmax(const Table *d_tab, const LearnSpan &S, hipStream_t s, StageEvents ev)
{
    const int grid = (int)((S.npx / 4u + 255u) / 256u);
    const auto kernel = S.masks ? (S.n > 2 ? k_minmax<true, 4> : S.n == 2 ? k_minmax<true, 2> : k_minmax<true, 1>)
                                : (S.n > 2 ? k_minmax<false, 4> : S.n == 2 ? k_minmax<false, 2> : k_minmax<false, 1>);
    FIZI_LAUNCH(kernel, grid, 256, 0, s, ev, d_tab, S);
    return hipGetLastError();
}

hipError_t launch_classify(const Table *d_tab, int total_tiles, int n_cu, const Tuning &t, hipStream_t s,
                           StageEvents ev)
{
    if (total_tiles <= 0)
        return hipSuccess;
    const int grid = min(total_tiles, n_cu * t.grid_per_cu);
    Table *tab = const_cast<Table *>(d_tab);
    switch (t.cls_iters) {
    case 1: FIZI_LAUNCH(k_classify<1>, grid, 256, 0, s, ev, tab); break;
    case 2: FIZI_LAUNCH(k_classify<2>, grid, 256, 0, s, ev, tab); break;
    case 8: FIZI_LAUNCH(k_classify<8>, grid, 256, 0, s, ev, tab); break;
    default: FIZI_LAUNCH(k_classify<4>, grid, 256, 0, s, ev, tab); break;
    }
    return hipGetLastError();
}

// Frames of one span workgroup: 16, so that a pixel's box is unpacked once
// for 16 frames, unless that leaves fewer workgroups than about one resident
// round (seven 256-thread workgroups per CU): then 8, or 4. With 4 / 8 / 16 /
// 32 frames 64 of 1920x1080 take 87 / 78 / 75 / 74 us (a longer list of inverse
// gains for the last 1%), 16 of 1280x720 (900 tiles) 13.8 / 12.2 / 12.9.
hipError_t launch_classify_span(const Table *d_tab, const SpanJobs &S, const Job &J, int n_cu, hipStream_t s,
                                StageEvents ev)
{
    FrameSpan F{};
    F.frames = S.frame;
    F.frame_stride = S.frame_bytes;
    F.raw = S.raw;
    F.raw_words = S.raw_bytes / sizeof(uint64_t);
    F.bgmin = J.bgmin;
    F.bgmax = J.bgmax;
    F.npx = (uint32_t)J.W * (uint32_t)J.H;
    F.n = S.n;
    F.delta = J.delta;
    F.S1 = J.S1;
    F.S0 = J.S0;
    F.scaled = J.scaled;
    F.lum2 = J.lum2;
    F.S_q16 = J.S_q16;
    F.hue = hue_form(J.hue);
    if (F.n <= 0)
        return hipSuccess;
    const int tiles = (int)((F.npx + 1023u) / 1024u);
    int per = kSpanFrames;
    while (per > 4 && (long long)tiles * ((F.n + per - 1) / per) < 7ll * n_cu)
        per /= 2;
    per = std::min(per, F.n);
    const dim3 grid((unsigned)tiles, (unsigned)((F.n + per - 1) / per));
    if (F.n == 1) {
        if (F.scaled)
            FIZI_LAUNCH(k_classify_one<kScaled>, tiles, 256, 0, s, ev, d_tab, F, J.hue);
        else if (F.lum2)
            FIZI_LAUNCH(k_classify_one<kCorrectedLum>, tiles, 256, 0, s, ev, d_tab, F, J.hue);
        else
            FIZI_LAUNCH(k_classify_one<kCorrected>, tiles, 256, 0, s, ev, d_tab, F, J.hue);
        return hipGetLastError();
    }
    if (F.scaled)
        FIZI_LAUNCH(k_classify_span<kScaled>, grid, 256, 0, s, ev, d_tab, F, per);
    else if (F.lum2)
        FIZI_LAUNCH(k_classify_span<kCorrectedLum>, grid, 256, 0, s, ev, d_tab, F, per);
    else
        FIZI_LAUNCH(k_classify_span<kCorrected>, grid, 256, 0, s, ev, d_tab, F, per);
    return hipGetLastError();
}

hipError_t launch_morph(const Table *d_tab, int total_tiles, int items, int max_wd, int max_ops, int n_cu,
                        const Tuning &t, hipStream_t s, StageEvents ev)
{
    if (total_tiles <= 0)
        return hipSuccess;
    const int waves = 256 / kWave;
    const int grid = min((total_tiles + waves - 1) / waves, n_cu * t.grid_per_cu);
    Table *tab = const_cast<Table *>(d_tab);
    const bool wide = max_wd > kWave, deep = max_ops > 4;
    const bool regs = t.morph_rows == 8 || t.morph_rows == 16;
    if (regs && wide && deep && !items) {
        if (t.morph_rows == 16)
            FIZI_LAUNCH(k_morph_mixed<16>, grid, 256, 0, s, ev, tab);
        else
            FIZI_LAUNCH(k_morph_mixed<8>, grid, 256, 0, s, ev, tab);
        return hipGetLastError();
    }
    if (regs && !(wide && deep)) {
        if (t.morph_rows == 16) {
            if (wide)
                FIZI_LAUNCH((k_morph_regs<16, 4, 2>), grid, 256, 0, s, ev, tab, total_tiles, items);
            else if (!deep)
                FIZI_LAUNCH((k_morph_regs<16, 4, 1>), grid, 256, 0, s, ev, tab, total_tiles, items);
            else if (max_ops <= 8)
                FIZI_LAUNCH((k_morph_regs<16, 8, 1>), grid, 256, 0, s, ev, tab, total_tiles, items);
            else
                FIZI_LAUNCH((k_morph_regs<16, 12, 1>), grid, 256, 0, s, ev, tab, total_tiles, items);
        } else if (wide) {
            FIZI_LAUNCH((k_morph_regs<8, 4, 2>), grid, 256, 0, s, ev, tab, total_tiles, items);
        } else if (!deep) {
            FIZI_LAUNCH((k_morph_regs<8, 4, 1>), grid, 256, 0, s, ev, tab, total_tiles, items);
        } else if (max_ops <= 8) {
            FIZI_LAUNCH((k_morph_regs<8, 8, 1>), grid, 256, 0, s, ev, tab, total_tiles, items);
        } else {
            FIZI_LAUNCH((k_morph_regs<8, 12, 1>), grid, 256, 0, s, ev, tab, total_tiles, items);
        }
        return hipGetLastError();
    }
    if (!wide && !deep)
        FIZI_LAUNCH((k_morph<4, 1>), grid, 256, 0, s, ev, tab);
    else if (!wide)
        FIZI_LAUNCH((k_morph<4 * kMaxMorphIters, 1>), grid, 256, 0, s, ev, tab);
    else if (!deep)
        FIZI_LAUNCH((k_morph<4, 2>), grid, 256, 0, s, ev, tab);
    else
        FIZI_LAUNCH((k_morph<4 * kMaxMorphIters, 2>), grid, 256, 0, s, ev, tab);
    return hipGetLastError();
}

hipError_t launch_resolve(const Table *d_tab, int njobs, hipStream_t s, StageEvents ev, const ChainSpan *chain,
                          bool small)
{
    if (njobs <= 0)
        return hipSuccess;
    // consecutive tracked frames of one stream: every frame's forest and
    // largest component at once, then the tracking chain in frame order
    Table *tab = const_cast<Table *>(d_tab);
    const int defer = chain ? 1 : 0;
    if (small)
        FIZI_LAUNCH(k_resolve<kResolveThreadsSmall>, njobs, kResolveThreadsSmall, 0, s, ev, tab, defer);
    else
        FIZI_LAUNCH(k_resolve<kResolveThreads>, njobs, kResolveThreads, 0, s, ev, tab, defer);
    if (chain) {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        k_track_chain<<<1, kResolveThreads, 0, s>>>(tab, *chain);
    }
    return hipGetLastError();
}

// Blocks per CU of the persistent step: what the kernel's registers and LDS
// allow (wave64, 512 VGPRs per SIMD lane in granules of 8, four SIMDs and
// 160 KiB of LDS per CU, eight waves per SIMD: four for the smallest form's 128
// VGPRs and 34 KiB), so that the whole grid is resident; at most eight.
template <int KMAX, int NC>
int flow_blocks_per_cu()
{
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_flow<KMAX, NC>, 256, 0) != hipSuccess)
        nb = 1;
    return std::max(1, std::min(nb, 8));
}

template <int KMAX, int NC>
hipError_t launch_flow_t(Table *tab, int n_cu, PersistState *ps, hipStream_t s, StageEvents ev)
{
    static int per_cu = -1;
    if (per_cu < 0)
        per_cu = flow_blocks_per_cu<KMAX, NC>();
    FIZI_LAUNCH((k_flow<KMAX, NC>), per_cu * n_cu, 256, 0, s, ev, tab, ps);
    return hipGetLastError();
}

hipError_t launch_persistent(const Table *d_tab, int max_wd, int max_ops, int n_cu, const Tuning &t,
                             uint8_t *persist, hipStream_t s, StageEvents ev)
{
    (void)t;
    Table *tab = const_cast<Table *>(d_tab);
    PersistState *ps = reinterpret_cast<PersistState *>(persist);
    const bool wide = max_wd > kWave, deep = max_ops > 4;
    if (!wide && !deep)
        return launch_flow_t<4, 1>(tab, n_cu, ps, s, ev);
    if (!wide)
        return launch_flow_t<4 * kMaxMorphIters, 1>(tab, n_cu, ps, s, ev);
    if (!deep)
        return launch_flow_t<4, 2>(tab, n_cu, ps, s, ev);
    return launch_flow_t<4 * kMaxMorphIters, 2>(tab, n_cu, ps, s, ev);
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t s)
{
    if (n == 0)
        return hipSuccess;
    const size_t grid = std::min<size_t>((n + 255) / 256, 65535);
    k_fill_u32<<<(unsigned)grid, 256, 0, s>>>(p, v, n);
    return hipGetLastError();
}

}  // namespace fizi
