// Internal layout shared by the HIP kernels and the C-ABI host code.
//
// Work is described by a job table in device memory: one Job per frame to
// process (a frame of a context's stream, or a learning frame), with the
// pointers to its inputs, outputs and scratch, its geometry and thresholds,
// and a few accumulators the kernels update atomically. The host fills the
// table in pinned memory and copies it to the device ahead of the kernels,
// which also zeroes the accumulators for that call (batch steps), or the gain
// kernel writes it on the device (consecutive frames of one stream). Every kernel walks a flat
// list of tiles (grid-stride) and finds a tile's job by binary search in a
// prefix array, so one launch covers frames of any mix of resolutions and a
// launch's shape does not depend on the work it is given. The persistent
// step instead takes work items from an ordered queue (see TableHeader).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fizi.h"
#include "fizi_shapes.h"

namespace fizi {

constexpr int kMaxJobs = 256;          // jobs per table
constexpr uint16_t kYrefClipped = 0xFFFFu;
constexpr int kMaxMorphIters = 3;      // open_iters, close_iters <= 3
constexpr int kGainSlots = 32;         // gain sums are spread over 32 accumulators
constexpr int kGainRows = 4;           // sampled rows per gain tile
constexpr int kShortBand = 4;          // morphology band height of launches too small to fill the device

// Skin-hue test on one RGB triple, without division (Section 3.1 (iii)).
// For a hue a, let d_a be an RGB colour of hue a. The determinant
// D(a, p) = det[(1,1,1), d_a, p] = kr (R - B) + kg (G - B) is positive exactly
// when the hue of p lies in the open half-turn (a, a + 180) and zero when it
// is a or a + 180, because the hexcone hue is a monotone, odd-symmetric
// re-parametrisation of the angle around the gray axis. The closed interval
// [a1, a2] of length L is then
//   L = 0:        D1 == 0 and p points along d_a1 (3 d.p - sum(d) sum(p) > 0)
//   0 < L < 180:  D1 >= 0 and D2 <= 0
//   L = 180:      D1 >= 0
//   L > 180:      D1 >= 0 or D2 <= 0
// always together with chroma > 0.
struct HueTest {
    int32_t k1r, k1g;          // D(a1, p) coefficients
    int32_t k2r, k2g;          // D(a2, p) coefficients
    int32_t dr, dg, db, dsum;  // d_a1 (scaled by 6000) for the one-point case
    int32_t mode;              // 0: L = 0, 1: 0 < L < 180, 2: L = 180, 3: L > 180
    int32_t pad;
};

// The same test without a case distinction: hue in [a1, a2] exactly when
// (D1' >= 0 and D2' <= 0 and D3' > 0) differs from flip, each D' a form
// k (R - B) + k (G - B) + c. 0 < L < 180: D1, D2, and D3' = 1. L = 180: D2' = 0.
// L > 180, the complement of D1 < 0 and D2 > 0: D1' = -D1 - 1, D2' = 1 - D2,
// flipped. L = 0: D1' = D2' = D1 and D3' = 3 d.p - sum(d) sum(p), which does
// not change when a gray is added to p and so is such a form too. |k| <= 18000.
struct HueForm {
    int32_t k1r, k1g, c1, k2r, k2g, c2, k3r, k3g, c3, flip;
};

// Temporal tracking state of one stream (device memory): the previous
// frame's centroid pixel, valid when that frame had a hand, and the click
// debouncer (bit 0: the reported click; bits 8..15: consecutive frames whose
// own click differs from it).
struct TrackState {
    int32_t valid, x, y;
    uint32_t click;
};

struct Job {
    const uint8_t *frame;      // H*W*3
    const uint8_t *bgmin;      // H*W*3
    const uint8_t *bgmax;      // H*W*3
    const uint16_t *yref;      // ceil(H/rs) * W
    uint64_t *raw;             // H*Wd words: AND of the three masks
    uint64_t *fizi;            // H*Wd words: after opening and closing
    uint64_t *hand;            // H*Wd words or null
    uint32_t *parent;          // W*H: union-find parents by run (run_cap), then component areas by root run
    uint32_t *bflag;           // per row band of the persistent step: epoch when classified
    uint32_t *index;           // W*H: run of a run's first pixel (valid there)
    uint2 *runs;               // run_cap runs (first pixel, last pixel | link flag)
    uint2 *links;              // link_cap pairs of run starts to join
    fizi_pointer *out;         // one pointer
    fizi_pointer *hout;        // its slot in a host ring (pinned, device-mapped), or null
    TrackState *track;         // the stream's tracking state, or null (largest component)
    uint64_t frame_index;
    int32_t W, H, Wd, rs;
    uint32_t run_cap, link_cap;
    uint32_t epoch;            // this dispatch's number for its scratch slot (never 0)
    int32_t band;              // morphology band height (rows)
    int32_t mgroup;            // morphology lanes per row: 64, or 16 / 32 to pack 4 / 2 bands per wave
    int32_t delta, S1, open_it, close_it, min_area, fill_pm, glo, ghi;
    int32_t scaled;            // thresholds scaled by the gain instead of corrected pixels
    uint32_t S_q16;            // max(S * 2^16, 1): the gray tolerance against (max - min) * inv
    int32_t debounce;          // tracked streams: frames a change of the click needs
    uint32_t track_r2;         // tracked streams: squared radius of the nearest-component pick
    int32_t S0;                // gray tolerance S as given
    int32_t lum2;              // over-exposure filter: 2 lum_hi, 0 when off
    HueTest hue;
    // accumulators (zero when the table is uploaded)
    // gain sums over usable sampled pixels (tables uploaded by a batch):
    // tile t adds to slot t % kGainSlots (fewer same-address atomics); 32 bits
    // hold a slot's share of the largest frame, 2^21 pixels of at most 1020
    // (64 tiles of 2^15). Spans sum in 64 bits elsewhere (SpanJobs).
    alignas(8) uint32_t num[kGainSlots];
    uint32_t den[kGainSlots];
    uint32_t nruns, nlinks;           // reserved together by one 64-bit add where both are known
    uint32_t flags, nflag;
    uint32_t gain_done, morph_done;   // persistent step: finished gain tiles, morphology bands
    uint32_t ginv;                    // persistent step and spans: 0x80000000 | inverse gain, once known
    uint32_t pick;                    // deferred tracking: root run of the largest component (or none)
};

// The persistent step's queue: segments of work items, in order
//   gain(o0), ..., gain(o[n-1]), bands(o0), ..., bands(o[n-1])
// over the jobs o sorted by size, largest first. A gain item is one gain
// tile; a band item is 4 * band rows: classify them, then run the
// morphology of the band above (and, for the last band, of this one) and,
// when a frame's last band is done, its components. An item only ever waits
// for items earlier in the queue.
struct TableHeader {
    int32_t njobs;
    int32_t flow_nseg;                    // 2 * njobs
    int32_t gain_pre[kMaxJobs + 1];   // gain tiles (kGainRows sampled rows)
    int32_t cls_pre[kMaxJobs + 1];    // classify tiles
    int32_t mor_pre[kMaxJobs + 1];    // morphology items (64 / mgroup bands each)
    int32_t flow_pre[2 * kMaxJobs + 1];   // first item of each queue segment
    int32_t flow_seg[2 * kMaxJobs];       // (job << 1) | (0: gain, 1: bands)
};

struct Table {
    TableHeader h;
    Job jobs[kMaxJobs];
};

static_assert(sizeof(TableHeader) % 8 == 0, "job array alignment");

// What classify needs of consecutive frames of one stream (a context's
// launch): one model, one geometry, one set of thresholds, frames and raw
// masks at fixed strides. Passed by value.
struct FrameSpan {
    const uint8_t *frames;     // frame i at frames + i * frame_stride
    size_t frame_stride;
    uint64_t *raw;             // raw mask of frame i at raw + i * raw_words
    size_t raw_words;
    const uint8_t *bgmin, *bgmax;
    uint32_t npx;
    int32_t n;
    int32_t delta, S1, S0, scaled, lum2;
    uint32_t S_q16;
    HueForm hue;
};
HueForm hue_form(const HueTest &h);

// The most runs a mask can have.
__host__ __device__ inline uint32_t run_capacity(int32_t W, int32_t H) { return (uint32_t)W * (uint32_t)H / 2u; }
// Joins across band and segment borders that are kept; beyond this many, runs
// are flagged for the component stage instead.
__host__ __device__ inline uint32_t link_capacity(int32_t W, int32_t H) { return (uint32_t)W * (uint32_t)H / 8u; }

// Launch shapes (tunable per resolution class).
struct Tuning {
    int cls_iters;      // classify tile = 1024 * cls_iters pixels (1, 2, 4, 8)
    int morph_rows;     // morphology band height (8, 16, 32, 64)
    int grid_per_cu;    // resident blocks per CU for the streaming kernels
    int short_bands = 1;   // launches too small to fill the device take short morphology bands
};

// Whether the morphology of a launch (tuned band height, widest frame in
// words, most stages of a job) holds a job's bands (ops stages) in registers
// with their halo: bands of 8 or 16 rows, and of the short height in such a
// launch, but in launches of frames of more than 64 words and of more than four
// stages only jobs of at most four. The others stream their bands. Only bands
// in registers share a wave on narrow frames.
inline bool morph_in_regs(int morph_rows, int max_wd, int max_ops, int ops)
{
    const bool wide = max_wd > 64, deep = max_ops > 4;
    return (morph_rows == 8 || morph_rows == 16) && !(wide && deep && ops > 4);
}

inline int cls_tile_px(const Tuning &t) { return 1024 * t.cls_iters; }

// Counters of the persistent step (device memory, zero between launches).
struct PersistState {
    unsigned int next;       // next queue item of the current launch
    unsigned int finished;   // blocks done with the current launch
    unsigned int error;      // a bounded wait gave up (sticky until read)
    unsigned int pad[61];
};
inline size_t persist_state_bytes() { return sizeof(PersistState); }

// Optional start/stop events taken from a kernel's own dispatch (measurement).
struct StageEvents {
    hipEvent_t start = nullptr;
    hipEvent_t stop = nullptr;
};

// Launches go through hipExtLaunchKernelGGL so that, when the caller asks for
// it, the start/stop events are taken from the kernel's own dispatch. `ev`
// is evaluated more than once: pass a variable.
#define FIZI_LAUNCH(kern, grid, block, lds, s, ev, ...)                                              \
    do {                                                                                           \
        if ((ev).start || (ev).stop)                                                               \
            hipExtLaunchKernelGGL(kern, dim3(grid), dim3(block), lds, s, (ev).start, (ev).stop, 0, \
                                  __VA_ARGS__);                                                    \
        else                                                                                       \
            hipLaunchKernelGGL(kern, dim3(grid), dim3(block), lds, s, __VA_ARGS__);                \
    } while (0)

// Scratch of the gain kernel of spans: per frame an arrival count (a cache
// line each: sharing lines cost 6 us over 64 frames), 0 between launches, then
// the launch's partial sums, reference and frame luminance of part p of frame
// i at pair i parts + p.
constexpr int kArrivedStride = 32;
constexpr size_t kArrivedWords = (size_t)kMaxJobs * kArrivedStride;
constexpr size_t kGainScratchBytes = kArrivedWords * sizeof(uint32_t) + (size_t)kGainParts * 2 * sizeof(GainSum);

// A launch over n consecutive frames of one stream: what the kernels after the
// front read of its first job, and the strides to the next ones. The gain
// kernel writes the job table from it, so that nothing is uploaded, and nothing
// in the state block is taken for an address that the launch itself has not
// written: the block is the caller's, who may fill it from another context's.
// Kernel arguments are kept few: 700 bytes of them cost 8 to 15 us a launch.
struct SpanJobs {
    const uint8_t *frame;
    size_t frame_bytes;
    uint64_t *raw, *fizi, *hand;        // hand null: none
    size_t raw_bytes, fizi_words, hand_words, slot_bytes;
    fizi_pointer *out, *ring;           // ring[k & ring_mask]: the host ring's place of frame index k
    TrackState *track;
    uint32_t *parent, *index;
    uint2 *runs, *links;
    uint64_t frame_index;
    uint16_t *yref;
    uint32_t ring_mask;
    int32_t table;                      // whether to write the table (not when learning)
    int32_t min_area, fill_pm, debounce;
    uint32_t track_r2;
    int16_t open_it, close_it;
    int32_t n, W, H, rs;
    int32_t band, mgroup;
    int32_t mor_items;                  // morphology items of one frame
    int32_t glo, ghi;
    uint32_t *arrived;                  // gain scratch, see kArrivedStride
    int32_t make_yref;                  // learning: the reference is frame 0, written to yref
    HueTest hue;
};

// Consecutive frames that widen a model; their inverse gains lie in a table
// (k_gain_span). masks: null, or each frame's pixels to keep out.
struct LearnSpan {
    const uint8_t *frames;
    size_t frame_bytes;
    const uint64_t *masks;
    uint8_t *bgmin, *bgmax;
    uint32_t npx;
    int32_t n, reset;
};

// Consecutive tracked frames of one stream for the tracking chain: frame j's
// outputs and forest follow the first one's by the strides given, so that the
// chain's loads need no job looked up before them.
struct ChainSpan {
    fizi_pointer *out, *ring;           // as SpanJobs
    TrackState *track;
    const uint64_t *fizi;
    size_t fizi_words;
    const uint32_t *parent, *index;     // of the first frame; run_cap parents, then the areas
    size_t slot_bytes;
    uint64_t frame_index;
    uint32_t ring_mask, run_cap, amin, r2;
    int32_t n, W, H, debounce;
};

// Kernel launchers (fizi_kernels.hip). Each returns the hipError_t of its launch.
hipError_t launch_gain(const Table *d_tab, int total_tiles, int n_cu, const Tuning &t,
                       hipStream_t s, StageEvents ev = {});
// Gain of a span's frames; builds its table.
hipError_t launch_gain_span(Table *d_tab, const SpanJobs &S, hipStream_t s, StageEvents ev = {});
hipError_t launch_minmax(const Table *d_tab, const LearnSpan &S, hipStream_t s, StageEvents ev = {});
hipError_t launch_classify(const Table *d_tab, int total_tiles, int n_cu, const Tuning &t,
                           hipStream_t s, StageEvents ev = {});
hipError_t launch_classify_span(const Table *d_tab, const SpanJobs &S, const Job &first, int n_cu, hipStream_t s,
                                StageEvents ev = {});
// items: morphology items of each job when they are all the same (a span), 0
// to look a band's job up in the table.
hipError_t launch_morph(const Table *d_tab, int total_tiles, int items, int max_wd, int max_ops, int n_cu,
                        const Tuning &t, hipStream_t s, StageEvents ev = {});
// chain: null, or the tracked frames of one stream that the jobs are, settled
// in order by a kernel after the component stage; small: 256-thread
// workgroups, for a launch that runs beside a streaming kernel.
hipError_t launch_resolve(const Table *d_tab, int njobs, hipStream_t s, StageEvents ev = {},
                          const ChainSpan *chain = nullptr, bool small = false);
hipError_t launch_persistent(const Table *d_tab, int max_wd, int max_ops, int n_cu, const Tuning &t,
                             uint8_t *persist, hipStream_t s, StageEvents ev = {});
hipError_t launch_fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t s);

}  // namespace fizi
