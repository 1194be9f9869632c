// C ABI of the single-stream context: learn_background, process_frames,
// get_pointer (include/fizi.h).
#include <algorithm>
#include <new>

#include "fizi_host.h"

using namespace fizi;

namespace {

constexpr int kRing = 65536;   // pointers kept for get_pointer (a power of two)
constexpr int kRecs = 64;

// State block: model | job tables | gain scratch | chunk pointers | chunk
// scratch slots | a second raw-mask buffer per slot (consecutive chunks of a
// call alternate between the two, so that a chunk's classify never writes the
// bits the previous chunk's morphology is reading).
struct CtxLayout {
    size_t model, tables, arrived, ptrs, slots, slot_stride, raw2, raw2_stride, total;
};

CtxLayout ctx_layout(const fizi_geom &g, const fizi_params &p, int chunk)
{
    CtxLayout L{};
    size_t off = 0;
    L.model = off;
    off += align256(model_bytes(g, p));
    L.tables = off;
    off += TableRing::device_bytes();
    L.arrived = off;
    off += align256(kGainScratchBytes);
    L.ptrs = off;
    off += align256((size_t)chunk * sizeof(fizi_pointer));
    L.slot_stride = align256(slot_bytes(g));
    L.slots = off;
    off += (size_t)chunk * L.slot_stride;
    L.raw2_stride = align256((size_t)g.height * (g.width / 64) * 8);
    L.raw2 = off;
    off += (size_t)chunk * L.raw2_stride;
    L.total = align256(off);
    return L;
}

}  // namespace

struct fizi_ctx {
    Model m;
    int chunk = 0;
    Tuning tune{};
    uint8_t *d = nullptr;
    CtxLayout L{};
    int device = 0;
    int n_cu = 0;
    // job tables in device memory, written by the gain kernel of each launch
    // and taken in turn: a launch's table is read until its back half is
    // done, which the caller's stream joins before the second launch after it
    int next_tab = 0;
    StageClock clk;
    // the last kRing pointers, indexed by frame: pinned, coherent host memory
    // that the component kernels store each final pointer into (d_ring is
    // its device-side address), so that no copy follows them
    fizi_pointer *h_ring = nullptr;
    fizi_pointer *d_ring = nullptr;
    // frames [f0, f1) are in the host pointer ring once `ev` (recorded after
    // the kernels that store them, default fences: the host reads what they
    // wrote) is done
    struct Rec {
        uint64_t f0, f1;
        hipEvent_t ev;
        bool valid;
    } recs[kRecs] = {};
    int next_rec = 0;
    // order_ev, or the record event of a call whose last launch ran on its
    // own stream, marks the end of the last call on its stream
    hipEvent_t order_ev = nullptr, last_ev = nullptr;
    hipStream_t last_stream = nullptr;
    bool have_last = false;
    uint64_t next_frame = 0;
    // calls of several chunks: the back half of a chunk (morphology,
    // components) on a side stream beside the next chunk's front
    hipStream_t side = nullptr;
    hipEvent_t cls_ev[2] = {};
    // pipelined calls (fizi_set_pipelined): a call leaves its last chunk's
    // back half on the side stream; the next call joins it after its first
    // classify (or fizi_flush does), and chunks keep alternating raw buffers
    // across calls
    bool pipe_calls = false;
    int parity = 0;      // raw buffer of the next chunk
    hipEvent_t pend_join = nullptr;  // end of the back half not yet joined, or null
};

namespace {

// Calls on different streams run one after the other.
int order_after_previous(fizi_ctx *c, hipStream_t s)
{
    if (c->have_last && c->last_stream != s)
        FIZI_HIP(hipStreamWaitEvent(s, c->last_ev, 0));
    return FIZI_OK;
}

// Marks the end of a call on s; done: an event already recorded there, or null.
int mark_last(fizi_ctx *c, hipStream_t s, hipEvent_t done = nullptr)
{
    if (!done) {
        FIZI_HIP(hipEventRecord(c->order_ev, s));
        done = c->order_ev;
    }
    c->last_ev = done;
    c->last_stream = s;
    c->have_last = true;
    return FIZI_OK;
}

// Orders s after the back half a pipelined call left pending.
int join_pending(fizi_ctx *c, hipStream_t s)
{
    if (c->pend_join) {
        FIZI_HIP(hipStreamWaitEvent(s, c->pend_join, 0));
        c->pend_join = nullptr;
    }
    return FIZI_OK;
}

// Joins a pending back half on the stream of the last call and waits for
// all of the context's work.
int drain(fizi_ctx *c)
{
    if (c->pend_join) {
        FIZI_TRY(join_pending(c, c->last_stream));
        FIZI_TRY(mark_last(c, c->last_stream));
    }
    if (c->have_last)
        FIZI_HIP(hipEventSynchronize(c->last_ev));
    return FIZI_OK;
}

// The next table of the ring.
Table *take_table(fizi_ctx *c)
{
    Table *t = reinterpret_cast<Table *>(c->d + c->L.tables + (size_t)c->next_tab * align256(sizeof(Table)));
    c->next_tab = (c->next_tab + 1) % kTabSlots;
    return t;
}

}  // namespace

extern "C" {

int fizi_default_params(fizi_params *out)
{
    if (!out)
        return fail(FIZI_EINVAL, "null output");
    out->alpha1_cdeg = 33000;
    out->alpha2_cdeg = 7500;
    out->gray_S = 20;
    out->bg_delta = 10;
    out->open_iters = 1;
    out->close_iters = 1;
    out->min_area = 1;
    out->click_fill_permille = 700;
    out->gain_row_stride = 8;
    out->gain_lo_q16 = 32768;
    out->gain_hi_q16 = 131072;
    out->brightness_mode = 0;
    out->click_debounce = 0;
    out->track_radius = 64;
    out->lum_hi = 0;
    return FIZI_OK;
}

int fizi_validate(const fizi_geom *geom, const fizi_params *params) { return validate(geom, params); }

size_t fizi_state_bytes(const fizi_geom *geom, const fizi_params *params, int32_t chunk_frames)
{
    if (validate(geom, params) != FIZI_OK || chunk_frames < 1 || chunk_frames > kMaxJobs)
        return 0;
    return ctx_layout(*geom, *params, chunk_frames).total;
}

int fizi_state_layout(const fizi_geom *geom, const fizi_params *params, int32_t chunk_frames,
                      fizi_layout *out)
{
    FIZI_TRY(validate(geom, params));
    if (chunk_frames < 1 || chunk_frames > kMaxJobs || !out)
        return fail(FIZI_EINVAL, "chunk_frames must be in [1, 256] and out non-null");
    const CtxLayout L = ctx_layout(*geom, *params, chunk_frames);
    Model m;
    model_at(m, *geom, *params, nullptr);
    out->bgmin = L.model + (uint64_t)(uintptr_t)m.bgmin;
    out->bgmax = L.model + (uint64_t)(uintptr_t)m.bgmax;
    out->yref = L.model + (uint64_t)(uintptr_t)m.yref;
    out->yref_rows = (uint64_t)m.yref_rows;
    out->total = L.total;
    return FIZI_OK;
}

int fizi_create(const fizi_geom *geom, const fizi_params *params, int32_t chunk_frames,
                void *d_state, size_t state_bytes, void *stream, fizi_ctx **out)
{
    FIZI_TRY(validate(geom, params));
    if (!out || !d_state)
        return fail(FIZI_EINVAL, "null d_state or out");
    if (chunk_frames < 1 || chunk_frames > kMaxJobs)
        return fail(FIZI_EINVAL, "chunk_frames must be in [1, 256]");
    if (reinterpret_cast<uintptr_t>(d_state) % 256 != 0)
        return fail(FIZI_EINVAL, "d_state must be 256-byte aligned");
    const CtxLayout L = ctx_layout(*geom, *params, chunk_frames);
    if (state_bytes < L.total)
        return fail(FIZI_ENOMEM, "state block smaller than fizi_state_bytes()");
    fizi_ctx *c = new (std::nothrow) fizi_ctx();
    if (!c)
        return fail(FIZI_ENOMEM, "host allocation failed");
    c->chunk = chunk_frames;
    c->d = static_cast<uint8_t *>(d_state);
    c->L = L;
    model_at(c->m, *geom, *params, c->d + L.model);
    c->tune = tuning_for(geom->width, morph_ops(*params), false);
    int rc = device_cu_count(&c->device, &c->n_cu);
    if (rc == FIZI_OK) {
        hipError_t e = hipHostMalloc(reinterpret_cast<void **>(&c->h_ring), sizeof(fizi_pointer) * kRing,
                                     hipHostMallocMapped | hipHostMallocCoherent);
        if (e == hipSuccess)
            e = hipHostGetDevicePointer(reinterpret_cast<void **>(&c->d_ring), c->h_ring, 0);
        if (e == hipSuccess)
            e = hipEventCreateWithFlags(&c->order_ev, kDeviceOrderEvent);
        for (int i = 0; i < kRecs && e == hipSuccess; ++i)
            e = hipEventCreateWithFlags(&c->recs[i].ev, hipEventDisableTiming);
        for (int k = 0; k < 2 && e == hipSuccess; ++k)
            e = hipEventCreateWithFlags(&c->cls_ev[k], kDeviceOrderEvent);
        if (e == hipSuccess)
            e = hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking);
        if (e == hipSuccess)
            e = launch_fill_u32(reinterpret_cast<uint32_t *>(c->d + L.arrived), 0u, kArrivedWords,
                                static_cast<hipStream_t>(stream));
        if (e != hipSuccess)
            rc = fail(FIZI_EHIP, std::string("fizi_create: ") + hipGetErrorString(e));
    }
    if (rc == FIZI_OK)
        rc = mark_last(c, static_cast<hipStream_t>(stream));
    if (rc != FIZI_OK) {
        const std::string msg = fizi_last_error();
        fizi_destroy(c);
        return fail(rc, msg);
    }
    *out = c;
    return FIZI_OK;
}

int learn_background(fizi_ctx *c, const uint8_t *d_frames, int32_t n_frames, int32_t reset, void *stream)
{
    if (!c || !d_frames)
        return fail(FIZI_EINVAL, "null context or frames");
    if (reinterpret_cast<uintptr_t>(d_frames) % 4 != 0)
        return fail(FIZI_EINVAL, "frames must be 4-byte aligned");
    if (n_frames < 1)
        return fail(FIZI_EINVAL, "n_frames must be >= 1");
    if (!reset && !c->m.learned)
        return fail(FIZI_ESTATE, "learning without reset needs a learned model");
    hipStream_t s = static_cast<hipStream_t>(stream);
    FIZI_TRY(order_after_previous(c, s));
    FIZI_TRY(join_pending(c, s));
    FIZI_TRY(learn_model(c->m, take_table(c), reinterpret_cast<uint32_t *>(c->d + c->L.arrived), c->tune, d_frames, n_frames, reset, s, &c->clk));
    return mark_last(c, s);
}

int relearn_background(fizi_ctx *c, const uint8_t *d_frames, int32_t n_frames, const uint64_t *d_fizi_bits,
                       void *stream)
{
    if (!c || !d_frames || !d_fizi_bits)
        return fail(FIZI_EINVAL, "null context, frames or masks");
    if (reinterpret_cast<uintptr_t>(d_frames) % 4 != 0 || reinterpret_cast<uintptr_t>(d_fizi_bits) % 8 != 0)
        return fail(FIZI_EINVAL, "frames must be 4-byte and masks 8-byte aligned");
    if (n_frames < 1)
        return fail(FIZI_EINVAL, "n_frames must be >= 1");
    if (!c->m.learned)
        return fail(FIZI_ESTATE, "relearn_background before learn_background");
    hipStream_t s = static_cast<hipStream_t>(stream);
    FIZI_TRY(order_after_previous(c, s));
    // the masks may come from a call whose back half is still pending
    FIZI_TRY(join_pending(c, s));
    FIZI_TRY(learn_model(c->m, take_table(c), reinterpret_cast<uint32_t *>(c->d + c->L.arrived), c->tune, d_frames, n_frames, 0, s, &c->clk, d_fizi_bits));
    return mark_last(c, s);
}

int process_frames(fizi_ctx *c, const uint8_t *d_frames, int32_t n_frames, uint64_t *d_fizi_bits,
                   uint64_t *d_hand_bits, fizi_pointer *d_pointers, void *stream)
{
    if (!c || !d_frames)
        return fail(FIZI_EINVAL, "null context or frames");
    if (reinterpret_cast<uintptr_t>(d_frames) % 4 != 0)
        return fail(FIZI_EINVAL, "frames must be 4-byte aligned");
    if (n_frames < 1)
        return fail(FIZI_EINVAL, "n_frames must be >= 1");
    if (!c->m.learned)
        return fail(FIZI_ESTATE, "process_frames before learn_background");
    hipStream_t s = static_cast<hipStream_t>(stream);
    FIZI_TRY(order_after_previous(c, s));
    const size_t W = c->m.g.width, H = c->m.g.height, px = W * H, words = H * (W / 64);
    fizi_pointer *internal = reinterpret_cast<fizi_pointer *>(c->d + c->L.ptrs);
    // several chunks: each chunk's back half runs beside the next chunk's
    // front (on the side stream; s joins it before the call ends, or, with
    // pipelined calls, after the next call's first classify)
    const bool pipelined = c->pipe_calls || n_frames > c->chunk;
    int par = c->pipe_calls ? c->parity : 0;
    hipEvent_t prev_join = c->pipe_calls ? c->pend_join : nullptr, last = nullptr;
    for (int f0 = 0; f0 < n_frames; f0 += c->chunk) {
        const int k = std::min(c->chunk, n_frames - f0);
        const uint64_t fbase = c->next_frame + (uint64_t)f0;
        // a launch whose morphology, in short bands of one wave each, needs
        // at most one wave per SIMD is bound by the length of one wave's
        // chain of rows rather than by the total work: it takes that shape
        // (13 row steps per wave against 17 for 8-row bands). Larger launches
        // keep the tuned shape, which repeats fewer halo rows.
        const bool short_chain =
            c->tune.short_bands && (size_t)k * ((H + kShortBand - 1) / kShortBand) <= (size_t)c->n_cu * 4;
        // the launch's first job, and the strides to the next ones
        Job J;
        fill_job(c->m, short_chain ? kShortBand : c->tune.morph_rows, J,
                 !short_chain && morph_in_regs(c->tune.morph_rows, (int)(W / 64), morph_ops(c->m.p), morph_ops(c->m.p)));
        set_scratch(J, slot_at(c->m.g, c->d + c->L.slots));
        if (pipelined && par)
            J.raw = reinterpret_cast<uint64_t *>(c->d + c->L.raw2);
        J.frame = d_frames + (size_t)f0 * px * 3;
        if (d_fizi_bits)
            J.fizi = d_fizi_bits + (size_t)f0 * words;
        J.hand = d_hand_bits ? d_hand_bits + (size_t)f0 * words : nullptr;
        J.out = d_pointers ? d_pointers + f0 : internal;
        J.hout = c->d_ring;
        J.frame_index = fbase;
        SpanJobs S = span_jobs(J, k, reinterpret_cast<uint32_t *>(c->d + c->L.arrived));
        S.table = 1;
        if (!d_fizi_bits)
            S.fizi_words = c->L.slot_stride / sizeof(uint64_t);
        S.slot_bytes = c->L.slot_stride;
        S.raw_bytes = pipelined && par ? c->L.raw2_stride : c->L.slot_stride;
        S.ring_mask = kRing - 1;
        Table *tab = take_table(c);
        FIZI_TRY(span_front(tab, S, J, c->n_cu, s, &c->clk));
        // the stream the chunk's back half goes to
        hipStream_t bs = s;
        if (pipelined) {
            FIZI_HIP(hipEventRecord(c->cls_ev[par], s));
            FIZI_HIP(hipStreamWaitEvent(c->side, c->cls_ev[par], 0));
            bs = c->side;
        }
        FIZI_TRY(span_back(tab, S, J, morph_ops(c->m.p), c->tune, c->n_cu, bs, &c->clk, pipelined));
        // the ring holds a chunk's pointers once its back half is done
        fizi_ctx::Rec &r = c->recs[c->next_rec];
        c->next_rec = (c->next_rec + 1) % kRecs;
        r.f0 = fbase;
        r.f1 = fbase + k;
        FIZI_HIP(hipEventRecord(r.ev, bs));
        r.valid = true;
        last = r.ev;
        if (pipelined) {
            // the chunk before this one is joined after this classify: the
            // next classify reuses its raw buffers
            if (prev_join)
                FIZI_HIP(hipStreamWaitEvent(s, prev_join, 0));
            prev_join = r.ev;
            par ^= 1;
        }
    }
    c->next_frame += (uint64_t)n_frames;
    if (!pipelined)
        return mark_last(c, s, last);
    if (c->pipe_calls) {
        c->pend_join = prev_join;
        c->parity = par;
    } else {
        FIZI_HIP(hipStreamWaitEvent(s, prev_join, 0));
    }
    return mark_last(c, s);
}

int get_pointer(fizi_ctx *c, int64_t frame_index, fizi_pointer *h_out)
{
    if (!c || !h_out)
        return fail(FIZI_EINVAL, "null context or output");
    if (frame_index < 0 || (uint64_t)frame_index >= c->next_frame)
        return fail(FIZI_ERANGE, "frame not submitted yet");
    if ((uint64_t)frame_index + kRing < c->next_frame)
        return fail(FIZI_ERANGE, "frame no longer kept (older than the last 65536)");
    // calls run in submission order, so the first recorded chunk that ends
    // after the frame finishes no earlier than the frame's own back half
    int best = -1;
    for (int i = 0; i < kRecs; ++i) {
        const fizi_ctx::Rec &r = c->recs[i];
        if (r.valid && r.f1 > (uint64_t)frame_index && (best < 0 || r.f0 < c->recs[best].f0))
            best = i;
    }
    if (best < 0)
        return fail(FIZI_ERANGE, "frame record missing");
    FIZI_HIP(hipEventSynchronize(c->recs[best].ev));
    *h_out = c->h_ring[(size_t)frame_index % kRing];
    return FIZI_OK;
}

int fizi_stage_timing(fizi_ctx *c, int32_t enable)
{
    if (!c)
        return fail(FIZI_EINVAL, "null context");
    return c->clk.enable(enable != 0);
}

int fizi_stage_times(fizi_ctx *c, double *h_ms, int64_t *h_launches)
{
    if (!c || !h_ms || !h_launches)
        return fail(FIZI_EINVAL, "null argument");
    return c->clk.read(h_ms, h_launches);
}

int fizi_set_tracking(fizi_ctx *c, int32_t enable)
{
    if (!c)
        return fail(FIZI_EINVAL, "null context");
    FIZI_TRY(drain(c));
    FIZI_HIP(launch_fill_u32(reinterpret_cast<uint32_t *>(c->m.track), 0u, sizeof(TrackState) / 4, nullptr));
    FIZI_HIP(hipStreamSynchronize(nullptr));
    c->m.tracking = enable != 0;
    return FIZI_OK;
}

int fizi_set_pipelined(fizi_ctx *c, int32_t enable)
{
    if (!c)
        return fail(FIZI_EINVAL, "null context");
    FIZI_TRY(drain(c));
    c->pipe_calls = enable != 0;
    c->parity = 0;
    return FIZI_OK;
}

int fizi_set_short_bands(fizi_ctx *c, int32_t enable)
{
    if (!c)
        return fail(FIZI_EINVAL, "null context");
    c->tune.short_bands = enable != 0;
    return FIZI_OK;
}

int fizi_flush(fizi_ctx *c, void *stream)
{
    if (!c)
        return fail(FIZI_EINVAL, "null context");
    hipStream_t s = static_cast<hipStream_t>(stream);
    FIZI_TRY(order_after_previous(c, s));
    FIZI_TRY(join_pending(c, s));
    return mark_last(c, s);
}

int fizi_destroy(fizi_ctx *c)
{
    if (!c)
        return FIZI_OK;
    if (c->have_last)
        (void)hipEventSynchronize(c->last_ev);
    // a pending back half, without touching the stream of the last call
    if (c->pend_join)
        (void)hipEventSynchronize(c->pend_join);
    c->clk.destroy();
    if (c->h_ring)
        (void)hipHostFree(c->h_ring);
    for (hipEvent_t e : {c->order_ev, c->cls_ev[0], c->cls_ev[1]})
        if (e)
            (void)hipEventDestroy(e);
    for (const fizi_ctx::Rec &r : c->recs)
        if (r.ev)
            (void)hipEventDestroy(r.ev);
    if (c->side)
        (void)hipStreamDestroy(c->side);
    delete c;
    return FIZI_OK;
}

}  // extern "C"
