// Shared host-side building blocks (see fizi_host.h).
#include <algorithm>
#include <climits>
#include <cstring>

#include "fizi_host.h"

namespace fizi {

namespace {
thread_local std::string g_err;
}

int fail(int code, const std::string &msg)
{
    g_err = msg;
    return code;
}

}  // namespace fizi

extern "C" const char *fizi_last_error(void) { return fizi::g_err.c_str(); }

namespace fizi {

namespace {

// Direction (scaled by 6000) of the hexcone colour of hue a centi-degrees.
void hue_dir(int a, int d[3])
{
    const int k = a / 6000, f = a - 6000 * k;
    switch (k) {
    case 0: d[0] = 6000; d[1] = f; d[2] = 0; break;
    case 1: d[0] = 6000 - f; d[1] = 6000; d[2] = 0; break;
    case 2: d[0] = 0; d[1] = 6000; d[2] = f; break;
    case 3: d[0] = 0; d[1] = 6000 - f; d[2] = 6000; break;
    case 4: d[0] = f; d[1] = 0; d[2] = 6000; break;
    default: d[0] = 6000; d[1] = 0; d[2] = 6000 - f; break;
    }
}

// det[(1,1,1), d, p] = R (dB - dG) + G (dR - dB) + B (dG - dR); the three
// coefficients sum to zero, so it is kr (R - B) + kg (G - B).
void hue_coef(int a, int32_t *kr, int32_t *kg)
{
    int d[3];
    hue_dir(a, d);
    *kr = d[2] - d[1];
    *kg = d[0] - d[2];
}

}  // namespace

HueTest make_hue(int a1, int a2)
{
    HueTest h{};
    hue_coef(a1, &h.k1r, &h.k1g);
    hue_coef(a2, &h.k2r, &h.k2g);
    int d[3];
    hue_dir(a1, d);
    h.dr = d[0];
    h.dg = d[1];
    h.db = d[2];
    h.dsum = d[0] + d[1] + d[2];
    const int L = ((a2 - a1) % 36000 + 36000) % 36000;
    h.mode = L == 0 ? 0 : (L < 18000 ? 1 : (L == 18000 ? 2 : 3));
    return h;
}

HueForm hue_form(const HueTest &h)
{
    HueForm f{h.k1r, h.k1g, 0, h.k2r, h.k2g, 0, 0, 0, 1, 0};
    switch (h.mode) {
    case 0:
        f.k2r = h.k1r;
        f.k2g = h.k1g;
        f.k3r = 3 * h.dr - h.dsum;
        f.k3g = 3 * h.dg - h.dsum;
        f.c3 = 0;
        break;
    case 2:
        f.k2r = f.k2g = 0;
        break;
    case 3:
        f = HueForm{-h.k1r, -h.k1g, -1, -h.k2r, -h.k2g, 1, 0, 0, 1, 1};
        break;
    default:
        break;
    }
    return f;
}

int validate(const fizi_geom *g, const fizi_params *p)
{
    if (!g || !p)
        return fail(FIZI_EINVAL, "null geometry or parameters");
    if (g->width < 64 || g->width % 64 != 0 || g->width > kMaxW)
        return fail(FIZI_EINVAL, "width must be a multiple of 64 in [64, 8192]");
    if (g->height < 1 || g->height > kMaxH)
        return fail(FIZI_EINVAL, "height must be in [1, 8192]");
    if (p->alpha1_cdeg < 0 || p->alpha1_cdeg >= 36000 || p->alpha2_cdeg < 0 || p->alpha2_cdeg >= 36000)
        return fail(FIZI_EINVAL, "alpha1_cdeg / alpha2_cdeg must be in [0, 36000)");
    if (p->gray_S < 0 || p->gray_S > 255)
        return fail(FIZI_EINVAL, "gray_S must be in [0, 255]");
    if (p->bg_delta < 0 || p->bg_delta > 255)
        return fail(FIZI_EINVAL, "bg_delta must be in [0, 255]");
    if (p->open_iters < 0 || p->open_iters > kMaxMorphIters || p->close_iters < 0 ||
        p->close_iters > kMaxMorphIters)
        return fail(FIZI_EINVAL, "open_iters / close_iters must be in [0, 3]");
    if (p->min_area < 0)
        return fail(FIZI_EINVAL, "min_area must be >= 0");
    if (p->click_fill_permille < 0 || p->click_fill_permille > 1000)
        return fail(FIZI_EINVAL, "click_fill_permille must be in [0, 1000]");
    if (p->gain_row_stride < 1 || p->gain_row_stride > 64)
        return fail(FIZI_EINVAL, "gain_row_stride must be in [1, 64]");
    if (p->gain_lo_q16 < 1 || p->gain_hi_q16 < p->gain_lo_q16 || p->gain_hi_q16 > (1 << 20))
        return fail(FIZI_EINVAL, "need 1 <= gain_lo_q16 <= gain_hi_q16 <= 2^20");
    if (p->brightness_mode != 0 && p->brightness_mode != 1)
        return fail(FIZI_EINVAL, "brightness_mode must be 0 or 1");
    if (p->click_debounce < 0 || p->click_debounce > 255)
        return fail(FIZI_EINVAL, "click_debounce must be in 0..255");
    if (p->track_radius < 0 || p->track_radius > 16384)
        return fail(FIZI_EINVAL, "track_radius must be in 0..16384");
    if (p->lum_hi != 0 && (p->lum_hi < 128 || p->lum_hi > 254))
        return fail(FIZI_EINVAL, "lum_hi must be 0 (off) or in 128..254");
    if (p->lum_hi != 0 && p->brightness_mode != 0)
        return fail(FIZI_EINVAL, "the over-exposure filter (lum_hi) works on corrected pixels: brightness_mode 0");
    return FIZI_OK;
}

int morph_ops(const fizi_params &p) { return 2 * (p.open_iters + p.close_iters); }

Tuning tuning_for(int max_width, int max_ops, bool batch)
{
    (void)max_width;
    (void)max_ops;
    Tuning t;
    t.cls_iters = 4;
    if (batch) {
        // the autotuner's pick on the 64-stream 640x480..3840x2160 workload
        // in the pipelined launch mode: 8 pixel groups per classify lane,
        // 16-row bands and a grid of 64 blocks per CU for the streaming
        // kernels (eight rounds of resident blocks even out the tail, and
        // leave slots free often enough for the back half that runs beside
        // them)
        t.cls_iters = 8;
        t.grid_per_cu = 64;
        t.morph_rows = 16;
    } else {
        // one stream (measured at 1920x1080): 8-row bands give a one-frame
        // call twice the morphology waves (p50 latency 0.10 ms against 0.13
        // with 16 rows) at the same chunked throughput
        t.grid_per_cu = 32;
        t.morph_rows = 8;
    }
    return t;
}

size_t model_bytes(const fizi_geom &g, const fizi_params &p)
{
    const size_t px = (size_t)g.width * g.height;
    const size_t rows = (g.height + p.gain_row_stride - 1) / p.gain_row_stride;
    return 2 * align256(px * 3) + align256(rows * g.width * 2) + align256(sizeof(TrackState));
}

void model_at(Model &m, const fizi_geom &g, const fizi_params &p, uint8_t *base)
{
    const size_t px = (size_t)g.width * g.height;
    m.g = g;
    m.p = p;
    m.hue = make_hue(p.alpha1_cdeg, p.alpha2_cdeg);
    m.yref_rows = (g.height + p.gain_row_stride - 1) / p.gain_row_stride;
    m.bgmin = base;
    m.bgmax = base + align256(px * 3);
    m.yref = reinterpret_cast<uint16_t *>(base + 2 * align256(px * 3));
    m.track = reinterpret_cast<TrackState *>(base + 2 * align256(px * 3) +
                                             align256((size_t)m.yref_rows * g.width * 2));
    m.learned = false;
    m.tracking = false;
}

size_t slot_bytes(const fizi_geom &g)
{
    const size_t px = (size_t)g.width * g.height, words = (size_t)g.height * (g.width / 64);
    return 2 * align256(words * 8) + 2 * align256(px * 4) + align256((px / 2) * 8) + align256((px / 8) * 8) +
           align256(flag_words(g) * 4);
}

Slot slot_at(const fizi_geom &g, uint8_t *base)
{
    const size_t px = (size_t)g.width * g.height, words = (size_t)g.height * (g.width / 64);
    Slot s;
    size_t o = 0;
    s.raw = reinterpret_cast<uint64_t *>(base + o);
    o += align256(words * 8);
    s.fz = reinterpret_cast<uint64_t *>(base + o);
    o += align256(words * 8);
    s.parent = reinterpret_cast<uint32_t *>(base + o);
    o += align256(px * 4);
    s.index = reinterpret_cast<uint32_t *>(base + o);
    o += align256(px * 4);
    s.runs = reinterpret_cast<uint2 *>(base + o);
    s.run_cap = run_capacity(g.width, g.height);
    o += align256((px / 2) * 8);
    s.links = reinterpret_cast<uint2 *>(base + o);
    s.link_cap = link_capacity(g.width, g.height);
    o += align256((px / 8) * 8);
    s.bflag = reinterpret_cast<uint32_t *>(base + o);
    s.nflags = flag_words(g);
    return s;
}

void fill_job(const Model &m, int band, Job &J, bool pack)
{
    std::memset(&J, 0, sizeof(J));
    J.bgmin = m.bgmin;
    J.bgmax = m.bgmax;
    J.yref = m.yref;
    J.W = m.g.width;
    J.H = m.g.height;
    J.Wd = m.g.width / 64;
    J.rs = m.p.gain_row_stride;
    J.band = band;
    // narrow frames share a wave between bands: 4 bands of at most 16 words,
    // or 2 of at most 32; not without an opening, where noise stays and its
    // runs, of all the wave's bands together, would fill a segment every row
    // (16 frames of 640x480 of noise: morphology 154 against 195 us, and the
    // joins left to the components)
    J.mgroup = !pack || m.p.open_iters == 0 ? 64 : (J.Wd <= 16 ? 16 : (J.Wd <= 32 ? 32 : 64));
    J.delta = m.p.bg_delta;
    J.S1 = std::max(m.p.gray_S, 1);
    J.open_it = m.p.open_iters;
    J.close_it = m.p.close_iters;
    J.min_area = m.p.min_area;
    J.fill_pm = m.p.click_fill_permille;
    J.glo = m.p.gain_lo_q16;
    J.ghi = m.p.gain_hi_q16;
    J.scaled = m.p.brightness_mode;
    J.S_q16 = std::max((uint32_t)m.p.gray_S << 16, 1u);
    J.debounce = m.p.click_debounce;
    J.track_r2 = (uint32_t)m.p.track_radius * (uint32_t)m.p.track_radius;
    J.S0 = m.p.gray_S;
    J.lum2 = 2 * m.p.lum_hi;
    J.hue = m.hue;
    J.track = m.tracking ? m.track : nullptr;
}

void set_scratch(Job &J, const Slot &s)
{
    J.raw = s.raw;
    J.fizi = s.fz;
    J.parent = s.parent;
    J.index = s.index;
    J.runs = s.runs;
    J.run_cap = s.run_cap;
    J.links = s.links;
    J.link_cap = s.link_cap;
    J.bflag = s.bflag;
}

void set_prefixes(Table &T, int njobs, const Tuning &t)
{
    T.h.njobs = njobs;
    T.h.gain_pre[0] = T.h.cls_pre[0] = T.h.mor_pre[0] = 0;
    const int ctile = cls_tile_px(t);
    for (int i = 0; i < njobs; ++i) {
        const Job &J = T.jobs[i];
        const long px = (long)J.W * J.H;
        const int rows = (J.H + J.rs - 1) / J.rs;
        T.h.gain_pre[i + 1] = T.h.gain_pre[i] + (rows + kGainRows - 1) / kGainRows;
        T.h.cls_pre[i + 1] = T.h.cls_pre[i] + (int)((px + ctile - 1) / ctile);
        const int bands = (J.H + J.band - 1) / J.band, per = 64 / J.mgroup;
        T.h.mor_pre[i + 1] = T.h.mor_pre[i] + (bands + per - 1) / per;
    }
    // the persistent step's queue: jobs by size, largest first; every gain
    // tile ahead of the bands, so that a band rarely waits for its frame's
    // gain
    int order[kMaxJobs];
    for (int i = 0; i < njobs; ++i)
        order[i] = i;
    std::stable_sort(order, order + njobs, [&](int a, int b) {
        return (long)T.jobs[a].W * T.jobs[a].H > (long)T.jobs[b].W * T.jobs[b].H;
    });
    int k = 0, item = 0;
    auto push = [&](int j, int type) {
        const int n = type == 0 ? T.h.gain_pre[j + 1] - T.h.gain_pre[j]
                                : (T.jobs[j].H + 4 * T.jobs[j].band - 1) / (4 * T.jobs[j].band);
        T.h.flow_pre[k] = item;
        T.h.flow_seg[k] = (j << 1) | type;
        item += n;
        ++k;
    };
    for (int i = 0; i < njobs; ++i)
        push(order[i], 0);
    for (int i = 0; i < njobs; ++i)
        push(order[i], 1);
    T.h.flow_nseg = k;
    T.h.flow_pre[k] = item;
}

int TableRing::init(uint8_t *d_base)
{
    for (int i = 0; i < kTabSlots; ++i) {
        d[i] = reinterpret_cast<Table *>(d_base + i * align256(sizeof(Table)));
        FIZI_HIP(hipHostMalloc(reinterpret_cast<void **>(&h[i]), sizeof(Table), hipHostMallocDefault));
        std::memset(h[i], 0, sizeof(Table));
        // the host only waits for the slot's kernels to be done with it
        FIZI_HIP(hipEventCreateWithFlags(&ev[i], kDeviceOrderEvent));
    }
    return FIZI_OK;
}

void TableRing::destroy()
{
    for (int i = 0; i < kTabSlots; ++i) {
        if (used[i] && ev[i])
            (void)hipEventSynchronize(ev[i]);
        if (h[i])
            (void)hipHostFree(h[i]);
        if (ev[i])
            (void)hipEventDestroy(ev[i]);
        h[i] = nullptr;
        ev[i] = nullptr;
    }
}

int TableRing::take(int *slot)
{
    const int s = next;
    next = (next + 1) % kTabSlots;
    if (used[s])
        FIZI_HIP(hipEventSynchronize(ev[s]));
    *slot = s;
    return FIZI_OK;
}

int TableRing::finish(int slot, hipStream_t s)
{
    FIZI_HIP(hipEventRecord(ev[slot], s));
    used[slot] = true;
    return FIZI_OK;
}

int StageClock::enable(bool want)
{
    if (want && !on) {
        for (int st = 0; st < FIZI_NSTAGES; ++st) {
            if (ev[st].empty()) {
                ev[st].resize(2 * kTimedLaunches, nullptr);
                for (auto &e : ev[st])
                    FIZI_HIP(hipEventCreate(&e));
            }
            used[st] = 0;
        }
    }
    on = want;
    return FIZI_OK;
}

StageEvents StageClock::next(int stage)
{
    StageEvents e;
    if (!on || used[stage] >= kTimedLaunches)
        return e;
    const int i = used[stage]++;
    e.start = ev[stage][2 * i];
    e.stop = ev[stage][2 * i + 1];
    return e;
}

int StageClock::read(double *ms, int64_t *n)
{
    for (int st = 0; st < FIZI_NSTAGES; ++st) {
        double tot = 0.0;
        for (int i = 0; i < used[st]; ++i) {
            FIZI_HIP(hipEventSynchronize(ev[st][2 * i + 1]));
            float t = 0.f;
            FIZI_HIP(hipEventElapsedTime(&t, ev[st][2 * i], ev[st][2 * i + 1]));
            tot += t;
        }
        ms[st] = tot;
        n[st] = used[st];
        used[st] = 0;
    }
    return FIZI_OK;
}

void StageClock::destroy()
{
    for (int st = 0; st < FIZI_NSTAGES; ++st) {
        for (auto &e : ev[st])
            if (e)
                (void)hipEventDestroy(e);
        ev[st].clear();
    }
}

int device_cu_count(int *device, int *n_cu)
{
    FIZI_HIP(hipGetDevice(device));
    FIZI_HIP(hipDeviceGetAttribute(n_cu, hipDeviceAttributeMultiprocessorCount, *device));
    return FIZI_OK;
}

SpanJobs span_jobs(const Job &J, int n, uint32_t *arrived)
{
    SpanJobs S{};
    const size_t px = (size_t)J.W * J.H;
    const int bands = (J.H + J.band - 1) / J.band, per = 64 / J.mgroup;
    S.frame = J.frame;
    S.frame_bytes = px * 3;
    S.raw = J.raw;
    S.fizi = J.fizi;
    S.hand = J.hand;
    S.fizi_words = S.hand_words = px / 64;
    S.out = J.out;
    S.ring = J.hout;
    S.track = J.track;
    S.parent = J.parent;
    S.index = J.index;
    S.runs = J.runs;
    S.links = J.links;
    S.min_area = J.min_area;
    S.fill_pm = J.fill_pm;
    S.debounce = J.debounce;
    S.track_r2 = J.track_r2;
    S.open_it = (int16_t)J.open_it;
    S.close_it = (int16_t)J.close_it;
    S.frame_index = J.frame_index;
    S.yref = const_cast<uint16_t *>(J.yref);
    S.n = n;
    S.W = J.W;
    S.H = J.H;
    S.rs = J.rs;
    S.band = J.band;
    S.mgroup = J.mgroup;
    S.mor_items = (bands + per - 1) / per;
    S.glo = J.glo;
    S.ghi = J.ghi;
    S.hue = J.hue;
    S.arrived = arrived;
    return S;
}

int span_front(Table *d_tab, const SpanJobs &S, const Job &first, int n_cu, hipStream_t s, StageClock *clk)
{
    auto ev = [&](int st) { return clk ? clk->next(st) : StageEvents{}; };
    FIZI_HIP(launch_gain_span(d_tab, S, s, ev(FIZI_STAGE_GAIN)));
    FIZI_HIP(launch_classify_span(d_tab, S, first, n_cu, s, ev(FIZI_STAGE_CLASSIFY)));
    return FIZI_OK;
}

int span_back(const Table *d_tab, const SpanJobs &S, const Job &first, int max_ops, const Tuning &t, int n_cu,
              hipStream_t s, StageClock *clk, bool beside)
{
    auto ev = [&](int st) { return clk ? clk->next(st) : StageEvents{}; };
    FIZI_HIP(launch_morph(d_tab, S.n * S.mor_items, S.mor_items, S.W / 64, max_ops, n_cu, t, s, ev(FIZI_STAGE_MORPH)));
    // tracked consecutive frames are resolved in order
    const bool tracked = S.n > 1 && S.track != nullptr;
    ChainSpan C{};
    if (tracked) {
        C.out = S.out;
        C.ring = S.ring;
        C.track = S.track;
        C.fizi = S.fizi;
        C.fizi_words = S.fizi_words;
        C.parent = first.parent;
        C.index = first.index;
        C.slot_bytes = S.slot_bytes;
        C.frame_index = S.frame_index;
        C.ring_mask = S.ring_mask;
        C.run_cap = first.run_cap;
        C.amin = (uint32_t)std::max(first.min_area, 0);
        C.r2 = first.track_r2;
        C.n = S.n;
        C.W = S.W;
        C.H = S.H;
        C.debounce = first.debounce;
    }
    FIZI_HIP(launch_resolve(d_tab, S.n, s, ev(FIZI_STAGE_RESOLVE), tracked ? &C : nullptr, beside));
    return FIZI_OK;
}

int learn_model(Model &m, Table *d_tab, uint32_t *arrived, const Tuning &t, const uint8_t *frames, int n, int reset,
                hipStream_t s, StageClock *clk, const uint64_t *masks)
{
    const size_t px = (size_t)m.g.width * m.g.height;
    for (int f0 = 0; f0 < n; f0 += kMaxJobs) {
        const int k = std::min(kMaxJobs, n - f0);
        Job J;
        fill_job(m, t.morph_rows, J, false);
        J.frame = frames + (size_t)f0 * px * 3;
        SpanJobs S = span_jobs(J, k, arrived);
        S.make_yref = reset && f0 == 0;
        FIZI_HIP(launch_gain_span(d_tab, S, s));
        const LearnSpan L{J.frame, px * 3, masks ? masks + (size_t)f0 * (px / 64) : nullptr, m.bgmin, m.bgmax,
                          (uint32_t)px, k, (reset && f0 == 0) ? 1 : 0};
        FIZI_HIP(launch_minmax(d_tab, L, s, clk ? clk->next(FIZI_STAGE_LEARN) : StageEvents{}));
    }
    m.learned = true;
    return FIZI_OK;
}

int run_front(const Table *d_tab, const Table &h, int njobs, const Tuning &t, int n_cu, bool fixed_grid,
              hipStream_t s, StageClock *clk)
{
    auto ev = [&](int st) { return clk ? clk->next(st) : StageEvents{}; };
    const int big = INT_MAX / 2;
    FIZI_HIP(launch_gain(d_tab, fixed_grid ? big : h.h.gain_pre[njobs], n_cu, t, s, ev(FIZI_STAGE_GAIN)));
    FIZI_HIP(launch_classify(d_tab, fixed_grid ? big : h.h.cls_pre[njobs], n_cu, t, s,
                             ev(FIZI_STAGE_CLASSIFY)));
    return FIZI_OK;
}

int run_back(const Table *d_tab, const Table &h, int njobs, int max_jobs, int max_wd, int max_ops,
             const Tuning &t, int n_cu, bool fixed_grid, hipStream_t s, StageClock *clk, bool beside)
{
    auto ev = [&](int st) { return clk ? clk->next(st) : StageEvents{}; };
    const int big = INT_MAX / 2;
    FIZI_HIP(launch_morph(d_tab, fixed_grid ? big : h.h.mor_pre[njobs], 0, max_wd, max_ops, n_cu, t, s,
                          ev(FIZI_STAGE_MORPH)));
    FIZI_HIP(launch_resolve(d_tab, fixed_grid ? max_jobs : njobs, s, ev(FIZI_STAGE_RESOLVE), nullptr, beside));
    return FIZI_OK;
}

int run_pipeline(const Table *d_tab, const Table &h, int njobs, int max_jobs, int max_wd, int max_ops,
                 const Tuning &t, int n_cu, bool fixed_grid, hipStream_t s, StageClock *clk)
{
    FIZI_TRY(run_front(d_tab, h, njobs, t, n_cu, fixed_grid, s, clk));
    return run_back(d_tab, h, njobs, max_jobs, max_wd, max_ops, t, n_cu, fixed_grid, s, clk);
}

}  // namespace fizi
