// Host side of the Downstream tracking + vertexing library: the C ABI of
// include/ds.h, argument validation, launch configuration and the launch
// modes (one launch per event, or one persistent work-stealing launch).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "ds.h"
#include "ds_kernels.h"

namespace {

constexpr int MAX_STREAM_SLOTS = 64;
constexpr int ITEMS_PER_SEED = 3;
constexpr int CLONE_BLOCK = 256;
constexpr size_t LDS_CU = 160 * 1024, LDS_STATIC = 256;   // of a compute unit; a tracking workgroup's static share
constexpr size_t LDS_GRAIN = 1280;   // granule of LDS allocation (three workgroups fit a unit to 53 760 bytes)
constexpr int SIMD_REGS = 512, SIMD_WAVES = 8;   // vector registers per lane of a SIMD, in blocks of eight; its wavefronts
constexpr int TRACK_BLOCKS[] = {64, 128, 192, 256, 512, 1024};
// tracking kernel instantiations of one block size
enum { TRK_PLAIN, TRK_CANDS, TRK_VTX, TRK_DV1, TRK_DV1_VTX, TRK_VTX_XTR, TRK_DV1_VTX_XTR, TRK_KINDS };
constexpr int ITEMS_MAX = 16;    // items per seed that LDS left over is spent on
constexpr size_t LDS_LIMIT = 160 * 1024 - 256;   // gfx950: 160 KiB per workgroup, minus static use
constexpr float PRESCREEN_MARGIN = 0.1f;         // mm, see the float32 error bound of the pair prescreen

struct Launch {
    int block, wg_per_cu, bins;
};
enum { SET_BLOCK = 1, SET_WG = 2, SET_BINS = 4 };
constexpr Launch TRACK_LAUNCH{256, 3, 1024};
constexpr Launch VERTEX_LAUNCH{256, 4, 0};   // workgroup per event, four resident per CU

constexpr int MAX_DEVICES = 64;
constexpr int STATIC_HDR = 64;   // ints: [0] the tracking and [2] the vertexing work counter
constexpr int STATIC_INTS = STATIC_HDR + ds::ORDER_WS + DS_STATIC_MAX_EVENTS;

// Largest-first event order of one stream slot: ORDER_WS ints of bin counts,
// then the order of up to `cap` events; and the smaller ones that came before it.
struct OrderWs {
    int *p = nullptr;
    int cap = 0;
    int *old[24] = {};   // (each at least twice the one before, the first of 1 024 events)
    int n_old = 0;
};

}  // namespace

// ds_process_static's workspace, for callers that cannot allocate: the work
// counters, then the largest-first order's bin counts (ORDER_WS ints),
// then the order of up to DS_STATIC_MAX_EVENTS events; 1.06 MB.  Every device
// the library runs on holds its own copy until the process ends.  On the host
// the name stands for no device address: host code uses only the address
// static_scratch() looked up for the device.
static __device__ __align__(256) int scratch[STATIC_INTS];

namespace {

std::mutex g_scratch_mu;
int *g_scratch[MAX_DEVICES] = {};

// The current device's copy of `scratch` (looked up once per device; the
// device must be current).
ds_status static_scratch(int device, int **p)
{
    if (device < 0 || device >= MAX_DEVICES) return DS_E_CAPACITY;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[device]) {
        void *q = nullptr;
        if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) return DS_E_DEVICE;
        g_scratch[device] = static_cast<int *>(q);
    }
    *p = g_scratch[device];
    return DS_OK;
}

}  // namespace

struct ds_ctx {
    int device = 0;
    int *scratch = nullptr;    // this device's static workspace (ds_process_static)
    int n_cu = 256;
    bool loaded = false;
    ds::DevGeom G{};
    double u_min = -1000.0, u_max = 1000.0;
    double ghost_threshold = 0.5;
    bool clone_kill = false;
    int algorithm = 0;             // 0: Dv0 window search, 1: Dv1 triplet search
    float *d_W = nullptr;    // ghost-killer weights, per-lane MFMA order (mlp_lane_layout)
    float *d_Wrow = nullptr; // the same, row-major (the candidate rows' per-lane network)
    float *d_WL = nullptr;   // trigger-line networks
    int *d_counters = nullptr;  // [MAX_STREAM_SLOTS][4]
    std::map<void *, int> slots;
    OrderWs order_ws[MAX_STREAM_SLOTS];
    int event_order = DS_ORDER_INPUT;   // persistent launches: DS_ORDER_*
    int fused_step = 1;                 // ds_process: one fused launch (1) or tracking then vertexing (0)
    int trk_waves[std::size(TRACK_BLOCKS)][TRK_KINDS] = {};   // set_kernel_attributes
    Launch trk = TRACK_LAUNCH;
    int trk_set = 0;           // which of them ds_set_launch set (SET_*); a launch chooses the others (choose_shape)
    Launch vtx = VERTEX_LAUNCH;
    std::mutex mu;
};

namespace {

ds_status dev_err(hipError_t e) { return e == hipSuccess ? DS_OK : DS_E_DEVICE; }

size_t round16(size_t v) { return (v + 15) & ~size_t(15); }

// Dynamic LDS of the tracking kernel, mirroring its carve: hits, bucket
// bounds (the fused vertexing's kept tracks lie over them), then the seed
// constants ... item buffers (one region: phase C's feature tiles and the
// fused vertexing's survivor masks reuse it), then clone killing's notes.
struct TrackLayout {
    size_t sc;      // seed constants: start of the reusable region
    size_t total;
};

TrackLayout track_layout(int hcap, int nb, int nb3, int map_ints, int block, int scap, int icap, int tcap, bool clone)
{
    TrackLayout L;
    size_t off = (size_t)hcap * 4;
    off = round16(off + (size_t)hcap * 2);
    off = round16(off + (size_t)(3 * nb + nb3 + 1) * 2);
    off = std::max(round16(off + (size_t)map_ints * 4), ds::fused_kept_bytes(tcap));
    off += ds::FIT_TAB * 8 + (size_t)(block / 64) * ds::ROW_QUEUE * 2;
    L.sc = off;
    off += (size_t)scap * sizeof(ds::SeedConst);
    off += (size_t)scap * 8;
    off = round16(off + (size_t)scap * 4);
    off = round16(off + (size_t)icap * 4);
    L.total = round16(off + (size_t)icap * 12) + (clone ? ds::clone_lds_bytes(tcap) : 0);
    return L;
}

// The footprint that decides whether an event of the declared size is taken
// (DS_E_CAPACITY beyond LDS_LIMIT): every lane of the workgroup with its seed,
// ITEMS_PER_SEED items of 12 bytes per lane, 24 bytes per kept track and 6 for
// its row where they do not fit beside the pair loop's buffer.  The launch's
// own layout (plan_track) is never larger.
size_t capacity_lds(int hcap, int nb, int nb3, int block, int tcap)
{
    const int icap = std::max(block * ITEMS_PER_SEED, ds::MAX_L3);
    const size_t head = round16(round16((size_t)hcap * 6) + (size_t)(3 * nb + nb3 + 1) * 2);
    const size_t region = round16((size_t)block * (sizeof(ds::SeedConst) + 12)) + round16((size_t)icap * 4) +
                          round16((size_t)icap * 8);
    size_t kept = 0;
    if (tcap > 0) {
        size_t ring = 4;
        while (ring < 4 * (size_t)block * 6) ring *= 2;
        const size_t rows = round16((size_t)tcap * 6 + 4);
        kept = round16((size_t)tcap * 24) + (region >= ring + rows ? 0 : rows);
    }
    return head + region + kept;
}

// k_vertex: the survivor masks of the pair loop, then the event's kept tracks
size_t vertex_lds(int tcap, int block)
{
    return sizeof(int) * (size_t)ds::vtx_mask_ints(block) + ds::kept_lds_bytes(tcap);
}

// The footprint that decides whether ds_vertex takes events of the declared
// size: 30 bytes per seed beside a buffer of six pairs per lane, rounded up to
// a power of two.  vertex_lds is never larger.
size_t vertex_capacity_lds(int tcap, int block)
{
    size_t pairs = 1;
    while (pairs < 6 * (size_t)block) pairs *= 2;
    return round16((size_t)tcap * 24) + round16((size_t)tcap * 6 + 4) + 4 * pairs;
}

// (of v near the largest int: the largest multiple)
int round_up(int v, int m) { return v > INT_MAX - m ? INT_MAX / m * m : ((v + m - 1) / m) * m; }

// LDS that a workgroup of the tracking kernel takes from its compute unit.
size_t lds_taken(size_t dynamic) { return (dynamic + LDS_STATIC + LDS_GRAIN - 1) / LDS_GRAIN * LDS_GRAIN; }

ds_status slot_for(ds_ctx *c, void *stream, int **counters, int *slot = nullptr)
{
    auto it = c->slots.find(stream);
    int s;
    if (it == c->slots.end()) {
        if ((int)c->slots.size() >= MAX_STREAM_SLOTS) return DS_E_CAPACITY;
        s = (int)c->slots.size();
        c->slots[stream] = s;
    } else {
        s = it->second;
    }
    *counters = c->d_counters + 4 * s;
    if (slot) *slot = s;
    return DS_OK;
}

// The largest-first workspace of a stream slot for n events, made and grown on
// demand.  A workspace is never freed before the context: launches in flight and
// graphs that a caller has captured may hold it (they double, so that the old
// ones together are no larger than the last).  While the stream is being
// captured nothing is allocated: null, the caller then takes input order.
ds_status order_workspace(ds_ctx *c, int slot, int n, hipStream_t s, int **ws)
{
    OrderWs &o = c->order_ws[slot];
    *ws = o.p;
    if (o.cap >= n) return DS_OK;
    *ws = nullptr;
    hipStreamCaptureStatus cap_status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap_status) != hipSuccess || cap_status != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return DS_OK;
    }
    const int cap = (int)std::max<long long>({n, 1024, std::min(2LL * o.cap, 1LL << 30)});
    int *p = nullptr;
    if (hipMalloc(&p, sizeof(int) * ((size_t)ds::ORDER_WS + (size_t)cap)) != hipSuccess) return DS_E_NOMEM;
    if (o.p) o.old[o.n_old++] = o.p;
    o.p = p;
    o.cap = cap;
    *ws = p;
    return DS_OK;
}

ds_status check_events(const ds_events *ev)
{
    if (!ev) return DS_E_ARG;
    if (ev->n_events < 0 || ev->n_seeds < 0 || ev->n_hits < 0 || ev->max_seeds_per_event < 0 ||
        ev->max_hits_per_event < 0)
        return DS_E_ARG;
    if (ev->n_events == 0) return DS_OK;
    if (!ev->seed_off || !ev->hit_off) return DS_E_ARG;
    if (ev->n_seeds > 0 && (!ev->sx || !ev->sy || !ev->stx || !ev->sty || !ev->sqop)) return DS_E_ARG;
    if (ev->n_hits > 0 && !ev->hu) return DS_E_ARG;
    return DS_OK;
}

ds_status check_extras(const ds_ctx *c, const ds_vertices *v)
{
    const bool any = v->m_pipi || v->m_ppi || v->line[0] || v->line[1] || v->line[2] || v->line[3];
    if (!any) return DS_OK;
    if (!(v->m_pipi && v->m_ppi && v->line[0] && v->line[1] && v->line[2] && v->line[3])) return DS_E_ARG;
    return c->d_WL ? DS_OK : DS_E_STATE;
}

ds_status check_tracks(const ds_tracks *t, int n_seeds, bool need_score)
{
    if (!t || !t->flags) return DS_E_ARG;
    if (n_seeds == 0) return DS_OK;
    if (!t->x || !t->y || !t->tx || !t->ty || !t->qop || !t->chi2 || !t->nhits) return DS_E_ARG;
    for (int L = 0; L < 4; ++L)
        if (!t->hit[L]) return DS_E_ARG;
    if (need_score && !t->score) return DS_E_ARG;
    return DS_OK;
}

// ---------------------------------------------------------------- kernels

template <int B>
hipError_t launch_track_b(const ds::TrackArgs &a, const ds::DevGeom &G, int grid, size_t lds, hipStream_t s)
{
    const ds::TrackKernArgs k{a, G};
    if (a.cmax > 0)
        hipLaunchKernelGGL((ds::k_track<B, true, false, false>), dim3(grid), dim3(B), lds, s, k);
    else if (a.hsec && a.vcount && a.m_pipi)
        hipLaunchKernelGGL((ds::k_track<B, false, true, true, true>), dim3(grid), dim3(B), lds, s, k);
    else if (a.hsec && a.vcount)
        hipLaunchKernelGGL((ds::k_track<B, false, true, true>), dim3(grid), dim3(B), lds, s, k);
    else if (a.hsec)
        hipLaunchKernelGGL((ds::k_track<B, false, false, true>), dim3(grid), dim3(B), lds, s, k);
    else if (a.vcount && a.m_pipi)
        hipLaunchKernelGGL((ds::k_track<B, false, true, false, true>), dim3(grid), dim3(B), lds, s, k);
    else if (a.vcount)
        hipLaunchKernelGGL((ds::k_track<B, false, true, false>), dim3(grid), dim3(B), lds, s, k);
    else
        hipLaunchKernelGGL((ds::k_track<B, false, false, false>), dim3(grid), dim3(B), lds, s, k);
    return hipGetLastError();
}

hipError_t launch_track(int block, const ds::TrackArgs &a, const ds::DevGeom &G, int grid, size_t lds,
                        hipStream_t s)
{
    switch (block) {
    case 64: return launch_track_b<64>(a, G, grid, lds, s);
    case 128: return launch_track_b<128>(a, G, grid, lds, s);
    case 192: return launch_track_b<192>(a, G, grid, lds, s);
    case 256: return launch_track_b<256>(a, G, grid, lds, s);
    case 512: return launch_track_b<512>(a, G, grid, lds, s);
    default: return launch_track_b<1024>(a, G, grid, lds, s);
    }
}

template <int B>
hipError_t launch_vertex_b(const ds::VertexArgs &a, const ds::DevGeom &G, int grid, size_t lds, hipStream_t s)
{
    if (a.m_pipi)
        hipLaunchKernelGGL((ds::k_vertex<B, true>), dim3(grid), dim3(B), lds, s, a, G);
    else
        hipLaunchKernelGGL((ds::k_vertex<B, false>), dim3(grid), dim3(B), lds, s, a, G);
    return hipGetLastError();
}

hipError_t launch_vertex(int block, const ds::VertexArgs &a, const ds::DevGeom &G, int grid, size_t lds,
                         hipStream_t s)
{
    switch (block) {
    case 64: return launch_vertex_b<64>(a, G, grid, lds, s);
    case 128: return launch_vertex_b<128>(a, G, grid, lds, s);
    case 256: return launch_vertex_b<256>(a, G, grid, lds, s);
    default: return launch_vertex_b<512>(a, G, grid, lds, s);
    }
}

// Allow every instantiation the full LDS of a gfx950 workgroup.  waves: the
// wavefronts of each tracking kernel that the registers of a compute unit hold.
hipError_t set_kernel_attributes(int (*waves)[TRK_KINDS])
{
    const void *fns[] = {   // (TRACK_BLOCKS times TRK_KINDS first)
#define DS_TRACK_FNS(B)                                                                                     \
    reinterpret_cast<const void *>(&ds::k_track<B, false, false, false>),                                   \
        reinterpret_cast<const void *>(&ds::k_track<B, true, false, false>),                                \
        reinterpret_cast<const void *>(&ds::k_track<B, false, true, false>),                                \
        reinterpret_cast<const void *>(&ds::k_track<B, false, false, true>),                                \
        reinterpret_cast<const void *>(&ds::k_track<B, false, true, true>),                                 \
        reinterpret_cast<const void *>(&ds::k_track<B, false, true, false, true>),                          \
        reinterpret_cast<const void *>(&ds::k_track<B, false, true, true, true>)
        DS_TRACK_FNS(64), DS_TRACK_FNS(128), DS_TRACK_FNS(192), DS_TRACK_FNS(256), DS_TRACK_FNS(512),
        DS_TRACK_FNS(1024),
#undef DS_TRACK_FNS
        reinterpret_cast<const void *>(&ds::k_vertex<64, false>),
        reinterpret_cast<const void *>(&ds::k_vertex<128, false>),
        reinterpret_cast<const void *>(&ds::k_vertex<256, false>),
        reinterpret_cast<const void *>(&ds::k_vertex<512, false>),
        reinterpret_cast<const void *>(&ds::k_vertex<64, true>),
        reinterpret_cast<const void *>(&ds::k_vertex<128, true>),
        reinterpret_cast<const void *>(&ds::k_vertex<256, true>),
        reinterpret_cast<const void *>(&ds::k_vertex<512, true>),
        reinterpret_cast<const void *>(&ds::k_clone<CLONE_BLOCK>)};
    for (const void *f : fns) {
        hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_LIMIT);
        if (e != hipSuccess) return e;
    }
    for (size_t k = 0; k < std::size(TRACK_BLOCKS) * TRK_KINDS; ++k) {
        hipFuncAttributes at;
        hipError_t e = hipFuncGetAttributes(&at, fns[k]);
        if (e != hipSuccess) return e;
        waves[k / TRK_KINDS][k % TRK_KINDS] = 4 * std::min(SIMD_WAVES, SIMD_REGS / round_up(std::max(at.numRegs, 8), 8));
    }
    return hipSuccess;
}

// Seeds or hits of a mean event, as far as the host can tell: the arrays' length
// over the number of events, unless that is more than the largest event (a part
// of a resident batch); then a third of the largest, as in uneven batches
// (1 000 of the arrays of 20 000 uneven events: 157 us with the arrays' mean,
// which looks like alike and full events, 119 with a third).
double mean_of(int length, int n_events, int most)
{
    const double mean = (double)length / std::max(n_events, 1);
    return mean <= most ? mean : most / 3.0;
}

struct VertexPlan {
    ds::VertexArgs a;
    int block, grid;
    size_t lds;
};

// A tracking launch's workgroup size, bins and LDS capacities.
struct TrackShape {
    bool dv1, clone;
    int nsec, max_seeds, hcap, tcap, wcap, want;   // given
    const int (*kinds)[TRK_KINDS];                 // ds_ctx::trk_waves
    int kind;
    int asked, block, bins, nb, nbu, nb3, nbu3, map_words, scap, icap, resident, wg_per_cu;
    TrackLayout L;

    int waves() const
    {
        size_t k = 0;
        while (TRACK_BLOCKS[k] != block) ++k;
        return kinds[k][kind];
    }

    int map_ints() const { return dv1 ? nsec * map_words : 0; }

    void set_bins(int b)
    {
        bins = b;
        nbu = dv1 ? std::max(4, (4 * bins - nsec - 4) / (3 * nsec)) : bins;
        nb = dv1 ? nsec * nbu + 1 : nbu;
        nbu3 = dv1 ? 1 : nbu;
        nb3 = dv1 ? nsec + 1 : nb;
    }

    bool fits()
    {
        L = track_layout(hcap, nb, nb3, map_ints(), block, scap, icap, tcap, clone);
        return L.total <= LDS_LIMIT;
    }

    // The layout at `block` lanes and `bins` bins.  Seeds of a chunk: no more than the largest event has.
    // Items of a chunk: at least all triplets of one seed (Dv1), or a third of its first-window hits (Dv0:
    // they are listed in the items' 12 result bytes), and room for the network's features of every seed,
    // which reuse the seed-constant ... item region, as do the fused pair loop's survivor masks.  A mean
    // event's items (`want`) in one chunk are worth a resident workgroup (10 000 events of 150 seeds, 600
    // hits, 1 024 bins: 285 us with room for them and three per unit, 325 with two chunks and four), not
    // half of them; the LDS then left over goes to items too.  (Measured with the kept tracks behind the items.)
    bool lay_out(int block_, int bins_)
    {
        block = block_;
        set_bins(bins_);
        scap = std::min(block, round_up(std::max(max_seeds, 1), 16));
        auto least = [&]() {
            const int spare = (scap + 15) / 16 * ds::MLP_TILE * 4 - scap * (int)(sizeof(ds::SeedConst) + 12);
            // (Dv1 keeps 16 bytes and 128 triplet flags per seed, and 128 queued probes per wavefront, over the
            // result bytes while it counts)
            const int flags = (scap * 32 + block / 64 * 512 + 11) / 12;
            // (clone killing's hash chains lie over the seeds and items)
            const int chains = clone ? (ds::clone_hash_words(tcap) * 4 - scap * 52 + 15) / 16 : 0;
            return round_up(std::max({chains, (wcap + 2) / 3, dv1 ? std::max(wcap, flags) : 0,
                                      (std::max(spare, ds::VTX_PAD) + 15) / 16, tcap / 64 + 4}), 16);
        };
        // the map of UTaX: 1 024 u bins per sector, 2 048 where a sector may hold more than a hundred hits
        map_words = hcap / 4 > 100 * nsec ? 64 : 32;
        icap = least();
        // the fullest events: a coarser map, fewer seeds in a chunk, then fewer bins
        while (dv1 && !fits() && map_words > 1) map_words /= 2;
        while (!fits() && scap > 16) {
            scap = std::max(16, scap / 32 * 16);
            icap = least();
        }
        while (!fits() && bins > 8) set_bins(bins / 2);
        if (L.total > LDS_LIMIT) return false;
        auto residents = [&]() { return std::max(1, std::min((int)(LDS_CU / lds_taken(L.total)), waves() * 64 / block)); };
        const int floor_icap = icap, most = std::min(residents(), 16 * 64 / block);
        icap = std::max(icap, std::min(round_up(want, 16), ds::MAX_ITEMS));
        if (!fits() || 2 * residents() <= most) {
            icap = floor_icap;
            (void)fits();
        }
        resident = residents();
        const size_t room = std::min(LDS_CU / resident / LDS_GRAIN * LDS_GRAIN - LDS_STATIC, LDS_LIMIT);
        if (room > L.total)
            icap = std::min(icap + (int)(room - L.total) / 16 / 16 * 16, std::max(icap, std::min(ITEMS_MAX * scap, ds::MAX_ITEMS)));
        return fits();
    }
};

// A prepared launch: arguments, shape, and the per-event variant.
struct TrackPlan {
    ds::TrackArgs a;
    int block, grid;
    size_t lds;
    int *order_ws = nullptr;   // persistent launch in largest-first order: its workspace
    int tiers = 1;             // in that order: launches, one per class of event sizes
    TrackShape tier[ds::MAX_TIERS];
    int n_cu = 256;
};

// The launch's shape: what ds_set_launch set, and for the rest:
//  - Few events (no more than compute units, or twice as many): each has a
//    unit to itself and the call lasts as long as its longest event, so more
//    lanes per event.  64 uneven events of 148 seeds and 583 hits per layer
//    on average: 70 us with 256 lanes, 46 with 512, 41 with 1 024; one such
//    event: 19.0, 17.2, 17.9; one of 51 seeds and 3 011 hits: 43, 36, 32.
//    Below some 128 hits per layer the wider workgroups' barriers cost more
//    than they give (14 events of 61 seeds, 71 hits: 15.1, 15.8, 17.2).
//  - Many events: as many resident wavefronts as the registers allow.  Where
//    the events are alike and LDS holds one or two of them per unit, that
//    takes 1 024 or 512 lanes (500 events of 300 seeds, 4 800 hits: 469 us
//    with 256 lanes, 388, 345; 5 000 of 300 seeds, 1 200 hits, tracking and
//    vertexing: 650, 521, 682); events far below the declared largest would
//    leave such workgroups idle (20 000 uneven ones: 865, 1 190, 1 215).
//  - 1 024 bins per layer, 512 where that lets another workgroup in (4 000
//    events of 150 seeds, 600 hits, clones killed: 147 us at 1 024 bins and
//    three per unit, 129 at 512 and four; without clone killing four fit at
//    either, 243 and 247 us for 10 000 events); Dv1 also 256 (10 000 events:
//    444 us at 1 024 bins and three per unit, 382 at 256 and four).
//  - as many workgroups per unit as are resident: one more waits for the end
//    of the launch with the event it was given.  Resident by LDS and by the
//    registers of the launch's own kernel (66 to 111 of them, so seven to four
//    wavefronts per SIMD): 1 111 events of 77 seeds, 333 hits, found, scored
//    and vertexed in three calls: 57 us with four per unit, where 87 events
//    wait for a second round, 49 with seven.
void choose_shape(const ds_ctx *c, const ds_events *ev, TrackShape &t)
{
    const Launch &set = c->trk;
    const bool auto_block = !(c->trk_set & SET_BLOCK), auto_bins = !(c->trk_set & SET_BINS);
    auto lay_out = [&](int block) {
        if (!t.lay_out(block, set.bins)) return false;
        for (int bins = 512; auto_bins && set.bins == 1024 && bins >= (t.dv1 ? 256 : 512); bins /= 2) {
            TrackShape h = t;
            if (h.lay_out(block, bins) && h.resident > t.resident) t = h;
        }
        return true;
    };
    bool ok = lay_out(set.block);
    if (auto_block && ok && ev->n_events > 0) {
        const double most = ev->max_hits_per_event / 4.0;
        const double hits = mean_of(ev->n_hits, ev->n_events, ev->max_hits_per_event) / 4.0;
        const double large = std::max(hits, std::min(most, 4.0 * hits) / 2.0);
        int block = set.block;
        if (ev->n_events <= c->n_cu && large >= 800.0) block = 1024;
        else if (ev->n_events <= 2 * c->n_cu && large >= 128.0) block = 512;
        if (2.0 * hits >= most && t.resident <= 2) block = std::max(block, t.resident == 1 ? 1024 : 512);
        for (; block > set.block && !lay_out(block); block /= 2) {}
        if (block <= set.block) (void)lay_out(set.block);
    }
    t.wg_per_cu = (c->trk_set & SET_WG) ? set.wg_per_cu : t.resident;
}

// Largest-first batches of events far below their largest: the events in
// classes of size, each in a launch with the lanes and LDS that it needs (the
// order kernels sort by class first).  One launch sized for the largest event
// holds two workgroups of 256 lanes per unit for all of them.  Classes: events
// that fit four such workgroups per unit; those up to two fifths of the way
// from there to the largest, with 512 lanes, two workgroups; and the rest, one
// of 512.  20 000 events of 148 seeds, 583 hits per layer on average, up to
// 466 and 7 137: 747 us in one launch, 663 in three over several batches; one
// batch repeated, 619 (640 with the middle class ending at a third of the way,
// 687 at half; 648 where the small class takes what fits three per unit).
int choose_tiers(const ds_ctx *c, const ds_events *ev, TrackShape *t)
{
    const TrackShape all = t[0];
    if (c->event_order != DS_ORDER_LARGEST_FIRST || (c->trk_set & (SET_BLOCK | SET_WG)) || ev->n_events < 16 * c->n_cu ||
        2.0 * mean_of(ev->n_hits, ev->n_events, ev->max_hits_per_event) >= ev->max_hits_per_event || all.block * all.resident >= 4 * 256)
        return 1;
    auto shape = [&](int sixteenths, int block, TrackShape &q) {
        q = all;
        q.max_seeds = round_up((int)((long long)all.max_seeds * sixteenths / 16), 16);
        q.hcap = round_up(all.hcap / 16 * sixteenths, 16);
        q.tcap = all.tcap ? q.max_seeds : 0;
        if (!q.lay_out(block, all.bins)) return false;
        q.wg_per_cu = q.resident;
        return true;
    };
    int k = 15, m;
    while (k > 4 && !(shape(k, 256, t[2]) && t[2].resident >= 4)) --k;
    if (k <= 4) return 1;
    m = (3 * k + 2 * 16) / 5;
    while (m > k && !(shape(m, 512, t[1]) && t[1].resident >= 2)) --m;
    if (m <= k || !shape(16, 512, t[0])) {
        t[0] = all;
        return 1;
    }
    t[0].max_seeds = all.max_seeds;
    return 3;
}

// The launch arguments that come from the shape.
void apply_shape(const ds_ctx *c, const TrackShape &t, ds::TrackArgs &a)
{
    a.hcap = t.hcap;
    a.scap = t.scap;
    a.icap = t.icap;
    a.wcap = t.wcap;
    a.tcap = t.tcap;
    a.nb = t.nb;
    a.nbu = t.nbu;
    a.inv_bw = (float)((double)t.nbu / (c->u_max - c->u_min));
    a.bin_off = (float)(-(double)a.inv_bw * c->u_min);
    a.nb3 = t.nb3;
    a.nbu3 = t.nbu3;
    a.inv_bw3 = (float)((double)t.nbu3 / (c->u_max - c->u_min));
    a.bin_off3 = (float)(-(double)a.inv_bw3 * c->u_min);
    a.fine = t.dv1 ? 1 : t.asked / t.bins;
    a.map_ints = t.map_ints();
    a.map_words = t.map_words;
    a.map_inv = (float)(32.0 * t.map_words / (c->u_max - c->u_min));
    a.map_off = (float)(-(double)a.map_inv * c->u_min);
}

ds_status plan_track(ds_ctx *c, const ds_events *ev, const ds_tracks *out, int fuse, int *counters, TrackPlan *p,
                     int vertex_fused = 0, bool cand_rows = false, bool clone = false)
{
    // Dv1 buckets hits by (layer, Y sector, u bin) plus one bucket per layer
    // for sector ids out of range; candidate rows always follow Dv0
    const bool dv1 = c->algorithm == 1 && !cand_rows;
    if (dv1 && !ev->hit_sector) return DS_E_ARG;
    // Dv1 reads layer 3 by whole sectors (one u bin each); layers 0-2 share the
    // rest of the 4 x bins bucket budget
    const int nsec = c->G.nsec;
    TrackShape t;
    t.dv1 = dv1;
    t.clone = clone;
    t.nsec = nsec;
    t.kinds = c->trk_waves;
    t.kind = cand_rows ? TRK_CANDS
             : dv1     ? (vertex_fused == 2 ? TRK_DV1_VTX_XTR : vertex_fused ? TRK_DV1_VTX : TRK_DV1)
                       : (vertex_fused == 2 ? TRK_VTX_XTR : vertex_fused ? TRK_VTX : TRK_PLAIN);
    t.max_seeds = ev->max_seeds_per_event;
    t.hcap = round_up(std::max(ev->max_hits_per_event, 1), 16);
    if (t.hcap > 65535) return DS_E_CAPACITY;   // 16-bit LDS positions and bucket bounds
    t.tcap = vertex_fused ? round_up(std::max(ev->max_seeds_per_event, 1), 16) : 0;
    if (t.tcap > 32767) return DS_E_CAPACITY;   // 15-bit kept-track indices
    t.set_bins(c->trk.bins);
    t.asked = c->trk.bins;
    if (capacity_lds(t.hcap, t.nb, t.nb3, c->trk.block, t.tcap) > LDS_LIMIT) return DS_E_CAPACITY;
    t.wcap = std::max(c->trk.block * ITEMS_PER_SEED, ds::MAX_L3);
    // items of a mean event: the UTbX hits in the first windows, with a margin (Dv1 has room for all
    // triplets of a seed, more than that)
    const double hits = mean_of(ev->n_hits, ev->n_events, ev->max_hits_per_event) / 4.0;
    const double seeds = mean_of(ev->n_seeds, ev->n_events, ev->max_seeds_per_event);
    const double per_seed = std::min((double)c->G.max_l3, 0.4 + hits * 2.0 * (c->G.w1c0 + 0.15 * c->G.w1c1) /
                                                              (c->u_max - c->u_min));
    t.want = (int)std::min(32.0 + 1.1 * seeds * std::max(per_seed, 1.0), (double)ds::MAX_ITEMS);
    choose_shape(c, ev, t);
    if (t.L.total > LDS_LIMIT) return DS_E_CAPACITY;
    ds::TrackArgs &a = p->a;
    std::memset(&a, 0, sizeof(a));
    a.n_events = ev->n_events;
    a.n_seeds = ev->n_seeds;
    a.n_hits = ev->n_hits;
    a.max_seeds = ev->max_seeds_per_event;
    a.max_hits = ev->max_hits_per_event;
    a.seed_off = ev->seed_off;
    a.sx = ev->sx;
    a.sy = ev->sy;
    a.stx = ev->stx;
    a.sty = ev->sty;
    a.sqop = ev->sqop;
    a.hit_off = ev->hit_off;
    a.hu = ev->hu;
    a.x = out->x;
    a.y = out->y;
    a.tx = out->tx;
    a.ty = out->ty;
    a.qop = out->qop;
    a.chi2 = out->chi2;
    a.score = out->score;
    a.h0 = out->hit[0];
    a.h1 = out->hit[1];
    a.h2 = out->hit[2];
    a.h3 = out->hit[3];
    a.nhits = out->nhits;
    a.cand = out->cand;
    a.flags = out->flags;
    a.counter = counters;
    a.W = c->d_W;
    a.fuse_mlp = fuse && !clone ? 1 : 0;
    a.clone = clone ? 1 : 0;
    a.ev_single = -1;
    a.tier = -1;
    apply_shape(c, t, a);
    a.hsec = dv1 ? ev->hit_sector : nullptr;
    a.map_reach = (float)(c->G.w2c0 + std::fabs(c->G.w2c1) * ds::MAP_QOP) + ds::MAP_MARGIN;
    a.map_range = ds::map_range(c->G.ffac[0]);
    p->block = t.block;
    p->grid = std::max(1, std::min(ev->n_events, c->n_cu * t.wg_per_cu));
    p->lds = t.L.total;
    p->tier[0] = t;
    p->tiers = choose_tiers(c, ev, p->tier);
    p->n_cu = c->n_cu;
    p->order_ws = nullptr;
    return DS_OK;
}

// A persistent launch takes the events largest first when the context says so
// (ws: the slot's workspace; the order kernels run ahead of the launch).
void set_order(TrackPlan &p, int *ws)
{
    p.order_ws = ws;
    p.a.order = ws ? ws + ds::ORDER_WS : nullptr;
}

ds_status plan_order(ds_ctx *c, int slot, int mode, hipStream_t s, TrackPlan &p)
{
    if (mode == DS_MODE_PER_EVENT || c->event_order != DS_ORDER_LARGEST_FIRST || p.a.n_events < 2) return DS_OK;
    int *ws = nullptr;
    const ds_status st = order_workspace(c, slot, p.a.n_events, s, &ws);
    if (st == DS_OK) set_order(p, ws);
    return st;
}

ds_status plan_vertex(ds_ctx *c, const ds_events *ev, const ds_tracks *trk, float score_max, const ds_vertices *out,
                      int *counters, VertexPlan *p)
{
    int tcap = round_up(std::max(ev->max_seeds_per_event, 1), 64);
    if (tcap > 32767) return DS_E_CAPACITY;   // 15-bit kept-track indices
    const size_t lds = vertex_lds(tcap, c->vtx.block);
    if (vertex_capacity_lds(tcap, c->vtx.block) > LDS_LIMIT) return DS_E_CAPACITY;
    ds::VertexArgs &a = p->a;
    std::memset(&a, 0, sizeof(a));
    a.n_events = ev->n_events;
    a.n_seeds = ev->n_seeds;
    a.max_seeds = ev->max_seeds_per_event;
    a.seed_off = ev->seed_off;
    a.sqop = ev->sqop;
    a.x = trk->x;
    a.y = trk->y;
    a.tx = trk->tx;
    a.ty = trk->ty;
    a.qop = trk->qop;
    a.score = trk->score;
    a.nhits = trk->nhits;
    a.score_max = score_max;
    a.vcap = out->cap_per_event;
    a.vcount = out->count;
    a.vi = out->i;
    a.vj = out->j;
    a.vx = out->x;
    a.vy = out->y;
    a.vz = out->z;
    a.vdoca = out->doca;
    a.voverflow = out->overflow;
    a.flags = out->flags;
    a.counter = counters + 2;
    a.ev_single = -1;
    a.tcap = tcap;
    a.m_pipi = out->m_pipi;
    a.m_ppi = out->m_ppi;
    a.line0 = out->line[0];
    a.line1 = out->line[1];
    a.line2 = out->line[2];
    a.line3 = out->line[3];
    a.WL = c->d_WL;
    p->block = c->vtx.block;
    p->grid = std::max(1, std::min(ev->n_events, c->n_cu * c->vtx.wg_per_cu));
    p->lds = lds;
    return DS_OK;
}

ds::GhostArgs ghost_args(ds_ctx *c, const ds_events *ev, const ds_tracks *trk)
{
    ds::GhostArgs a;
    std::memset(&a, 0, sizeof(a));
    a.n_events = ev->n_events;
    a.n_seeds = ev->n_seeds;
    a.n_hits = ev->n_hits;
    a.seed_off = ev->seed_off;
    a.sx = ev->sx;
    a.sy = ev->sy;
    a.stx = ev->stx;
    a.sty = ev->sty;
    a.sqop = ev->sqop;
    a.hit_off = ev->hit_off;
    a.hu = ev->hu;
    a.x = trk->x;
    a.y = trk->y;
    a.tx = trk->tx;
    a.ty = trk->ty;
    a.qop = trk->qop;
    a.chi2 = trk->chi2;
    a.h0 = trk->hit[0];
    a.h1 = trk->hit[1];
    a.h2 = trk->hit[2];
    a.h3 = trk->hit[3];
    a.nhits = trk->nhits;
    a.score = trk->score;
    a.flags = trk->flags;
    a.W = c->d_W;
    return a;
}

hipError_t launch_ghost(ds_ctx *c, const ds::GhostArgs &a, hipStream_t s)
{
    const int grid = std::max(1, std::min(a.n_events, c->n_cu * 8));
    hipLaunchKernelGGL(ds::k_ghost<128>, dim3(grid), dim3(128), 0, s, a, c->G);
    return hipGetLastError();
}

ds_status clone_args(const ds_events *ev, const ds_tracks *trk, ds::CloneArgs *a, size_t *lds)
{
    std::memset(a, 0, sizeof(*a));
    const int tcap = round_up(std::max(ev->max_seeds_per_event, 1), 64);
    *lds = (size_t)tcap * 16 * (CLONE_BLOCK / 64);
    if (*lds > LDS_LIMIT) return DS_E_CAPACITY;
    a->n_events = ev->n_events;
    a->n_seeds = ev->n_seeds;
    a->max_seeds = ev->max_seeds_per_event;
    a->seed_off = ev->seed_off;
    a->x = trk->x;
    a->y = trk->y;
    a->tx = trk->tx;
    a->ty = trk->ty;
    a->qop = trk->qop;
    a->chi2 = trk->chi2;
    a->score = trk->score;
    a->h0 = trk->hit[0];
    a->h1 = trk->hit[1];
    a->h2 = trk->hit[2];
    a->h3 = trk->hit[3];
    a->nhits = trk->nhits;
    a->cand = trk->cand;
    a->flags = trk->flags;
    a->tcap = tcap;
    return DS_OK;
}

hipError_t launch_clone(ds_ctx *c, const ds::CloneArgs &a, size_t lds, hipStream_t s)
{
    const int waves = CLONE_BLOCK / 64;
    const int grid = std::max(1, std::min((a.n_events + waves - 1) / waves, c->n_cu * 8));
    hipLaunchKernelGGL(ds::k_clone<CLONE_BLOCK>, dim3(grid), dim3(CLONE_BLOCK), lds, s, a);
    return hipGetLastError();
}

// The largest-first order of the batch into ws + ORDER_WS (two small launches).
hipError_t launch_order(const TrackPlan &p, hipStream_t s)
{
    ds::OrderArgs o;
    std::memset(&o, 0, sizeof(o));
    o.seed_off = p.a.seed_off;
    o.hit_off = p.a.hit_off;
    o.n = p.a.n_events;
    o.tiers = p.tiers;
    for (int k = 0; k < p.tiers; ++k) {
        o.max_seeds[k] = p.tier[k].max_seeds;
        o.max_hits[k] = p.tier[k].hcap;
    }
    while (((std::min(p.a.max_seeds, 1 << 20) + std::min(p.a.max_hits, 1 << 20) / 8) >> o.shift) >= ds::ORDER_BINS / o.tiers)
        ++o.shift;
    o.ws = p.order_ws;
    o.order = p.order_ws + ds::ORDER_WS;
    hipLaunchKernelGGL(ds::k_order_count, dim3(ds::ORDER_ROWS), dim3(ds::ORDER_BLOCK), 0, s, o);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ds::k_order_place, dim3(ds::ORDER_ROWS), dim3(ds::ORDER_BLOCK), 0, s, o);
    return hipGetLastError();
}

hipError_t run_track(ds_ctx *c, const TrackPlan &p, int mode, hipStream_t s)
{
    if (mode == DS_MODE_PER_EVENT) {
        ds::TrackArgs a = p.a;
        for (int e = 0; e < a.n_events; ++e) {
            a.ev_single = e;
            hipError_t err = launch_track(p.block, a, c->G, 1, p.lds, s);
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    }
    if (p.a.order) {
        hipError_t e = launch_order(p, s);
        if (e != hipSuccess) return e;
    }
    if (p.a.order && p.tiers > 1) {
        ds::TrackArgs a = p.a;
        a.ends = p.order_ws + ds::ORDER_ROWS * ds::ORDER_BINS;
        for (a.tier = 0; a.tier < p.tiers; ++a.tier) {
            const TrackShape &t = p.tier[a.tier];
            apply_shape(c, t, a);
            hipError_t e = launch_track(t.block, a, c->G, std::min(a.n_events, c->n_cu * t.wg_per_cu), t.L.total, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    return launch_track(p.block, p.a, c->G, p.grid, p.lds, s);
}

hipError_t run_vertex(ds_ctx *c, const VertexPlan &p, int mode, hipStream_t s)
{
    if (mode == DS_MODE_PER_EVENT) {
        ds::VertexArgs a = p.a;
        for (int e = 0; e < a.n_events; ++e) {
            a.ev_single = e;
            hipError_t err = launch_vertex(p.block, a, c->G, 1, p.lds, s);
            if (err != hipSuccess) return err;
        }
        return hipSuccess;
    }
    return launch_vertex(p.block, p.a, c->G, p.grid, p.lds, s);
}

// Argument checks of ds_process / ds_process_static (host side, before any launch).
ds_status check_process(ds_ctx *c, const ds_events *ev, const ds_tracks *trk, const ds_vertices *out, int mode)
{
    if (!c) return DS_E_ARG;
    if (!c->loaded) return DS_E_STATE;
    if (mode < DS_MODE_PER_EVENT || mode > DS_MODE_GRAPH) return DS_E_ARG;
    ds_status st = check_events(ev);
    if (st != DS_OK) return st;
    st = check_tracks(trk, ev->n_seeds, true);
    if (st != DS_OK) return st;
    if (!out || out->cap_per_event < 0 || !out->overflow || !out->flags) return DS_E_ARG;
    if (ev->n_events == 0) return DS_OK;
    if (!out->count) return DS_E_ARG;
    if (out->cap_per_event > 0 && (!out->i || !out->j || !out->x || !out->y || !out->z || !out->doca))
        return DS_E_ARG;
    return check_extras(c, out);
}

// Enqueue the whole step on s: work counters at `counters` ([0] tracking,
// [2] vertexing), the largest-first order in order_ws (null: input order).
// Nothing here allocates.  DS_MODE_GRAPH enqueues the same launches as
// DS_MODE_PERSISTENT: one fused, or tracking, the two of clone killing and
// vertexing; with largest-first order two more ahead, and up to three in place
// of the tracking one, so eight at most.  Replaying them from a cached hipGraph
// cost 25 us a call against 4 us per launch (100 events: 28.8 us a step
// replayed, 16.2 direct; 10 000 events: 394 and 383; clone killing with its
// four launches, 50 events: 86.7 and 79.7).
ds_status process_enqueue(ds_ctx *c, const ds_events *ev, const ds_tracks *trk, float score_max,
                          const ds_vertices *out, int mode, hipStream_t s, int *counters, int *order_ws)
{
    const bool ck = c->clone_kill;
    TrackPlan tp;
    ds_status st = plan_track(c, ev, trk, ck ? 0 : 1, counters, &tp);
    if (st != DS_OK) return st;
    if (mode != DS_MODE_PER_EVENT) set_order(tp, order_ws);
    VertexPlan vp;
    st = plan_vertex(c, ev, trk, score_max, out, counters, &vp);
    if (st != DS_OK) return st;
    ds::CloneArgs ca;
    size_t clds = 0;
    ds::GhostArgs ga = ghost_args(c, ev, trk);
    if (ck) {
        st = clone_args(ev, trk, &ca, &clds);
        if (st != DS_OK) return st;
    }
    if (mode != DS_MODE_PER_EVENT && c->fused_step) {
        // one launch: tracking, clone killing, ghost-killer and vertexing fused per event (events too large
        // for the clone notes beside the kept tracks: four launches)
        TrackPlan fp;
        st = plan_track(c, ev, trk, 1, counters, &fp, out->m_pipi ? 2 : 1, false, ck);
        if (st != DS_OK && !ck) return st;
        if (st == DS_OK) {
            set_order(fp, tp.order_ws);
            ds::TrackArgs &a = fp.a;
            a.score_max = score_max;
            a.vcap = out->cap_per_event;
            a.vcount = out->count;
            a.vi = out->i;
            a.vj = out->j;
            a.vx = out->x;
            a.vy = out->y;
            a.vz = out->z;
            a.vdoca = out->doca;
            a.voverflow = out->overflow;
            a.vflags = out->flags;
            a.m_pipi = out->m_pipi;
            a.m_ppi = out->m_ppi;
            a.line0 = out->line[0];
            a.line1 = out->line[1];
            a.line2 = out->line[2];
            a.line3 = out->line[3];
            a.WL = c->d_WL;
            return dev_err(run_track(c, fp, mode, s));
        }
    }
    hipError_t e = run_track(c, tp, mode, s);
    if (e == hipSuccess && ck) e = launch_clone(c, ca, clds, s);
    if (e == hipSuccess && ck) e = launch_ghost(c, ga, s);
    if (e == hipSuccess) e = run_vertex(c, vp, mode, s);
    return dev_err(e);
}

}  // namespace

extern "C" {

const char *ds_status_str(ds_status s)
{
    switch (s) {
    case DS_OK: return "DS_OK";
    case DS_E_ARG: return "DS_E_ARG: invalid argument";
    case DS_E_STATE: return "DS_E_STATE: geometry not loaded";
    case DS_E_NOMEM: return "DS_E_NOMEM: allocation failed";
    case DS_E_CAPACITY: return "DS_E_CAPACITY: size beyond library capacity";
    case DS_E_DEVICE: return "DS_E_DEVICE: HIP runtime error";
    }
    return "unknown ds_status";
}

ds_status ds_create(ds_ctx **ctx, int device)
{
    if (!ctx) return DS_E_ARG;
    *ctx = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return DS_E_ARG;
    if (hipSetDevice(device) != hipSuccess) return DS_E_DEVICE;
    ds_ctx *c = new (std::nothrow) ds_ctx();
    if (!c) return DS_E_NOMEM;
    c->device = device;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) == hipSuccess && prop.multiProcessorCount > 0)
        c->n_cu = prop.multiProcessorCount;
    ds_status sst = static_scratch(device, &c->scratch);
    if (sst != DS_OK) {
        delete c;
        return sst;
    }
    if (hipMalloc(&c->d_counters, sizeof(int) * 4 * MAX_STREAM_SLOTS) != hipSuccess) {
        delete c;
        return DS_E_NOMEM;
    }
    if (set_kernel_attributes(c->trk_waves) != hipSuccess ||
        hipMemset(c->d_counters, 0, sizeof(int) * 4 * MAX_STREAM_SLOTS) != hipSuccess) {
        (void)hipFree(c->d_counters);
        delete c;
        return DS_E_DEVICE;
    }
    *ctx = c;
    return DS_OK;
}

void ds_destroy(ds_ctx *c)
{
    if (!c) return;
    (void)hipSetDevice(c->device);
    if (c->d_W) (void)hipFree(c->d_W);
    if (c->d_Wrow) (void)hipFree(c->d_Wrow);
    if (c->d_WL) (void)hipFree(c->d_WL);
    if (c->d_counters) (void)hipFree(c->d_counters);
    for (auto &o : c->order_ws) {
        for (int k = 0; k < o.n_old; ++k) (void)hipFree(o.old[k]);
        if (o.p) (void)hipFree(o.p);
    }
    delete c;
}

ds_status ds_load_geometry(ds_ctx *c, const ds_geometry *g, const float *w, size_t nw)
{
    if (!c || !g || !w || nw != (size_t)ds::NWEIGHTS) return DS_E_ARG;
    if (g->max_l3 < 0 || g->max_l3 > ds::MAX_L3 || g->newton_iters < 0 || g->newton_iters > 16) return DS_E_ARG;
    for (int L = 0; L < 3; ++L)
        if (g->n_closest[L] < 0 || g->n_closest[L] > ds::MAX_CLOSEST) return DS_E_ARG;
    if (!(g->u_max > g->u_min) || !(g->sigma_hit > 0.0) || g->z_magnet == g->z_layer[3]) return DS_E_ARG;
    for (int L = 0; L < 3; ++L)
        if (!(g->z_layer[L] < g->z_layer[L + 1])) return DS_E_ARG;
    if (g->algorithm != 0 && g->algorithm != 1) return DS_E_ARG;
    // Dv1: at most 15 sectors (4-bit spans) and a tolerance band narrower than
    // a sector, so that a seed is compatible with at most two of them
    if (g->algorithm == 1 && (g->n_sectors < 1 || g->n_sectors > 15 || !(g->sector_h > 0.0) ||
                              !(g->sector_tol >= 0.0) || !(2.0 * g->sector_tol < g->sector_h) ||
                              !std::isfinite(g->sector_y0)))
        return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    // launches already enqueued on any stream read the resident weights: let
    // them finish before they are replaced
    if (hipDeviceSynchronize() != hipSuccess) return DS_E_DEVICE;
    ds::DevGeom G{};
    for (int L = 0; L < 4; ++L) {
        G.zl[L] = g->z_layer[L];
        G.tana[L] = g->tan_stereo[L];
        G.dz[L] = g->z_layer[L] - g->z_ref;
    }
    G.zm = g->z_magnet;
    G.zs = g->z_seed;
    G.zref = g->z_ref;
    G.mk = g->polarity * g->kick;
    G.inv_sigma2 = 1.0 / (g->sigma_hit * g->sigma_hit);
    G.inv_5sigma = 1.0 / (5.0 * g->sigma_hit);
    G.w1c0 = g->w1_c0;
    G.w1c1 = g->w1_c1;
    G.w2c0 = g->w2_c0;
    G.w2c1 = g->w2_c1;
    for (int L = 0; L < 3; ++L) G.ffac[L] = (g->z_magnet - g->z_layer[L]) / (g->z_magnet - g->z_layer[3]);
    const int masks[4] = {11, 13, 14, 15};
    for (int k = 0; k < 4; ++k) {
        double n = 0, sz = 0, szz = 0;
        for (int L = 0; L < 4; ++L)
            if ((masks[k] >> L) & 1) {
                n += 1;
                sz += G.dz[L];
                szz += G.dz[L] * G.dz[L];
            }
        G.fit_sz[k] = sz;
        G.fit_inv_det[k] = 1.0 / (n * szz - sz * sz);
        G.fit_inv_n[k] = 1.0 / n;
    }
    G.zm_ref = g->z_magnet - g->z_ref;
    G.zm_seed = g->z_magnet - g->z_seed;
    G.zref_seed = g->z_ref - g->z_seed;
    G.gc0 = g->gamma_c0;
    G.gc1 = g->gamma_c1;
    G.fp = g->fringe_polarity;
    G.doca_max = g->doca_max;
    const float thr = (float)g->doca_max + PRESCREEN_MARGIN;
    G.prescreen_r = thr;
    G.prescreen_thr2 = thr * thr;
    G.max_l3 = g->max_l3;
    for (int L = 0; L < 3; ++L) {
        G.ncl[L] = g->n_closest[L];
        G.nw[L] = std::max(g->n_closest[L], 1);
    }
    G.newton_iters = g->newton_iters;
    G.nsec = g->algorithm == 1 ? g->n_sectors : 1;
    G.sec_y0 = g->sector_y0;
    G.sec_h = g->algorithm == 1 ? g->sector_h : 1.0;
    G.sec_inv = 1.0 / G.sec_h;
    G.sec_tol = g->sector_tol;
    // the ghost-killer network is evaluated on the matrix cores: its weights go
    // to the device in the per-lane order of the MFMA operands
    std::vector<float> wm(ds::MLP_WM);
    ds::mlp_lane_layout(w, wm.data());
    if (!c->d_W && hipMalloc(&c->d_W, sizeof(float) * ds::MLP_WM) != hipSuccess) return DS_E_NOMEM;
    if (hipMemcpy(c->d_W, wm.data(), sizeof(float) * ds::MLP_WM, hipMemcpyHostToDevice) != hipSuccess)
        return DS_E_DEVICE;
    if (!c->d_Wrow && hipMalloc(&c->d_Wrow, sizeof(float) * ds::NWEIGHTS) != hipSuccess) return DS_E_NOMEM;
    if (hipMemcpy(c->d_Wrow, w, sizeof(float) * ds::NWEIGHTS, hipMemcpyHostToDevice) != hipSuccess)
        return DS_E_DEVICE;
    c->G = G;
    c->u_min = g->u_min;
    c->u_max = g->u_max;
    c->ghost_threshold = g->ghost_threshold;
    c->clone_kill = g->clone_kill != 0;
    c->algorithm = g->algorithm;
    c->loaded = true;
    return DS_OK;
}

ds_status ds_find_tracks(ds_ctx *c, const ds_events *ev, const ds_tracks *out, int mode, int fuse, void *stream)
{
    if (!c) return DS_E_ARG;
    if (!c->loaded) return DS_E_STATE;
    if (mode < DS_MODE_PER_EVENT || mode > DS_MODE_GRAPH) return DS_E_ARG;
    ds_status st = check_events(ev);
    if (st != DS_OK) return st;
    st = check_tracks(out, ev->n_seeds, fuse != 0);
    if (st != DS_OK) return st;
    if (ev->n_events == 0) return DS_OK;
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int *counters, slot;
    st = slot_for(c, stream, &counters, &slot);
    if (st != DS_OK) return st;
    TrackPlan p;
    st = plan_track(c, ev, out, fuse, counters, &p);
    if (st != DS_OK) return st;
    st = plan_order(c, slot, mode, s, p);
    if (st != DS_OK) return st;
    return dev_err(run_track(c, p, mode, s));
}

ds_status ds_ghost_kill(ds_ctx *c, const ds_events *ev, const ds_tracks *trk, void *stream)
{
    if (!c) return DS_E_ARG;
    if (!c->loaded) return DS_E_STATE;
    ds_status st = check_events(ev);
    if (st != DS_OK) return st;
    st = check_tracks(trk, ev->n_seeds, true);
    if (st != DS_OK) return st;
    if (ev->n_events == 0) return DS_OK;
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    return dev_err(launch_ghost(c, ghost_args(c, ev, trk), reinterpret_cast<hipStream_t>(stream)));
}

ds_status ds_kill_clones(ds_ctx *c, const ds_events *ev, const ds_tracks *trk, void *stream)
{
    if (!c) return DS_E_ARG;
    if (!c->loaded) return DS_E_STATE;
    ds_status st = check_events(ev);
    if (st != DS_OK) return st;
    st = check_tracks(trk, ev->n_seeds, false);
    if (st != DS_OK) return st;
    if (ev->n_events == 0) return DS_OK;
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    ds::CloneArgs a;
    size_t lds;
    st = clone_args(ev, trk, &a, &lds);
    if (st != DS_OK) return st;
    return dev_err(launch_clone(c, a, lds, reinterpret_cast<hipStream_t>(stream)));
}

int ds_candidate_slots(ds_ctx *c)
{
    if (!c || !c->loaded) return 0;
    return c->G.max_l3 * c->G.nw[0] * c->G.nw[1] * c->G.nw[2];
}

ds_status ds_score_candidates(ds_ctx *c, const ds_events *ev, const ds_candidates *out, void *stream)
{
    if (!c) return DS_E_ARG;
    if (!c->loaded) return DS_E_STATE;
    ds_status st = check_events(ev);
    if (st != DS_OK) return st;
    if (!out || !out->flags || out->capacity < 0) return DS_E_ARG;
    if (ev->n_events == 0) return DS_OK;
    const int cmax = c->G.max_l3 * c->G.nw[0] * c->G.nw[1] * c->G.nw[2];
    if (cmax <= 0) return DS_OK;
    if ((long long)out->capacity < (long long)ev->n_seeds * cmax) return DS_E_CAPACITY;
    if (ev->n_seeds > 0) {
        if (!out->seed || !out->cand || !out->nhits || !out->x || !out->y || !out->tx || !out->ty || !out->qop ||
            !out->chi2 || !out->score)
            return DS_E_ARG;
        for (int L = 0; L < 4; ++L)
            if (!out->hit[L]) return DS_E_ARG;
    }
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int *counters;
    st = slot_for(c, stream, &counters);
    if (st != DS_OK) return st;
    ds_tracks none;
    std::memset(&none, 0, sizeof(none));
    none.flags = out->flags;
    TrackPlan p;
    st = plan_track(c, ev, &none, 0, counters, &p, false, true);
    if (st != DS_OK) return st;
    p.a.cmax = cmax;
    p.a.r_seed = out->seed;
    p.a.r_cand = out->cand;
    p.a.r_nhits = out->nhits;
    p.a.r_h0 = out->hit[0];
    p.a.r_h1 = out->hit[1];
    p.a.r_h2 = out->hit[2];
    p.a.r_h3 = out->hit[3];
    p.a.r_x = out->x;
    p.a.r_y = out->y;
    p.a.r_tx = out->tx;
    p.a.r_ty = out->ty;
    p.a.r_qop = out->qop;
    p.a.r_chi2 = out->chi2;
    p.a.r_score = out->score;
    p.a.Wrow = c->d_Wrow;   // each candidate is scored where it is written
    const long long rows = (long long)ev->n_seeds * cmax;
    if (rows > 0) {
        const int grid = (int)std::min<long long>((rows + 255) / 256, (long long)c->n_cu * 16);
        hipLaunchKernelGGL(ds::k_clear_rows, dim3(grid), dim3(256), 0, s, out->nhits, rows);
        if (hipGetLastError() != hipSuccess) return DS_E_DEVICE;
    }
    return dev_err(run_track(c, p, DS_MODE_PERSISTENT, s));
}

ds_status ds_vertex(ds_ctx *c, const ds_events *ev, const ds_tracks *trk, float score_max, const ds_vertices *out,
                    int mode, void *stream)
{
    if (!c) return DS_E_ARG;
    if (!c->loaded) return DS_E_STATE;
    if (mode < DS_MODE_PER_EVENT || mode > DS_MODE_GRAPH) return DS_E_ARG;
    ds_status st = check_events(ev);
    if (st != DS_OK) return st;
    st = check_tracks(trk, ev->n_seeds, true);
    if (st != DS_OK) return st;
    if (!out || out->cap_per_event < 0 || !out->overflow || !out->flags) return DS_E_ARG;
    if (ev->n_events == 0) return DS_OK;
    if (!out->count) return DS_E_ARG;
    if (out->cap_per_event > 0 && (!out->i || !out->j || !out->x || !out->y || !out->z || !out->doca))
        return DS_E_ARG;
    st = check_extras(c, out);
    if (st != DS_OK) return st;
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int *counters;
    st = slot_for(c, stream, &counters);
    if (st != DS_OK) return st;
    VertexPlan p;
    st = plan_vertex(c, ev, trk, score_max, out, counters, &p);
    if (st != DS_OK) return st;
    return dev_err(run_vertex(c, p, mode, s));
}

ds_status ds_process(ds_ctx *c, const ds_events *ev, const ds_tracks *trk, float score_max, const ds_vertices *out,
                     int mode, void *stream)
{
    ds_status st = check_process(c, ev, trk, out, mode);
    if (st != DS_OK || ev->n_events == 0) return st;
    if (std::isnan(score_max)) score_max = (float)c->ghost_threshold;
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int *counters, slot;
    st = slot_for(c, stream, &counters, &slot);
    if (st != DS_OK) return st;
    int *order_ws = nullptr;
    if (mode != DS_MODE_PER_EVENT && c->event_order == DS_ORDER_LARGEST_FIRST && ev->n_events >= 2) {
        st = order_workspace(c, slot, ev->n_events, s, &order_ws);
        if (st != DS_OK) return st;
    }
    return process_enqueue(c, ev, trk, score_max, out, mode, s, counters, order_ws);
}

ds_status ds_process_static(ds_ctx *c, const ds_events *ev, const ds_tracks *trk, float score_max,
                            const ds_vertices *out, void *stream)
{
    ds_status st = check_process(c, ev, trk, out, DS_MODE_PERSISTENT);
    if (st != DS_OK) return st;
    if (ev->n_events > DS_STATIC_MAX_EVENTS) return DS_E_CAPACITY;
    if (ev->n_events == 0) return DS_OK;
    if (std::isnan(score_max)) score_max = (float)c->ghost_threshold;
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // the device's static array (its address, looked up at ds_create): the work
    // counters start at zero, whatever an earlier call left there (a fill
    // kernel, not a memset node, so that a caller may capture the call)
    int *sp = c->scratch;
    hipLaunchKernelGGL(ds::k_fill_i32, dim3(8), dim3(256), 0, s, sp, 0, STATIC_HDR + ds::ORDER_WS);
    if (hipGetLastError() != hipSuccess) return DS_E_DEVICE;
    int *order_ws = (c->event_order == DS_ORDER_LARGEST_FIRST && ev->n_events >= 2) ? sp + STATIC_HDR : nullptr;
    return process_enqueue(c, ev, trk, score_max, out, DS_MODE_PERSISTENT, s, sp, order_ws);
}

ds_status ds_load_lines(ds_ctx *c, const float *w, size_t nw)
{
    if (!c || !w || nw != (size_t)(4 * ds::LINE_NW)) return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    if (hipSetDevice(c->device) != hipSuccess) return DS_E_DEVICE;
    if (!c->d_WL && hipMalloc(&c->d_WL, sizeof(float) * 4 * ds::LINE_NW) != hipSuccess) return DS_E_NOMEM;
    if (hipMemcpy(c->d_WL, w, sizeof(float) * 4 * ds::LINE_NW, hipMemcpyHostToDevice) != hipSuccess)
        return DS_E_DEVICE;
    return DS_OK;
}

ds_status ds_set_launch(ds_ctx *c, int kernel, int block, int wg_per_cu, int bins)
{
    if (!c || (kernel != 0 && kernel != 1)) return DS_E_ARG;
    if (block != 0 && block != 64 && block != 128 && block != 192 && block != 256 && block != 512) return DS_E_ARG;
    if (kernel == 1 && block == 192) return DS_E_ARG;   // tracking only
    if (wg_per_cu < 0 || wg_per_cu > 16) return DS_E_ARG;
    if (bins != 0 && (kernel != 0 || bins < 64 || bins > 4096 || (bins & (bins - 1)))) return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    Launch &L = kernel == 0 ? c->trk : c->vtx;
    Launch n = L;
    if (block) n.block = block;
    if (wg_per_cu) n.wg_per_cu = wg_per_cu;
    if (bins) n.bins = bins;
    if (kernel == 0) c->trk_set |= (block ? SET_BLOCK : 0) | (wg_per_cu ? SET_WG : 0) | (bins ? SET_BINS : 0);
    L = n;
    return DS_OK;
}

ds_status ds_reset_launch(ds_ctx *c, int kernel)
{
    if (!c || (kernel != 0 && kernel != 1)) return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    if (kernel == 0) {
        c->trk = TRACK_LAUNCH;
        c->trk_set = 0;
    } else {
        c->vtx = VERTEX_LAUNCH;
    }
    return DS_OK;
}

ds_status ds_set_event_order(ds_ctx *c, int order)
{
    if (!c || (order != DS_ORDER_INPUT && order != DS_ORDER_LARGEST_FIRST)) return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    c->event_order = order;
    return DS_OK;
}

ds_status ds_set_step_fusion(ds_ctx *c, int fused)
{
    if (!c || (fused != 0 && fused != 1)) return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    c->fused_step = fused;
    return DS_OK;
}

ds_status ds_get_step_fusion(ds_ctx *c, int *fused)
{
    if (!c || !fused) return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    *fused = c->fused_step;
    return DS_OK;
}

ds_status ds_get_event_order(ds_ctx *c, int *order)
{
    if (!c || !order) return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    *order = c->event_order;
    return DS_OK;
}

ds_status ds_get_launch(ds_ctx *c, int kernel, int *block, int *wg_per_cu, int *bins)
{
    if (!c || (kernel != 0 && kernel != 1) || !block || !wg_per_cu || !bins) return DS_E_ARG;
    std::lock_guard<std::mutex> lock(c->mu);
    const Launch &L = kernel == 0 ? c->trk : c->vtx;
    *block = L.block;
    *wg_per_cu = L.wg_per_cu;
    *bins = L.bins;
    return DS_OK;
}

}  // extern "C"
