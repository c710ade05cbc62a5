// Device code of the Downstream tracking + two-track vertexing library for
// gfx950 (MI355X).  Included once, by ds_api.hip.
//
// Method (Kholoimov et al., arXiv:2503.13092):
//   * magnet-point (single kink) extrapolation of SciFi seeds to the UT
//     ("Algorithm Design", eq. 1 and the magnet-point text after it);
//   * Dv0 search: a first window in UTbX, then for each of up to 10 closest
//     UTbX hits a refined line through the hit and the magnet point, with the
//     closest UTaX hit and the two closest UTaU and UTbV hits;
//   * candidates scored by a least-squares chi2, best one per seed;
//   * ghost-killer MLP ("Ghost-Killer Neural Network");
//   * two-track vertexing: eq. 3/eq. 4 trajectories, Newton-Raphson PCA
//     ("Vertexing Two Downstream Tracks").
//
// Numerics.  Window searches, fits and vertex refinement run in float64 (on
// CDNA4 the float64 FMA rate equals the unpacked float32 rate), in the frame
// of the seed's un-kicked straight line x_S(z): a hit's residual is
// rho = u - c_L with c_L = x_S(z_L) - y(z_L)*tan(alpha_L).  In that frame the
// kinked prediction is MP*K*q/p*(z_M - z) and the refined line through a
// UTbX hit and the magnet point is rho_3*(z_M - z)/(z_M - z_3), because x_S
// passes through the magnet point.  The ghost-killer runs in float32 on
// features computed in float64 from the stored float32 track.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ds {

constexpr int NF = 17, NH1 = 32, NH2 = 16;
constexpr int NWEIGHTS = NH1 * NF + NH1 + NH2 * NH1 + NH2 + NH2 + 1;  // 1121
// Per-lane weight words of mlp_score_wave (lane l, group g = l / 16, n = l % 16):
// [u * 5 + s] = W1[16 u + n][4 s + g] (b1 in input column 17, zeros past it),
// [MLP_A2 + 4 u + r] = W2[n][16 u + 4 g + r], [MLP_B2 + r] = b2[4 g + r],
// [MLP_W3 + r] = W3[4 g + r], [MLP_B3] = b3; stored as float4 q of lane l at
// (q * 64 + l).
constexpr int MLP_K1 = 20, MLP_A2 = 10, MLP_B2 = 18, MLP_W3 = 22, MLP_B3 = 26;
constexpr int MLP_LANE_WORDS = 28;
constexpr int MLP_WM = 64 * MLP_LANE_WORDS;

// Host side: the per-lane order from the row-major parameters W1, b1, W2, b2, W3, b3.
inline void mlp_lane_layout(const float *w, float *wm)
{
    const float *W1 = w, *b1 = W1 + NH1 * NF, *W2 = b1 + NH1, *b2 = W2 + NH2 * NH1, *W3 = b2 + NH2, *b3 = W3 + NH2;
    for (int l = 0; l < 64; ++l) {
        const int g = l / 16, n = l % 16;
        float v[MLP_LANE_WORDS] = {};
        for (int u = 0; u < 2; ++u)
            for (int s = 0; s < MLP_K1 / 4; ++s) {
                const int j = 16 * u + n, k = 4 * s + g;
                v[u * (MLP_K1 / 4) + s] = k < NF ? W1[j * NF + k] : (k == NF ? b1[j] : 0.0f);
            }
        for (int u = 0; u < 2; ++u)
            for (int r = 0; r < 4; ++r) v[MLP_A2 + 4 * u + r] = W2[n * NH1 + 16 * u + 4 * g + r];
        for (int r = 0; r < 4; ++r) {
            v[MLP_B2 + r] = b2[4 * g + r];
            v[MLP_W3 + r] = W3[4 * g + r];
        }
        v[MLP_B3] = b3[0];
        for (int k = 0; k < MLP_LANE_WORDS; ++k) wm[((k / 4) * 64 + l) * 4 + k % 4] = v[k];
    }
}

constexpr int MAX_L3 = 16;
constexpr int MAX_CLOSEST = 2;
constexpr int MAX_ITEMS = 8176;   // 13-bit item numbers
constexpr int F_BAD_OFFSETS = 1, F_CAPACITY = 2, F_NONFINITE = 4;
constexpr int LINE_NF = 12, LINE_NH = 32;
constexpr int LINE_NW = LINE_NH * LINE_NF + LINE_NH + LINE_NH + 1;  // 449 per network

// Geometry after host-side preprocessing (passed by value as a kernel argument).
struct DevGeom {
    double zl[4], tana[4];
    double zm, zs, zref;
    double mk;            // polarity * kick
    double inv_sigma2;
    double inv_5sigma;    // residual feature scale 1/(5 sigma)
    double w1c0, w1c1, w2c0, w2c1;
    double ffac[3];       // (z_M - z_L)/(z_M - z_3)
    double dz[4];         // z_L - z_ref
    // least-squares constants of the four valid layer sets {0,1,3}, {0,2,3}, {1,2,3}, {0,1,2,3}
    double fit_sz[4], fit_inv_det[4], fit_inv_n[4];
    double zm_ref, zm_seed, zref_seed;   // z_M - z_ref, z_M - z_seed, z_ref - z_seed
    double gc0, gc1, fp;                 // eq. 3
    double doca_max;
    float prescreen_r, prescreen_thr2;   // doca_max + margin and its square, for the float32 pair prescreen
    int max_l3;
    int ncl[3];
    int nw[3];                           // max(ncl, 1): radix of the candidate index
    int newton_iters;
    // Dv1 Y sectors: band k = [sec_y0 + k sec_h, sec_y0 + (k + 1) sec_h), k < nsec
    double sec_y0, sec_h, sec_inv, sec_tol;   // sec_inv = 1 / sec_h
    int nsec;
};

struct TrackArgs {
    int n_events, n_seeds, n_hits, max_seeds, max_hits;
    const int *seed_off;
    const float *sx, *sy, *stx, *sty, *sqop;
    const int *hit_off;
    const float *hu;
    float *x, *y, *tx, *ty, *qop, *chi2, *score;
    int *h0, *h1, *h2, *h3, *nhits, *cand, *flags;
    int *counter;        // events taken beyond the first of each workgroup (persistent launch)
    const float *W;      // ghost-killer parameters (resident)
    int fuse_mlp;
    int fine;            // Dv0: bins that the context asks for per bin of the launch (a power of two)
    int clone;           // fused vertexing: clones are killed between an event's tracks and their scores
    int ev_single;       // >= 0: this launch processes only that event
    int hcap;            // LDS hit capacity of the launch
    int scap;            // LDS capacity for the seeds of one chunk (at most the workgroup size)
    int icap;            // LDS capacity for the (seed, UTbX hit) items of one seed chunk
    int wcap;            // first-window hits (Dv0) or axial triplets (Dv1) of one seed beyond which it is
                         // truncated and flagged
    // candidate-scoring mode: rows [n_seeds * cmax], row = seed * cmax + candidate index
    int cmax;
    int *r_seed, *r_cand, *r_nhits, *r_h0, *r_h1, *r_h2, *r_h3;
    float *r_x, *r_y, *r_tx, *r_ty, *r_qop, *r_chi2, *r_score;
    const float *Wrow;   // candidate rows: the ghost-killer weights W1, b1, W2, b2, W3, b3 row-major
    // fused vertexing (ds_process): kept tracks of an event go to LDS as they are written
    int tcap;            // LDS capacity for kept tracks of one event
    float score_max;
    int vcap;
    int *vcount, *vi, *vj;
    float *vx, *vy, *vz, *vdoca;
    int *voverflow, *vflags;
    float *m_pipi, *m_ppi, *line0, *line1, *line2, *line3;
    const float *WL;
    int nb;              // buckets of layers 0-2: u bins (Dv0) or sectors x u bins + 1 (Dv1)
    int nbu;             // u bins (per sector) of layers 0-2
    float inv_bw, bin_off;    // bin = floor(u * inv_bw + bin_off), clamped to [0, nbu)
    int nb3, nbu3;       // the same for layer 3 (UTbX), stored after layers 0-2; Dv1 reads it
    float inv_bw3, bin_off3;  // by whole sectors only, so it has one u bin per sector
    const uint8_t *hsec; // Dv1: Y sector of every hit (null for Dv0)
    int map_ints;        // Dv1: LDS words of the map of UTaX, words per sector and its u bins (32 to a word)
    int map_words;
    float map_inv, map_off, map_reach, map_range;
    const int *order;    // persistent launch: events in this order (a permutation), null = input order
    const int *ends;     // largest-first order in classes: their ends in it
    int tier;            // the class of this launch (-1: all events)
};

struct GhostArgs {
    int n_events, n_seeds, n_hits;
    const int *seed_off;
    const float *sx, *sy, *stx, *sty, *sqop;
    const int *hit_off;
    const float *hu;
    const float *x, *y, *tx, *ty, *qop, *chi2;
    const int *h0, *h1, *h2, *h3, *nhits;
    float *score;
    int *flags;
    const float *W;
};

struct CloneArgs {
    int n_events, n_seeds, max_seeds;
    const int *seed_off;
    float *x, *y, *tx, *ty, *qop, *chi2, *score;
    int *h0, *h1, *h2, *h3, *nhits, *cand, *flags;
    int tcap;            // LDS capacity (seeds) per wavefront
};

struct VertexArgs {
    int n_events, n_seeds, max_seeds;
    const int *seed_off;
    const float *sqop;
    const float *x, *y, *tx, *ty, *qop, *score;
    const int *nhits;
    float score_max;
    int vcap;
    int *vcount, *vi, *vj;
    float *vx, *vy, *vz, *vdoca;
    int *voverflow, *flags;
    int *counter;        // events taken beyond the first of each workgroup (persistent launch)
    int ev_single;
    int tcap;            // LDS capacity for kept tracks
    // after-vertex outputs (nullable): masses (MeV) and the four trigger-line scores
    float *m_pipi, *m_ppi, *line0, *line1, *line2, *line3;
    const float *WL;     // trigger-line networks, 4 x (W1[32][12], b1[32], W2[32], b2)
};

// The tracking kernel's arguments as one block.
struct TrackKernArgs {
    TrackArgs a;
    DevGeom G;
};

// ----------------------------------------------------------------- helpers

// The launch's argument block, reached through an opaque copy of its address.
// Loads through the returned reference cannot move above the call, so a
// persistent kernel re-reads uniform arguments (scalar loads) in the phase that
// uses them instead of keeping all of them live, and spilled to vector lanes,
// across its whole loop.
template <typename T>
__device__ __forceinline__ const T &kernel_args()
{
    typedef const __attribute__((address_space(4))) T *cptr;
    cptr p = (cptr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const T *)p;
}

// The lane's index in its workgroup, opaque: what is derived from it is
// computed in the phase that uses it.  Hoisted out of the persistent loop,
// those addresses held a quarter of the registers and spilled.
__device__ __forceinline__ int fresh_tid()
{
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// A value that every lane holds alike (read from LDS, say), made known to the
// compiler as one: branches on it are then scalar.  Event and chunk counts
// taken as lane values made the persistent loop's branches masked ones, with
// some thirty registers carried around it for values no lane needed.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Workgroup barrier ordering LDS traffic only: unlike __syncthreads it does not
// wait for the wave's outstanding global stores.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive sum over the 64 lanes of a wavefront, in lane order: four doubling
// row shifts within rows of 16 lanes, then the row broadcasts of lanes 15 and
// 31 (DPP, no LDS traffic).  Lanes outside a shift's source read 0.
__device__ __forceinline__ int wave_inclusive_sum(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2, 3
    return x;
}

template <int BLOCK>
__device__ __forceinline__ int block_exclusive_scan(int v, int *s_wsum, int *total)
{
    const int tid = fresh_tid(), lane = tid & 63, wid = tid >> 6;
    const int x = wave_inclusive_sum(v);
    if (lane == 63) s_wsum[wid] = x;
    lds_barrier();
    int off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w) {
        int s = s_wsum[w];
        off += (w < wid) ? s : 0;
        tot += s;
    }
    lds_barrier();
    *total = uniform(tot);
    return off + x - v;
}

// Bin of u: floor(u * inv + off) clamped to [0, top], one rounding and so
// monotone in u (the same function for hits and window edges).
struct Bins {
    float inv, off, top;
};

__device__ __forceinline__ int bin_of(const Bins &b, float u)
{
    return (int)__builtin_amdgcn_fmed3f(fmaf(u, b.inv, b.off), 0.0f, b.top);
}

// A refined window's parameters (a launch's, read once per phase: re-read from
// the argument segment in its loop they cost three scalar round trips per item).
struct WindowArgs {
    double w2c0, w2c1;
    int nb, nbu, nsec;
    Bins bins;
};

__device__ __forceinline__ bool finite5(float a, float b, float c, float d, float e)
{
    return isfinite(a) && isfinite(b) && isfinite(c) && isfinite(d) && isfinite(e);
}

// Window order of hits: (|u - m|, u, index within the layer run), lexicographic.
__device__ __forceinline__ bool key_less(double da, float ua, int ia, double db, float ub, int ib)
{
    return da < db || (da == db && (ua < ub || (ua == ub && ia < ib)));
}

// Window order of the hit at LDS position p (distance d, coordinate u) against
// the kept hit at position pk (distance dk; pk < 0: empty slot).
__device__ __forceinline__ bool before(const float *hu_s, const uint16_t *hidx_s, double d, float u, int p, double dk, int pk)
{
    if (d != dk || pk < 0) return d < dk || pk < 0;
    const float uk = hu_s[pk];
    if (u != uk) return u < uk;
    return hidx_s[p] < hidx_s[pk];
}

// The window's bin bounds in float32: m and W rounded (errors below 1e-4 mm
// for |m| < 2000 mm) and widened by 1e-3 mm, so the buckets always cover
// [m - W, m + W] (a superset: membership is decided on |u - m| <= W in float64).
__device__ __forceinline__ void window_bins(const Bins &b, double m, double W, int &b_lo, int &b_hi)
{
    const float mf = (float)m, wf = (float)W + 1e-3f;
    b_lo = bin_of(b, mf - wf);
    b_hi = bin_of(b, mf + wf);
}

// LDS positions [p_lo, p_hi) of the buckets of `layer` covering [m - W, m + W]
// (a superset of the window: membership is decided on |u - m| <= W).
__device__ __forceinline__ void bin_range(const uint16_t *E, int layer, const WindowArgs &w, double m, double W, int &p_lo,
                                 int &p_hi)
{
    int b_lo, b_hi;
    window_bins(w.bins, m, W, b_lo, b_hi);
    p_lo = E[layer * w.nb + b_lo];
    p_hi = E[layer * w.nb + b_hi + 1];
}

__device__ __forceinline__ Bins track_bins(const TrackArgs &a) { return Bins{a.inv_bw, a.bin_off, (float)(a.nbu - 1)}; }

// LDS range of the UTbX buckets covering [m - W, m + W], cut down around m
// where it holds many more than the `most` closest hits that are used: the
// smallest run of buckets b(m) - r .. b(m) + r with that many hits bounds their
// distance by r + 1 bucket widths, so buckets b(m) -+ (r + 2) hold every hit
// that can be among them (the wide training windows of 100 mm: 14 hits a seed
// instead of 70 at 600 hits per layer).  Not at the ends, whose buckets also
// hold the hits beyond the binned range, and not for ranges beyond wcap, whose
// seeds may have to be flagged.
__device__ __forceinline__ void first_window_range(const uint16_t *E, const TrackArgs &a, int most, double m, double W,
                                                   int &p_lo, int &p_hi)
{
    const int nb = a.nb;
    int b_lo, b_hi;
    const Bins bins = track_bins(a);
    window_bins(bins, m, W, b_lo, b_hi);
    const uint16_t *E3 = E + 3 * nb;
    p_lo = E3[b_lo];
    p_hi = E3[b_hi + 1];
    if (p_hi - p_lo <= 2 * most || p_hi - p_lo > a.wcap) return;
    const int b = bin_of(bins, (float)m);
    int r = 0;
    while (b - r > b_lo && b + r < b_hi && (int)E3[b + r + 1] - (int)E3[b - r] < most) ++r;
    if (b - r - 2 <= b_lo || b + r + 2 >= b_hi) return;
    p_lo = E3[b - r - 2];
    p_hi = E3[b + r + 3];
}

// The bins that the context asks for, where the launch takes wider ones.
__device__ __forceinline__ Bins fine_bins(const TrackArgs &a)
{
    return Bins{(float)a.fine * a.inv_bw, (float)a.fine * a.bin_off, (float)(a.fine * a.nbu - 1)};
}

// The first `n` hits inside the first window |u - m| <= W of a range [p_lo, p_hi)
// that holds more, into list[0 .. n) as d0 + position, in the order of the bins
// that the context asks for: all hits of the launch's bins before the one that
// holds the n-th, and of that one by its parts.  (A seed beyond its limit, one
// lane: which hits it keeps must not depend on the launch's bins.)
__device__ __forceinline__ void list_first(const float *hu_s, const uint16_t *E, const TrackArgs &a, double m, double W,
                                           int p_lo, int p_hi, int n, uint32_t d0, uint32_t *list)
{
    const Bins fb = fine_bins(a);
    auto inside = [&](int p) { return fabs((double)hu_s[p] - m) <= W; };
    int last = p_lo;
    for (int k = 0; last < p_hi; ++last) {
        k += inside(last) ? 1 : 0;
        if (k == n) break;
    }
    const int b = bin_of(track_bins(a), hu_s[last]);
    const int q_lo = max(p_lo, (int)E[3 * a.nb + b]), q_hi = min(p_hi, (int)E[3 * a.nb + b + 1]);
    int w = 0;
    for (int p = p_lo; p < q_lo; ++p)
        if (inside(p)) list[w++] = d0 + (uint32_t)p;
    for (int part = a.fine * b; w < n && part != INT_MAX;) {
        int next = INT_MAX;
        for (int p = q_lo; p < q_hi; ++p) {
            if (!inside(p)) continue;
            const int f = bin_of(fb, hu_s[p]);
            if (f == part && w < n) list[w++] = d0 + (uint32_t)p;
            if (f > part) next = min(next, f);
        }
        part = next;
    }
}

// Candidate key for the per-seed reduction: more hits first, then lower chi2
// (non-negative double bits are monotone; the 8 lowest mantissa bits are
// dropped), then lower candidate index.
__device__ __forceinline__ unsigned long long pack_key(int n, double chi2, int c)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(chi2);
    return ((unsigned long long)(4 - n) << 63) | ((b >> 8) << 7) | (unsigned long long)c;
}

struct SeedConst {
    double c[4];     // c_L = x_S(z_L) - y(z_L) tan(alpha_L)
    float q;         // seed q/p (window widths and the kinked prediction)
    uint16_t lo, hi; // LDS range of the UTbX buckets covering the first window
};

// Least-squares constants of the four valid layer sets (masks 11, 13, 14, 15)
// as an LDS table: a lane's set is read with three 8-byte loads, where
// selecting it from scalar registers took 18 vector instructions.
constexpr int ROW_QUEUE = 128;   // candidates a wavefront queues for fitting: below 64 left over and 64 more
constexpr int FIT_TAB = 12;   // sum of dz, 1/det of the normal equations, 1/n, four sets each

__device__ __forceinline__ void fit_table(const DevGeom &G, double *tab)
{
    const int t = threadIdx.x;
    if (t < 4) {
        tab[t] = G.fit_sz[t];
        tab[4 + t] = G.fit_inv_det[t];
        tab[8 + t] = G.fit_inv_n[t];
    }
}

// Straight-line least squares rho_L ~ alpha + beta dz_L over the layer set
// `mask`; rho_L must be 0 for a layer outside the set (it then adds nothing to
// the sums, and its weight 0 keeps it out of chi2).
__device__ __forceinline__ void fit_set(const DevGeom &G, const double *tab, int mask, const double rho[4], double &alpha,
                               double &beta, double &chi2)
{
    const int k = (mask == 15) ? 3 : (mask == 14) ? 2 : (mask == 13) ? 1 : 0;
    const double f_sz = tab[k], f_idet = tab[4 + k], f_in = tab[8 + k], f_n = (mask == 15) ? 4.0 : 3.0;
    double sr = 0.0, szr = 0.0;
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        sr += rho[L];
        szr = fma(G.dz[L], rho[L], szr);
    }
    beta = (f_n * szr - f_sz * sr) * f_idet;
    alpha = (sr - beta * f_sz) * f_in;
    double c2 = 0.0;
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        const double r = rho[L] - alpha - beta * G.dz[L];
        c2 = fma(r, r * (((mask >> L) & 1) ? 1.0 : 0.0), c2);
    }
    chi2 = c2 * G.inv_sigma2;
}

// ------------------------------------------------------------ ghost-killer

// Features of a stored track (float32 values), its seed and its hits.
__device__ __forceinline__ void ghost_features(const DevGeom &G, float xf, float yf, float txf, float tyf, float qf,
                                      float c2f, int nh, float sxf, float syf, float stxf, float styf, float sqf,
                                      const float hu4[4], int hasmask, float f[NF])
{
    f[0] = xf * 1e-3f;
    f[1] = yf * 1e-3f;
    f[2] = txf * (1.0f / 0.3f);
    f[3] = tyf * (1.0f / 0.3f);
    f[4] = qf * 2.0f;
    f[5] = c2f * 0.1f;
    f[6] = ((float)nh - 3.5f) * 2.0f;
    f[7] = sxf * (1.0f / 3000.0f);
    f[8] = syf * (1.0f / 3000.0f);
    f[9] = stxf * 2.0f;
    f[10] = styf * 2.0f;
    f[11] = sqf * 2.0f;
    const double x = xf, y = yf, tx = txf, ty = tyf;
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        double r = 0.0;
        if ((hasmask >> L) & 1) {
            double yl = fma(ty, G.dz[L], y);
            double xhat = fma(yl, G.tana[L], (double)hu4[L]);
            r = (xhat - fma(tx, G.dz[L], x)) * G.inv_5sigma;
        }
        f[12 + L] = (float)r;
    }
    double xm_trk = fma(tx, G.zm_ref, x);
    double xm_seed = fma((double)stxf, G.zm_seed, (double)sxf);
    f[16] = (float)(xm_trk - xm_seed);
}

// Read-only, wave-uniform parameters: loads through the constant address
// space become scalar loads and the weights feed the FMAs as SGPR operands.
typedef const __attribute__((address_space(4))) float cfloat;

// The ghost-killer network of one lane on the vector ALUs, its weights read
// through the scalar cache (the same for every lane): for the candidate rows,
// each scored where its lane writes it (fit_rows has up to 64 of them at once;
// the matrix-core network would sum them in another order).  Hidden layer 1 is
// consumed as it is produced (h2 accumulates over it in unit order).
__device__ __forceinline__ float mlp_score_lane(const float *Wg, const float f[NF])
{
    asm volatile("" : "+s"(Wg));   // keeps the weight loads beside their uses
    cfloat *W1 = (cfloat *)(Wg), *b1 = W1 + NH1 * NF, *W2 = b1 + NH1, *b2 = W2 + NH2 * NH1, *W3 = b2 + NH2,
           *b3 = W3 + NH2;
    float h2[NH2];
#pragma unroll
    for (int k = 0; k < NH2; ++k) h2[k] = b2[k];
#pragma unroll
    for (int j = 0; j < NH1; ++j) {
        float z = b1[j];
#pragma unroll
        for (int k = 0; k < NF; ++k) z = fmaf(W1[j * NF + k], f[k], z);
        const float h = fmaxf(z, 0.0f);
#pragma unroll
        for (int k = 0; k < NH2; ++k) h2[k] = fmaf(W2[k * NH1 + j], h, h2[k]);
    }
    float z = b3[0];
#pragma unroll
    for (int k = 0; k < NH2; ++k) z = fmaf(W3[k], fmaxf(h2[k], 0.0f), z);
    return 1.0f / (1.0f + __expf(-z));
}

// The ghost-killer network ("Ghost-Killer Neural Network": 17 inputs, ReLU
// hidden layers of 32 and 16, sigmoid output) of a wavefront's 64 rows, one
// row per lane, on the matrix cores.  Both hidden layers are products
// H^T = W X^T of v_mfma_f32_16x16x4_f32 tiles: 16 units x 16 rows per tile,
// 4 inputs per step.  In a tile, lane l holds row (l % 16) of its block and
// input / unit index 4 (l / 16) + r, so a lane's own 17 features are first
// transposed across the four 16-lane groups (permlane swaps), and the layer-1
// output is already in the layer-2 operand layout.  The weights come in the
// per-lane order built by mlp_lane_layout.  Every output element is the same
// sequence of operations wherever its row sits, so a track's score does not
// depend on its lane.
typedef float f32x4 __attribute__((ext_vector_type(4)));

// lanes 32..63 of a <-> lanes 0..31 of b
__device__ __forceinline__ void lane_swap32(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// odd 16-lane groups of a <-> even 16-lane groups of b
__device__ __forceinline__ void lane_swap16(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// This lane's weight words of mlp_score_wave.
__device__ __forceinline__ void mlp_lane_weights(const float *Wm, float w[MLP_LANE_WORDS])
{
    const int lane = fresh_tid() & 63;
    const float4 *W4 = reinterpret_cast<const float4 *>(Wm);
#pragma unroll
    for (int q = 0; q < MLP_LANE_WORDS / 4; ++q) {
        const float4 v = W4[q * 64 + lane];
        w[4 * q] = v.x;
        w[4 * q + 1] = v.y;
        w[4 * q + 2] = v.z;
        w[4 * q + 3] = v.w;
    }
}

// The network on 16 rows already in the MFMA layout: x[s] holds, in 16-lane
// group j, input 4 s + j of row l % 16 (inputs past the 17 features: the bias
// column 1, then zeros; all zeros for rows without a track).  All 64 lanes
// call it together; every group gets the rows' scores.
__device__ __forceinline__ float mlp_block(const float w[MLP_LANE_WORDS], const float x[MLP_K1 / 4])
{
    f32x4 h[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) h[u] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < MLP_K1 / 4; ++s)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            h[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u * (MLP_K1 / 4) + s], x[s], h[u], 0, 0, 0);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) h[u][r] = fmaxf(h[u][r], 0.0f);
    f32x4 o = f32x4{w[MLP_B2], w[MLP_B2 + 1], w[MLP_B2 + 2], w[MLP_B2 + 3]};
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) o = __builtin_amdgcn_mfma_f32_16x16x4f32(w[MLP_A2 + 4 * u + r], h[u][r], o, 0, 0, 0);
    float p = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) p = fmaf(w[MLP_W3 + r], fmaxf(o[r], 0.0f), p);
    // sum over the four groups: (g0 + g2) + (g1 + g3), in every group
    float c = p, d = p;
    lane_swap32(c, d);
    const float p2 = c + d;
    c = p2;
    d = p2;
    lane_swap16(c, d);
    const float z = c + d + w[MLP_B3];
    return 1.0f / (1.0f + __expf(-z));
}

// The network on each lane's own 17 features f (registers).  All 64 lanes
// must call it together (wave-uniform control flow).  Lanes with row == false
// contribute zeros; every lane gets its own row's score.
__device__ __forceinline__ float mlp_score_wave(const float w[MLP_LANE_WORDS], const float f[NF], bool row)
{
    const unsigned long long rows = __ballot(row);
    // layer-1 inputs padded to 20: the features, 1 (the bias column), zeros
    float x[MLP_K1];
#pragma unroll
    for (int k = 0; k < MLP_K1; ++k) x[k] = (row && k < NF) ? f[k] : (row && k == NF) ? 1.0f : 0.0f;
    // per step s, (register 4s + j, group b) -> (register 4s + b, group j): then
    // x[4s + b] holds, in group j, input 4s + j of the row of lane 16 b + l % 16
#pragma unroll
    for (int s = 0; s < MLP_K1 / 4; ++s) {
        lane_swap32(x[4 * s], x[4 * s + 2]);
        lane_swap32(x[4 * s + 1], x[4 * s + 3]);
        lane_swap16(x[4 * s], x[4 * s + 1]);
        lane_swap16(x[4 * s + 2], x[4 * s + 3]);
    }
    float score = 0.5f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if (((rows >> (16 * b)) & 0xffffull) == 0) continue;   // no row in this block
        const float xb[MLP_K1 / 4] = {x[b], x[4 + b], x[8 + b], x[12 + b], x[16 + b]};
        const float v = mlp_block(w, xb);
        score = ((threadIdx.x & 63) >> 4) == b ? v : score;
    }
    return score;
}

// Features of 16 rows in LDS, in the operand layout: feature k of row r of a
// block at T[16 k + r], so that group j's lanes read input 4 s + j of the 16
// rows as consecutive words.
constexpr int MLP_TILE = NF * 16;   // floats per block

__device__ __forceinline__ void mlp_tile_store(float *T, int row, const float f[NF])
{
    T += (row >> 4) * MLP_TILE + (row & 15);
#pragma unroll
    for (int k = 0; k < NF; ++k) T[16 * k] = f[k];
}

// The network on a block's tile T, its first `rows` rows (1 to 16); all 64
// lanes together.  The scores of the rows replace the first feature.
__device__ __forceinline__ void mlp_score_tile(const float w[MLP_LANE_WORDS], float *T, int rows)
{
    const int lane = fresh_tid() & 63, grp = lane >> 4, r = lane & 15;
    const bool row = r < rows;
    float x[MLP_K1 / 4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = row ? T[16 * (4 * s + grp) + r] : 0.0f;
    // inputs 16..19: feature 16 (group 0), the bias column (group 1), zeros
    const float v = T[16 * 16 + r];
    x[4] = !row ? 0.0f : grp == 0 ? v : (grp == 1 ? 1.0f : 0.0f);
    const float score = mlp_block(w, x);
    if (grp == 0 && row) T[r] = score;   // (this wavefront's reads are done: its LDS operations complete in order)
}

// The network on the workgroup's rows, at most one per lane (features f),
// gathered to dense rows in T; the 16-row blocks are shared out to all
// wavefronts.  T may lie over data that every lane has read.  The lane's score.
template <int BLOCK>
__device__ __forceinline__ float mlp_score_rows(const float *W, float *T, int *s_wsum, bool row, const float f[NF])
{
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned long long rm = __ballot(row);
    if (lane == 0) s_wsum[wave] = __popcll(rm);
    lds_barrier();
    int first = 0, n = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / 64; ++w) {
        const int c = uniform(s_wsum[w]);
        first += w < wave ? c : 0;
        n += c;
    }
    const int r = first + __builtin_amdgcn_mbcnt_hi((unsigned)(rm >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)rm, 0));
    if (row) mlp_tile_store(T, r, f);
    float mw[MLP_LANE_WORDS];
    mlp_lane_weights(W, mw);   // (in flight at the barrier)
    lds_barrier();
    for (int b = wave; 16 * b < n; b += BLOCK / 64) mlp_score_tile(mw, T + b * MLP_TILE, min(16, n - 16 * b));
    lds_barrier();
    return row ? T[(r >> 4) * MLP_TILE + (r & 15)] : 0.0f;
}

// ------------------------------------------------------------------ track

__device__ __forceinline__ void write_empty_track(const TrackArgs &a, int i)
{
    if (!a.x) return;  // candidate-scoring mode writes no track slots
    a.x[i] = 0.0f;
    a.y[i] = 0.0f;
    a.tx[i] = 0.0f;
    a.ty[i] = 0.0f;
    a.qop[i] = 0.0f;
    a.chi2[i] = 0.0f;
    if (a.fuse_mlp) a.score[i] = 0.0f;
    a.h0[i] = -1;
    a.h1[i] = -1;
    a.h2[i] = -1;
    a.h3[i] = -1;
    a.nhits[i] = 0;
    if (a.cand) a.cand[i] = -1;
}

// First-window centre in UTbX: the kinked prediction of the seed.  One
// expression for every use, so that membership tests agree bit for bit.
__device__ __forceinline__ double window1_centre(const DevGeom &G, double c3, double q)
{
    return fma(G.mk * q, G.zm - G.zl[3], c3);
}

// Seed constants of the residual frame.
__device__ __forceinline__ bool seed_frame(const DevGeom &G, float fsx, float fsy, float fstx, float fsty, float fsq,
                                  SeedConst &sc)
{
    if (!finite5(fsx, fsy, fstx, fsty, fsq)) return false;
    const double sx = fsx, sy = fsy, stx = fstx, sty = fsty;
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        const double dzs = G.zl[L] - G.zs;
        const double xs = fma(stx, dzs, sx);
        const double yl = fma(sty, dzs, sy);
        sc.c[L] = fma(-yl, G.tana[L], xs);
    }
    sc.q = fsq;
    sc.lo = sc.hi = 0;
    return true;
}

// ------------------------------------------------------------------ Dv1

// Y sectors compatible with height y: those whose band
// [y0 + k h, y0 + (k + 1) h) overlaps [y - tol, y + tol]; klo > khi (15, 0)
// when none does.  The same floor as the definition.
__device__ __forceinline__ void sector_range(const DevGeom &G, double y, int &klo, int &khi)
{
    // a multiplication by 1/h stands in for the division except beside a band boundary, where its
    // rounding could tell (eight float64 divisions per seed were a third of the staging time)
    auto bands = [&](double d) {
        const double q = d * G.sec_inv;
        return fabs(q - rint(q)) < 1e-9 ? d / G.sec_h : q;
    };
    const double a = bands(y - G.sec_tol - G.sec_y0);
    const double b = bands(y + G.sec_tol - G.sec_y0);
    const double fa = floor(a), fb = floor(b), top = (double)(G.nsec - 1);
    if (fb < 0.0 || fa > top) {
        klo = 15;
        khi = 0;
        return;
    }
    klo = fa < 0.0 ? 0 : (int)fa;
    khi = fb > top ? G.nsec - 1 : (int)fb;
}

// Dv1 keeps the four layers' sector ranges in the seed constants, 4 + 4 bits
// per layer (lo: layers 0 and 1, hi: layers 2 and 3).
__device__ __forceinline__ void seed_sectors(const DevGeom &G, float fsy, float fsty, SeedConst &sc)
{
    uint32_t packed = 0;
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        const double yl = fma((double)fsty, G.zl[L] - G.zs, (double)fsy);
        int klo, khi;
        sector_range(G, yl, klo, khi);
        packed |= (uint32_t)(klo | (khi << 4)) << (8 * L);
    }
    sc.lo = (uint16_t)(packed & 0xffffu);
    sc.hi = (uint16_t)(packed >> 16);
}

__device__ __forceinline__ void sector_span(const SeedConst &sc, int L, int &klo, int &khi)
{
    const uint32_t v = (((uint32_t)sc.lo | ((uint32_t)sc.hi << 16)) >> (8 * L)) & 0xffu;
    klo = (int)(v & 15u);
    khi = (int)(v >> 4);
}

// LDS ranges of the buckets of layer L, sectors klo..khi (at most two), whose
// u bins cover [m - W, m + W]; buckets are (layer, sector, u bin).  Branch-free:
// the four bounds are read at sector indices clamped into the layer's buckets
// and dropped when the sector is not in the span.
__device__ __forceinline__ void sector_bins(const uint16_t *E, const WindowArgs &w, int L, int klo, int khi, double m, double W,
                                   int &lo0, int &len0, int &lo1, int &len1)
{
    int b_lo, b_hi;
    window_bins(w.bins, m, W, b_lo, b_hi);
    const int base0 = L * w.nb + (int)__umul24(min(klo, w.nsec - 1), w.nbu);
    const int base1 = L * w.nb + (int)__umul24(min(klo + 1, w.nsec - 1), w.nbu);
    const int e0 = E[base0 + b_lo], e1 = E[base0 + b_hi + 1], e2 = E[base1 + b_lo], e3 = E[base1 + b_hi + 1];
    const bool in0 = klo <= khi, in1 = klo + 1 <= khi;
    lo0 = in0 ? e0 : 0;
    len0 = in0 ? e1 - e0 : 0;
    lo1 = in1 ? e2 : 0;
    len1 = in1 ? e3 - e2 : 0;
}

__device__ __forceinline__ WindowArgs window_args(const TrackArgs &a, const DevGeom &G)
{
    return WindowArgs{G.w2c0, G.w2c1, a.nb, a.nbu, G.nsec, track_bins(a)};
}

// Does the line through the magnet point and the UTbX hit at p3 meet a UTaX
// hit of a compatible sector within W (the axial triplet)?
__device__ __forceinline__ bool dv1_triplet(double ffac, const WindowArgs &w, const float *hu_s, const uint16_t *E,
                                   const SeedConst &sc, int p3)
{
    const double W = fma(w.w2c1, fabs((double)sc.q), w.w2c0);
    const double m = fma((double)hu_s[p3] - sc.c[3], ffac, sc.c[0]);
    int klo, khi, lo0, len0, lo1, len1;
    sector_span(sc, 0, klo, khi);
    sector_bins(E, w, 0, klo, khi, m, W, lo0, len0, lo1, len1);
    const int n = len0 + len1;
    bool hit = false;
    for (int kb = 0; kb < n && !hit; kb += 4) {
        float u[4];   // (places past the end read what follows in LDS and are dropped)
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = hu_s[kb + j < len0 ? lo0 + kb + j : lo1 + (kb + j - len0)];
#pragma unroll
        for (int j = 0; j < 4; ++j) hit |= (kb + j < n) & (fabs((double)u[j] - m) <= W);
    }
    return hit;
}

// Dv1's map of UTaX: a bit per (Y sector, u bin), `words` words per sector, set
// where the window of a seed with |q/p| up to MAP_QOP could reach a hit from
// that bin.  One LDS word per sector and a dozen vector instructions rule out
// nine probes in ten; those that remain (about half of them triplets) are
// gathered, 64 to a pass, for the exact test.  Testing every probe exactly took
// 75 instructions each, more than half of the launch (10 000 events of 150
// seeds, 600 hits per layer: 653 to 439 us).
struct SectorMap {
    uint32_t *bits;   // n_sectors * words
    int words;
    Bins bins;
    float reach;      // the widest window it serves, with the margin of float32 projections
    float range;      // coordinates up to which float32 projections are within that margin
};

constexpr float MAP_QOP = 0.5f;      // seeds of more are tested exactly throughout
constexpr float MAP_MARGIN = 2e-2f;

// Coordinates below which the float32 projection of map_maybe is within two
// thirds of MAP_MARGIN for a projection factor f: its error is at most 2^-24
// (f (4 |c3| + 3 |u|) + 2 |c0|).  16 384 mm for factors up to 1.2, less for a
// magnet point close to UTbX.
inline float map_range(double f) { return (float)(16384.0 * fmin(1.0, 12.0 / (8.0 * fabs(f) + 2.4))); }

__device__ __forceinline__ void map_set(const SectorMap &m, int nsec, float u, int sec)
{
    if (sec >= nsec) return;
    int b0 = bin_of(m.bins, u - m.reach);
    const int b1 = bin_of(m.bins, u + m.reach);
    uint32_t *w = m.bits + __umul24(sec, m.words) + (b0 >> 5);
    for (; b1 - b0 > 31; b0 = (b0 | 31) + 1) atomicOr(w++, ~0u << (b0 & 31));
    const uint32_t run = ~0u >> (31 - (b1 - b0));
    const int sh = b0 & 31;
    atomicOr(w, run << sh);
    if (sh + b1 - b0 > 31) atomicOr(w + 1, run >> (32 - sh));
}

// What the triplet look-up needs of a seed: its UTbX range, and its projection
// to UTaX in float32 with the first words of its one or two sectors in the map.
struct alignas(16) MapSeed {
    float c0, c3;
    uint32_t range;   // LDS position | number of hits << 16
    uint32_t words;   // first word of the lower sector | of the upper one << 15 | exact << 31
};

__device__ __forceinline__ MapSeed map_seed(const SectorMap &m, int nsec, const SeedConst &sc, int p_lo, int n)
{
    MapSeed s;
    s.c0 = (float)sc.c[0];
    s.c3 = (float)sc.c[3];
    int klo, khi;
    sector_span(sc, 0, klo, khi);
    s.range = (uint32_t)p_lo | ((klo <= khi ? (uint32_t)n : 0u) << 16);
    const bool exact = fmaxf(fabsf(s.c0), fabsf(s.c3)) > m.range || fabsf(sc.q) > MAP_QOP;   // outside what the map serves
    s.words = __umul24(min(klo, nsec - 1), m.words) | (__umul24(khi, m.words) << 15) | (exact ? 1u << 31 : 0u);
    return s;
}

// False only if no hit of the seed's sectors can lie within its window of the
// line through the magnet point and a UTbX hit at u (map_range bounds the
// projection's float32 error).
__device__ __forceinline__ bool map_maybe(const SectorMap &m, const MapSeed &s, float ffac, float u)
{
    const int b = bin_of(m.bins, fmaf(u - s.c3, ffac, s.c0));
    const uint32_t *w = m.bits + (b >> 5);
    const uint32_t bits = w[s.words & 0x7fffu] | w[(s.words >> 15) & 0x7fffu];
    return (((bits >> (b & 31)) & 1u) != 0u) | (fabsf(u) > m.range) | ((int)s.words < 0);
}

// Candidate key of Dv1: the candidate index holds the UTbX hit's index in its
// layer run, 20 bits; 43 bits of chi2 above it.
__device__ __forceinline__ unsigned long long pack_key_dv1(int n, double chi2, int c)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(chi2);
    return ((unsigned long long)(4 - n) << 63) | ((b >> 20) << 20) | (unsigned long long)c;
}

// The refined window of an item (a seed and one of its UTbX hits, LDS position
// p3) in layer L (wavefront-uniform): LDS positions of its two closest hits,
// packed low and high, 0xffff for none.  Hits are ordered by the float32-rounded
// distance (rounding is monotone, so a strictly smaller rounded distance is a
// strictly smaller distance); window membership is always the float64 test.
//
// A unit of work is one layer of one item, a lane each: a lane that walked the
// three layers together held three windows in registers (168 in all, three
// waves per SIMD) and ran as long as the longest of 192 windows; the units are
// spread evenly over the wavefronts and read four positions per LDS round trip
// (the kernels hold 66 to 111 registers now, seven to four waves).
template <bool DV1>
__device__ __forceinline__ uint32_t window_best2(const WindowArgs &w, double ffac, const float *hu_s,
                                                 const uint16_t *hidx_s, const uint16_t *E, const SeedConst &sc, int L,
                                                 int p3)
{
    const double W2 = fma(w.w2c1, fabs((double)sc.q), w.w2c0);
    const double m = fma((double)hu_s[p3] - sc.c[3], ffac, sc.c[L]);
    int lo, len0, lo1 = 0, len;   // up to two LDS ranges (Dv1: one per compatible Y sector)
    if (DV1) {
        int klo, khi, l1;
        sector_span(sc, L, klo, khi);
        sector_bins(E, w, L, klo, khi, m, W2, lo, len0, lo1, l1);
        len = len0 + l1;
    } else {
        int hi;
        bin_range(E, L, w, m, W2, lo, hi);
        len0 = len = hi - lo;
    }
    auto at = [&](int k) { return (!DV1 || k < len0) ? lo + k : lo1 + (k - len0); };
    // the three smallest keys: the float32-rounded distance, its last byte replaced by the hit's place in
    // the range (~0: none)
    uint32_t k0 = ~0u, k1 = ~0u, k2 = ~0u;
    for (int kb = 0; kb < len; kb += 4) {
        float u[4];   // (places past the end read what follows in LDS and are dropped)
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = hu_s[at(kb + j)];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double d = fabs((double)u[j] - m);
            const bool in = (kb + j < len) & (d <= W2);
            const uint32_t key = in ? (__float_as_uint((float)d) & ~255u) | (uint32_t)(kb + j) : ~0u;
            k2 = max(min(k2, key), k1);   // the middle of (k1, k2, key), k1 <= k2
            k1 = max(min(k1, key), k0);
            k0 = min(k0, key);
        }
    }
    int r0 = k0 != ~0u ? at((int)(k0 & 255u)) : -1, r1 = k1 != ~0u ? at((int)(k1 & 255u)) : -1;
    // distances that agree but for the last byte (exact ties among them), and ranges whose places do not
    // fit a byte, are settled on the full key (|delta| in float64, u, index)
    const bool close = (k1 != ~0u) & (((k0 ^ k1) < 256u) | ((k1 ^ k2) < 256u));
    if (__builtin_expect(__ballot(close | (len > 256)) != 0ull, 0)) {
        if (close | (len > 256)) {
            r0 = r1 = -1;
            for (int k = 0; k < len; ++k) {
                const int p = at(k);
                const float u = hu_s[p];
                const double d = fabs((double)u - m);
                if (!(d <= W2)) continue;
                if (before(hu_s, hidx_s, d, u, p, r0 >= 0 ? fabs((double)hu_s[r0] - m) : INFINITY, r0)) {
                    r1 = r0;
                    r0 = p;
                } else if (before(hu_s, hidx_s, d, u, p, r1 >= 0 ? fabs((double)hu_s[r1] - m) : INFINITY, r1)) {
                    r1 = p;
                }
            }
        }
    }
    return (uint32_t)(r0 & 0xffff) | ((uint32_t)r1 << 16);
}

// An item's options: per layer 0-2 how many of its window's hits take part
// (n_closest caps them), and the layer set of its candidates, the same for all
// of them (a layer either has hits, and all its options are hits, or stands
// for "no hit").  cands: how many candidates it has, 0 when the set is not
// valid (3 hits, one of them in UTaX or UTaU; with Dv1 the UTaX hit of the
// axial triplet).
struct ItemOptions {
    int n0, n1, n2, mask, cands;
};

template <bool DV1>
__device__ __forceinline__ ItemOptions item_options(const DevGeom &G, uint32_t w0, uint32_t w1, uint32_t w2)
{
    auto found = [](uint32_t w, int ncl) { return min(ncl, (int)((w & 0xffffu) != 0xffffu) + (int)((w >> 16) != 0xffffu)); };
    ItemOptions o;
    o.n0 = found(w0, G.ncl[0]);
    o.n1 = found(w1, G.ncl[1]);
    o.n2 = found(w2, G.ncl[2]);
    o.mask = 8 | (o.n0 > 0 ? 1 : 0) | (o.n1 > 0 ? 2 : 0) | (o.n2 > 0 ? 4 : 0);
    const bool ok = __popc(o.mask) >= 3 && (o.mask & (DV1 ? 1 : 3)) != 0;
    o.cands = ok ? max(o.n0, 1) * max(o.n1, 1) * max(o.n2, 1) : 0;
    return o;
}

// LDS positions (-1: no hit) of candidate t of an item, in candidate-index
// order (UTaX option slowest), and its part (i0 nw1 + i1) nw2 + i2 of the index.
__device__ __forceinline__ int candidate_hits(const DevGeom &G, const ItemOptions &o, uint32_t w0, uint32_t w1,
                                              uint32_t w2, int t, int bp[3])
{
    const int b2 = o.n2 > 1 ? 1 : 0, b1 = o.n1 > 1 ? 1 : 0;   // bits that the options take in t
    const int i2 = b2 ? t & 1 : 0, i1 = b1 ? (t >> b2) & 1 : 0, i0 = t >> (b1 + b2);
    auto hit = [](uint32_t w, int n, int i) { return n > 0 ? (int)(i ? w >> 16 : w & 0xffffu) : -1; };
    bp[0] = hit(w0, o.n0, i0);
    bp[1] = hit(w1, o.n1, i1);
    bp[2] = hit(w2, o.n2, i2);
    return (i0 * G.nw[1] + i1) * G.nw[2] + i2;
}

// Residuals of a candidate's hits in the seed frame (0 for a layer without).
__device__ __forceinline__ void candidate_rho(const float *hu_s, const SeedConst &sc, const int bp[4], double rho[4])
{
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        const double r = (double)hu_s[max(bp[L], 0)] - sc.c[L];
        rho[L] = bp[L] >= 0 ? r : 0.0;
    }
}

// Rank of the UTbX hit at p3 among the seed's first-window hits (by the
// window key), or -1 if it is outside the window.
__device__ __forceinline__ int first_window_rank(const DevGeom &G, const float *hu_s, const uint16_t *hidx_s,
                                        const SeedConst &sc, int p3)
{
    const double W1 = fma(G.w1c1, fabs((double)sc.q), G.w1c0);
    const double m3 = window1_centre(G, sc.c[3], (double)sc.q);
    const float u3 = hu_s[p3];
    const double d3 = fabs((double)u3 - m3);
    if (!(d3 <= W1)) return -1;
    const int i3 = hidx_s[p3];
    int rank = 0;
    // four positions per LDS round trip
    for (int p0 = sc.lo; p0 < sc.hi; p0 += 4) {
        float u[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) u[j] = hu_s[p0 + j < sc.hi ? p0 + j : p3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = p0 + j;
            const double d = fabs((double)u[j] - m3);
            if (p < sc.hi && (d < d3 || (d == d3 && p != p3 && key_less(d, u[j], (int)hidx_s[p], d3, u3, i3)))) ++rank;
        }
    }
    return rank;
}

// The float32 track record of a fitted candidate; its ghost score is set by
// the caller (mlp_score_wave of the features, 0 without the network).
struct StoredTrack {
    float x, y, tx, ty, qop, chi2, score;
};

// A seed's float32 parameters.
struct SeedRaw {
    float x, y, tx, ty, qop;
};

__device__ __forceinline__ SeedRaw load_seed(const TrackArgs &a, int i)
{
    return SeedRaw{a.sx[i], a.sy[i], a.stx[i], a.sty[i], a.sqop[i]};
}

// f (optional): the track's ghost-killer features.
__device__ __forceinline__ StoredTrack stored_track(const DevGeom &G, const SeedRaw &sd, int n, double al, double be,
                                           double c2, const float *hu_s, const int bp[4], float *f)
{
    const float fsx = sd.x, fsy = sd.y, fstx = sd.tx, fsty = sd.ty, fsq = sd.qop;
    const double sx = fsx, sy = fsy, stx = fstx, sty = fsty;
    StoredTrack t;
    t.x = (float)(fma(stx, G.zref_seed, sx) + al);
    t.tx = (float)(stx + be);
    t.y = (float)fma(sty, G.zref_seed, sy);
    t.ty = fsty;
    t.qop = (G.mk != 0.0) ? (float)(-be / G.mk) : fsq;
    t.chi2 = (float)c2;
    t.score = 0.0f;
    if (f) {
        float hu4[4];
        int mask = 0;
#pragma unroll
        for (int L = 0; L < 4; ++L) {
            hu4[L] = bp[L] >= 0 ? hu_s[bp[L]] : 0.0f;
            mask |= bp[L] >= 0 ? (1 << L) : 0;
        }
        ghost_features(G, t.x, t.y, t.tx, t.ty, t.qop, t.chi2, n, fsx, fsy, fstx, fsty, fsq, hu4, mask, f);
    }
    return t;
}

// Write the selected candidate (LDS positions bp, -1 = none) as seed i's
// track, all but its ghost score.
__device__ __forceinline__ StoredTrack write_track(const TrackArgs &a, const DevGeom &G, const double *tab, int i,
                                                   const SeedRaw &sd, const SeedConst &sc, const float *hu_s,
                                                   const uint16_t *hidx_s, const int bp[4], int c)
{
    const int mask = (bp[0] >= 0 ? 1 : 0) | (bp[1] >= 0 ? 2 : 0) | (bp[2] >= 0 ? 4 : 0) | 8;
    const int n = __popc(mask);
    double rho[4];
    candidate_rho(hu_s, sc, bp, rho);
    double al, be, c2;
    fit_set(G, tab, mask, rho, al, be, c2);
    const StoredTrack t = stored_track(G, sd, n, al, be, c2, hu_s, bp, nullptr);
    a.x[i] = t.x;
    a.y[i] = t.y;
    a.tx[i] = t.tx;
    a.ty[i] = t.ty;
    a.qop[i] = t.qop;
    a.chi2[i] = t.chi2;
    a.h0[i] = bp[0] >= 0 ? (int)hidx_s[bp[0]] : -1;
    a.h1[i] = bp[1] >= 0 ? (int)hidx_s[bp[1]] : -1;
    a.h2[i] = bp[2] >= 0 ? (int)hidx_s[bp[2]] : -1;
    a.h3[i] = (int)hidx_s[bp[3]];
    a.nhits[i] = n;
    if (a.cand) a.cand[i] = c;
    return t;
}

// One row per (seed, candidate index) of the candidate-scoring mode.
__device__ __forceinline__ void write_candidate_row(const TrackArgs &a, const DevGeom &G, int i, int n, int c, double al,
                                           double be, double c2, const float *hu_s, const uint16_t *hidx_s,
                                           const int bp[4])
{
    float f[NF];
    const StoredTrack t = stored_track(G, load_seed(a, i), n, al, be, c2, hu_s, bp, f);
    const size_t r = (size_t)i * (size_t)a.cmax + (size_t)c;
    a.r_seed[r] = i;
    a.r_cand[r] = c;
    a.r_nhits[r] = n;
    a.r_h0[r] = bp[0] >= 0 ? (int)hidx_s[bp[0]] : -1;
    a.r_h1[r] = bp[1] >= 0 ? (int)hidx_s[bp[1]] : -1;
    a.r_h2[r] = bp[2] >= 0 ? (int)hidx_s[bp[2]] : -1;
    a.r_h3[r] = (int)hidx_s[bp[3]];
    a.r_x[r] = t.x;
    a.r_y[r] = t.y;
    a.r_tx[r] = t.tx;
    a.r_ty[r] = t.ty;
    a.r_qop[r] = t.qop;
    a.r_chi2[r] = t.chi2;
    a.r_score[r] = mlp_score_lane(a.Wrow, f);
}

// The launch's binning parameters, read once per event and held in scalar
// registers (opaque to the compiler, which would otherwise re-load them from
// the argument segment, a scalar round trip, at every use).
struct BinParams {
    int nb, nbu, nb3, nbu3;
    Bins b, b3;
};

template <typename T>
__device__ __forceinline__ T opaque_uniform(T v)
{
    asm volatile("" : "+s"(v));
    return v;
}

__device__ __forceinline__ BinParams bin_params(const TrackArgs &a)
{
    BinParams b;
    b.nb = opaque_uniform(a.nb);
    b.nbu = opaque_uniform(a.nbu);
    b.nb3 = opaque_uniform(a.nb3);
    b.nbu3 = opaque_uniform(a.nbu3);
    b.b = Bins{opaque_uniform(a.inv_bw), opaque_uniform(a.bin_off), (float)(b.nbu - 1)};
    b.b3 = Bins{opaque_uniform(a.inv_bw3), opaque_uniform(a.bin_off3), (float)(b.nbu3 - 1)};
    return b;
}

// Bucket of a hit: (layer, u bin) for Dv0; (layer, Y sector, u bin) for Dv1,
// with one last bucket per layer for sector ids outside [0, nsec).
template <bool DV1>
__device__ __forceinline__ int hit_bucket(const BinParams &bp, int nsec, int L, float u, int sec)
{
    const bool l3 = DV1 && L == 3;   // Dv0's layer 3 has the common layout
    int b = L * bp.nb + bin_of(l3 ? bp.b3 : bp.b, u);
    // (24-bit products: a 32-bit one takes four times as long)
    if (DV1) b = sec < nsec ? b + (int)__umul24(sec, l3 ? bp.nbu3 : bp.nbu) : L * bp.nb + nsec * (l3 ? bp.nbu3 : bp.nbu);
    return b;
}

// The hits of one staging round of a layer that WPL wavefronts share, for
// wavefront `sub` of them (slot j: hit r 64 HPT WPL + 64 (j WPL + sub) + lane
// of the run at `base`, n hits): their u and, for Dv1, their Y sectors, loaded
// with them (not again at each use).
template <bool DV1, int HPT, int WPL>
__device__ __forceinline__ void load_round(const TrackArgs &a, int base, int n, int r, int sub, float u[HPT],
                                           uint32_t sp[HPT])
{
    // one lane pointer and constant offsets: no per-slot address registers to
    // keep; slot j is in the run iff lane < lim - 64 WPL j
    const int lane = fresh_tid() & 63;
    const int skip = r * 64 * HPT * WPL + 64 * sub, lim = n - skip;
    const float *hp = a.hu + base + skip + lane;
#pragma unroll
    for (int j = 0; j < HPT; ++j) u[j] = (lane < lim - 64 * WPL * j) ? hp[64 * WPL * j] : 0.0f;
    if (DV1) {
        const uint8_t *sp8 = a.hsec + base + skip + lane;
#pragma unroll
        for (int j = 0; j < HPT; ++j) sp[j] = (lane < lim - 64 * WPL * j) ? (uint32_t)sp8[64 * WPL * j] : 0u;
    }
}

// Bucket bounds are 16-bit (an event's hits in LDS stay below 2^16): E[i] += 1
// through a 32-bit LDS atomic on the pair of bounds that holds it, returning
// the old E[i]; the low half never reaches 2^16, so it never carries into the
// high one.
__device__ __forceinline__ int bkt_add(uint16_t *E, int i)
{
    uint32_t *w = reinterpret_cast<uint32_t *>(E) + (i >> 1);
    const int sh = (i & 1) * 16;
    return (int)((atomicAdd(w, 1u << sh) >> sh) & 0xffffu);
}

// Zero the n 16-bit bounds at EL (one wavefront): 16-byte stores over the
// aligned middle, single bounds at the two ends.
__device__ __forceinline__ void zero_bounds(uint16_t *EL, int n)
{
    const int lane = fresh_tid() & 63;
    const int head = (int)((16 - (reinterpret_cast<uintptr_t>(EL) & 15)) & 15) / 2;   // bounds before 16-B alignment
    const int h = min(head, n);
    if (lane < h) EL[lane] = 0;
    const int nv = (n - h) / 8;   // whole 8-bound (16-byte) groups
    uint4 *V = reinterpret_cast<uint4 *>(EL + h);
    for (int q = lane; q < nv; q += 64) V[q] = make_uint4(0u, 0u, 0u, 0u);
    for (int b = h + 8 * nv + lane; b < n; b += 64) EL[b] = 0;
}

// Exclusive prefix, offset by `carry`, of the n 16-bit counts at EL (one
// wavefront), two counts per lane per step: a lane reads the pair (b, b + 1)
// of its 32-bit word, the wavefront sums the pairs (DPP, no LDS traffic) and
// the lane writes both starts back; eight independent 128-bound pieces per
// round, then the carries.  EL may start at an odd bound: the first and last
// bounds outside whole words go on their own.
__device__ __forceinline__ void scan_bounds(uint16_t *EL, int n, int carry)
{
    const int lane = fresh_tid() & 63;
    int first = 0;
    if (reinterpret_cast<uintptr_t>(EL) & 2) {   // EL[0] is the high half of a word
        first = n > 0 ? (int)EL[0] : 0;
        if (lane == 0 && n > 0) EL[0] = (uint16_t)carry;
        carry += first;
        ++EL;
        --n;
    }
    uint32_t *W = reinterpret_cast<uint32_t *>(EL);
    const int nw = n / 2;
    for (int w0 = 0; w0 < nw; w0 += 512) {
        uint32_t pr[8];
        int v[8], incl[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int w = w0 + 64 * j + lane;
            pr[j] = w < nw ? W[w] : 0u;
            v[j] = (int)(pr[j] & 0xffffu) + (int)(pr[j] >> 16);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) incl[j] = wave_inclusive_sum(v[j]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int w = w0 + 64 * j + lane;
            const int s0 = carry + incl[j] - v[j], s1 = s0 + (int)(pr[j] & 0xffffu);
            if (w < nw) W[w] = (uint32_t)s0 | ((uint32_t)s1 << 16);
            carry += __builtin_amdgcn_readlane(incl[j], 63);
        }
    }
    if ((n & 1) && lane == 0) EL[n - 1] = (uint16_t)carry;   // a last bound in the low half of a word
}

// The whole workgroup: the n hits at hu_s, hidx_s in the order of their indices
// (a bitonic sort in place; with the first step of each merge mirrored, every
// exchange puts the smaller index first, so n may be any number).
template <int BLOCK>
__device__ __forceinline__ void sort_run(float *hu_s, uint16_t *hidx_s, int n)
{
    const int tid = fresh_tid();
    for (int k = 2; k < 2 * n; k *= 2)
        for (int j = k; j > 1; j /= 2) {
            for (int i = tid; i < n; i += BLOCK) {
                const int p = j == k ? i ^ (k - 1) : i ^ (j / 2);
                if (p > i && p < n && hidx_s[p] < hidx_s[i]) {
                    const uint16_t x = hidx_s[i];
                    const float u = hu_s[i];
                    hidx_s[i] = hidx_s[p];
                    hu_s[i] = hu_s[p];
                    hidx_s[p] = x;
                    hu_s[p] = u;
                }
            }
            lds_barrier();
        }
}

// Order the hits of every bucket of one layer by their index in the run: the
// order a single wavefront places them in, where several share the layer.  It
// decides exact ties of unranked first-window hits.  A lane per bucket; buckets
// of more than CROWDED hits (few bins, or hits beyond the binned range) are left
// to sort_crowded: 2 in the returned bits, 4 for some of more than WAVE_RUN.
constexpr int CROWDED = 32, WAVE_RUN = 256;

__device__ __forceinline__ int sort_buckets(float *hu_s, uint16_t *hidx_s, const uint16_t *EL, int nb, int first, int lanes)
{
    int left = 0;
    for (int b = first; b < nb; b += lanes) {
        const int s = EL[b], e = EL[b + 1];
        left |= e - s > WAVE_RUN ? 4 : e - s > CROWDED ? 2 : 0;
        if (e - s < 2 || e - s > CROWDED) continue;
        for (int i = s + 1; i < e; ++i) {
            const float u = hu_s[i];
            const uint16_t x = hidx_s[i];
            int p = i;
            for (; p > s && hidx_s[p - 1] > x; --p) {
                hu_s[p] = hu_s[p - 1];
                hidx_s[p] = hidx_s[p - 1];
            }
            if (p != i) {
                hu_s[p] = u;
                hidx_s[p] = x;
            }
        }
    }
    return left;
}

// One wavefront: the n <= WAVE_RUN hits at hu_s, hidx_s in the order of their
// indices, each put at the place that the smaller indices leave it.
__device__ __forceinline__ void rank_run(float *hu_s, uint16_t *hidx_s, int n)
{
    const int lane = fresh_tid() & 63;
    float u[WAVE_RUN / 64];
    uint16_t x[WAVE_RUN / 64];
    int r[WAVE_RUN / 64] = {};
#pragma unroll
    for (int q = 0; q < WAVE_RUN / 64; ++q) {
        const int i = min(64 * q + lane, n - 1);
        u[q] = hu_s[i];
        x[q] = hidx_s[i];
    }
#pragma unroll 4
    for (int j = 0; j < n; ++j) {
        const uint16_t xj = hidx_s[j];
#pragma unroll
        for (int q = 0; q < WAVE_RUN / 64; ++q) r[q] += xj < x[q] ? 1 : 0;
    }
    wave_sync();
#pragma unroll
    for (int q = 0; q < WAVE_RUN / 64; ++q)
        if (64 * q + lane < n) {
            hu_s[r[q]] = u[q];
            hidx_s[r[q]] = x[q];
        }
}

// The buckets that sort_buckets left, dealt to the wavefronts, or (`whole`)
// those of more than WAVE_RUN hits, by the workgroup together.  40 events of
// 2 600 hits a layer in 64 bins, nearly all of them crowded: 93 us a step, 76
// with the bins left as they came, 246 with a wavefront's 64 bins in turn.
template <int BLOCK>
__device__ __forceinline__ void sort_crowded(float *hu_s, uint16_t *hidx_s, const uint16_t *EL, int nb, bool whole)
{
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int turn = 0;
    for (int b0 = 0; b0 < nb; b0 += 64) {
        const int b = min(b0 + lane, nb - 1), s = EL[b], n = b0 + lane < nb ? EL[b + 1] - s : 0;
        for (unsigned long long m = __ballot(whole ? n > WAVE_RUN : (n > CROWDED) & (n <= WAVE_RUN)); m != 0ull; m &= m - 1) {
            const int k = __ffsll((long long)m) - 1;
            const int at = __builtin_amdgcn_readlane(s, k), len = __builtin_amdgcn_readlane(n, k);
            if (whole)
                sort_run<BLOCK>(hu_s + at, hidx_s + at, len);
            else if (turn++ % (BLOCK / 64) == wave)
                rank_run(hu_s + at, hidx_s + at, len);
        }
    }
}

// Stage one event's hits: count a layer's hits into its buckets, scan the
// counts (two buckets per lane per step, DPP sums) and place the hits.  Up to
// seven wavefronts: a wavefront per layer, with no workgroup barrier until the
// end (a wavefront's LDS operations complete in order).  Eight and sixteen
// wavefronts, taken where few events leave each its latency: two and four per
// layer, a barrier between the passes.  Same result as a workgroup counting
// sort: E[b] = start of bucket b, E[3*nb + nb3] = count.  *s_bad must be 0 on
// entry.
template <int BLOCK, bool DV1, typename Between>
__device__ __forceinline__ bool stage_hits_w(const TrackArgs &a, int nsec, const SectorMap &map, int hb, const int hl[4],
                                             int nh, float *hu_s, uint16_t *hidx_s, uint16_t *E, int *s_bad,
                                             Between &&between)
{
    constexpr int NW = BLOCK / 64, WPL = NW >= 8 ? NW / 4 : 1;   // wavefronts per layer
    constexpr int HPT = 16 / WPL;                                // hits per lane per round: 1 024 hits of a layer
    static_assert(NW < 8 || NW % 4 == 0, "whole wavefronts per layer");
    // readfirstlane: the layer index is then known to be wavefront-uniform
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the first layer's loads are in flight while `between` runs
    const int L0 = wave / WPL, sub = wave % WPL;
    int L = L0;
    int lo = L < 4 ? hl[L] : 0, n = L < 4 ? (L < 3 ? hl[L + 1] : nh) - hl[L] : 0;
    float u[HPT];
    uint32_t sp[HPT];
    load_round<DV1, HPT, WPL>(a, hb + lo, n, 0, sub, u, sp);
    // Dv1: every lane a few of UTaX's hits for the map (one wavefront with the whole layer kept the others
    // waiting for half of its counting)
    constexpr int MAP_HPT = 4;
    float mu[MAP_HPT];
    uint32_t ms[MAP_HPT];
    const int n0 = hl[1] - hl[0];
    if (DV1) {
#pragma unroll
        for (int j = 0; j < MAP_HPT; ++j) {
            const int k = tid + j * BLOCK;
            mu[j] = k < n0 ? a.hu[hb + k] : 0.0f;
            ms[j] = k < n0 ? (uint32_t)a.hsec[hb + k] : 255u;
        }
        for (int i = tid; i < nsec * map.words; i += BLOCK) map.bits[i] = 0u;
    }
    if (tid == 0) E[0] = 0;
    between();
    const BinParams bp = bin_params(a);
    if (DV1) {
        lds_barrier();
#pragma unroll
        for (int j = 0; j < MAP_HPT; ++j)
            if (j * BLOCK < n0) map_set(map, nsec, mu[j], (int)ms[j]);
        for (int k = tid + MAP_HPT * BLOCK; k < n0; k += BLOCK) map_set(map, nsec, a.hu[hb + k], (int)a.hsec[hb + k]);
    }
    bool bad = false;
    int left = 0;
    for (; L < 4; L += NW / WPL) {
        if (L != L0) {   // a further layer of this wavefront (fewer than four wavefronts)
            lo = hl[L];
            n = (L < 3 ? hl[L + 1] : nh) - lo;
            load_round<DV1, HPT, WPL>(a, hb + lo, n, 0, sub, u, sp);
        }
        uint16_t *EL = E + 1 + L * bp.nb;   // EL[b]: count, then end, of bucket (L, b)
        const int nb = (DV1 && L == 3) ? bp.nb3 : bp.nb;
        if (sub == 0) zero_bounds(EL, nb);
        if (WPL > 1) lds_barrier();
        constexpr int ROUND = 64 * HPT * WPL;
        const int rounds = (n + ROUND - 1) / ROUND;
        for (int r = 0; r < rounds; ++r) {
            if (r > 0) load_round<DV1, HPT, WPL>(a, hb + lo, n, r, sub, u, sp);
#pragma unroll
            for (int j = 0; j < HPT; ++j) {
                const int k0 = r * ROUND + 64 * (j * WPL + sub);
                if (k0 >= n) break;   // uniform: no lane has slot j
                if (k0 + lane < n) {
                    // (an event with a non-finite hit is dropped as a whole: its hits may go anywhere)
                    bad |= !isfinite(u[j]);
                    bkt_add(E, hit_bucket<DV1>(bp, nsec, L, u[j], DV1 ? (int)sp[j] : 0) + 1);
                }
            }
        }
        if (WPL > 1) lds_barrier();
        if (sub == 0) scan_bounds(EL, nb, lo);
        if (WPL > 1) lds_barrier();
        // placing pass: EL[b] advances to the end of bucket b
        for (int r = 0; r < rounds; ++r) {
            if (rounds > 1) load_round<DV1, HPT, WPL>(a, hb + lo, n, r, sub, u, sp);
#pragma unroll
            for (int j = 0; j < HPT; ++j) {
                const int k0 = r * ROUND + 64 * (j * WPL + sub);
                if (k0 >= n) break;
                if (k0 + lane < n) {
                    const int pos = bkt_add(E, hit_bucket<DV1>(bp, nsec, L, u[j], DV1 ? (int)sp[j] : 0) + 1);
                    hu_s[pos] = u[j];
                    hidx_s[pos] = (uint16_t)(k0 + lane);
                }
            }
        }
        if (WPL > 1 && !DV1) {
            lds_barrier();
            left = sort_buckets(hu_s, hidx_s, E + 3 * bp.nb, bp.nb, tid, BLOCK);
        }
    }
    if (bad | (left != 0)) atomicOr(s_bad, left | (bad ? 1 : 0));
    lds_barrier();
    const int state = uniform(*s_bad);
    if (WPL > 1 && !DV1 && __builtin_expect(state > 1, 0)) {
        uint16_t *E3 = E + 3 * bp.nb;
        if (state & 2) sort_crowded<BLOCK>(hu_s, hidx_s, E3, bp.nb, false);
        if (state & 4) sort_crowded<BLOCK>(hu_s, hidx_s, E3, bp.nb, true);
        lds_barrier();
    }
    return (state & 1) == 0;
}

__device__ __forceinline__ bool pca64(const DevGeom &G, double x1, double y1, double tx1, double ty1, double g1, double x2,
                             double y2, double tx2, double ty2, double g2, double &vx, double &vy, double &vz,
                             double &doca, double &s_out, double &t_out);
__device__ __forceinline__ void vertex_extras(const DevGeom &G, const float *WLg, float4 A, float4 B, double g1, double g2,
                                     float q1, float q2, double s, double t, float4 V, float out[6]);

// LDS of the vertexing's survivor masks, in ints, beside the kept tracks (the
// fused step lays them over buffers that are dead by then).
__host__ __device__ constexpr int vtx_mask_ints(int block) { return 8 * block; }

// Kept tracks of one event in LDS, the vertexing input.  Positive-charge
// tracks fill st/q/slot from the front and negative ones from the back, each
// list in slot order (the o-th negative at tcap - 1 - o).  row[r] describes
// the r-th kept track in slot order: its index o in its charge list, | 0x8000
// when positive; the tracks of the other charge before it number r - o, so its
// partners of higher slot are that list's entries from r - o on.
// The pair loop reads up to 31 entries past either end of its run: at least
// VTX_PAD bytes of the workgroup's LDS lie before and after st.
struct Kept {
    float4 *st;      // x, y, tx, ty at the UT midpoint
    float *q;        // fitted q/p
    int *slot;       // slot << 1 | positive seed charge
    uint16_t *row;
};

constexpr int VTX_PAD = 512;

__host__ __device__ constexpr size_t kept_lds_bytes(int tcap)
{
    return tcap <= 0 ? 0
           : 10 * tcap >= VTX_PAD ? ((size_t)tcap * 26 + 15) & ~(size_t)15
                                  : (size_t)tcap * 16 + VTX_PAD;
}

// In the fused step the list starts VTX_PAD bytes into the workgroup's LDS.
__host__ __device__ constexpr size_t fused_kept_bytes(int tcap) { return tcap <= 0 ? 0 : VTX_PAD + kept_lds_bytes(tcap); }

__device__ __forceinline__ Kept kept_carve(unsigned char *base, int tcap)
{
    Kept k;
    k.st = reinterpret_cast<float4 *>(base);
    k.q = reinterpret_cast<float *>(base + (size_t)tcap * 16);
    k.slot = reinterpret_cast<int *>(base + (size_t)tcap * 20);
    k.row = reinterpret_cast<uint16_t *>(base + (size_t)tcap * 24);
    return k;
}

// Appends this chunk's kept tracks (at most one per lane, lanes in slot
// order).  n and np (kept so far, positive so far) are workgroup-uniform and
// advanced; tcap < 32768 (LDS holds far fewer).
template <int BLOCK>
__device__ __forceinline__ void kept_append(const Kept &K, int tcap, bool kept, bool positive, float4 st, float q,
                                            int slot, int &n, int &np, int *s_wsum)
{
    int tot;
    const int ex = block_exclusive_scan<BLOCK>(kept ? (positive ? 0x10001 : 1) : 0, s_wsum, &tot);
    if (kept) {
        const int r = n + (ex & 0xffff);
        const int pb = np + (ex >> 16);   // positive tracks before this one
        const int o = positive ? pb : r - pb;
        const int pos = positive ? o : tcap - 1 - o;
        K.st[pos] = st;
        K.q[pos] = q;
        K.slot[pos] = (slot << 1) | (positive ? 1 : 0);
        K.row[r] = (uint16_t)(o | (positive ? 0x8000 : 0));
    }
    n += tot & 0xffff;
    np += tot >> 16;
}

// The kept tracks of slots [s0, s1) of the event, as this workgroup's lanes
// wrote them, appended.
template <int BLOCK>
__device__ __forceinline__ void keep_stored(const TrackArgs &a, const Kept &K, int s0, int s1, int &n, int &np, int *s_wsum)
{
    __syncthreads();   // the tracks that other wavefronts wrote are visible
    for (int b = s0; b < s1; b += BLOCK) {
        const int i = b + fresh_tid();
        bool kept = false;
        float4 st = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float q = 0.0f, sq = 0.0f;
        if (i < s1) {
            kept = a.nhits[i] > 0 && a.score[i] < a.score_max;
            st = make_float4(a.x[i], a.y[i], a.tx[i], a.ty[i]);
            q = a.qop[i];
            sq = a.sqop[i];
        }
        kept_append<BLOCK>(K, a.tcap, kept, sq > 0.0f, st, q, i - s0, n, np, s_wsum);
    }
}

// Sign bit set: the pair may lie within doca_max.  Straight trajectories: the
// distance of the two lines is |w.n|/|n|, n = d1 x d2; near-parallel pairs
// always pass.  The float32 error stays far below the margin in prescreen_thr2.
__device__ __forceinline__ float pair_near(const DevGeom &G, float4 A, float4 B)
{
    const float wx = A.x - B.x, wy = A.y - B.y;
    const float nx = A.w - B.w, ny = B.z - A.z;
    const float nz = fmaf(A.z, B.w, -(A.w * B.z));
    const float wn = fmaf(wx, nx, wy * ny);
    const float nn = fmaf(nx, nx, fmaf(ny, ny, nz * nz));
    return fminf(fmaf(wn, wn, -(G.prescreen_thr2 * nn)), nn - 1e-6f);
}

// The same for eq. 4 trajectories, x(s) = x + tx s + g s^2, y(s) = y + ty s,
// z = s.  Two points closer than R have |s - t| < R, so the y coordinates
// confine s to s0 +- w around the crossing of the straight y projections, and
// within that interval the x separation, a parabola, cannot fall below its
// value at s0 less its slope's and curvature's reach.  Where even that is
// beyond R (1 + the slope of the second track), no point of the two curves is
// within R, whatever the Newton steps do.  The float32 rounding of s0 and of
// the parabola is added as slack; comparisons with a NaN (parallel y
// projections, infinities) pass.
__device__ __forceinline__ float pair_near_curved(const DevGeom &G, float4 A, float gA, float4 B, float gB)
{
    const float R = G.prescreen_r;
    const float dx = A.x - B.x, dy = A.y - B.y, vx = A.z - B.z, vy = A.w - B.w, dg = gA - gB;
    const float iv = __builtin_amdgcn_rcpf(vy);
    const float s0 = -dy * iv, as = fabsf(s0);
    const float w = fmaf(fmaf(R, fabsf(B.w), R) * fabsf(iv), 1.00001f, 2e-6f * as);
    const float t1 = vx * s0, ag = fabsf(gA) + fabsf(gB), g2 = ag * as * as;
    const float q = fmaf(dg * s0, s0, dx + t1);
    const float slope = fabsf(fmaf(2.0f * dg, s0, vx));
    const float reach = fmaf(fmaf(fabsf(dg), w, slope), w, R * fmaf(ag, R + 2.0f * (as + w), 1.0f + fabsf(B.z)));
    const float slack = 1e-6f * (fabsf(dx) + fabsf(t1) + g2 + fmaf(2.0f * ag, as, fabsf(vx)) * (w + as));
    return fabsf(q) > reach * 1.00001f + slack ? 1.0f : -1.0f;
}

// Survivor bits of one task: a lane's row against ns <= 32 of its partners
// (uniform, a multiple of 4), the s-th partner at bit s.  A positive row
// walks its partners backwards (they lie from the back of the list), so that
// every lane's reads advance by the same constant.
template <bool CURVED>
__device__ __forceinline__ uint32_t vtx_task_bits(const DevGeom &G, const Kept &K, int first, int ns, bool fwd,
                                                  float4 A, float gA)
{
    uint32_t m = 0;
    const float4 *p = K.st + first;
    const float *pq = K.q + first;
    for (int s = 0; s < ns; s += 4) {
        float4 B[4];
        float gB[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            B[j] = p[s + j];
            // entries outside the list hold other data: their bits are dropped by the caller
            if (CURVED) gB[j] = -(float)G.fp * fmaf((float)G.gc1 * 1e-3f, pq[s + j], (float)G.gc0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float d = CURVED ? pair_near_curved(G, A, gA, B[j], gB[j]) : pair_near(G, A, B[j]);
            m = __builtin_amdgcn_alignbit(m, __float_as_uint(d), 31);   // (m << 1) | sign of d
        }
    }
    return fwd ? __builtin_bitreverse32(m << (32 - ns)) : m;
}

// Vertexing of one event by the whole workgroup.  Only opposite-charge pairs
// are visited: row r of the pair triangle (the r-th kept track in slot order)
// holds its opposite-charge partners of higher slot, a run of the other charge
// list, so rows in slot order with their partners in list order enumerate the
// pairs in (i, j) order.
//   1. Masks.  A wavefront takes 64 rows, a lane each, against 32 partners of
//      every row (a broadcast LDS read per charge and step), and keeps one bit
//      per pair that passes the float32 prescreen: 16 vector instructions and
//      one LDS read per pair.  A lane-per-pair loop over pair ranks took 76:
//      its row searches, addresses and masks were most of the work (the step of
//      5 000 events, 300 seeds and 1 200 hits per layer each, all pairs: 0.892
//      to 0.818 ms).  Curved trajectories, which had no prescreen and sent every
//      pair to the float64 fit, pass 0.2 to 3 % of them (3 001 uneven events
//      with masses and trigger lines: 1.909 to 0.326 ms).
//   2. The rows' bit counts are scanned; the survivors' ranks then run in
//      (i, j) order, and a survivor is found from its rank by a search of the
//      row starts and a select in the row's mask words.
//   3. Survivors are fitted a workgroup at a time (float64 Newton PCA, a lane
//      per pair) and the passing ones written in rank order, the first vcap.
// The masks of `words` ints at `mem` hold a panel of rows (all of them for
// events of usual size); larger events take several panels.  XTR: also the
// masses and trigger-line scores of each vertex.
// Args: TrackArgs (fused step) or VertexArgs (standalone): the vertex outputs
// vcap, vcount, vi, vj, vx, vy, vz, vdoca, voverflow, the extras' outputs, WL
// and the seeds' sqop under the same names.  n kept tracks, np of them
// positive, in K (kept_append), visible to every lane.
template <int BLOCK, bool XTR, typename Args>
__device__ __forceinline__ void vertex_event_block(const Args &a, const DevGeom &G, int e, int s0, int n, int np,
                                          const Kept &K, int tcap, int *mem, int words, int *s_wsum)
{
    constexpr int NW = BLOCK / 64;
    const int tid = fresh_tid(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool curved = (G.fp != 0.0);
    const int nn = n - np;   // negative tracks
    int out_n = 0;           // workgroup-uniform
    for (int r0 = 0; np > 0 && nn > 0 && r0 < n;) {
        // longest row from r0 on: the partners left in either list
        auto longest = [&](int r) {
            const int d = K.row[r], o = d & 0x7fff;
            return __builtin_amdgcn_readfirstlane(max(nn - ((d & 0x8000) ? r - o : o), np - ((d & 0x8000) ? o : r - o)));
        };
        const int segs = (longest(r0) + 31) >> 5;
        if (segs <= 0) break;
        const int fit_rows = (words - 1) / (segs + 1);
        const int rows = min(n - r0, fit_rows >= 64 ? fit_rows & ~63 : fit_rows);
        int *R = mem;                                                    // rows + 1 survivor ranks
        uint32_t *M = reinterpret_cast<uint32_t *>(mem + rows + 1);      // mask word of (segment, row)
        const int nrb = (rows + 63) >> 6;
        for (int t = wave; t < nrb * segs; t += NW) {
            const int rb = t / segs, seg = t - rb * segs;
            const int left = longest(r0 + 64 * rb) - 32 * seg;
            if (left <= 0) continue;   // no row of the block reaches this segment (its words are not read)
            const int ns = min(32, (left + 3) & ~3);
            const int rr = 64 * rb + lane, r = r0 + min(rr, rows - 1);
            const int d = K.row[r], o = d & 0x7fff;
            const bool positive = (d & 0x8000) != 0;
            const int len = (positive ? nn : np) - (r - o) - 32 * seg;   // this row's partners in the segment
            const int q0 = r - o + 32 * seg;
            const int own = positive ? o : tcap - 1 - o;
            // a row without partners here reads from the list's start
            const int first = len <= 0 ? 0 : positive ? tcap - q0 - ns : q0;
            const float4 A = K.st[own];
            uint32_t m;
            if (curved)
                m = vtx_task_bits<true>(G, K, first, ns, !positive, A,
                                        -(float)G.fp * fmaf((float)G.gc1 * 1e-3f, K.q[own], (float)G.gc0));
            else
                m = vtx_task_bits<false>(G, K, first, ns, !positive, A, 0.0f);
            m &= len >= 32 ? ~0u : len <= 0 ? 0u : (1u << len) - 1u;
            if (rr < rows) M[seg * rows + rr] = m;
        }
        lds_barrier();
        int total = 0;
        for (int b = 0; b < rows; b += BLOCK) {
            const int rr = b + tid;
            int c = 0;
            if (rr < rows) {
                const int r = r0 + rr, d = K.row[r];
                const int len = ((d & 0x8000) ? nn : np) - (r - (d & 0x7fff));
                for (int s = 0; 32 * s < len; ++s) c += __popc(M[s * rows + rr]);
            }
            int tot;
            const int ex = block_exclusive_scan<BLOCK>(c, s_wsum, &tot);
            if (rr < rows) R[rr] = total + ex;
            total += tot;
        }
        if (tid == 0) R[rows] = total;
        lds_barrier();
        const int top = 1 << (31 - __builtin_clz(rows));   // highest power of two <= rows
        for (int b = 0; b < total; b += BLOCK) {
            const int k = b + tid;
            int pass = 0, ia = 0, ib = 0;
            float4 V = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            float2 ST = make_float2(0.0f, 0.0f);
            if (k < total) {
                // the row of rank k: the last one that starts at or below it
                int rr = 0;
                for (int step = top; step > 0; step >>= 1)
                    if (rr + step < rows && R[rr + step] <= k) rr += step;
                int left = k - R[rr], s = 0;
                uint32_t m = M[rr];
                for (int c = __popc(m); left >= c; c = __popc(m)) {
                    left -= c;
                    m = M[++s * rows + rr];
                }
                for (; left > 0; --left) m &= m - 1;
                const int r = r0 + rr, d = K.row[r], o = d & 0x7fff;
                const int q = r - o + 32 * s + __ffs(m) - 1;   // partner's index in its list
                ia = (d & 0x8000) ? o : tcap - 1 - o;
                ib = (d & 0x8000) ? tcap - 1 - q : q;
                const float4 A = K.st[ia], B = K.st[ib];
                const double g1 = -G.fp * (G.gc0 + G.gc1 * ((double)K.q[ia] * 1e-3));
                const double g2 = -G.fp * (G.gc0 + G.gc1 * ((double)K.q[ib] * 1e-3));
                double vx, vy, vz, dd, ps, pt;
                const bool good = pca64(G, A.x, A.y, A.z, A.w, g1, B.x, B.y, B.z, B.w, g2, vx, vy, vz, dd, ps, pt);
                pass = (good && (dd < G.doca_max)) ? 1 : 0;
                V = make_float4((float)vx, (float)vy, (float)vz, (float)dd);
                ST = make_float2((float)ps, (float)pt);
            }
            int tot2;
            const int opos = block_exclusive_scan<BLOCK>(pass, s_wsum, &tot2);
            if (pass) {
                const int m2 = out_n + opos;
                if (m2 < a.vcap) {
                    const size_t o = (size_t)e * (size_t)a.vcap + (size_t)m2;
                    a.vi[o] = K.slot[ia] >> 1;
                    a.vj[o] = K.slot[ib] >> 1;
                    a.vx[o] = V.x;
                    a.vy[o] = V.y;
                    a.vz[o] = V.z;
                    a.vdoca[o] = V.w;
                    if constexpr (XTR) {
                        const float4 TA = K.st[ia], TB = K.st[ib];
                        const double g1 = -G.fp * (G.gc0 + G.gc1 * ((double)K.q[ia] * 1e-3));
                        const double g2 = -G.fp * (G.gc0 + G.gc1 * ((double)K.q[ib] * 1e-3));
                        float ex[6];
                        vertex_extras(G, a.WL, TA, TB, g1, g2, a.sqop[s0 + (K.slot[ia] >> 1)],
                                      a.sqop[s0 + (K.slot[ib] >> 1)], ST.x, ST.y, V, ex);
                        a.m_pipi[o] = ex[0];
                        a.m_ppi[o] = ex[1];
                        a.line0[o] = ex[2];
                        a.line1[o] = ex[3];
                        a.line2[o] = ex[4];
                        a.line3[o] = ex[5];
                    }
                }
            }
            out_n += tot2;
        }
        r0 += rows;
        if (r0 < n) lds_barrier();   // the panel's masks are read
    }
    if (tid == 0) {
        a.vcount[e] = out_n < a.vcap ? out_n : a.vcap;
        if (out_n > a.vcap) atomicAdd(a.voverflow, out_n - a.vcap);
    }
}

// ------------------------------------------------------- clones, fused step
//
// Clone killing inside the fused launch: an event's tracks are noted in LDS as
// they are found, by slot; after its last chunk every track looks for a better
// one that shares more than two hits, killed ones are rewritten as "no track",
// and the survivors are scored and kept.  Two tracks that share three of four
// hits share one in UTaX or UTaU, so a track meets all its rivals in two hash
// chains, one per layer (k_clone compares every pair of the event).  As
// launches of their own the three steps read the tracks back from HBM and set
// the vertexing up again, and every one ends in a tail of few workgroups:
// 4 000 events of 150 seeds, 600 hits: 270 us with them, 148 in this launch.
struct CloneNotes {
    unsigned long long *hits;   // four 16-bit hit indices, 0xffff: none
    float *chi2;
    int *n;                     // number of hits; 0: no track
};

constexpr int CLONE_HASH = 256;

__host__ __device__ constexpr size_t clone_lds_bytes(int tcap) { return (size_t)tcap * 16; }

// LDS words of the hash chains (over the region that is dead by then).
__host__ __device__ constexpr int clone_hash_words(int tcap) { return 2 * CLONE_HASH + (tcap * 6 + 3) / 4; }

__device__ __forceinline__ CloneNotes clone_carve(unsigned char *base, int tcap)
{
    CloneNotes c;
    c.hits = reinterpret_cast<unsigned long long *>(base);
    c.chi2 = reinterpret_cast<float *>(c.hits + tcap);
    c.n = reinterpret_cast<int *>(c.chi2 + tcap);
    return c;
}

__device__ __forceinline__ void clone_record(const CloneNotes &c, int slot, bool found, const int bp[4],
                                             const uint16_t *hidx_s, float chi2)
{
    unsigned long long p = 0;
    int n = 0;
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        const bool has = found && bp[L] >= 0;
        p |= (unsigned long long)(has ? (unsigned)hidx_s[max(bp[L], 0)] : 0xffffu) << (16 * L);
        n += has ? 1 : 0;
    }
    c.hits[slot] = p;
    c.chi2[slot] = chi2;
    c.n[slot] = n;
}

// Track j kills track k: more than two shared hits, and more hits, or as many
// and a lower chi2, or both equal and a lower slot.
__device__ __forceinline__ bool clone_kills(const CloneNotes &c, int j, int k)
{
    const unsigned long long pj = c.hits[j], pk = c.hits[k];
    int shared = 0;
#pragma unroll
    for (int L = 0; L < 4; ++L) {
        const unsigned h = (unsigned)(pk >> (16 * L)) & 0xffffu;
        shared += (h != 0xffffu && h == ((unsigned)(pj >> (16 * L)) & 0xffffu)) ? 1 : 0;
    }
    if (shared <= 2) return false;
    const int nj = c.n[j], nk = c.n[k];
    const float cj = c.chi2[j], ck = c.chi2[k];
    return nj > nk || (nj == nk && (cj < ck || (cj == ck && j < k)));
}

// The event's tracks (noted, and written without scores): kills, then scores
// of the survivors and the kept list, in passes of scap slots.  `region`: dead
// LDS for the hash chains, then the network's rows.
template <int BLOCK>
__device__ __forceinline__ void kill_and_score(const TrackArgs &a, const DevGeom &G, int s0, int s1, const int ho[5],
                                               const Kept &K, const CloneNotes &c, uint32_t *region, int *s_wsum,
                                               int &nk, int &nkp)
{
    const int tid = fresh_tid(), n = s1 - s0;
    uint32_t *heads = region;
    uint16_t *next = reinterpret_cast<uint16_t *>(region + 2 * CLONE_HASH), *dead = next + 2 * n;
    __syncthreads();   // the tracks that other wavefronts wrote are visible
    for (int b = tid; b < 2 * CLONE_HASH; b += BLOCK) heads[b] = 0xffffu;
    lds_barrier();
    auto hit = [&](int k, int L) { return (unsigned)(c.hits[k] >> (16 * L)) & 0xffffu; };
    for (int k = tid; k < n; k += BLOCK)
        for (int L = 0; L < 2; ++L) {
            const unsigned h = hit(k, L);
            if (h != 0xffffu) next[L * n + k] = (uint16_t)atomicExch(&heads[L * CLONE_HASH + (h & (CLONE_HASH - 1))], (uint32_t)k);
        }
    lds_barrier();
    for (int k = tid; k < n; k += BLOCK) {
        bool killed = false;
        for (int L = 0; L < 2; ++L) {
            const unsigned h = hit(k, L);
            if (h == 0xffffu) continue;
            for (unsigned j = heads[L * CLONE_HASH + (h & (CLONE_HASH - 1))]; j != 0xffffu && !killed; j = next[L * n + j])
                killed = (int)j != k && clone_kills(c, (int)j, k);
        }
        dead[k] = killed ? 1 : 0;
    }
    lds_barrier();
    for (int k = tid; k < n; k += BLOCK)   // (all pairs are judged on the tracks as found)
        if (dead[k]) c.n[k] = -1;
    lds_barrier();
    for (int b = 0; b < n; b += a.scap) {
        const int k = b + tid, i = s0 + k;
        const bool have = tid < a.scap && k < n;
        const int nh = have ? c.n[k] : 0;
        const bool row = nh > 0;
        float f[NF] = {}, sq = 0.0f, qop = 0.0f;
        float4 st = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (row) {
            float hu4[4];
            int has = 0;
            const unsigned long long p = c.hits[k];
#pragma unroll
            for (int L = 0; L < 4; ++L) {
                const unsigned h = (unsigned)(p >> (16 * L)) & 0xffffu;
                hu4[L] = h != 0xffffu ? a.hu[ho[L] + (int)h] : 0.0f;
                has |= h != 0xffffu ? 1 << L : 0;
            }
            st = make_float4(a.x[i], a.y[i], a.tx[i], a.ty[i]);
            qop = a.qop[i];
            sq = a.sqop[i];
            ghost_features(G, st.x, st.y, st.z, st.w, qop, c.chi2[k], nh, a.sx[i], a.sy[i], a.stx[i], a.sty[i], sq, hu4, has,
                           f);
        } else if (have) {
            if (nh < 0) write_empty_track(a, i);
            a.score[i] = 0.0f;
        }
        const float score = mlp_score_rows<BLOCK>(a.W, reinterpret_cast<float *>(region), s_wsum, row, f);
        if (row) a.score[i] = score;
        kept_append<BLOCK>(K, a.tcap, row && score < a.score_max, sq > 0.0f, st, qop, k, nk, nkp, s_wsum);
    }
}

// Event of launch iteration `iter`, n_events or more when there is none left.
// A persistent launch gives each workgroup the event of its own index first
// and the rest by a work counter: with every event taken from the counter, a
// launch opened with as many device-wide atomics on one address as it has
// workgroups (finding, scoring and vertexing 1 111 small events in three
// calls: 98 to 57 us without; the fused 10 000-event launch 0.324 to 0.308 ms),
// and a launch of no more events than workgroups needs no counter at all.
// Every workgroup fails exactly once, so the counter ends at n_events - 1
// before the last failing grab, which sets it back to zero for the next launch.
// tier >= 0: only the events of that class of the order (ends: the classes').
__device__ __forceinline__ int grab_event(int *counter, int n_events, int ev_single, const int *order, int tier,
                                          const int *ends, int iter)
{
    if (ev_single >= 0) return iter == 0 ? ev_single : n_events;
    const int grid = (int)gridDim.x;
    const int first = tier > 0 ? ends[tier - 1] : 0, n = (tier >= 0 ? ends[tier] : n_events) - first;
    int k = (int)blockIdx.x;
    if (iter > 0) {
        if (n <= grid) return n_events;
        const int c = atomicAdd(counter, 1);
        if (c == n - 1) atomicExch(counter, 0);
        k = grid + c;
    }
    if (k >= n) return n_events;
    return order ? order[first + k] : k;
}

// One whole wave: the event of iteration `iter` and its offsets into LDS,
// s_nx = {event, seed_off[e], seed_off[e + 1], hit_off[4e .. 4e + 4]}.
__device__ __forceinline__ void fetch_event(const TrackArgs &a, int iter, int lane, int *s_nx)
{
    int en = 0;
    if (lane == 0) en = grab_event(a.counter, a.n_events, a.ev_single, a.order, a.tier, a.ends, iter);
    en = __builtin_amdgcn_readfirstlane(en);
    if (lane == 0) s_nx[0] = en;
    if (lane < 7 && en < a.n_events) s_nx[1 + lane] = lane < 2 ? a.seed_off[en + lane] : a.hit_off[4 * en + lane - 2];
}

// XTR (with VTX): the fused vertexing also writes masses and trigger-line scores.
template <int BLOCK, bool CANDS, bool VTX, bool DV1, bool XTR = false>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(CANDS ? 2 : 4))) void k_track(TrackKernArgs)
{
    static_assert(!(CANDS && DV1), "candidate rows follow Dv0");
    static_assert(!XTR || VTX, "extras come with the fused vertexing");
    const TrackArgs &a0 = kernel_args<TrackKernArgs>().a;
    extern __shared__ __align__(16) unsigned char smem[];
    size_t off = 0;
    float *hu_s = reinterpret_cast<float *>(smem + off);
    off += (size_t)a0.hcap * 4;
    uint16_t *hidx_s = reinterpret_cast<uint16_t *>(smem + off);
    off = (off + (size_t)a0.hcap * 2 + 15) & ~(size_t)15;
    uint16_t *E = reinterpret_cast<uint16_t *>(smem + off);
    off = (off + (size_t)(3 * a0.nb + a0.nb3 + 1) * 2 + 15) & ~(size_t)15;
    uint32_t *map_s = reinterpret_cast<uint32_t *>(smem + off);   // Dv1 (no words otherwise)
    off = (off + (size_t)a0.map_ints * 4 + 15) & ~(size_t)15;
    // the fused vertexing's kept tracks lie over hits, bounds and map: they are listed when the event's last
    // chunk has been fitted.  (Behind the items they took 26 bytes per seed of the largest event, and with
    // them a resident workgroup per unit: 10 000 events of 150 seeds, 600 hits: 282 us with three, 243 with four;
    // 20 000 uneven events of up to 466 seeds, 865 and 753 us.)
    if (VTX) off = max(off, fused_kept_bytes(a0.tcap));
    double *s_fit = reinterpret_cast<double *>(smem + off);
    off += FIT_TAB * 8;
    uint16_t *s_rows = reinterpret_cast<uint16_t *>(smem + off);   // candidates waiting for their fit, per wavefront
    off += (size_t)(BLOCK / 64) * ROW_QUEUE * 2;
    SeedConst *s_c = reinterpret_cast<SeedConst *>(smem + off);
    off += (size_t)a0.scap * sizeof(SeedConst);
    unsigned long long *s_key = reinterpret_cast<unsigned long long *>(smem + off);
    off += (size_t)a0.scap * 8;
    int *s_base = reinterpret_cast<int *>(smem + off);
    off = (off + (size_t)a0.scap * 4 + 15) & ~(size_t)15;
    // items: seed (10 bits) << 16 | LDS position of its UTbX hit (~0: dropped), then the three
    // layers' window results; first-window hits that have to be ranked are listed there before
    uint32_t *it_desc = reinterpret_cast<uint32_t *>(smem + off);
    off = (off + (size_t)a0.icap * 4 + 15) & ~(size_t)15;
    uint32_t *it_res = reinterpret_cast<uint32_t *>(smem + off);
    off = (off + (size_t)a0.icap * 12 + 15) & ~(size_t)15;
    // (the vertexing's survivor masks lie over the seed constants and items)
    const uint32_t items_end = (uint32_t)off;
    __shared__ int s_nx[8];   // next event and its offsets (fetch_event)
    __shared__ int s_bad, s_nacc, s_nitems, s_npre, s_nkept, s_nkpos;
    __shared__ int s_over;   // Dv0: a seed of the chunk has more than max_l3 first-window hits
    __shared__ int s_long;   // Dv1: a seed of the chunk has more than 128 UTbX hits
    __shared__ int s_cut;    // Dv1: the chunk's first seed has more than wcap triplets
    __shared__ int s_wsum[BLOCK / 64];
    {
        const int tid = fresh_tid();
        if (tid < 64) fetch_event(a0, 0, tid, s_nx);
        fit_table(kernel_args<TrackKernArgs>().G, s_fit);
        if (tid == 0) s_over = 0;
    }

    // The next event is fetched while this one is processed: its index (the
    // work counter's atomic) and offsets arrive during phase B, where the
    // last wave, the one with the fewest items, waits for them.
    lds_barrier();
    for (int iter = 0;; ++iter) {
        const TrackKernArgs &Ke = kernel_args<TrackKernArgs>();
        const TrackArgs &a = Ke.a;
        const DevGeom &G = Ke.G;
        const int e = uniform(s_nx[0]), tid = fresh_tid();
        if (e >= a.n_events) break;
        const int s0 = uniform(s_nx[1]), s1 = uniform(s_nx[2]);
        int ho[5];
#pragma unroll
        for (int L = 0; L < 5; ++L) ho[L] = uniform(s_nx[3 + L]);
        if (tid == 0) s_bad = 0;
        lds_barrier();   // s_nx read by every wave before it is refilled
        const bool seeds_ok = (0 <= s0) && (s0 <= s1) && (s1 <= a.n_seeds);
        bool runs_ok = (0 <= ho[0]) && (ho[4] <= a.n_hits), hits_ok = true;
#pragma unroll
        for (int L = 0; L < 4; ++L) {
            runs_ok = runs_ok && (ho[L] <= ho[L + 1]);
            hits_ok = hits_ok && (ho[L + 1] - ho[L] <= 65535);
        }
        hits_ok = hits_ok && runs_ok;
        const int nh = ho[4] - ho[0];
        int bad = 0;
        if (!seeds_ok || !hits_ok) bad = F_BAD_OFFSETS;
        else if (nh > a.hcap || nh > a.max_hits || s1 - s0 > a.max_seeds) bad = F_CAPACITY;
        if (bad) {
            if (tid == 0) atomicOr(a.flags, bad);
            if (VTX && tid == 0) a.vcount[e] = 0;
            // (the flags of the vertexing launch that follows the others when clones are killed)
            if (VTX && a.clone && tid == 0 && (!seeds_ok || s1 - s0 > a.max_seeds))
                atomicOr(a.vflags, seeds_ok ? F_CAPACITY : F_BAD_OFFSETS);
            if (seeds_ok)
                for (int i = s0 + tid; i < s1; i += BLOCK) {
                    write_empty_track(a, i);
                    if (VTX && a.clone && runs_ok) a.score[i] = 0.0f;
                }
            if (tid < 64) fetch_event(a, iter + 1, tid, s_nx);
            lds_barrier();
            continue;
        }
        if (s1 == s0) {
            if (VTX && tid == 0) a.vcount[e] = 0;
            if (tid < 64) fetch_event(a, iter + 1, tid, s_nx);
            lds_barrier();
            continue;
        }
        int hl[4];
#pragma unroll
        for (int L = 0; L < 4; ++L) hl[L] = ho[L] - ho[0];
        // seed frames of the first chunk, computed while the hits are loading;
        // the seeds are loaded first, so that the frames wait for them alone
        const SectorMap map = DV1 ? SectorMap{map_s, a.map_words, Bins{a.map_inv, a.map_off, (float)(32 * a.map_words - 1)},
                                              a.map_reach, a.map_range}
                                  : SectorMap{};
        const bool have0 = tid < min(s1 - s0, a.scap);
        SeedRaw sd0{};
        if (have0) sd0 = load_seed(a, s0 + tid);
        auto first_frames = [&]() {
            if (have0) {
                SeedConst sc{};
                if (!seed_frame(G, sd0.x, sd0.y, sd0.tx, sd0.ty, sd0.qop, sc)) {
                    atomicOr(a.flags, F_NONFINITE);
                    sc.q = __int_as_float(0x7fc00000);   // NaN: no frame
                } else if (DV1) {
                    seed_sectors(G, sd0.y, sd0.ty, sc);
                }
                s_c[tid] = sc;
            }
        };
        if (!stage_hits_w<BLOCK, DV1>(a, G.nsec, map, ho[0], hl, nh, hu_s, hidx_s, E, &s_bad, first_frames)) {
            if (tid == 0) atomicOr(a.flags, F_NONFINITE);
            if (VTX && tid == 0) a.vcount[e] = 0;
            for (int i = s0 + tid; i < s1; i += BLOCK) {
                write_empty_track(a, i);
                if (VTX && a.clone) a.score[i] = 0.0f;
            }
            if (tid < 64) fetch_event(a, iter + 1, tid, s_nx);
            lds_barrier();
            continue;
        }

        // seeds in chunks of at most scap, shortened so that their items fit
        for (int sc0 = s0; sc0 < s1;) {
            const TrackKernArgs &Kc = kernel_args<TrackKernArgs>();
            const TrackArgs &a = Kc.a;
            const DevGeom &G = Kc.G;
            const int n_chunk = min(a.scap, s1 - sc0), tid = fresh_tid();
            if (tid == 0) {
                s_nacc = n_chunk;
                s_nitems = s_npre = INT_MAX;
                s_long = s_cut = 0;
            }
            // phase A: lane per seed, the UTbX bucket range of its first window;
            // every hit of the range inside the window becomes an item (seed, hit)
            const int i = sc0 + tid;
            const bool have = tid < n_chunk;
            // (the seed constants stay in LDS: the first chunk's were left there during staging)
            SeedConst &sc = s_c[have ? tid : 0];
            double m3 = 0.0, W1 = 0.0;
            int n_rng = 0, p_lo = 0, p_hi = 0;
            if (have) {
                if (sc0 != s0) {
                    SeedConst f{};
                    if (!seed_frame(G, a.sx[i], a.sy[i], a.stx[i], a.sty[i], a.sqop[i], f)) {
                        atomicOr(a.flags, F_NONFINITE);
                        f.q = __int_as_float(0x7fc00000);   // NaN: no frame
                    } else if (DV1) {
                        seed_sectors(G, a.sy[i], a.sty[i], f);
                    }
                    sc = f;
                }
                const float q = sc.q;
                if (q == q) {
                    if (DV1) {
                        // Dv1: every UTbX hit of the compatible sectors, no momentum window
                        int klo, khi;
                        sector_span(sc, 3, klo, khi);
                        if (klo <= khi) {
                            p_lo = E[3 * a.nb + klo * a.nbu3];
                            p_hi = E[3 * a.nb + (khi + 1) * a.nbu3];
                        }
                    } else if (G.max_l3 > 0) {
                        m3 = window1_centre(G, sc.c[3], (double)q);
                        W1 = fma(G.w1c1, fabs((double)q), G.w1c0);
                        first_window_range(E, a, G.max_l3, m3, W1, p_lo, p_hi);
                    }
                    n_rng = p_hi - p_lo;
                }
                if (!DV1) {   // Dv1 keeps its sector spans in lo / hi
                    sc.lo = (uint16_t)p_lo;
                    sc.hi = (uint16_t)p_hi;
                }
            }
            // an item per UTbX hit inside the first window (Dv0) or per axial triplet (Dv1)
            auto is_item = [&](int p) { return fabs((double)hu_s[p] - m3) <= W1; };
            int n_win = 0;
            uint32_t in_mask = 0;   // Dv0: in-window flags of the range's first 32 hits
            // Dv1 looks its axial triplets up in the map of UTaX, sixteen lanes per seed (tens of UTbX hits
            // each), and tests those that the map does not rule out, 64 at a time
            int *s_cnt = reinterpret_cast<int *>(s_key);    // free until the scan below
            // triplet flags of a seed's first 128 UTbX hits, kept for the write pass (free until phase B)
            unsigned long long *s_mask = reinterpret_cast<unsigned long long *>(it_res);
            MapSeed *s_ms = reinterpret_cast<MapSeed *>(s_mask + 2 * a.scap);
            // readfirstlane: the compiler then knows the wavefront index is uniform
            const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
            const WindowArgs wa = DV1 ? window_args(a, G) : WindowArgs{};
            const double ff0 = G.ffac[0];
            const float ff0f = (float)ff0;
            if (DV1) {
                if (have) {
                    s_ms[tid] = map_seed(map, G.nsec, sc, p_lo, n_rng);
                    s_mask[2 * tid] = s_mask[2 * tid + 1] = 0ull;
                    s_cnt[tid] = 0;
                }
                lds_barrier();
                if (have && n_rng > 128) s_long = 1;   // (cleared by lane 0 before this barrier, read after the next)
                uint32_t *queue = reinterpret_cast<uint32_t *>(s_ms + a.scap) + wave * 128;
                int qn = 0;   // queued probes (wavefront-uniform)
                auto test = [&](int n) {
                    if (lane < n) {
                        const uint32_t d = queue[lane];
                        const int sl = (int)(d >> 16), p = (int)(d & 0xffffu);
                        if (dv1_triplet(ff0, wa, hu_s, E, s_c[sl], p)) {
                            const int k = p - (int)(s_ms[sl].range & 0xffffu);
                            if (k < 128)
                                atomicOr(reinterpret_cast<uint32_t *>(s_mask) + 4 * sl + (k >> 5), 1u << (k & 31));
                            else
                                atomicAdd(&s_cnt[sl], 1);
                        }
                    }
                };
                auto append = [&](bool maybe, int sl, int p) {
                    const unsigned long long m = __ballot(maybe);
                    if (m == 0ull) return;
                    const int pos = qn + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                                    __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
                    if (maybe) queue[pos] = ((uint32_t)sl << 16) | (uint32_t)p;
                    qn += __popcll(m);
                    if (qn < 64) return;
                    wave_sync();
                    test(64);
                    qn -= 64;
                    const uint32_t rest = queue[64 + lane];
                    wave_sync();
                    queue[lane] = rest;
                };
                // four seeds at a time, two hits of a lane at once, so that their LDS round trips overlap; a
                // lane past its seed's hits looks up the last one (without any: hit 0) and is masked off
                const int l16 = lane & 15;
                for (int s4 = 4 * wave; s4 < n_chunk; s4 += 4 * (BLOCK / 64)) {
                    const int sl = s4 + (lane >> 4);
                    const MapSeed ms = s_ms[min(sl, n_chunk - 1)];
                    const int plo = (int)(ms.range & 0xffffu), nr = sl < n_chunk ? (int)(ms.range >> 16) : 0;
                    int longest = nr;   // of the four
#pragma unroll
                    for (int g = 0; g < 4; ++g) longest = max(longest, __builtin_amdgcn_readlane(nr, 16 * g));
                    for (int k0 = 0; k0 < uniform(longest); k0 += 32) {
                        const int ka = k0 + l16, kb = ka + 16;
                        const int pa = plo + max(min(ka, nr - 1), 0), pb = plo + max(min(kb, nr - 1), 0);
                        const float ua = hu_s[pa], ub = hu_s[pb];
                        const bool ma = map_maybe(map, ms, ff0f, ua), mb = map_maybe(map, ms, ff0f, ub);
                        append((ka < nr) & ma, sl, pa);
                        append((kb < nr) & mb, sl, pb);
                    }
                }
                wave_sync();
                test(qn);
                lds_barrier();
                n_win = have ? s_cnt[tid] + __popcll(s_mask[2 * tid]) + __popcll(s_mask[2 * tid + 1]) : 0;
            } else {
                // four positions per LDS round trip
                for (int k0 = 0; k0 < n_rng; k0 += 4) {
                    float u[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) u[j] = hu_s[k0 + j < n_rng ? p_lo + k0 + j : p_lo];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int k = k0 + j;
                        const bool in = k < n_rng && fabs((double)u[j] - m3) <= W1;
                        n_win += in ? 1 : 0;
                        in_mask |= (in && k < 32) ? 1u << k : 0u;
                    }
                }
            }
            // a seed takes an item per triplet up to wcap (Dv1), or per first-window hit up to max_l3 (Dv0):
            // with more hits than that, and for candidate rows, whose index holds the rank, its hits are
            // listed and ranked first
            const int n_fin = min(n_win, DV1 ? a.wcap : G.max_l3), n_all = n_win;
            if (!DV1 && (CANDS ? n_win > 0 : n_win > n_fin)) s_over = 1;
            int tot, tot_pre = 0, pre = 0;
            const int excl = block_exclusive_scan<BLOCK>(n_fin, s_wsum, &tot);
            const bool over = !DV1 && uniform(s_over);   // uniform: written before a barrier
            // (no more than wcap hits of a seed are listed: the places below the next seed's are all written)
            if (over) pre = block_exclusive_scan<BLOCK>(min(n_win, a.wcap), s_wsum, &tot_pre);
            const int pcap = 3 * a.icap;
            bool acc = have && (excl + n_fin <= a.icap) && n_win <= a.wcap && (!over || pre + n_win <= pcap);
            if (tid == 0 && have && !acc) {
                // one seed alone has more hits than its limit: keep the first ones (flagged)
                atomicOr(a.flags, F_CAPACITY);
                n_win = a.wcap;
                acc = true;
                if (DV1) s_cut = 1;   // (cleared by this lane, read behind a barrier)
            }
            // acceptance is a prefix of the chunk; only the (rare) refused seeds
            // touch the shared counters: the first refused one ends the chunk
            // and its exclusive offsets are the chunk's counts
            if (have && !acc) {
                atomicMin(&s_nacc, tid);
                atomicMin(&s_nitems, excl);
                if (over) atomicMin(&s_npre, pre);
            }
            if (acc) {
                s_key[tid] = ~0ull;
                s_base[tid] = excl;
                if (!DV1) {
                    uint32_t *list = over ? it_res + pre : it_desc + excl;
                    // (the items of a seed that needs no ranks carry their place in the list)
                    const uint32_t d0 = ((uint32_t)tid << 16) | (uint32_t)p_lo;
                    const uint32_t step = over && !CANDS && n_win <= G.max_l3 ? 1u << 26 : 0u;
                    if (n_rng <= 32) {
                        uint32_t m = in_mask;
                        for (int w = 0; m != 0 && w < n_win; ++w) {
                            const int k = __ffs(m) - 1;
                            m &= m - 1;
                            list[w] = d0 + (uint32_t)k + (uint32_t)(w + 1) * step;
                        }
                    } else if (__builtin_expect(a.fine > 1 && n_all > a.wcap, 0)) {
                        list_first(hu_s, E, a, m3, W1, p_lo, p_hi, n_win, (uint32_t)tid << 16, list);
                    } else {
                        for (int k = 0, w = 0; k < n_rng && w < n_win; ++k) {
                            if (is_item(p_lo + k)) {
                                list[w] = d0 + (uint32_t)k + (uint32_t)(w + 1) * step;
                                ++w;
                            }
                        }
                    }
                    // the places of a seed's items decide exact ties in chi2: with wider bins than the
                    // context asks for, hits of one bin are put in the order of its parts
                    if (a.fine > 1 && n_win > 1 && n_win <= G.max_l3) {
                        const Bins fb = fine_bins(a);
                        auto part = [&](uint32_t d) { return bin_of(fb, hu_s[d & 0xffffu]); };
                        for (int w = 1; w < n_win; ++w) {
                            const uint32_t d = list[w] & 0x3ffffffu;
                            const int b = part(d);
                            int p = w;
                            for (; p > 0 && part(list[p - 1]) > b; --p)
                                list[p] = (list[p - 1] & 0x3ffffffu) + (uint32_t)(p + 1) * step;
                            if (p < w) list[p] = d + (uint32_t)(p + 1) * step;
                        }
                    }
                    if (over)   // (a truncated seed does not fill all of its ranks)
                        for (int w = 0; w < n_fin; ++w) it_desc[excl + w] = ~0u;
                } else {
                    // Dv1, lane per seed: the triplets among the first 128 UTbX hits,
                    // from the counting pass's flags, in hit order
                    int w = 0;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        unsigned long long m = 64 * j < n_rng ? s_mask[2 * tid + j] : 0ull;
                        for (; m != 0 && w < n_fin; ++w) {
                            const int k = 64 * j + __ffsll((long long)m) - 1;
                            m &= m - 1;
                            it_desc[excl + w] = ((uint32_t)tid << 16) | (uint32_t)(p_lo + k);
                        }
                    }
                }
            }
            if (DV1 && uniform(s_long)) {   // uniform: written before a barrier
                // seeds with more than 128 UTbX hits: the rest of their triplets, a
                // wavefront per seed, after the flagged ones
                lds_barrier();
                // a truncated seed keeps its first triplets in the order of its hits' sectors and indices.
                // Where several wavefronts placed the layer, its sectors are put in that order first; the
                // chunk's other seeds, found in the former one, then come in the next chunk
                const bool redo = BLOCK >= 512 && uniform(s_cut);
                if (__builtin_expect(redo, 0)) {
                    int klo, khi;
                    sector_span(s_c[0], 3, klo, khi);
                    klo = uniform(klo);
                    khi = uniform(khi);
                    for (int k = klo; k <= khi; ++k) {
                        const int p0 = uniform(E[3 * a.nb + k]), p1 = uniform(E[3 * a.nb + k + 1]);
                        sort_run<BLOCK>(hu_s + p0, hidx_s + p0, p1 - p0);
                    }
                    if (tid == 0) {
                        s_nacc = 1;
                        s_nitems = a.wcap;
                    }
                    lds_barrier();
                }
                const int nacc_w = uniform(s_nacc), nit_w = uniform(min(min(tot, s_nitems), a.icap));
                for (int sl = wave; sl < nacc_w; sl += BLOCK / 64) {
                    const int pk = uniform((int)s_ms[sl].range), plo = pk & 0xffff, nr = pk >> 16;
                    if (nr <= 128) continue;
                    const SeedConst &scw = s_c[sl];
                    const int base = s_base[sl], cap = (sl + 1 < nacc_w ? s_base[sl + 1] : nit_w) - base;
                    int w = redo ? 0 : __popcll(s_mask[2 * sl]) + __popcll(s_mask[2 * sl + 1]);
                    for (int k0 = redo ? 0 : 128; k0 < nr && w < cap; k0 += 64) {
                        const bool f = k0 + lane < nr && dv1_triplet(ff0, wa, hu_s, E, scw, plo + k0 + lane);
                        const unsigned long long m = __ballot(f);
                        const int pre = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                                   __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
                        if (f && w + pre < cap)
                            it_desc[base + w + pre] = ((uint32_t)sl << 16) | (uint32_t)(plo + k0 + lane);
                        w += __popcll(m);
                    }
                }
            }
            lds_barrier();
            const int nacc = uniform(s_nacc), n_items = uniform(min(min(tot, s_nitems), a.icap));
            if (sc0 == s0 && tid >= BLOCK - 64) fetch_event(a, iter + 1, tid - (BLOCK - 64), s_nx);
            if (over) {
                // phase B0: lane per listed hit, its rank in the seed's window is its place among the items
                // (seeds with no more hits than are used keep their list's order)
                const int n_pre = uniform(min(min(tot_pre, s_npre), pcap));
                for (int it = fresh_tid(); it < n_pre; it += BLOCK) {
                    const uint32_t d = it_res[it] & 0x3ffffffu;
                    const int sl = (int)(d >> 16), w = (int)(it_res[it] >> 26);
                    const int r = w > 0 ? w - 1 : first_window_rank(G, hu_s, hidx_s, s_c[sl], (int)(d & 0xffffu));
                    if (r >= 0 && r < G.max_l3) it_desc[s_base[sl] + r] = d;
                }
                lds_barrier();
                if (tid == 0) s_over = 0;   // (read by every wave before the barrier)
            }
            // phase B1: a unit is 64 items in one refined window's layer
            {
                const TrackKernArgs &Ki = kernel_args<TrackKernArgs>();
                const TrackArgs &a = Ki.a;
                const DevGeom &G = Ki.G;
                const int nblk = (n_items + 63) >> 6, lane = fresh_tid() & 63, icap = a.icap;
                const WindowArgs wa = window_args(a, G);
                const double ff[3] = {G.ffac[0], G.ffac[1], G.ffac[2]};
                for (int u = wave, L = 0, b = wave; u < 3 * nblk; u += BLOCK / 64, b += BLOCK / 64) {
                    while (b >= nblk) {
                        b -= nblk;
                        ++L;
                    }
                    const int it = 64 * b + lane;
                    if (it < n_items) {
                        const uint32_t d = it_desc[it];
                        if (d != ~0u)
                            it_res[L * icap + it] = window_best2<DV1>(wa, L == 0 ? ff[0] : L == 1 ? ff[1] : ff[2], hu_s,
                                                                      hidx_s, E, s_c[d >> 16], L, (int)(d & 0xffffu));
                    }
                }
            }
            lds_barrier();
            // phase B2: the valid items' candidates, queued per wavefront and fitted 64 at a time, a lane each
            {
                const TrackKernArgs &Ki = kernel_args<TrackKernArgs>();
                const TrackArgs &a = Ki.a;
                const DevGeom &G = Ki.G;
                const int lane = fresh_tid() & 63;
                uint16_t *rows = s_rows + wave * ROW_QUEUE;
                int qn = 0;   // queued candidates (wavefront-uniform)
                auto fit_rows = [&](int n) {
                    const bool row = lane < n;
                    const int r = rows[lane], it = r & 0x1fff, t = r >> 13;
                    int bp[4] = {-1, -1, -1, 0}, c = 0, sl = 0, mask = 8;
                    double al = 0.0, be = 0.0, c2 = 0.0;
                    if (row) {
                        const uint32_t d = it_desc[it];
                        sl = (int)(d >> 16);
                        bp[3] = (int)(d & 0xffffu);
                        const uint32_t w0 = it_res[it], w1 = it_res[a.icap + it], w2 = it_res[2 * a.icap + it];
                        const ItemOptions o = item_options<DV1>(G, w0, w1, w2);
                        const int r3 = DV1 ? (int)hidx_s[bp[3]] : it - s_base[sl];
                        c = r3 * (G.nw[0] * G.nw[1] * G.nw[2]) + candidate_hits(G, o, w0, w1, w2, t, bp);
                        mask = o.mask;
                        double rho[4];
                        candidate_rho(hu_s, s_c[sl], bp, rho);
                        fit_set(G, s_fit, mask, rho, al, be, c2);
                    }
                    if (CANDS) {
                        if (row) write_candidate_row(a, G, sc0 + sl, __popc(mask), c, al, be, c2, hu_s, hidx_s, bp);
                    } else if (row) {
                        atomicMin(&s_key[sl], DV1 ? pack_key_dv1(__popc(mask), c2, c) : pack_key(__popc(mask), c2, c));
                    }
                };
                for (int b = wave; 64 * b < n_items; b += BLOCK / 64) {
                    const int it = 64 * b + lane;
                    int n = 0;
                    if (it < n_items && it_desc[it] != ~0u)
                        n = item_options<DV1>(G, it_res[it], it_res[a.icap + it], it_res[2 * a.icap + it]).cands;
                    for (int t = 0;; ++t) {
                        const unsigned long long m = __ballot(t < n);
                        if (m == 0ull) break;
                        const int pos = qn + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                                        __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
                        if (t < n) rows[pos] = (uint16_t)(it | (t << 13));
                        qn += __popcll(m);
                        if (qn >= 64) {
                            wave_sync();
                            fit_rows(64);
                            qn -= 64;
                            const uint16_t rest = rows[64 + lane];
                            wave_sync();
                            rows[lane] = rest;
                        }
                    }
                }
                if (qn > 0) {
                    wave_sync();
                    fit_rows(qn);
                }
            }
            {
            const int tid = fresh_tid(), i = sc0 + tid;
            // the seed parameters of phase C are loaded before the barrier: their
            // latency overlaps the wait
            SeedRaw sd{};
            if (!CANDS && tid < nacc) sd = load_seed(a, i);
            lds_barrier();
            // phase C: lane per seed, write the winner; then its ghost score, the
            // network run by each wavefront with a winner as a whole
            bool won = false;
            StoredTrack t{};
            int wbp[4] = {-1, -1, -1, -1};
            if (!CANDS && tid < nacc) {
                const int per_r3 = G.nw[0] * G.nw[1] * G.nw[2];
                const unsigned long long key = s_key[tid];
                if (key == ~0ull) {
                    write_empty_track(a, i);
                } else {
                    const int c = (int)(key & (DV1 ? 0xfffffull : 127ull));
                    const int b0 = s_base[tid], b1 = tid + 1 < nacc ? s_base[tid + 1] : n_items;
                    int it = b0 + c / per_r3, cw = c;
                    if (DV1) {
                        // the seed's item whose UTbX hit has the winning index
                        const int i3 = c / per_r3;
                        it = b0;
                        for (int k = b0; k < b1; ++k)
                            if (it_desc[k] != ~0u && (int)hidx_s[it_desc[k] & 0xffffu] == i3) it = k;
                    }
                    // (hits that were not ranked stand in window order: the position orders only exact
                    // ties, and the winner alone is ranked where its index is asked for)
                    const uint32_t w0 = it_res[it], w1 = it_res[a.icap + it], w2 = it_res[2 * a.icap + it];
                    const ItemOptions o = item_options<DV1>(G, w0, w1, w2);
                    const int rest = c % per_r3, i2 = rest % G.nw[2], i1 = (rest / G.nw[2]) % G.nw[1],
                              i0 = rest / (G.nw[2] * G.nw[1]);
                    int bp[4];
                    bp[0] = o.n0 > 0 ? (int)(i0 ? w0 >> 16 : w0 & 0xffffu) : -1;
                    bp[1] = o.n1 > 0 ? (int)(i1 ? w1 >> 16 : w1 & 0xffffu) : -1;
                    bp[2] = o.n2 > 0 ? (int)(i2 ? w2 >> 16 : w2 & 0xffffu) : -1;
                    bp[3] = (int)(it_desc[it] & 0xffffu);
                    if (!DV1 && a.cand)
                        cw = first_window_rank(G, hu_s, hidx_s, s_c[tid], bp[3]) * per_r3 + rest;
                    t = write_track(a, G, s_fit, i, sd, s_c[tid], hu_s, hidx_s, bp, cw);
                    won = true;
#pragma unroll
                    for (int L = 0; L < 4; ++L) wbp[L] = bp[L];
                }
            }
            if (!CANDS && a.fuse_mlp) {
                // the network on the chunk's tracks: their features go over the seed constants, keys and
                // items (all read by now)
                float f[NF] = {};
                if (won) {
                    float hu4[4];
                    int mask = 0;
#pragma unroll
                    for (int L = 0; L < 4; ++L) {
                        hu4[L] = hu_s[max(wbp[L], 0)];
                        mask |= wbp[L] >= 0 ? (1 << L) : 0;
                    }
                    ghost_features(G, t.x, t.y, t.tx, t.ty, t.qop, t.chi2, __popc(mask), sd.x, sd.y, sd.tx, sd.ty,
                                   sd.qop, hu4, mask, f);
                }
                const float score = mlp_score_rows<BLOCK>(a.W, reinterpret_cast<float *>(s_c), s_wsum, won, f);
                if (won) {
                    t.score = score;
                    a.score[i] = score;
                }
            }
            if (VTX && a.clone && tid < nacc) clone_record(clone_carve(smem + items_end, a.tcap), i - s0, won, wbp, hidx_s, t.chi2);
            if (VTX && !a.clone && sc0 + nacc == s1) {
                // kept tracks listed in slot order, split by seed charge: the earlier chunks' as they were
                // written, then this one's
                const bool kept = won && t.score < a.score_max;
                const Kept K = kept_carve(smem + VTX_PAD, a.tcap);
                int nk = 0, nkp = 0;
                if (sc0 > s0) keep_stored<BLOCK>(a, K, s0, sc0, nk, nkp, s_wsum);
                kept_append<BLOCK>(K, a.tcap, kept, sd.qop > 0.0f, make_float4(t.x, t.y, t.tx, t.ty), t.qop, i - s0, nk, nkp,
                                   s_wsum);
                if (tid == 0) {
                    s_nkept = nk;
                    s_nkpos = nkp;
                }
            }
            }
            lds_barrier();
            sc0 += nacc;
        }
        if (VTX && kernel_args<TrackKernArgs>().a.clone) {
            const TrackKernArgs &Kf = kernel_args<TrackKernArgs>();
            int nk = 0, nkp = 0;
            kill_and_score<BLOCK>(Kf.a, Kf.G, s0, s1, ho, kept_carve(smem + VTX_PAD, Kf.a.tcap), clone_carve(smem + items_end, Kf.a.tcap),
                                  reinterpret_cast<uint32_t *>(s_c), s_wsum, nk, nkp);
            if (fresh_tid() == 0) {
                s_nkept = nk;
                s_nkpos = nkp;
            }
            lds_barrier();
        }
        if (VTX) {
            const TrackKernArgs &Kv = kernel_args<TrackKernArgs>();
            vertex_event_block<BLOCK, XTR>(Kv.a, Kv.G, e, s0, uniform(s_nkept), uniform(s_nkpos), kept_carve(smem + VTX_PAD, Kv.a.tcap),
                                           Kv.a.tcap, reinterpret_cast<int *>(s_c),
                                           (int)(items_end - (uint32_t)((unsigned char *)s_c - smem)) / 4, s_wsum);
        }
    }
}

// ------------------------------------------------------------ event order
//
// Largest-first order of a batch for the persistent launches: a counting sort
// of a work estimate (seeds + hits / 8), descending, within classes of events
// that a launch of their own takes (OrderArgs).  ORDER_ROWS workgroups count
// their events in LDS and leave a row of counts each; the same workgroups then
// place them from the rows' sums.  Nothing has to be cleared between calls and
// no global atomic is taken (20 000 events: 4 and 16.5 us for the two launches
// with atomic counts and cursors, 4.6 and 6.0 so).  Events of one bin in any order
// (results do not depend on the processing order).
constexpr int ORDER_BINS = 256, ORDER_ROWS = 8, ORDER_BLOCK = 1024, MAX_TIERS = 3;
constexpr int ORDER_WS = ORDER_ROWS * ORDER_BINS + 64;   // ints ahead of the order array; the classes' ends are the last

struct OrderArgs {
    const int *seed_off, *hit_off;
    int n, tiers;                     // events; classes (the last one's are the smallest)
    int max_seeds[MAX_TIERS], max_hits[MAX_TIERS];   // largest event of a class (class 0 takes all)
    int shift;                        // of the work estimate, so that it has 256 / tiers bins
    int *ws, *order;
};

__device__ __forceinline__ int order_bin(const OrderArgs &a, int e)
{
    const int s = a.seed_off[e + 1] - a.seed_off[e], h = a.hit_off[4 * e + 4] - a.hit_off[4 * e];
    int c = 0;
    // (bad offsets: the first class, which has the declared limits)
    while (c + 1 < a.tiers && 0 <= s && s <= a.max_seeds[c + 1] && 0 <= h && h <= a.max_hits[c + 1]) ++c;
    const int bins = ORDER_BINS / a.tiers;
    return c * bins + bins - 1 - min((min(max(s, 0), 1 << 20) + min(max(h, 0), 1 << 20) / 8) >> a.shift, bins - 1);
}

__global__ __launch_bounds__(ORDER_BLOCK) void k_order_count(OrderArgs a)
{
    __shared__ int h[ORDER_BINS];
    const int t = threadIdx.x;
    if (t < ORDER_BINS) h[t] = 0;
    __syncthreads();
    for (int e = blockIdx.x * ORDER_BLOCK + t; e < a.n; e += gridDim.x * ORDER_BLOCK) atomicAdd(&h[order_bin(a, e)], 1);
    __syncthreads();
    if (t < ORDER_BINS) a.ws[blockIdx.x * ORDER_BINS + t] = h[t];
}

__global__ __launch_bounds__(ORDER_BLOCK) void k_order_place(OrderArgs a)
{
    __shared__ int at[ORDER_BINS];
    __shared__ int s_wsum[ORDER_BLOCK / 64];
    const int t = threadIdx.x;
    int all = 0, mine = 0;   // of bin t: every workgroup's events, the earlier workgroups'
    if (t < ORDER_BINS) {
#pragma unroll
        for (int r = 0; r < ORDER_ROWS; ++r) {
            const int c = a.ws[r * ORDER_BINS + t];
            all += c;
            mine += r < (int)blockIdx.x ? c : 0;
        }
    }
    int tot;
    const int start = block_exclusive_scan<ORDER_BLOCK>(all, s_wsum, &tot);
    if (t < ORDER_BINS) at[t] = start + mine;
    const int bins = ORDER_BINS / a.tiers;
    if (blockIdx.x == 0 && t < a.tiers * bins && (t + 1) % bins == 0) a.ws[ORDER_ROWS * ORDER_BINS + t / bins] = start + all;
    __syncthreads();
    for (int e = blockIdx.x * ORDER_BLOCK + t; e < a.n; e += gridDim.x * ORDER_BLOCK) {
        const int pos = atomicAdd(&at[order_bin(a, e)], 1);
        if (pos < a.n) a.order[pos] = e;   // (always)
    }
}

// Sets n ints to v (graph-safe: a kernel, not a memset node).
__global__ void k_fill_i32(int *p, int v, int n)
{
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) p[k] = v;
}

// Marks every candidate row empty (nhits 0) before a candidate-scoring pass.
__global__ void k_clear_rows(int *r_nhits, long long n)
{
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long long)gridDim.x * blockDim.x)
        r_nhits[k] = 0;
}

// Standalone ghost-killer: one workgroup per event (grid-stride), lane per seed.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_ghost(GhostArgs a, DevGeom G)
{
    for (int e = blockIdx.x; e < a.n_events; e += gridDim.x) {
        const int s0 = a.seed_off[e], s1 = a.seed_off[e + 1];
        int ho[5];
#pragma unroll
        for (int L = 0; L < 5; ++L) ho[L] = a.hit_off[4 * e + L];
        bool ok = (0 <= s0) && (s0 <= s1) && (s1 <= a.n_seeds) && (0 <= ho[0]) && (ho[4] <= a.n_hits);
#pragma unroll
        for (int L = 0; L < 4; ++L) ok = ok && (ho[L] <= ho[L + 1]);
        if (!ok) {
            if (threadIdx.x == 0) atomicOr(a.flags, F_BAD_OFFSETS);
            continue;
        }
        // uniform trip count: the network runs on whole wavefronts
        for (int ib = s0; ib < s1; ib += BLOCK) {
            const int i = ib + (int)threadIdx.x;
            bool row = false;
            float f[NF];
            if (i < s1) {
                const int nh = a.nhits[i];
                const int hh[4] = {a.h0[i], a.h1[i], a.h2[i], a.h3[i]};
                float hu4[4];
                int has = 0;
                bool hit_ok = true;
#pragma unroll
                for (int L = 0; L < 4; ++L) {
                    hu4[L] = 0.0f;
                    if (hh[L] >= 0) {
                        if (hh[L] < ho[L + 1] - ho[L]) {
                            hu4[L] = a.hu[ho[L] + hh[L]];
                            has |= 1 << L;
                        } else {
                            hit_ok = false;
                        }
                    }
                }
                if (nh > 0 && !hit_ok) atomicOr(a.flags, F_BAD_OFFSETS);
                row = nh > 0 && hit_ok;
                if (row)
                    ghost_features(G, a.x[i], a.y[i], a.tx[i], a.ty[i], a.qop[i], a.chi2[i], nh, a.sx[i], a.sy[i],
                                   a.stx[i], a.sty[i], a.sqop[i], hu4, has, f);
                else
                    a.score[i] = 0.0f;
            }
            if (__ballot(row) != 0) {
                float mw[MLP_LANE_WORDS];
                mlp_lane_weights(a.W, mw);
                const float sc = mlp_score_wave(mw, f, row);
                if (row) a.score[i] = sc;
            }
        }
    }
}

// ----------------------------------------------------------------- vertex

// Newton-Raphson point of closest approach in float64.  Offsets s, t are
// z - z_ref on each trajectory.  Returns false for (near-)parallel tracks or
// a singular Newton system.
__device__ __forceinline__ bool pca64(const DevGeom &G, double x1, double y1, double tx1, double ty1, double g1, double x2,
                             double y2, double tx2, double ty2, double g2, double &vx, double &vy, double &vz,
                             double &doca, double &s_out, double &t_out)
{
    const double wx = x1 - x2, wy = y1 - y2;
    const double nx = ty1 - ty2, ny = tx2 - tx1, nz = tx1 * ty2 - ty1 * tx2;
    const double nn = nx * nx + ny * ny + nz * nz;
    if (nn < 1e-12) return false;
    // w x d = (wy, -wx, wx*ty - wy*tx) for w = (wx, wy, 0), d = (tx, ty, 1)
    const double inn = 1.0 / nn;
    const double base = wy * nx - wx * ny;
    double s = -(base + (wx * ty2 - wy * tx2) * nz) * inn;
    double t = -(base + (wx * ty1 - wy * tx1) * nz) * inn;
    for (int it = 0; it < G.newton_iters; ++it) {
        const double X1 = x1 + tx1 * s + g1 * s * s, Y1 = y1 + ty1 * s;
        const double X2 = x2 + tx2 * t + g2 * t * t, Y2 = y2 + ty2 * t;
        const double Dx = X1 - X2, Dy = Y1 - Y2, Dz = s - t;
        const double p1x = tx1 + 2.0 * g1 * s, p2x = tx2 + 2.0 * g2 * t;
        const double gr1 = Dx * p1x + Dy * ty1 + Dz;
        const double gr2 = -(Dx * p2x + Dy * ty2 + Dz);
        const double h11 = p1x * p1x + ty1 * ty1 + 1.0 + 2.0 * g1 * Dx;
        const double h22 = p2x * p2x + ty2 * ty2 + 1.0 - 2.0 * g2 * Dx;
        const double h12 = -(p1x * p2x + ty1 * ty2 + 1.0);
        const double det = h11 * h22 - h12 * h12;
        const double tr = h11 + h22;
        if (fabs(det) < 1e-12 * tr * tr) return false;
        const double idet = 1.0 / det;
        const double ds = (h22 * gr1 - h12 * gr2) * idet;
        const double dt = (h11 * gr2 - h12 * gr1) * idet;
        s -= ds;
        t -= dt;
    }
    const double X1 = x1 + tx1 * s + g1 * s * s, Y1 = y1 + ty1 * s;
    const double X2 = x2 + tx2 * t + g2 * t * t, Y2 = y2 + ty2 * t;
    const double Dx = X1 - X2, Dy = Y1 - Y2, Dz = s - t;
    vx = 0.5 * (X1 + X2);
    vy = 0.5 * (Y1 + Y2);
    vz = G.zref + 0.5 * (s + t);
    doca = sqrt(Dx * Dx + Dy * Dy + Dz * Dz);
    s_out = s;
    t_out = t;
    return true;
}

// Invariant masses of a vertex (pi+ pi-, and p pi with the faster track as the
// proton; MeV) from the seed momenta and the trajectory tangents at the points
// of closest approach (offsets s, t from z_ref), then the four trigger-line
// networks (12 -> 32 ReLU -> 1 sigmoid, float32) on the pair and the vertex.
__device__ __forceinline__ void vertex_extras(const DevGeom &G, const float *WLg, float4 A, float4 B, double g1, double g2,
                                     float q1, float q2, double s, double t, float4 V, float out[6])
{
    const double MPI = 0.13957039, MPR = 0.93827209;
    const double d1x = (double)A.z + 2.0 * g1 * s, d1y = A.w, d2x = (double)B.z + 2.0 * g2 * t, d2y = B.w;
    const double n1 = sqrt(d1x * d1x + d1y * d1y + 1.0), n2 = sqrt(d2x * d2x + d2y * d2y + 1.0);
    const double p1 = 1.0 / fabs((double)q1), p2 = 1.0 / fabs((double)q2);
    const double Sx = p1 * d1x / n1 + p2 * d2x / n2;
    const double Sy = p1 * d1y / n1 + p2 * d2y / n2;
    const double Sz = p1 / n1 + p2 / n2;
    const double ss = Sx * Sx + Sy * Sy + Sz * Sz;
    const double e1 = sqrt(p1 * p1 + MPI * MPI), e2 = sqrt(p2 * p2 + MPI * MPI);
    double m2 = (e1 + e2) * (e1 + e2) - ss;
    const double mpipi = 1000.0 * sqrt(m2 > 0.0 ? m2 : 0.0);
    const double ep = p1 >= p2 ? sqrt(p1 * p1 + MPR * MPR) + e2 : sqrt(p2 * p2 + MPR * MPR) + e1;
    m2 = ep * ep - ss;
    const double mppi = 1000.0 * sqrt(m2 > 0.0 ? m2 : 0.0);
    out[0] = (float)mpipi;
    out[1] = (float)mppi;
    float f[LINE_NF];
    f[0] = (float)log(p1);
    f[1] = (float)log(p2);
    f[2] = (float)(d1x / 0.3);
    f[3] = (float)(d1y / 0.3);
    f[4] = (float)(d2x / 0.3);
    f[5] = (float)(d2y / 0.3);
    f[6] = V.z * 1e-3f;
    f[7] = sqrtf(V.x * V.x + V.y * V.y) * 0.01f;
    f[8] = V.w;
    f[9] = (float)((mpipi - 497.6) * 0.01);
    f[10] = (float)((mppi - 1115.7) * 0.01);
    f[11] = (float)sqrt(Sx * Sx + Sy * Sy);
    asm volatile("" : "+s"(WLg));
    cfloat *WL = (cfloat *)(WLg);
#pragma unroll
    for (int l = 0; l < 4; ++l) {
        cfloat *W = WL + l * LINE_NW, *b1 = W + LINE_NH * LINE_NF, *w2 = b1 + LINE_NH, *b2 = w2 + LINE_NH;
        float z = b2[0];
#pragma unroll
        for (int j = 0; j < LINE_NH; ++j) {
            float a = b1[j];
#pragma unroll
            for (int k = 0; k < LINE_NF; ++k) a = fmaf(W[j * LINE_NF + k], f[k], a);
            z = fmaf(w2[j], fmaxf(a, 0.0f), z);
        }
        out[2 + l] = 1.0f / (1.0f + __expf(-z));
    }
}

// Standalone vertexing (ds_vertex): a workgroup per event (work-stolen); the
// event's kept tracks (nhits > 0, score < score_max) are compacted into LDS in
// slot order, then the pairs go through vertex_event_block, the routine of the
// fused step.  LDS: the survivor masks, then the kept tracks (kept_lds_bytes).
template <int BLOCK, bool XTR>
__global__ __launch_bounds__(BLOCK) void k_vertex(VertexArgs a, DevGeom G)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int MASK = vtx_mask_ints(BLOCK);
    static_assert(MASK * 4 >= VTX_PAD, "the pair loop may read VTX_PAD bytes ahead of the kept tracks");
    int *mask = reinterpret_cast<int *>(smem);
    const Kept K = kept_carve(smem + MASK * 4, a.tcap);
    __shared__ int s_nx[3];   // next event and its seed offsets
    __shared__ int s_wsum[BLOCK / 64];
    const int tid = threadIdx.x;
    // the next event and its offsets, by one wave, while the others work
    auto fetch = [&](int iter) {
        const int lane = tid & 63;
        int en = 0;
        if (lane == 0) en = grab_event(a.counter, a.n_events, a.ev_single, nullptr, -1, nullptr, iter);
        en = __builtin_amdgcn_readfirstlane(en);
        if (lane == 0) s_nx[0] = en;
        if (lane < 2 && en < a.n_events) s_nx[1 + lane] = a.seed_off[en + lane];
    };
    if (tid < 64) fetch(0);
    lds_barrier();
    for (int iter = 0;; ++iter) {
        const int e = uniform(s_nx[0]), s0 = uniform(s_nx[1]), s1 = uniform(s_nx[2]);
        if (e >= a.n_events) break;
        lds_barrier();   // s_nx read by every wave before it is refilled
        const bool ok = (0 <= s0) && (s0 <= s1) && (s1 <= a.n_seeds);
        if (!ok || s1 - s0 > a.tcap || s1 - s0 > a.max_seeds) {
            if (tid == 0) {
                atomicOr(a.flags, ok ? F_CAPACITY : F_BAD_OFFSETS);
                a.vcount[e] = 0;
            }
            if (tid >= BLOCK - 64) fetch(iter + 1);
            lds_barrier();
            continue;
        }
        // kept tracks, in slot order per seed charge
        int n = 0, np = 0;
        for (int base = s0; base < s1; base += BLOCK) {
            const int i = base + tid;
            const bool kept = (i < s1) && (a.nhits[i] > 0) && (a.score[i] < a.score_max);
            float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            float qv = 0.0f;
            bool positive = false;
            if (kept) {
                v = make_float4(a.x[i], a.y[i], a.tx[i], a.ty[i]);
                qv = a.qop[i];
                positive = a.sqop[i] > 0.0f;
            }
            kept_append<BLOCK>(K, a.tcap, kept, positive, v, qv, i - s0, n, np, s_wsum);
        }
        if (tid >= BLOCK - 64) fetch(iter + 1);
        lds_barrier();   // the kept tracks are visible
        vertex_event_block<BLOCK, XTR>(a, G, e, s0, n, np, K, a.tcap, mask, MASK, s_wsum);
        lds_barrier();   // the event's LDS is free again
    }
}

// Clone killing: one wavefront per event.  A found track is killed when
// another found track of the event shares more than two UT hits with it and
// has more hits, or as many and a lower chi2, or both equal and a lower slot.
// Decisions are taken on LDS copies, so the kills of one event do not depend
// on each other; a killed track is written as "no track".
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_clone(CloneArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    unsigned char *wb = smem + (size_t)wid * (size_t)a.tcap * 16;
    unsigned long long *hp = reinterpret_cast<unsigned long long *>(wb);
    int *nh = reinterpret_cast<int *>(wb + (size_t)a.tcap * 8);
    float *c2 = reinterpret_cast<float *>(wb + (size_t)a.tcap * 12);
    const int waves = (int)gridDim.x * (BLOCK / 64);
    for (int e = (int)blockIdx.x * (BLOCK / 64) + wid; e < a.n_events; e += waves) {
        const int s0 = a.seed_off[e], s1 = a.seed_off[e + 1];
        const bool ok = (0 <= s0) && (s0 <= s1) && (s1 <= a.n_seeds);
        if (!ok || s1 - s0 > a.tcap || s1 - s0 > a.max_seeds) {
            if (lane == 0) atomicOr(a.flags, ok ? F_CAPACITY : F_BAD_OFFSETS);
            continue;
        }
        const int n = s1 - s0;
        for (int k = lane; k < n; k += 64) {
            const int i = s0 + k;
            const int h[4] = {a.h0[i], a.h1[i], a.h2[i], a.h3[i]};
            unsigned long long p = 0;
#pragma unroll
            for (int L = 0; L < 4; ++L)
                p |= (unsigned long long)(h[L] >= 0 ? ((unsigned)h[L] & 0xffffu) : 0xffffu) << (16 * L);
            hp[k] = p;
            nh[k] = a.nhits[i];
            c2[k] = a.chi2[i];
        }
        wave_sync();
        for (int k = lane; k < n; k += 64) {
            const int nk = nh[k];
            if (nk <= 0) continue;
            const unsigned long long pk = hp[k];
            const float ck = c2[k];
            bool killed = false;
            for (int j = 0; j < n && !killed; ++j) {
                const int nj = nh[j];
                if (j == k || nj <= 0) continue;
                const unsigned long long pj = hp[j];
                int shared = 0;
#pragma unroll
                for (int L = 0; L < 4; ++L) {
                    const unsigned hk = (unsigned)(pk >> (16 * L)) & 0xffffu;
                    shared += (hk != 0xffffu && hk == ((unsigned)(pj >> (16 * L)) & 0xffffu)) ? 1 : 0;
                }
                if (shared <= 2) continue;
                const float cj = c2[j];
                killed = nj > nk || (nj == nk && (cj < ck || (cj == ck && j < k)));
            }
            if (killed) {
                const int i = s0 + k;
                a.x[i] = 0.0f;
                a.y[i] = 0.0f;
                a.tx[i] = 0.0f;
                a.ty[i] = 0.0f;
                a.qop[i] = 0.0f;
                a.chi2[i] = 0.0f;
                if (a.score) a.score[i] = 0.0f;
                a.h0[i] = -1;
                a.h1[i] = -1;
                a.h2[i] = -1;
                a.h3[i] = -1;
                a.nhits[i] = 0;
                if (a.cand) a.cand[i] = -1;
            }
        }
        wave_sync();
    }
}

}  // namespace ds
