// Pixel objects and track candidates (Sec. 2.1 of the paper and its
// kernel-flow figure, Sec. 3): pixel line segments (pLS, seeds of four
// pixel hits) linked to the kept quintuplets (pT5) and to the triplets
// (pT3), cross-cleaning of the collections, and the track candidates.
//
// Readings of the paper taken here (it gives no formula):
//  - a pLS links to an object inside a window around its direction (tangent
//    at the beam line, cot theta) when the chain of its four pixel hits and
//    the object's anchors passes an r-phi chi2 about the circle through its
//    first hit and two anchors and an r-z chi2 about the straight line in
//    arc length (score = their sum);
//  - inside the pT5 collection, and then inside the pT3 collection built
//    from the pLS that no surviving pT5 uses, a candidate survives iff no
//    candidate sharing one of its hits (pixel or outer) has a smaller
//    (score, seed, hit tuple) key;
//  - cross-cleaning in the paper's order: pT3 near a pT5 in eta-phi or
//    sharing a hit with one; kept quintuplets near or sharing a hit with a
//    pT5 or cleaned pT3; unlinked pLS against all of them, then among
//    themselves (the smaller seed index keeps a shared pixel hit);
//  - track candidates: pT5, pT3, T5 and pLS left after cleaning.
//
// The collections are small (thousands per event) and a step's work takes a
// few microseconds, so what counts is how many launches and dependent loads
// there are: ten kernels (eleven for larger batches), each with enough lanes
// per object that its loads are one chain.  A wave takes a few seeds and scans
// the objects of their event from a per-event list; 16 lanes take a
// candidate, a wave an object of the cross-cleaning.  Per-hit minima use
// 64-bit atomics on (removal, score bits, seed), taken as soon as a candidate
// is accepted; ties on that key are resolved by the hit tuples.  List counters
// take one atomic per wave and list key (one address taking an atomic per
// object would serialise thousands of device-scope atomics).  Every per-event
// list is kept per (event, azimuth bin), so that a seed or an object scans only
// the bins its window or closeness reaches; the survivors of a step are marks
// on the entries of the seeds' or quintuplets' list and no list of their own.
// One PU200 event: 205 us in 20 launches with a pass, a count, a scan and a
// list per step, 88 us like this.
#include <algorithm>

#include "lst_access.hpp"
#include "lst_cuts.hpp"

namespace lst {

__device__ __forceinline__ int px_lane() { return threadIdx.x & 63; }

constexpr unsigned long long KEY_NONE = ~0ull;

// list `list` of pl_cnt / pl_off / pl_fill
__device__ __forceinline__ int32_t *pl(const EvDev &E, int32_t *base, int list)
{
    return base + (size_t)list * ((size_t)E.cap_ev * PX_NB + 1);
}

// azimuth bin of a direction (tangent t.x, t.y): floor((phi + pi) PX_NB /
// 2 pi), clamped; monotone in phi
constexpr float PX_PI = 3.14159265358979f;
__device__ __forceinline__ int phi_bin(float phi)
{
    const float b = (phi + PX_PI) * (PX_NB / (2.0f * PX_PI));
    return b > 0.0f ? (int)fminf(b, (float)(PX_NB - 1)) : 0;
}

__device__ __forceinline__ int dir_bin(const float4 &d) { return phi_bin(atan2f(d.y, d.x)); }

// The bins holding every direction within wphi of d in azimuth: [a0, b0]
// and, across the wrap at +-pi, [a1, b1] (empty when a1 > b1).  A NaN
// direction passes no window; it scans every bin.
__device__ __forceinline__ void window_bins(const float4 &d, float wphi, int &a0, int &b0, int &a1,
                                            int &b1)
{
    a0 = 0;
    b0 = PX_NB - 1;
    a1 = 1;
    b1 = 0;
    const float ph = atan2f(d.y, d.x);
    if (!(wphi < PX_PI) || !(ph == ph)) return;
    const float lo = ph - wphi, hi = ph + wphi;
    if (lo < -PX_PI) {
        b0 = phi_bin(hi);
        a1 = phi_bin(lo + 2.0f * PX_PI);
        b1 = PX_NB - 1;
    } else if (hi > PX_PI) {
        a0 = phi_bin(lo);
        a1 = 0;
        b1 = phi_bin(hi - 2.0f * PX_PI);
    } else {
        a0 = phi_bin(lo);
        b0 = phi_bin(hi);
    }
    // the two parts meet: every bin, once
    if (a1 <= b1 && (a1 <= b0 + 1 && b1 + 1 >= a0)) {
        a0 = 0;
        b0 = PX_NB - 1;
        a1 = 1;
        b1 = 0;
    }
}

// Add one to cnt[key] for every active lane with `act`: the lanes are
// grouped by key with ballots, then each group's first lane adds the group's
// size (the wave's atomics go out together: one memory round trip); returns
// each such lane's old value plus its rank in its group (its slot in a list
// being filled).
__device__ __forceinline__ int32_t agg_add(int32_t *cnt, int key, bool act)
{
    const int l = px_lane();
    const unsigned long long below = (1ull << l) - 1ull;
    int lead_of = l, rank = 0, size = 0;
    unsigned long long todo = __ballot(act);
    while (todo) {
        const int lead = __builtin_ctzll(todo);
        const int k = __builtin_amdgcn_readlane(key, lead);
        const unsigned long long grp = todo & __ballot(key == k);
        if ((grp >> l) & 1ull) {
            lead_of = lead;
            rank = (int)__popcll(grp & below);
        }
        if (l == lead) size = (int)__popcll(grp);
        todo &= ~grp;
    }
    int32_t base = 0;
    if (size > 0) base = atomicAdd(&cnt[key], size);
    base = __shfl(base, lead_of, 64);
    return base + rank;
}

// Objects handed to one wave, consecutive, in the one-wave-per-object passes
constexpr int PX_WCHUNK = 2;

// ---------------------------------------------------------------- input
// A pixel batch as sent (px_pack_words) into its arrays: hit indices made
// batch-wide, each seed's event and its index there.
__global__ __launch_bounds__(BLOCK) void k_px_take(EvDev E, int n_ev)
{
    const int32_t *p = (const int32_t *)E.px_pack;
    const int n_px = p[0], n_sd = p[1];
    const int32_t *px_off = p + 2, *sd_off = px_off + n_ev + 1;
    const float *x = (const float *)(sd_off + n_ev + 1), *y = x + n_px, *z = y + n_px;
    const int32_t *seeds = (const int32_t *)(z + n_px);
    const int t0 = blockIdx.x * BLOCK + threadIdx.x, st = gridDim.x * BLOCK;
    if (t0 == 0) {
        ((int32_t *)E.desc)[D_NPX] = n_px;
        ((int32_t *)E.desc)[D_NSEEDS] = n_sd;
    }
    for (int i = t0; i <= n_ev; i += st) {
        E.px_off[i] = px_off[i];
        E.sd_off[i] = sd_off[i];
    }
    for (int i = t0; i < n_px; i += st) {
        E.px_x[i] = x[i];
        E.px_y[i] = y[i];
        E.px_z[i] = z[i];
    }
    for (int q = t0; q < n_sd; q += st) {
        int lo = 0, hi = n_ev - 1;   // last event whose first seed is at or before q
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (sd_off[mid] <= q) lo = mid; else hi = mid - 1;
        }
        for (int k = 0; k < 4; ++k) E.sd_hits[4 * q + k] = px_off[lo] + seeds[4 * q + k];
        E.sd_ev[q] = lo;
        E.sd_local[q] = q - sd_off[lo];
    }
}

// ---------------------------------------------------------------- setup
// every per-event list count, the per-hit minima and flags, seed state and
// direction
__global__ __launch_bounds__(BLOCK) void k_px_init(EvDev E)
{
    if (upstream_overflow(E)) return;
    const int t0 = blockIdx.x * BLOCK + threadIdx.x, st = gridDim.x * BLOCK;
    const int n_px = E.desc[D_NPX], n_sd = E.desc[D_NSEEDS];
    const int n_hits = (int)E.gc[GC_N_SORTED];
    const int n_pl = PXL_COUNT * (E.cap_ev * PX_NB + 1);
    for (int i = t0; i < n_pl; i += st) {
        E.pl_cnt[i] = 0;
        E.pl_fill[i] = 0;
    }
    for (int i = t0; i < n_sd; i += st) {
        E.sd_c5[i] = make_int2(0, 0);
        E.sd_c3[i] = make_int2(0, 0);
    }
    for (int i = t0; i < n_hits; i += st) {
        E.hmin_o[i] = KEY_NONE;
        E.hflag_o[i] = 0;
    }
    for (int i = t0; i < n_px; i += st) {
        E.hmin_p[i] = KEY_NONE;
        E.hflag_p[i] = 0;
    }
    for (int i = t0; i < n_sd; i += st) {
        E.sd_used[i] = 0;
        E.sd_keep[i] = 0;
        // seed direction
        const int32_t a = E.sd_hits[4 * i], d = E.sd_hits[4 * i + 3];
        E.sd_dir[i] = pls_dir(E.px_x[a], E.px_y[a], E.px_z[a], E.px_x[d], E.px_y[d], E.px_z[d]);
    }
}

__device__ __forceinline__ int md_event(const EvDev &E, int32_t md, int n_mod)
{
    return E.md_slot[md] / n_mod;
}

// The passes over the listed objects: kept quintuplets, triplets and seeds
// side by side, a block of threads of one kind at a time (list PXL_*, index v
// of n in it).
struct PxBlocks {
    uint32_t n5, n3, ns, b5, b3, bs;
    __device__ PxBlocks(const EvDev &E, uint32_t *s_pre5, uint32_t *s_pre3)
    {
        n5 = obj_prefix(E, OT_T5, s_pre5);
        n3 = obj_prefix(E, OT_T3, s_pre3);
        ns = (uint32_t)E.desc[D_NSEEDS];
        b5 = (n5 + BLOCK - 1) / BLOCK;
        b3 = b5 + (n3 + BLOCK - 1) / BLOCK;
        bs = b3 + (ns + BLOCK - 1) / BLOCK;
    }
    __device__ int list(uint32_t b, uint32_t &v, uint32_t &n) const
    {
        const int k = b < b5 ? PXL_K5 : b < b3 ? PXL_K3 : PXL_SD;
        v = (b - (k == PXL_K5 ? 0u : k == PXL_K3 ? b5 : b3)) * BLOCK + threadIdx.x;
        n = k == PXL_K5 ? n5 : k == PXL_K3 ? n3 : ns;
        return k;
    }
};

// directions of the kept quintuplets and of every triplet; with the seeds,
// counted per (event, azimuth bin)
__global__ __launch_bounds__(BLOCK) void k_obj_dir(EvDev E, int n_mod)
{
    __shared__ uint32_t s_pre5[NSH + 1], s_pre3[NSH + 1];
    if (upstream_overflow(E)) return;
    const PxBlocks B(E, s_pre5, s_pre3);
    for (uint32_t b = blockIdx.x; b < B.bs; b += gridDim.x) {
        uint32_t v, n;
        const int list = B.list(b, v, n);
        bool act = v < n;
        int key = 0;
        if (act && list == PXL_K5) {
            const int32_t t = obj_at(E, OT_T5, s_pre5, v);
            act = E.t5_keep[t] != 0;
            if (act) {
                const MdV A = load_md(E, E.t5_md0[t]), C = load_md(E, E.t5_md2[t]),
                          Q = load_md(E, E.t5_md4[t]);
                const float4 d = obj_dir(A, Q, bridge_curv(A, C, Q));
                E.t5_dir[t] = d;
                key = md_event(E, E.t5_md0[t], n_mod) * PX_NB + dir_bin(d);
            } else {
                E.t5_clean[t] = 0;
            }
        } else if (act && list == PXL_K3) {
            const int32_t t = obj_at(E, OT_T3, s_pre3, v);
            const float4 d = obj_dir(load_md(E, E.t3_a[t]), load_md(E, E.t3_c[t]), E.t3_k[t]);
            E.t3_dir[t] = d;
            key = md_event(E, E.t3_a[t], n_mod) * PX_NB + dir_bin(d);
        } else if (act) {
            key = E.sd_ev[v] * PX_NB + dir_bin(E.sd_dir[v]);
        }
        (void)agg_add(pl(E, E.pl_cnt, list), key, act);
    }
}

// exclusive scan of the lists' counts, one block per list; off[n] = the total
__global__ __launch_bounds__(1024) void k_pl_scan(EvDev E)
{
    __shared__ int32_t s_part[1024];
    if (upstream_overflow(E)) return;
    const int list = (int)blockIdx.x;
    const int n = E.desc[D_NEV] * PX_NB;
    const int32_t *cnt = pl(E, E.pl_cnt, list);
    int32_t *off = pl(E, E.pl_off, list);
    const int per = (n + 1023) / 1024;
    const int a = threadIdx.x * per, b = min(a + per, n);
    int32_t sum = 0;
    for (int e = a; e < b; ++e) sum += cnt[e];
    s_part[threadIdx.x] = sum;
    __syncthreads();
    // inclusive scan of the 1024 partial sums (doubling steps)
    for (int d = 1; d < 1024; d <<= 1) {
        const int32_t add = (int)threadIdx.x >= d ? s_part[threadIdx.x - d] : 0;
        __syncthreads();
        s_part[threadIdx.x] += add;
        __syncthreads();
    }
    int32_t run = s_part[threadIdx.x] - sum;
    for (int e = a; e < b; ++e) {
        off[e] = run;
        run += cnt[e];
    }
    if (threadIdx.x == 1023) off[n] = s_part[1023];
}

// Arenas of up to PX_SELF events scan their counts inside k_obj_fill: each
// block scans the few hundred counts for itself, one key per thread (block 0
// writes the offsets for the later kernels): 9.4 us against 10.7 after a scan
// of its own, itself 3.8 us and a launch.  Past one key per thread the scan
// grows with the events in every block, where one block per list does it once.
constexpr int PX_SELF = BLOCK / PX_NB;

// kept quintuplets, triplets and seeds into their per-(event, bin) lists
template <bool SELF>
__global__ __launch_bounds__(BLOCK) void k_obj_fill(EvDev E, int n_mod)
{
    __shared__ uint32_t s_pre5[NSH + 1], s_pre3[NSH + 1];
    __shared__ int32_t s_off[SELF ? PXL_COUNT : 1][BLOCK], s_w[PXL_COUNT][WAVES];
    if (upstream_overflow(E)) return;
    if constexpr (SELF) {
        const int l = px_lane(), w = (int)(threadIdx.x >> 6);
        int32_t c[PXL_COUNT], x[PXL_COUNT];
#pragma unroll
        for (int k = 0; k < PXL_COUNT; ++k)
            c[k] = x[k] = (int)threadIdx.x < E.cap_ev * PX_NB ? pl(E, E.pl_cnt, k)[threadIdx.x] : 0;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1)
#pragma unroll
            for (int k = 0; k < PXL_COUNT; ++k) {
                const int32_t up = __shfl_up(x[k], d, 64);
                x[k] += l >= d ? up : 0;
            }
#pragma unroll
        for (int k = 0; k < PXL_COUNT; ++k)
            if (l == 63) s_w[k][w] = x[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PXL_COUNT; ++k) {
            int32_t before = 0;
            for (int q = 0; q < w; ++q) before += s_w[k][q];
            const int32_t ex = before + x[k] - c[k];
            s_off[k][threadIdx.x] = ex;
            if (blockIdx.x == 0 && (int)threadIdx.x < E.cap_ev * PX_NB) {
                int32_t *off = pl(E, E.pl_off, k);
                off[threadIdx.x] = ex;
                if ((int)threadIdx.x == E.cap_ev * PX_NB - 1) off[threadIdx.x + 1] = ex + c[k];
            }
        }
    }
    const PxBlocks B(E, s_pre5, s_pre3);   // (its barrier also covers the offsets)
    for (uint32_t b = blockIdx.x; b < B.bs; b += gridDim.x) {
        uint32_t v, n;
        const int list = B.list(b, v, n);
        bool act = v < n;
        int key = 0;
        int32_t t = (int32_t)v;
        float4 d = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (act && list == PXL_K5) {
            t = obj_at(E, OT_T5, s_pre5, v);
            act = E.t5_keep[t] != 0;
            if (act) {
                d = E.t5_dir[t];
                key = md_event(E, E.t5_md0[t], n_mod) * PX_NB + dir_bin(d);
            }
        } else if (act && list == PXL_K3) {
            t = obj_at(E, OT_T3, s_pre3, v);
            d = E.t3_dir[t];
            key = md_event(E, E.t3_a[t], n_mod) * PX_NB + dir_bin(d);
        } else if (act) {
            d = E.sd_dir[t];
            key = E.sd_ev[t] * PX_NB + dir_bin(d);
        }
        int32_t at = agg_add(pl(E, E.pl_fill, list), key, act);
        if (!act) continue;
        if constexpr (SELF) at += s_off[list][key];
        else at += pl(E, E.pl_off, list)[key];
        if (list == PXL_K5) {
            E.pl_k5[at] = t;
            E.pl_k5d[at] = d;
        } else if (list == PXL_K3) {
            E.pl_k3[at] = t;
            E.pl_k3d[at] = d;
        } else {
            E.sd_pos[t] = at;
            E.pl_sdd[at] = d;
            E.pl_sdk[at] = 0;
        }
    }
}

// ---------------------------------------------------------------- linking
// the MDs of an outer object, inner to outer
template <int KIND>
__device__ __forceinline__ int32_t obj_md(const EvDev &E, int32_t t, int j)
{
    if constexpr (KIND == 5) return t5_md(E, t, j);
    else return j == 0 ? E.t3_a[t] : j == 1 ? E.t3_b[t] : E.t3_c[t];
}

// grouped position of outer hit j (0 .. 2 KIND - 1) of candidate c's object
template <int KIND>
__device__ __forceinline__ int32_t c_ohit(const EvDev &E, int32_t obj, int j)
{
    const int32_t m = obj_md<KIND>(E, obj, j >> 1);
    return (j & 1) ? E.md_hup[m] : E.md_hlo[m];
}

// A candidate's key among those that share a hit: score, then the seed's
// index in its event.  A score is a sum of squares over positive variances,
// so its sign bit is free; the top two bits order the three duplicate
// removals that share the per-hit minima, each below the ones before it (pT5
// 2, pT3 1, pLS 0), so that the minima need no reset in between.
template <int KIND>
__device__ __forceinline__ unsigned long long c_key(float score, int32_t seed_local)
{
    return ((unsigned long long)(KIND == 5 ? 2 : 1) << 62) |
           ((unsigned long long)(__float_as_uint(score) & 0x7fffffffu) << 31) | (uint32_t)seed_local;
}

// hit j of a candidate: pixel hits 0 .. 3, then the outer ones (may differ
// between lanes); its minimum, its flag
template <int KIND>
__device__ __forceinline__ int32_t c_hit(const EvDev &E, int32_t s, int32_t obj, int j)
{
    return j < 4 ? E.sd_hits[4 * s + j] : c_ohit<KIND>(E, obj, j - 4);
}

template <int KIND>
__device__ __forceinline__ unsigned long long *c_min(const EvDev &E, int32_t s, int32_t obj, int j)
{
    return (j < 4 ? E.hmin_p : E.hmin_o) + c_hit<KIND>(E, s, obj, j);
}

// NS seeds per wave: the objects of their events in the azimuth bins of their
// link windows are walked as one list, 64 at a time; those inside the window
// are queued in LDS, and the link chi2 runs on 64 of them together.  The chi2
// is what costs here (some thousand instructions, a few objects per chunk
// inside the window), so it runs on full waves and not once per chunk:
// one PU200 event, pT5 / pT3 23.5 / 21.6 us with the minima of the duplicate
// removal in a launch of their own (14.5 / 12.0), 24.8 / 27.2 with them here,
// 21.1 / 22.8 on blocks of 4 waves instead of 16, 15.7 / 18.2 with the queue.
// Two, four or eight seeds per wave: 16.6, 15.8, 18.9 us (pT5); one or two
// 18.0, 17.6 (pT3).
// A block reserves room for its round's candidates with one atomic; the queue
// is in seed order, so each seed's candidates are consecutive (its range in
// sd_c5 / sd_c3).  A wave with more than PX_STAGE candidates scans again and
// writes the rest directly.
constexpr int PX_LW = 4, PX_STAGE = 128;

template <int NS>
struct SmLink {
    int32_t obj[PX_LW][PX_STAGE];
    float score[PX_LW][PX_STAGE];
    uint8_t slot[PX_LW][PX_STAGE];
    int32_t qt[PX_LW][128];          // queue: object, seed of the wave
    uint8_t qs[PX_LW][128];
    float4 dir[PX_LW][NS];
    float pix[PX_LW][NS][12];        // its four hits
    uint32_t cnt[PX_LW], base;
};

template <int KIND, int NS>
__device__ __forceinline__ uint32_t link_scan(const EvDev &E, const Consts &K, const PixConsts &P,
                                              int s0, int n_sd, uint32_t (&n_of)[NS], SmLink<NS> &sm,
                                              int w, uint32_t write_base, bool second)
{
    constexpr int NP = 4 + KIND, IC = KIND == 5 ? 6 : 4, NR = 2 * NS;
    const int l = px_lane();
    const unsigned long long below = (1ull << l) - 1ull;
    const int32_t *off = pl(E, E.pl_off, KIND == 5 ? PXL_K5 : PXL_K3);
    const int32_t *lst = KIND == 5 ? E.pl_k5 : E.pl_k3;
    const float4 *dir = KIND == 5 ? E.pl_k5d : E.pl_k3d;   // in list order
    const float x2p = KIND == 5 ? P.x5p : P.x3p, x2z = KIND == 5 ? P.x5z : P.x3z;
    // the list ranges of the seeds' windows (two per seed: the wrap at +-pi)
    int32_t from = 0, len = 0;
    if (l < NR) {
        const int s = s0 + (l >> 1);
        if (s < n_sd && (KIND == 5 || !E.sd_used[s])) {
            const float4 d = E.sd_dir[s];
            const int ev = E.sd_ev[s];
            int a[2], b[2];
            window_bins(d, P.wphi, a[0], b[0], a[1], b[1]);
            const int lo = (l & 1) ? a[1] : a[0], hi = (l & 1) ? b[1] : b[0];
            if (lo <= hi) {
                from = off[ev * PX_NB + lo];
                len = off[ev * PX_NB + hi + 1] - from;
            }
            if (!(l & 1)) sm.dir[w][l >> 1] = d;
        }
    }
    if (l < 4 * NS && s0 + (l >> 2) < n_sd) {
        const int32_t h = E.sd_hits[4 * (s0 + (l >> 2)) + (l & 3)];
        float *x = &sm.pix[w][l >> 2][3 * (l & 3)];
        x[0] = E.px_x[h];
        x[1] = E.px_y[h];
        x[2] = E.px_z[h];
    }
    wave_lds_sync();
    int32_t st[NR], pre[NR + 1];
    pre[0] = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        st[r] = __builtin_amdgcn_readlane(from, r) - pre[r];
        pre[r + 1] = pre[r] + __builtin_amdgcn_readlane(len, r);
    }
    const int32_t tot = pre[NR];
#pragma unroll
    for (int q = 0; q < NS; ++q) n_of[q] = 0;
    uint32_t n_acc = 0;
    int qn = 0;
    // entry f of the joint list
    auto entry = [&](int32_t f, int &q, int32_t &t, float4 &d) {
        int32_t b = st[0];
        q = 0;
#pragma unroll
        for (int r = 1; r < NR; ++r)
            if (f >= pre[r]) {
                b = st[r];
                q = r >> 1;
            }
        if (f < tot) {
            t = lst[b + f];
            d = dir[b + f];
        }
    };
    // the link chi2 of the queue's first n <= 64
    auto link = [&](int n) {
        bool ok = false;
        float score = 0.0f;
        int32_t t = 0;
        int q = 0;
        if (l < n) {
            t = sm.qt[w][l];
            q = sm.qs[w][l];
            const float *x = sm.pix[w][q];
            LPt pts[NP];
#pragma unroll
            for (int k = 0; k < 4; ++k) pts[k] = lpt_px(x[3 * k], x[3 * k + 1], x[3 * k + 2]);
#pragma unroll
            for (int j = 0; j < KIND; ++j) pts[4 + j] = lpt_md(load_md(E, obj_md<KIND>(E, t, j)));
            ok = link_accept<NP, IC>(K, pts, P.sig2p, P.sigz, x2p, x2z, score);
        }
        const unsigned long long m = __ballot(ok);
        if (ok) {
            const uint32_t pos = n_acc + (uint32_t)__popcll(m & below);
            if (!second && pos < PX_STAGE) {
                sm.obj[w][pos] = t;
                sm.score[w][pos] = score;
                sm.slot[w][pos] = (uint8_t)q;
            } else if (second && pos >= PX_STAGE) {
                const uint32_t at = write_base + pos;
                if (at < (uint32_t)E.cap_pxc) {
                    const int32_t s = s0 + q;
                    (KIND == 5 ? E.c5_seed : E.c3_seed)[at] = s;
                    (KIND == 5 ? E.c5_obj : E.c3_obj)[at] = t;
                    (KIND == 5 ? E.c5_score : E.c3_score)[at] = score;
                    for (int j = 0; j < 4 + 2 * KIND; ++j)
                        atomicMin(c_min<KIND>(E, s, t, j), c_key<KIND>(score, E.sd_local[s]));
                }
            }
        }
        n_acc += (uint32_t)__popcll(m);
#pragma unroll
        for (int k = 0; k < NS; ++k) n_of[k] += (uint32_t)__popcll(m & __ballot(q == k));
    };
    int qx = 0;
    int32_t tn = 0;
    float4 dn = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    entry(l, qx, tn, dn);
    for (int32_t f0 = 0; f0 < tot; f0 += 64) {
        const int q = qx;
        const int32_t t = tn;
        const float4 dt = dn;
        entry(f0 + 64 + l, qx, tn, dn);   // loaded while this chunk is tested
        const bool in = f0 + l < tot && link_window(sm.dir[w][q], dt, P.wl2);
        const unsigned long long m = __ballot(in);
        if (in) {
            const int at = qn + (int)__popcll(m & below);
            sm.qt[w][at] = t;
            sm.qs[w][at] = (uint8_t)q;
        }
        qn += (int)__popcll(m);
        if (qn < 64) continue;
        wave_lds_sync();
        link(64);
        qn -= 64;
        const int32_t mt = sm.qt[w][64 + l];
        const uint8_t ms = sm.qs[w][64 + l];
        wave_lds_sync();
        if (l < qn) {
            sm.qt[w][l] = mt;
            sm.qs[w][l] = ms;
        }
    }
    wave_lds_sync();
    if (qn > 0) link(qn);
    wave_lds_sync();
    return n_acc;
}

template <int KIND, int NS>
__global__ __launch_bounds__(PX_LW * 64) void k_px_link(EvDev E, Consts K, PixConsts P)
{
    __shared__ SmLink<NS> sm;
    const int l = px_lane(), w = (int)(threadIdx.x >> 6);
    const int n = E.desc[D_NSEEDS];
    int32_t *c_seed = KIND == 5 ? E.c5_seed : E.c3_seed;
    int32_t *c_obj = KIND == 5 ? E.c5_obj : E.c3_obj;
    float *c_score = KIND == 5 ? E.c5_score : E.c3_score;
    int2 *sd_c = KIND == 5 ? E.sd_c5 : E.sd_c3;
    if (upstream_overflow(E)) return;
    for (int r0 = blockIdx.x * PX_LW * NS; r0 < n; r0 += gridDim.x * PX_LW * NS) {
        const int s0 = r0 + w * NS;
        uint32_t n_of[NS];
        const uint32_t n_acc = link_scan<KIND, NS>(E, K, P, s0, n, n_of, sm, w, 0u, false);
        if (l == 0) sm.cnt[w] = n_acc;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t tot = 0;
            for (int k = 0; k < PX_LW; ++k) tot += sm.cnt[k];
            sm.base = tot ? atomicAdd(&E.gc[KIND == 5 ? GC_PX5 : GC_PX3], tot) : 0u;
        }
        __syncthreads();
        uint32_t mine = sm.base;
        for (int k = 0; k < w; ++k) mine += sm.cnt[k];
        const uint32_t cap = (uint32_t)E.cap_pxc;
        if (l == 0 && mine + n_acc > cap) atomicOr(&E.gc[GC_OVERFLOW], 1u << OT_COUNT);
        uint32_t at = mine;   // each seed's range
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const uint32_t first = at < cap ? at : cap;
            at += n_of[q];
            const uint32_t last = at < cap ? at : cap;
            if (l == 0 && s0 + q < n) sd_c[s0 + q] = make_int2((int)first, (int)(last - first));
        }
        const uint32_t staged = n_acc < PX_STAGE ? n_acc : PX_STAGE;
        for (uint32_t k = l; k < staged; k += 64) {
            if (mine + k < cap) {
                c_seed[mine + k] = s0 + sm.slot[w][k];
                c_obj[mine + k] = sm.obj[w][k];
                c_score[mine + k] = sm.score[w][k];
            }
        }
        // into the minima of their hits, 16 lanes per candidate
        const int j = l & 15;
        for (uint32_t k = (uint32_t)(l >> 4); k < staged; k += 4)
            if (mine + k < cap && j < 4 + 2 * KIND) {
                const int32_t s = s0 + sm.slot[w][k];
                atomicMin(c_min<KIND>(E, s, sm.obj[w][k], j),
                          c_key<KIND>(sm.score[w][k], E.sd_local[s]));
            }
        if (n_acc > PX_STAGE)
            (void)link_scan<KIND, NS>(E, K, P, s0, n, n_of, sm, w, mine, true);
        __syncthreads();   // the stage is rewritten by the next round
    }
}

// ---------------------------------------------------------------- duplicate removal
template <int KIND>
__device__ __forceinline__ uint32_t n_cand(const EvDev &E)
{
    const uint32_t n = E.gc[KIND == 5 ? GC_PX5 : GC_PX3];
    return n < (uint32_t)E.cap_pxc ? n : (uint32_t)E.cap_pxc;
}

// per-event hit index of outer hit j of an object
template <int KIND>
__device__ __forceinline__ int32_t c_orig(const EvDev &E, int32_t obj, int j)
{
    return hit_orig(E, c_ohit<KIND>(E, obj, j));
}

// Lane j of the 16 of candidate c (act: there is one): does it survive among
// the candidates that share its hit j?  True for the lanes without a hit.
// Equal (score, seed): the smaller outer hit tuple wins; the seed's
// candidates are consecutive, lane j compares every 16th.
template <int KIND>
__device__ __forceinline__ bool c_keep16(const EvDev &E, uint32_t c, bool act, int32_t s, int32_t o,
                                         float sc, int32_t h, int j)
{
    const int g = px_lane() & 48;
    bool ok = true;
    if (act && j < 4 + 2 * KIND)
        ok = (j < 4 ? E.hmin_p : E.hmin_o)[h] == c_key<KIND>(sc, E.sd_local[s]);
    if ((((__ballot(ok) >> g) & 0xffffull) == 0xffffull) && act) {
        const int2 rg = (KIND == 5 ? E.sd_c5 : E.sd_c3)[s];
        for (uint32_t u = (uint32_t)(rg.x + j); u < (uint32_t)(rg.x + rg.y); u += 16) {
            if (u == c) continue;
            const float scu = KIND == 5 ? E.c5_score[u] : E.c3_score[u];
            if (__float_as_uint(scu) != __float_as_uint(sc)) continue;
            const int32_t ou = KIND == 5 ? E.c5_obj[u] : E.c3_obj[u];
            for (int k = 0; k < 2 * KIND; ++k) {
                const int32_t a = c_orig<KIND>(E, ou, k), b = c_orig<KIND>(E, o, k);
                if (a != b) {
                    if (a < b) ok = false;
                    break;
                }
            }
        }
    }
    return ok;
}

// ---------------------------------------------------------------- cross-cleaning
// any direction of the event's list, of an entry that takes(i), within dr2 of
// d: the whole wave scans the list's azimuth bins around d (half-width wdr) 64
// entries at a time (wave-uniform arguments)
template <class F>
__device__ __forceinline__ bool wave_near_any(const EvDev &E, int list, int ev, const float4 *dirs,
                                              const float4 &d, float dr2, float wdr, F &&takes)
{
    const int32_t *off = pl(E, E.pl_off, list);
    int a[2], b[2];
    window_bins(d, wdr, a[0], b[0], a[1], b[1]);
    for (int part = 0; part < 2; ++part) {
        if (a[part] > b[part]) continue;
        const int32_t i0 = off[ev * PX_NB + a[part]], i1 = off[ev * PX_NB + b[part] + 1];
        for (int32_t bb = i0; bb < i1; bb += 64) {
            const int32_t i = bb + px_lane();
            bool near = false;
            if (i < i1) {
                const float4 q = dirs[i];   // loaded along with the entry's state
                const bool in = takes(i);
                near = close_dir(d, q, dr2) && in;
            }
            if (__ballot(near)) return true;
        }
    }
    return false;
}

// the run of objects [first, last) of the wave in a one-wave-per-object pass
__device__ __forceinline__ void wave_run(uint32_t n, uint32_t &first, uint32_t &last, uint32_t &step)
{
    const uint32_t w = blockIdx.x * WAVES + (threadIdx.x >> 6);
    first = w * PX_WCHUNK;
    step = gridDim.x * WAVES * PX_WCHUNK;
    last = first + PX_WCHUNK < n ? first + PX_WCHUNK : n;
}

// Surviving pT5 and pT3, 16 lanes per candidate: one per hit, so that a
// candidate's reads take one chain of loads instead of one after another
// (PU200, pT5 / pT3: keep, mark and, for the pT3, clean 31 / 32 us with a
// thread per candidate and a launch each, 4.8 / 10.2 us here).
// Hits and seeds of a survivor are marked, 1 for a pT5 and 2 for a pT3; a
// seed's mark also goes to its place in the seeds' azimuth list, which is the
// list of the survivors' directions (a seed has one survivor at most).  A pT3
// near a pT5 or sharing a hit with one is a duplicate: it looks for ones
// only, so the marks of the pT3 set meanwhile don't matter to it.
template <int KIND>
__global__ __launch_bounds__(BLOCK) void k_pxd_keep(EvDev E, PixConsts P)
{
    constexpr uint8_t MARK = KIND == 5 ? 1 : 2;
    if (upstream_overflow(E)) return;
    const uint32_t n = n_cand<KIND>(E);
    const int l = px_lane(), j = l & 15, g = l & 48;
    for (uint32_t c0 = blockIdx.x * (BLOCK / 16); c0 < n; c0 += gridDim.x * (BLOCK / 16)) {
        const uint32_t c = c0 + (threadIdx.x >> 4);
        const bool act = c < n, hit = act && j < 4 + 2 * KIND;
        int32_t s = 0, o = 0, h = 0;
        float sc = 0.0f;
        if (act) {
            s = (KIND == 5 ? E.c5_seed : E.c3_seed)[c];
            o = (KIND == 5 ? E.c5_obj : E.c3_obj)[c];
            sc = (KIND == 5 ? E.c5_score : E.c3_score)[c];
        }
        if (hit) h = c_hit<KIND>(E, s, o, j);
        uint8_t *flag = (j < 4 ? E.hflag_p : E.hflag_o) + h;
        bool ok = c_keep16<KIND>(E, c, act, s, o, sc, h, j) && act;
        if (KIND == 3) {
            if (hit && *flag == 1) ok = false;
            unsigned long long m = __ballot(ok);
            for (int q = 0; q < 64; q += 16) {
                if (((m >> q) & 0xffffull) != 0xffffull) continue;
                const int sq = __builtin_amdgcn_readlane(s, q);
                if (wave_near_any(E, PXL_SD, E.sd_ev[sq], E.pl_sdd, E.sd_dir[sq], P.dr2, P.wdr,
                                  [&](int32_t i) { return E.pl_sdk[i] == 1; }) && g == q)
                    ok = false;
            }
        }
        const bool keep = ((__ballot(ok) >> g) & 0xffffull) == 0xffffull;
        if (act && j == 0) {
            (KIND == 5 ? E.c5_keep : E.c3_keep)[c] = keep;
            if (keep) {
                E.sd_used[s] = 1;
                E.pl_sdk[E.sd_pos[s]] = MARK;
            }
        }
        if (keep && hit) *flag = MARK;
    }
}

// kept quintuplets near, or sharing a hit with, a pT5 or cleaned pT3 (in list
// order: those left are the list's entries with pl_k5k set)
__global__ __launch_bounds__(BLOCK) void k_t5_clean(EvDev E, PixConsts P, int n_mod)
{
    if (upstream_overflow(E)) return;
    const uint32_t n5 = (uint32_t)pl(E, E.pl_off, PXL_K5)[E.desc[D_NEV] * PX_NB];
    const int l = px_lane();
    uint32_t first, last, step;
    wave_run(n5, first, last, step);
    for (; first < n5; first += step, last = first + PX_WCHUNK < n5 ? first + PX_WCHUNK : n5) {
        for (uint32_t v = first; v < last; ++v) {
            const int32_t t = E.pl_k5[v];
            const bool hit = l < 10 && E.hflag_o[c_ohit<5>(E, t, l)] != 0;
            bool keep = __ballot(hit) == 0ull;
            if (keep)
                keep = !wave_near_any(E, PXL_SD, md_event(E, E.t5_md0[t], n_mod), E.pl_sdd, E.pl_k5d[v],
                                      P.dr2, P.wdr, [&](int32_t i) { return E.pl_sdk[i] != 0; });
            if (l == 0) {
                E.t5_clean[t] = keep;
                E.pl_k5k[v] = keep;
            }
        }
    }
}

// unlinked pLS: a pixel hit held by a candidate, or near one, is a
// duplicate; the rest mark their pixel hits with their index (minimum)
__global__ __launch_bounds__(BLOCK) void k_pls_clean(EvDev E, PixConsts P)
{
    if (upstream_overflow(E)) return;
    const uint32_t n_sd = (uint32_t)E.desc[D_NSEEDS];
    const int l = px_lane();
    uint32_t first, last, step;
    wave_run(n_sd, first, last, step);
    for (; first < n_sd; first += step, last = first + PX_WCHUNK < n_sd ? first + PX_WCHUNK : n_sd) {
        for (uint32_t s = first; s < last; ++s) {
            if (E.sd_used[s]) continue;
            const bool hit = l < 4 && E.hflag_p[E.sd_hits[4 * s + l]] != 0;
            bool keep = __ballot(hit) == 0ull;
            const int ev = E.sd_ev[s];
            const float4 d = E.sd_dir[s];
            if (keep)
                keep = !wave_near_any(E, PXL_SD, ev, E.pl_sdd, d, P.dr2, P.wdr,
                                      [&](int32_t i) { return E.pl_sdk[i] != 0; });
            if (keep)
                keep = !wave_near_any(E, PXL_K5, ev, E.pl_k5d, d, P.dr2, P.wdr,
                                      [&](int32_t i) { return E.pl_k5k[i] != 0; });
            if (l == 0) E.sd_keep[s] = keep;
            if (keep && l < 4)
                atomicMin(&E.hmin_p[E.sd_hits[4 * s + l]], (unsigned long long)(uint32_t)E.sd_local[s]);
        }
    }
}

__global__ __launch_bounds__(BLOCK) void k_pls_keep(EvDev E)
{
    if (upstream_overflow(E)) return;
    const int n_sd = E.desc[D_NSEEDS];
    for (int s = blockIdx.x * BLOCK + threadIdx.x; s < n_sd; s += gridDim.x * BLOCK) {
        if (!E.sd_keep[s]) continue;
        const unsigned long long me = (unsigned long long)(uint32_t)E.sd_local[s];
        bool keep = true;
        for (int k = 0; k < 4; ++k) keep = keep && E.hmin_p[E.sd_hits[4 * s + k]] == me;
        E.sd_keep[s] = keep;
    }
}

// ---------------------------------------------------------------- launch
static int px_grid(int64_t work, int per_block)
{
    int64_t g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > GRID_MAX) g = GRID_MAX;
    return (int)g;
}

hipError_t launch_px_take(const EvDev &E, int n_ev, int64_t n_px, int64_t n_seeds, hipStream_t s)
{
    const int grid = px_grid(std::max<int64_t>(std::max(n_px, n_seeds), n_ev + 1), BLOCK);
    hipLaunchKernelGGL(k_px_take, dim3(grid), dim3(BLOCK), 0, s, E, n_ev);
    return hipGetLastError();
}

hipError_t launch_pixel(const EvDev &E, const Consts &K, const PixConsts &P, hipStream_t s)
{
    const int n_mod = E.cap_slots / E.cap_ev;
    const int g_hits = px_grid(std::max<int64_t>(E.cap_hits, E.cap_px), BLOCK);
    const int g_sd = px_grid(E.cap_seeds, BLOCK);
    // seeds per wave in the link scans: a pT5 window holds a few dozen kept
    // quintuplets, a pT3 window hundreds of triplets
    constexpr int PX_NS5 = 4, PX_NS3 = 2;
    const int g_link5 = px_grid(E.cap_seeds, PX_LW * PX_NS5);
    const int g_link3 = px_grid(E.cap_seeds, PX_LW * PX_NS3);
    const int g_obj = px_grid((int64_t)(E.rc[OT_T3] + E.rc[OT_T5]) * NSH + E.cap_seeds, BLOCK);
    const int g_keep = px_grid(E.cap_pxc, BLOCK / 16);
    // one wave per object, PX_WCHUNK objects per wave
    const int g_objw = px_grid((int64_t)E.rc[OT_T5] * NSH, WAVES * PX_WCHUNK);
    const int g_sdc = px_grid(E.cap_seeds, WAVES * PX_WCHUNK);
    hipLaunchKernelGGL(k_px_init, dim3(g_hits), dim3(BLOCK), 0, s, E);
    hipLaunchKernelGGL(k_obj_dir, dim3(g_obj), dim3(BLOCK), 0, s, E, n_mod);
    if (E.cap_ev <= PX_SELF) {
        hipLaunchKernelGGL(k_obj_fill<true>, dim3(g_obj), dim3(BLOCK), 0, s, E, n_mod);
    } else {
        hipLaunchKernelGGL(k_pl_scan, dim3(PXL_COUNT), dim3(1024), 0, s, E);
        hipLaunchKernelGGL(k_obj_fill<false>, dim3(g_obj), dim3(BLOCK), 0, s, E, n_mod);
    }
    hipLaunchKernelGGL((k_px_link<5, PX_NS5>), dim3(g_link5), dim3(PX_LW * 64), 0, s, E, K, P);
    hipLaunchKernelGGL(k_pxd_keep<5>, dim3(g_keep), dim3(BLOCK), 0, s, E, P);
    // pT3 from the seeds no pT5 uses
    hipLaunchKernelGGL((k_px_link<3, PX_NS3>), dim3(g_link3), dim3(PX_LW * 64), 0, s, E, K, P);
    hipLaunchKernelGGL(k_pxd_keep<3>, dim3(g_keep), dim3(BLOCK), 0, s, E, P);
    // cross-cleaning
    hipLaunchKernelGGL(k_t5_clean, dim3(g_objw), dim3(BLOCK), 0, s, E, P, n_mod);
    hipLaunchKernelGGL(k_pls_clean, dim3(g_sdc), dim3(BLOCK), 0, s, E, P);
    hipLaunchKernelGGL(k_pls_keep, dim3(g_sd), dim3(BLOCK), 0, s, E);
    return hipGetLastError();
}

}  // namespace lst
