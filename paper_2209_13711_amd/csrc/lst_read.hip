// Results for the host: one event's objects, or a field of them, packed into
// rows, and the per-event counts, computed where the arrays are.
//
// The object arrays are spread over 32 regions sized by the arena's
// capacities and hold all events of a batch, so copying them to the host to
// pick one event's objects there moves many times the result (a PU200-like
// event: 9 MB of arrays for 84 KB of kept quintuplets).  These kernels select
// and convert on the device and store the packed rows straight into pinned
// host memory: what crosses the bus is the result, and no copy command
// follows the kernel.  Rows keep the order of the arrays: regions in order,
// positions in order within a region.
//
// What bounds them is latency.  One PU200-like event: its kept quintuplets
// take 29 us from call to return (two launches of 5 and 7 us, the rest is
// launching, waiting and the host's copy), 830 us with the arrays copied to
// the host; its counts 24 us (9.1 us), 1,070 us before.  The kept quintuplets
// of 16 such events: 0.42 ms, 365 ms before.  One launch for the rows, each
// block waiting for the counts of those before it, took 10.2 us and gained
// nothing over the two.
#include <algorithm>

#include "lst_access.hpp"

namespace lst {

__device__ __forceinline__ int rd_lane() { return threadIdx.x & 63; }

// the chain's counters as the host getters need them (every thread of the block calls it)
__device__ __forceinline__ void put_header(const EvDev &E, ReadHdr *h)
{
    uint32_t group = 0;
    const uint4 *words = reinterpret_cast<const uint4 *>(E.gc + GC_GROUP);
    for (int i = threadIdx.x; i < GC_GROUP_WORDS / 4; i += blockDim.x) {
        const uint4 v = words[i];
        group |= v.x | v.y | v.z | v.w;
    }
    const bool fault = __syncthreads_or(group != 0u) != 0;
    for (int i = threadIdx.x; i < OT_COUNT * NSH; i += blockDim.x)
        h->shard[i / NSH][i % NSH] = E.gc[gc_shard(i / NSH, i % NSH)];
    if (threadIdx.x == 0) {
        h->overflow = E.gc[GC_OVERFLOW];
        h->error = E.gc[GC_ERROR] | (fault ? 4u : 0u);
    }
}

// exclusive sum over the block's threads (BLOCK of them) and the total
__device__ __forceinline__ uint32_t rd_block_scan(uint32_t v, uint32_t *s_w, uint32_t &total)
{
    const int l = rd_lane(), w = (int)(threadIdx.x >> 6);
    uint32_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t t = __shfl_up(x, d, 64);
        if (l >= d) x += t;
    }
    if (l == 63) s_w[w] = x;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        if (i < w) before += s_w[i];
        total += s_w[i];
    }
    __syncthreads();
    return before + x - v;
}

// ---------------------------------------------------------------- rows
// the first mini-doublet of an object
template <int TYPE>
__device__ __forceinline__ int32_t first_md(const EvDev &E, int32_t t)
{
    if constexpr (TYPE == OT_MD) return t;
    else if constexpr (TYPE == OT_SEG) return E.seg_in[t];
    else if constexpr (TYPE == OT_T3) return E.t3_a[t];
    else return E.t5_md0[t];
}

// object t belongs to the wanted rows: kept (when asked), and its module in
// the event's slots (a batch of one event needs no look)
template <int TYPE>
__device__ __forceinline__ bool wanted(const EvDev &E, const PackArgs &A, int32_t t)
{
    if (A.kept_only && !E.t5_keep[t]) return false;
    if (A.whole_batch) return true;
    const int32_t s = E.md_slot[first_md<TYPE>(E, t)];
    return s >= A.lo_slot && s < A.hi_slot;
}

// the block's share [first, last) of the n stored objects
__device__ __forceinline__ void block_share(uint32_t n, uint32_t &first, uint32_t &last)
{
    const uint32_t per = (n + gridDim.x - 1) / gridDim.x;
    first = min(blockIdx.x * per, n);
    last = min(first + per, n);
}

// wanted objects in each block's share
template <int TYPE>
__global__ __launch_bounds__(BLOCK) void k_pack_count(EvDev E, PackArgs A)
{
    __shared__ uint32_t s_pre[NSH + 1], s_n;
    if (objects_unusable(E)) return;
    if (threadIdx.x == 0) s_n = 0;
    const uint32_t n = obj_prefix(E, TYPE, s_pre);
    uint32_t first, last, mine = 0;
    block_share(n, first, last);
    for (uint32_t v0 = first; v0 < last; v0 += BLOCK) {
        const uint32_t v = v0 + threadIdx.x;
        const bool on = v < last && wanted<TYPE>(E, A, obj_at(E, TYPE, s_pre, v));
        mine += (uint32_t)__popcll(__ballot(on));
    }
    if (rd_lane() == 0 && mine) atomicAdd(&s_n, mine);
    __syncthreads();
    if (threadIdx.x == 0) E.rd_cnt[blockIdx.x] = s_n;
}

// word j of object t's row: hit j of its tuple, or word j of the field
template <int TYPE, int WIDTH, class T, bool TUPLE>
__device__ __forceinline__ T row_word(const EvDev &E, const PackArgs &A, int32_t t, uint32_t j)
{
    if constexpr (TUPLE) {
        const int d = (int)(j >> 1);
        int32_t m;
        if constexpr (TYPE == OT_MD) m = t;
        else if constexpr (TYPE == OT_SEG) m = d == 0 ? E.seg_in[t] : E.seg_out[t];
        else if constexpr (TYPE == OT_T3) m = d == 0 ? E.t3_a[t] : d == 1 ? E.t3_b[t] : E.t3_c[t];
        else m = t5_md(E, t, d);
        return hit_orig(E, (j & 1) ? E.md_hup[m] : E.md_hlo[m]);
    } else {
        return ((const T *)A.field)[(size_t)t * WIDTH + j];
    }
}

// the rows of each block's share after those of the blocks before it.  A
// tile of BLOCK objects lists its wanted ones in LDS; the block then walks
// the tile's output words, so that stores to the host are consecutive.
template <int TYPE, int WIDTH, class T, bool TUPLE>
__global__ __launch_bounds__(BLOCK) void k_pack_rows(EvDev E, PackArgs A)
{
    __shared__ uint32_t s_pre[NSH + 1], s_w[WAVES];
    __shared__ int32_t s_idx[BLOCK];
    if (blockIdx.x == 0) put_header(E, A.hdr);
    if (objects_unusable(E)) {
        if (blockIdx.x == 0 && threadIdx.x == 0) A.hdr->rows = 0;
        return;
    }
    const uint32_t n = obj_prefix(E, TYPE, s_pre);
    uint32_t mine = 0, before;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += BLOCK) mine += E.rd_cnt[b];
    (void)rd_block_scan(mine, s_w, before);
    uint32_t first, last;
    block_share(n, first, last);
    T *out = (T *)A.out;
    for (uint32_t v0 = first; v0 < last; v0 += BLOCK) {
        const uint32_t v = v0 + threadIdx.x;
        const int32_t t = v < last ? obj_at(E, TYPE, s_pre, v) : 0;
        const bool on = v < last && wanted<TYPE>(E, A, t);
        uint32_t rows;
        const uint32_t pos = rd_block_scan(on ? 1u : 0u, s_w, rows);
        if (on) s_idx[pos] = t;
        __syncthreads();
        const uint32_t room = before < A.cap_rows ? A.cap_rows - before : 0u;
        const uint32_t words = (rows < room ? rows : room) * WIDTH;
        for (uint32_t q = threadIdx.x; q < words; q += BLOCK)
            out[(size_t)before * WIDTH + q] =
                row_word<TYPE, WIDTH, T, TUPLE>(E, A, s_idx[q / WIDTH], q % WIDTH);
        before += rows;
        __syncthreads();   // s_idx is rewritten by the next tile
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) A.hdr->rows = before;
}

template <int TYPE, int WIDTH, class T, bool TUPLE>
static hipError_t pack(const EvDev &E, const PackArgs &A, hipStream_t s)
{
    const int64_t span = (int64_t)E.rc[TYPE] * NSH;
    const int grid = (int)std::min<int64_t>(PACK_BLOCKS, std::max<int64_t>(1, (span + BLOCK - 1) / BLOCK));
    hipLaunchKernelGGL(k_pack_count<TYPE>, dim3(grid), dim3(BLOCK), 0, s, E, A);
    hipLaunchKernelGGL((k_pack_rows<TYPE, WIDTH, T, TUPLE>), dim3(grid), dim3(BLOCK), 0, s, E, A);
    return hipGetLastError();
}

hipError_t launch_pack_tuples(const EvDev &E, int type, const PackArgs &A, hipStream_t s)
{
    switch (type) {
    case OT_MD: return pack<OT_MD, 2, int32_t, true>(E, A, s);
    case OT_SEG: return pack<OT_SEG, 4, int32_t, true>(E, A, s);
    case OT_T3: return pack<OT_T3, 6, int32_t, true>(E, A, s);
    default: return pack<OT_T5, 10, int32_t, true>(E, A, s);
    }
}

hipError_t launch_pack_field(const EvDev &E, int type, int row_bytes, const PackArgs &A, hipStream_t s)
{
    const bool t3 = type == OT_T3;
    switch (row_bytes) {
    case 1: return t3 ? pack<OT_T3, 1, uint8_t, false>(E, A, s) : pack<OT_T5, 1, uint8_t, false>(E, A, s);
    case 4: return t3 ? pack<OT_T3, 1, uint32_t, false>(E, A, s) : pack<OT_T5, 1, uint32_t, false>(E, A, s);
    case 4 * MLP_NIN:
        return t3 ? pack<OT_T3, MLP_NIN, uint32_t, false>(E, A, s)
                  : pack<OT_T5, MLP_NIN, uint32_t, false>(E, A, s);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------- pixel rows
// Track candidates (what < 0) or link candidates (0 pT5, 1 pT3) of one event
// as rows in lexicographic order.  The sources are taken as one list: pT5
// candidates, pT3 candidates, quintuplets, the event's seeds.  Three launches:
// wanted entries per block, their sort keys (first words of the row) into a
// list, and each row to the place its rank among the keys gives it.  The
// rank counts the smaller keys, n per row.  A PU200-like event (2,300 rows):
// 5.0, 6.6 and 24 us, 49 us from call to return; 1.3 ms with the pixel
// stage's arrays copied to the host and sorted there.
struct PxList {
    uint32_t n5, n3, nt, total;
    int32_t sd0;
};

// the list's lengths (every thread of the block calls it)
__device__ __forceinline__ PxList px_list(const EvDev &E, const PackArgs &A, uint32_t *s_pre)
{
    PxList L{};
    const uint32_t cap = (uint32_t)E.cap_pxc;
    if (A.what != 1) L.n5 = min(E.gc[GC_PX5], cap);
    if (A.what != 0) L.n3 = min(E.gc[GC_PX3], cap);
    L.total = L.n5 + L.n3;
    if (A.what < 0) {
        L.nt = t5_prefix(E, s_pre);
        L.sd0 = E.sd_off[A.event];
        L.total += L.nt + (uint32_t)(E.sd_off[A.event + 1] - L.sd0);
    }
    return L;
}

// entry v of the list: its source (0 pT5, 1 pT3, 2 T5, 3 pLS) and index there
struct PxEntry {
    int32_t src, i;
};

__device__ __forceinline__ PxEntry px_entry(const EvDev &E, const PxList &L, const uint32_t *s_pre,
                                            uint32_t v)
{
    if (v < L.n5) return PxEntry{0, (int32_t)v};
    if ((v -= L.n5) < L.n3) return PxEntry{1, (int32_t)v};
    if ((v -= L.n3) < L.nt) return PxEntry{2, t5_at(E, s_pre, v)};
    return PxEntry{3, L.sd0 + (int32_t)(v - L.nt)};
}

__device__ __forceinline__ bool px_wanted(const EvDev &E, const PackArgs &A, const PxEntry &e)
{
    switch (e.src) {
    case 0: return (A.what == 0 || E.c5_keep[e.i]) && E.sd_ev[E.c5_seed[e.i]] == A.event;
    case 1: return (A.what == 1 || E.c3_keep[e.i]) && E.sd_ev[E.c3_seed[e.i]] == A.event;
    case 2: {
        if (!E.t5_clean[e.i]) return false;
        const int32_t s = E.md_slot[E.t5_md0[e.i]];
        return s >= A.lo_slot && s < A.hi_slot;
    }
    default: return E.sd_keep[e.i] != 0;
    }
}

__device__ __forceinline__ int32_t px_seed(const EvDev &E, const PxEntry &e)
{
    return e.src == 0 ? E.sd_local[E.c5_seed[e.i]] : e.src == 1 ? E.sd_local[E.c3_seed[e.i]]
         : e.src == 2 ? -1 : E.sd_local[e.i];
}

// outer hit j (0..9) of the entry's object, -1 past its end
__device__ __forceinline__ int32_t px_hit(const EvDev &E, const PxEntry &e, int j)
{
    int32_t m;
    if (e.src == 1) {
        if (j >= 6) return -1;
        const int32_t o = E.c3_obj[e.i];
        m = j < 2 ? E.t3_a[o] : j < 4 ? E.t3_b[o] : E.t3_c[o];
    } else if (e.src == 3) {
        return -1;
    } else {
        m = t5_md(E, e.src == 0 ? E.c5_obj[e.i] : e.i, j >> 1);
    }
    return hit_orig(E, (j & 1) ? E.md_hup[m] : E.md_hlo[m]);
}

// word j of the entry's row: (type, seed, hits) or (seed, hits, score, kept)
__device__ __forceinline__ int32_t px_word(const EvDev &E, const PackArgs &A, const PxEntry &e, int j)
{
    if (A.what < 0) {
        // sources in the order of the track candidates' types
        if (j == 0) return e.src == 0 ? A.type_of[0] : e.src == 1 ? A.type_of[1]
                         : e.src == 2 ? A.type_of[2] : A.type_of[3];
        return j == 1 ? px_seed(E, e) : px_hit(E, e, j - 2);
    }
    if (j == 0) return px_seed(E, e);
    if (j < 11) return px_hit(E, e, j - 1);
    if (j == 11) return __float_as_int(e.src == 0 ? E.c5_score[e.i] : E.c3_score[e.i]);
    return e.src == 0 ? E.c5_keep[e.i] : E.c3_keep[e.i];
}

// the row's first words as an unsigned key in row order (every word is at
// least -1; types fit two bits, seeds 30)
__device__ __forceinline__ uint64_t px_key(const EvDev &E, const PackArgs &A, const PxEntry &e)
{
    const uint64_t seed = (uint64_t)(uint32_t)(px_seed(E, e) + 1);
    const uint64_t hit = (uint64_t)((uint32_t)px_hit(E, e, 0) + 1u);
    const uint64_t type = A.what < 0 ? (uint64_t)px_word(E, A, e, 0) : 0u;
    return (type << 62) | (seed << 32) | hit;
}

__global__ __launch_bounds__(BLOCK) void k_px_count(EvDev E, PackArgs A)
{
    __shared__ uint32_t s_pre[NSH + 1], s_n;
    if (objects_unusable(E)) return;
    if (threadIdx.x == 0) s_n = 0;
    const PxList L = px_list(E, A, s_pre);
    __syncthreads();
    uint32_t first, last, mine = 0;
    block_share(L.total, first, last);
    for (uint32_t v0 = first; v0 < last; v0 += BLOCK) {
        const uint32_t v = v0 + threadIdx.x;
        const bool on = v < last && px_wanted(E, A, px_entry(E, L, s_pre, v));
        mine += (uint32_t)__popcll(__ballot(on));
    }
    if (rd_lane() == 0 && mine) atomicAdd(&s_n, mine);
    __syncthreads();
    if (threadIdx.x == 0) E.rd_cnt[blockIdx.x] = s_n;
}

__global__ __launch_bounds__(BLOCK) void k_px_keys(EvDev E, PackArgs A)
{
    __shared__ uint32_t s_pre[NSH + 1], s_w[WAVES];
    if (objects_unusable(E)) return;
    const PxList L = px_list(E, A, s_pre);
    uint32_t mine = 0, before;
    for (uint32_t b = threadIdx.x; b < blockIdx.x; b += BLOCK) mine += E.rd_cnt[b];
    (void)rd_block_scan(mine, s_w, before);
    uint32_t first, last;
    block_share(L.total, first, last);
    for (uint32_t v0 = first; v0 < last; v0 += BLOCK) {
        const uint32_t v = v0 + threadIdx.x;
        PxEntry e{};
        bool on = false;
        if (v < last) {
            e = px_entry(E, L, s_pre, v);
            on = px_wanted(E, A, e);
        }
        uint32_t rows;
        const uint32_t pos = before + rd_block_scan(on ? 1u : 0u, s_w, rows);
        if (on) {
            E.rd_key[pos] = px_key(E, A, e);
            E.rd_src[pos] = make_int2(e.src, e.i);
        }
        before += rows;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) E.rd_cnt[PACK_BLOCKS] = before;
}

// row order of entries with equal keys, other than themselves
__device__ __forceinline__ bool px_less(const EvDev &E, const PackArgs &A, uint32_t a, uint32_t b)
{
    const int2 x = E.rd_src[a], y = E.rd_src[b];
    const PxEntry ea{x.x, x.y}, eb{y.x, y.y};
    for (int j = 0; j < A.width; ++j) {
        const int32_t p = px_word(E, A, ea, j), q = px_word(E, A, eb, j);
        if (p != q) return p < q;
    }
    return a < b;
}

// A wave ranks PX_RANK rows at a time: its lanes take the keys 64 at a time
// and compare each with all of the wave's rows.  (One thread per row over
// keys staged in LDS kept nine blocks busy: 197 us for 2,300 rows.)  PX_KEYS
// keys per lane are loaded before the first is compared, and equal keys (rare)
// are looked at after them: with the comparison of equal keys between the
// loads, each waited for the one before, 25.4 us for 2,300 rows against 13.1.
constexpr int PX_RANK = 4, PX_KEYS = 8;

__global__ __launch_bounds__(BLOCK) void k_px_rows(EvDev E, PackArgs A)
{
    if (blockIdx.x == 0) put_header(E, A.hdr);
    const uint32_t n = objects_unusable(E) ? 0u : E.rd_cnt[PACK_BLOCKS];
    if (blockIdx.x == 0 && threadIdx.x == 0) A.hdr->rows = n;
    if (n > A.cap_rows) return;   // the buffer grows and the rows are packed again
    const uint32_t l = (uint32_t)rd_lane(), width = (uint32_t)A.width;
    int32_t *out = (int32_t *)A.out;
    for (uint32_t r0 = (blockIdx.x * WAVES + (threadIdx.x >> 6)) * PX_RANK; r0 < n;
         r0 += gridDim.x * WAVES * PX_RANK) {
        uint64_t key[PX_RANK];
        uint32_t rank[PX_RANK];
#pragma unroll
        for (int i = 0; i < PX_RANK; ++i) {
            key[i] = r0 + i < n ? E.rd_key[r0 + i] : 0;
            rank[i] = 0;
        }
        for (uint32_t c0 = l; c0 < n; c0 += 64 * PX_KEYS) {
            uint64_t o[PX_KEYS];
#pragma unroll
            for (int k = 0; k < PX_KEYS; ++k) {
                const uint32_t c = c0 + 64 * k;
                o[k] = c < n ? E.rd_key[c] : ~0ull;
            }
            bool tie = false;
#pragma unroll
            for (int k = 0; k < PX_KEYS; ++k)
#pragma unroll
                for (int i = 0; i < PX_RANK; ++i) {
                    rank[i] += o[k] < key[i];
                    tie |= o[k] == key[i] && c0 + 64 * k != r0 + i;
                }
            if (!tie) continue;
#pragma unroll 1
            for (uint32_t c = c0; c < n && c < c0 + 64 * PX_KEYS; c += 64)
#pragma unroll
                for (int i = 0; i < PX_RANK; ++i)
                    if (E.rd_key[c] == key[i] && r0 + i < n && c != r0 + i && px_less(E, A, c, r0 + i))
                        ++rank[i];
        }
#pragma unroll
        for (int i = 0; i < PX_RANK; ++i)
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) rank[i] += __shfl_xor(rank[i], d, 64);
        const uint32_t words = min(n - r0, (uint32_t)PX_RANK) * width;
        for (uint32_t q = l; q < words; q += 64) {
            const uint32_t i = q / width, j = q - i * width;
            const uint32_t at = i == 0 ? rank[0] : i == 1 ? rank[1] : i == 2 ? rank[2] : rank[3];
            const int2 x = E.rd_src[r0 + i];
            out[(size_t)at * width + j] = px_word(E, A, PxEntry{x.x, x.y}, (int)j);
        }
    }
}
static_assert(PX_RANK == 4, "rank of the row in the loop above");

hipError_t launch_pack_pixel(const EvDev &E, const PackArgs &A, hipStream_t s)
{
    const int64_t most = 2 * (int64_t)E.cap_pxc + (int64_t)E.rc[OT_T5] * NSH + E.cap_seeds;
    const int grid = (int)std::min<int64_t>(PACK_BLOCKS, std::max<int64_t>(1, (most + BLOCK - 1) / BLOCK));
    hipLaunchKernelGGL(k_px_count, dim3(grid), dim3(BLOCK), 0, s, E, A);
    hipLaunchKernelGGL(k_px_keys, dim3(grid), dim3(BLOCK), 0, s, E, A);
    hipLaunchKernelGGL(k_px_rows, dim3(grid), dim3(BLOCK), 0, s, E, A);
    return hipGetLastError();
}

// ---------------------------------------------------------------- counts
// Sums per event, stored per block (no atomics on device memory, no clearing)
// and added up by a second kernel, or, for one event, by the host (23 KB: 2.5
// us less than the launch; 0.3 MB for 16 events: 100 us more).  The grid has a
// part for the module slots
// (candidates and number of mini-doublets, candidate segments: four threads
// per slot share its map edges) and one for each kind of stored object, one
// thread per object: its event, and the candidates it is the first half of
// (segments and triplets) or its flags (quintuplets).
//
// Bounded by the chain of dependent loads, so the objects are taken from
// their arrays directly, each load level once: walking them through their
// module's MDs (a thread per MD, a wave per 64 slots, a block per 64 slots)
// took 47, 55 and 35 us on a PU200-like event, the time of the densest
// modules.
constexpr int RC_SLOTS = BLOCK / 4;    // module slots of a block
constexpr int RC_EVENTS = 64;          // events of a block's table; more take further grid rows
constexpr int RC_OBJ = 3;              // sums of a block and event

__device__ __forceinline__ void slot_counts(const EvDev &E, const ModDev &M, int stage, uint64_t *part)
{
    __shared__ uint64_t s_sum[WAVES][RC_OBJ];
    const int n_mod = M.n_mod, nb = (n_mod + RC_SLOTS - 1) / RC_SLOTS;
    const int ev = blockIdx.x / nb, sl = (int)threadIdx.x >> 2, quarter = threadIdx.x & 3;
    const int m = (blockIdx.x - ev * nb) * RC_SLOTS + sl;
    const size_t base = (size_t)ev * n_mod;
    uint64_t sum[RC_OBJ] = {0, 0, 0};
    if (m < n_mod) {
        const size_t slot = base + m;
        const int32_t e0 = M.map_ptr[m] + quarter, e1 = M.map_ptr[m + 1];
        const uint32_t b0 = E.boff[2 * slot], b1 = E.boff[2 * slot + 1], b2 = E.boff[2 * slot + 2];
        if (stage >= 3) {
            const uint32_t mc = (uint32_t)E.md_cnt[slot];
            uint32_t outer = 0;
            if (mc)
#pragma unroll 8
                for (int32_t q = e0; q < e1; q += 4) outer += (uint32_t)E.md_cnt[base + M.map_col[q]];
            sum[2] = (uint64_t)mc * outer;
            if (quarter == 0) sum[1] = mc;
        }
        if (quarter == 0) sum[0] = (uint64_t)(b1 - b0) * (b2 - b1);
    }
    const int l = rd_lane(), w = (int)(threadIdx.x >> 6);
#pragma unroll
    for (int k = 0; k < RC_OBJ; ++k) {
        unsigned long long v = sum[k];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        if (l == 0) s_sum[w][k] = v;
    }
    __syncthreads();
    if (threadIdx.x < RC_OBJ) {
        uint64_t v = 0;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) v += s_sum[i][threadIdx.x];
        part[(size_t)blockIdx.x * RC_OBJ + threadIdx.x] = v;
    }
}

// objects of TYPE taken by block `b` of `blocks`; per event of the row
// [ev0, ev0 + RC_EVENTS) the number of objects and two more sums
template <int TYPE>
__device__ __forceinline__ void obj_counts(const EvDev &E, int n_mod, int n_ev, int ev0, int stage,
                                           uint32_t b, uint32_t blocks, uint64_t *part)
{
    __shared__ uint32_t s_pre[NSH + 1];
    __shared__ unsigned long long s_tab[RC_EVENTS][RC_OBJ];
    const uint32_t n_md = E.rc[OT_MD] * NSH;   // mini-doublets: after a fault an index may be any
    const int n_row = min(n_ev - ev0, RC_EVENTS);
    for (int i = threadIdx.x; i < n_row * RC_OBJ; i += BLOCK) s_tab[i / RC_OBJ][i % RC_OBJ] = 0;
    const uint32_t n = obj_prefix(E, TYPE, s_pre);   // (its barrier also covers the table)
    // sums of the thread's run of objects of one event, added to the table
    // when the event changes
    int run = -1;
    unsigned long long cnt = 0, s1 = 0, s2 = 0;
    auto flush = [&]() {
        if (run < 0) return;
        atomicAdd(&s_tab[run][0], cnt);
        if (s1) atomicAdd(&s_tab[run][1], s1);
        if (s2) atomicAdd(&s_tab[run][2], s2);
        cnt = s1 = s2 = 0;
    };
    for (uint32_t v = b * BLOCK + threadIdx.x; v < n; v += blocks * BLOCK) {
        const int32_t t = obj_at(E, TYPE, s_pre, v);
        int ev = 0;
        if (n_ev > 1) {
            const int32_t md = first_md<TYPE>(E, t);
            if ((uint32_t)md >= n_md) continue;
            ev = E.md_slot[md] / n_mod - ev0;
        }
        if (ev < 0 || ev >= n_row) continue;
        if (ev != run) {
            flush();
            run = ev;
        }
        ++cnt;
        if constexpr (TYPE == OT_SEG) {
            const int32_t md = E.seg_out[t];
            if ((uint32_t)md < n_md) s1 += (uint64_t)E.seg_cnt[md];
        }
        if constexpr (TYPE == OT_T3)
            if (stage >= 5) {
                const int32_t md = E.t3_c[t];
                if ((uint32_t)md < n_md) s1 += (uint64_t)E.t3_cnt[md];
            }
        if constexpr (TYPE == OT_T5) {
            if (stage >= 7) s1 += E.t5_keep[t];
            if (stage >= 8) s2 += E.t5_clean[t];
        }
    }
    flush();
    __syncthreads();
    for (int i = threadIdx.x; i < n_row * RC_OBJ; i += BLOCK)
        part[((size_t)b * n_ev + ev0) * RC_OBJ + i] = s_tab[i / RC_OBJ][i % RC_OBJ];
}

__global__ __launch_bounds__(BLOCK) void k_read_counts(EvDev E, ModDev M, int n_ev, int stage,
                                                       uint32_t n_slot_blocks, uint32_t n_obj_blocks,
                                                       ReadHdr *hdr, uint64_t *part)
{
    if (hdr && blockIdx.x == 0 && blockIdx.y == 0) put_header(E, hdr);
    if (upstream_overflow(E)) return;
    if (blockIdx.x < n_slot_blocks) {
        if (blockIdx.y == 0) slot_counts(E, M, stage, part);
        return;
    }
    const uint32_t i = blockIdx.x - n_slot_blocks, kind = i / n_obj_blocks, b = i % n_obj_blocks;
    uint64_t *out = part + (size_t)n_slot_blocks * RC_OBJ + (size_t)kind * n_obj_blocks * n_ev * RC_OBJ;
    const int ev0 = (int)blockIdx.y * RC_EVENTS;
    if (kind == 0) obj_counts<OT_SEG>(E, M.n_mod, n_ev, ev0, stage, b, n_obj_blocks, out);
    else if (kind == 1) obj_counts<OT_T3>(E, M.n_mod, n_ev, ev0, stage, b, n_obj_blocks, out);
    else obj_counts<OT_T5>(E, M.n_mod, n_ev, ev0, stage, b, n_obj_blocks, out);
}

// event blockIdx.x: the sums of its slot blocks and of the object blocks
__global__ __launch_bounds__(BLOCK) void k_add_counts(EvDev E, int n_ev, int kinds,
                                                      uint32_t n_slot_blocks, uint32_t n_obj_blocks,
                                                      ReadHdr *hdr, EventSums *out)
{
    __shared__ uint64_t s_sum[WAVES][4][RC_OBJ];
    if (blockIdx.x == 0) put_header(E, hdr);
    if (upstream_overflow(E)) return;
    const int ev = blockIdx.x, l = rd_lane(), w = (int)(threadIdx.x >> 6);
    const uint32_t per = n_slot_blocks / (uint32_t)n_ev;
    for (int k = 0; k < 4; ++k) {   // module slots, then the object kinds
        unsigned long long sum[RC_OBJ] = {0, 0, 0};
        const uint32_t nb = k == 0 ? per : k <= kinds ? n_obj_blocks : 0u;
        for (uint32_t b = threadIdx.x; b < nb; b += BLOCK) {
            const size_t at = k == 0 ? (size_t)ev * per + b
                                     : n_slot_blocks + ((size_t)(k - 1) * n_obj_blocks + b) * n_ev + ev;
#pragma unroll
            for (int j = 0; j < RC_OBJ; ++j) sum[j] += E.rd_part[at * RC_OBJ + j];
        }
#pragma unroll
        for (int j = 0; j < RC_OBJ; ++j) {
            unsigned long long v = sum[j];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
            if (l == 0) s_sum[w][k][j] = v;
        }
    }
    __syncthreads();
    if (threadIdx.x < 4 * RC_OBJ) {
        const int k = threadIdx.x / RC_OBJ, j = threadIdx.x % RC_OBJ;
        uint64_t v = 0;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) v += s_sum[i][k][j];
        out[ev].sum[k][j] = v;
    }
}

// The object part's blocks per kind: enough to take one event's objects in a
// pass or two, fewer for many events so that the sums stay small.
static uint32_t count_obj_blocks(int n_events)
{
    return (uint32_t)std::max(32, std::min(256, 4096 / n_events));
}

// sums that the blocks store for up to n_events events (blocks x events of
// count_obj_blocks is at most the larger of 4096 and 32 n_events)
size_t count_part_size(int n_mod, int n_events)
{
    const size_t slots = (size_t)n_events * ((n_mod + RC_SLOTS - 1) / RC_SLOTS);
    return (slots + 3 * std::max<size_t>(4096, 32 * (size_t)n_events)) * RC_OBJ;
}

static int counted_kinds(int stage) { return stage >= 6 ? 3 : stage >= 5 ? 2 : stage >= 4 ? 1 : 0; }

hipError_t launch_read_counts(const EvDev &E, const ModDev &M, int n_events, int stage, ReadHdr *hdr,
                              EventSums *out, hipStream_t s)
{
    const uint32_t slots = (uint32_t)n_events * ((M.n_mod + RC_SLOTS - 1) / RC_SLOTS);
    const uint32_t obj = count_obj_blocks(n_events);
    const int kinds = counted_kinds(stage);
    const dim3 grid(slots + kinds * obj, (n_events + RC_EVENTS - 1) / RC_EVENTS);
    const bool one = n_events == 1;   // the blocks' sums follow the event's in the host buffer
    hipLaunchKernelGGL(k_read_counts, grid, dim3(BLOCK), 0, s, E, M, n_events, stage, slots, obj,
                       one ? hdr : nullptr, one ? (uint64_t *)(out + 1) : E.rd_part);
    if (!one)
        hipLaunchKernelGGL(k_add_counts, dim3(n_events), dim3(BLOCK), 0, s, E, n_events, kinds, slots, obj,
                           hdr, out);
    return hipGetLastError();
}

void finish_counts(const ModDev &M, int n_events, int stage, EventSums *out)
{
    if (n_events != 1) return;
    const uint32_t slots = (M.n_mod + RC_SLOTS - 1) / RC_SLOTS, obj = count_obj_blocks(1);
    const uint64_t *part = (const uint64_t *)(out + 1);
    *out = EventSums{};
    for (int k = 0; k <= counted_kinds(stage); ++k)
        for (uint32_t b = 0; b < (k ? obj : slots); ++b, part += RC_OBJ)
            for (int j = 0; j < RC_OBJ; ++j) out->sum[k][j] += part[j];
}

size_t read_counts_bytes(const ModDev &M, int n_events)
{
    return n_events * sizeof(EventSums) +
           (n_events == 1 ? sizeof(uint64_t) * count_part_size(M.n_mod, 1) : 0);
}

}  // namespace lst
