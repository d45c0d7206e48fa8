// Properties by which the paper compares a sparsified graph with the
// original (Preliminaries): the sparsified subgraph itself, per-vertex
// triangle counts lambda_i, clustering c_i = lambda_i / (d_i (d_i - 1) / 2),
// C_G = the mean of c_i over d_i > 1 (Eq. cc), connected components, and the
// Spearman rank correlation of two per-vertex scores by the stated formula
// rho = 1 - 6 sum p_i^2 / (n (n^2 - 1)) (tied scores share the mean of
// their ranks).
#include "ad_internal.h"

#include <cstring>    // before rocPRIM: its host code calls memset

#include <rocprim/rocprim.hpp>

#include <algorithm>
#include <cstdint>

namespace ad {

constexpr int PBLOCK = 256;
constexpr int PREDUCE_BLOCKS = 1024;     // fixed grid: reductions in a fixed order

static unsigned pgrid(int64_t count) { return grid_for(std::max<int64_t>(1, count), PBLOCK); }

// ------------------------------------------------------------- subgraph --

__global__ void k_keep_u32(int64_t m, const uint8_t *__restrict__ keep, uint32_t *__restrict__ k32) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x)
        k32[e] = keep[e] ? 1u : 0u;
}

// Kept flag of every stored entry, as the input of the entry scan.
struct EntryKept {
    const uint8_t *keep;
    const int32_t *eid;
    __device__ uint32_t operator()(int64_t p) const { return keep[eid[p]] ? 1u : 0u; }
};
using EntryKeptIt = rocprim::transform_iterator<rocprim::counting_iterator<int64_t>, EntryKept, uint32_t>;
static EntryKeptIt entry_kept(const uint8_t *keep, const int32_t *eid) {
    return EntryKeptIt(rocprim::counting_iterator<int64_t>(0), EntryKept{keep, eid});
}

// The subgraph keeps the stored order, so pos[p] (kept entries before p)
// places entry p, and a row starts at pos of its first entry.
__global__ void k_sub_rows(int64_t n, int64_t nnz, const int64_t *__restrict__ row_ptr,
                           const int32_t *__restrict__ eid, const uint8_t *__restrict__ keep,
                           const uint32_t *__restrict__ pos, int64_t *__restrict__ sub_row_ptr) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t p = row_ptr[i];
        int64_t v = 0;
        if (p < nnz) v = pos[p];
        else if (nnz > 0) v = (int64_t)pos[nnz - 1] + (keep[eid[nnz - 1]] ? 1 : 0);
        sub_row_ptr[i] = v;
    }
}

__global__ void k_compact_entries(int64_t nnz, const int32_t *__restrict__ col, const float *__restrict__ w,
                                  const int32_t *__restrict__ eid, const uint8_t *__restrict__ keep,
                                  const uint32_t *__restrict__ new_id, const uint32_t *__restrict__ pos,
                                  int32_t *__restrict__ sub_col, float *__restrict__ sub_w,
                                  int32_t *__restrict__ sub_eid, int32_t *__restrict__ orig_edge) {
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz; p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t e = eid[p];
        if (!keep[e]) continue;
        const uint32_t q = pos[p];
        sub_col[q] = col[p];
        if (sub_w) sub_w[q] = w[p];
        sub_eid[q] = (int32_t)new_id[e];
        if (orig_edge) orig_edge[q] = e;
    }
}

// ------------------------------------------------------------ triangles --

// Triangles, each found once: with the vertices ordered by (degree, id), the
// triangle a < b < c is found at b, where c of a's upper neighbours N+(a), a in
// N-(b), is looked up among b's own, N+(b).  |N+(b)| is at most sqrt(2m) (each
// member has at least as many neighbours as b), so N+(b) fits a small table in LDS,
// with a count per entry for c's share; a's share is the walk's hits and b's
// their total.  Lookups: the sum over edges (a, b) of |N+(a)|.
// The table has 4-entry buckets at a load of a quarter or less, so that one
// 16-byte LDS read answers almost every lookup, hits included.
// What bounds it: the line requests of the walked rows and, for each edge, of
// the row's place and the share's atomic.  A search of one end's whole row
// per edge (3.6e9 lookups at n = 2^20, m = 16M, against 0.92e9 here, in a bitmap
// that left one workgroup per compute unit): 17.2 ms for that graph and
// its 30% selection together; 4.0 ms here.
constexpr int TRI_SMALL = 64;            // rows up to here: 16 lanes each; longer: a workgroup
constexpr int TRI_HUB = 4096;            // rows from here: TRI_SLICES workgroups
constexpr int TRI_SLICES = 16;
constexpr int TRI_CAP = 512;             // N+ entries in a workgroup's table (1,024: 10% slower, fewer
                                         // workgroups fit)
// More take further passes, each of which walks all rows of N-: where that would be three or
// more (dense graphs), a table of TRI_WIDE_CAP entries at half load, by TRI_WIDE_SLICES
// workgroups of TRI_WIDE_B.  Cliques of 2,000 and 4,000: 7.6 and 84 ms in passes of 512 (searching
// whole rows 7.0 and 51), 6.0 and 44 so; n = 4,000, m = 4.2M 20.0 and 16.2.  From one entry past
// TRI_CAP on, a clique of 1,000 would take 1.20 ms for 0.95.
constexpr int TRI_WIDE = 2 * TRI_CAP;    // N+ entries from which on a row is wide
constexpr int TRI_WIDE_CAP = 2048, TRI_WIDE_B = 512, TRI_WIDE_SLICES = 4;
constexpr int TRI_U = 8;                 // loads in flight per lane (4: 25% slower)
constexpr int TRI_TEAM = 16;
constexpr int32_t TRI_EMPTY = -1;

// Where N+(i) starts (below 2m < 2^32) and its length (below 2^16).
__device__ __forceinline__ uint64_t tri_place(int64_t start, int len) { return ((uint64_t)start << 16) | (uint64_t)len; }
__device__ __forceinline__ int64_t tri_start(uint64_t p) { return (int64_t)(p >> 16); }
__device__ __forceinline__ int tri_len(uint64_t p) { return (int)(p & 0xffffu); }

template <int SLOTS>
__device__ __forceinline__ int tri_bucket(int32_t x) {
    return (int)(((uint32_t)x * 0x9E3779B1u) >> 8) & (SLOTS / 4 - 1);
}

// Puts x, absent so far, into the table and returns its slot.  A bucket's
// slots fill in order.
template <int SLOTS>
__device__ __forceinline__ int tri_put(int32_t *key, int32_t x) {
    for (int s = 4 * tri_bucket<SLOTS>(x);; s = (s + 1) & (SLOTS - 1))
        if (atomicCAS(&key[s], TRI_EMPTY, x) == TRI_EMPTY) return s;
}

// x's slot if it lies in bucket b (whose keys are k), else -1.
__device__ __forceinline__ int tri_match(const int4 &k, int b, int32_t x) {
    return k.x == x ? 4 * b : (k.y == x ? 4 * b + 1 : (k.z == x ? 4 * b + 2 : (k.w == x ? 4 * b + 3 : -1)));
}

// Walks dir[q0], dir[q0 + step], ... < q1, counting each entry found; returns the hits.
template <int SLOTS>
__device__ __forceinline__ unsigned int tri_walk(const int32_t *__restrict__ dir, int64_t q0, int64_t q1, int step,
                                                 const int32_t *key, unsigned int *cnt) {
    unsigned int t = 0;
    for (; q0 < q1; q0 += (int64_t)TRI_U * step) {
        int32_t x[TRI_U];
#pragma unroll
        for (int u = 0; u < TRI_U; ++u) x[u] = q0 + u * step < q1 ? dir[q0 + u * step] : TRI_EMPTY;
        // every entry's bucket is read before the first is looked at
        int4 k[TRI_U];
        int b[TRI_U];
#pragma unroll
        for (int u = 0; u < TRI_U; ++u) {
            b[u] = tri_bucket<SLOTS>(x[u]);
            k[u] = ((const int4 *)key)[b[u]];
        }
#pragma unroll
        for (int u = 0; u < TRI_U; ++u) {
            if (x[u] == TRI_EMPTY) continue;
            int at = tri_match(k[u], b[u], x[u]);
            // a full bucket: the next ones (some bucket always has room, so the search ends)
            while (at < 0 && k[u].w != TRI_EMPTY) {
                b[u] = (b[u] + 1) & (SLOTS / 4 - 1);
                k[u] = ((const int4 *)key)[b[u]];
                at = tri_match(k[u], b[u], x[u]);
            }
            if (at >= 0) {
                atomicAdd(&cnt[at], 1u);
                ++t;
            }
        }
    }
    return t;
}

// Degrees, and the rows longer than TRI_SMALL: rows[0 ..] up to TRI_HUB entries
// (count[0]), rows[n ..] longer (count[1]).  One append per workgroup and list.
constexpr int TRI_LIST_B = 1024;

__global__ __launch_bounds__(TRI_LIST_B) void k_triangles_lists(int64_t n, const int64_t *__restrict__ row_ptr,
                                                                int32_t *__restrict__ deg, int32_t *__restrict__ rows,
                                                                unsigned int *__restrict__ count) {
    __shared__ unsigned int have[2], base[2];
    if (threadIdx.x < 2) have[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * TRI_LIST_B + threadIdx.x;
    const int64_t d = i < n ? row_ptr[i + 1] - row_ptr[i] : 0;
    if (i < n) deg[i] = (int32_t)d;
    const int c = d > TRI_HUB ? 1 : (d > TRI_SMALL ? 0 : -1);
    unsigned int at = 0;
    if (c >= 0) at = atomicAdd(&have[c], 1u);
    __syncthreads();
    if (threadIdx.x < 2 && have[threadIdx.x]) base[threadIdx.x] = atomicAdd(&count[threadIdx.x], have[threadIdx.x]);
    __syncthreads();
    if (c >= 0) rows[c * n + base[c] + at] = (int32_t)i;
}

// dir: every row with N+ first and N- after it, either in any order; place[i]:
// where N+(i) lies; wide: the rows with more than TRI_WIDE upper neighbours (count[2]).
// Bound by the gathers of the neighbours' degrees.
__global__ __launch_bounds__(PBLOCK) void k_triangles_orient(int64_t n, const int64_t *__restrict__ row_ptr,
                                                             const int32_t *__restrict__ col,
                                                             const int32_t *__restrict__ deg,
                                                             const int32_t *__restrict__ rows,
                                                             unsigned int *__restrict__ count,
                                                             int32_t *__restrict__ dir, uint64_t *__restrict__ place,
                                                             int32_t *__restrict__ wide) {
    __shared__ unsigned int n_up, n_down;
    const int lane = threadIdx.x & (WAVE - 1);
    for (int c = 0; c < 2; ++c) {
        const unsigned int nr = count[c];
        for (unsigned int h = blockIdx.x; h < nr; h += gridDim.x) {
            const int64_t i = rows[c * n + h];
            const int64_t b0 = row_ptr[i], b1 = row_ptr[i + 1];
            const int32_t di = (int32_t)(b1 - b0);
            if (threadIdx.x == 0) n_up = n_down = 0u;
            __syncthreads();
            for (int64_t q0 = b0; q0 < b1; q0 += 4 * PBLOCK) {
                int32_t j[4], dj[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t q = q0 + u * PBLOCK + threadIdx.x;
                    j[u] = q < b1 ? col[q] : -1;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) dj[u] = j[u] >= 0 ? deg[j[u]] : 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const bool up = j[u] >= 0 && (dj[u] > di || (dj[u] == di && j[u] > i));
                    const bool down = j[u] >= 0 && !up;
                    const unsigned long long mu = __ballot(up), md = __ballot(down);
                    unsigned int au = 0, ad = 0;
                    if (lane == 0) {
                        if (mu) au = atomicAdd(&n_up, (unsigned int)__popcll(mu));
                        if (md) ad = atomicAdd(&n_down, (unsigned int)__popcll(md));
                    }
                    au = __shfl(au, 0, WAVE);
                    ad = __shfl(ad, 0, WAVE);
                    const unsigned long long below = ((unsigned long long)1 << lane) - 1;
                    if (up) dir[b0 + au + __popcll(mu & below)] = j[u];
                    if (down) dir[b1 - 1 - ad - __popcll(md & below)] = j[u];
                }
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                place[i] = tri_place(b0, (int)n_up);
                if (n_up > (unsigned)TRI_WIDE) wide[atomicAdd(&count[2], 1u)] = (int32_t)i;
            }
            __syncthreads();
        }
    }
    const int sub = threadIdx.x % TRI_TEAM, shift = lane - sub;      // the team's first lane
    const unsigned long long below = ((unsigned long long)1 << sub) - 1;
    const int64_t teams = (int64_t)gridDim.x * (PBLOCK / TRI_TEAM);
    const int64_t n_pad = ceil_div_dev(n, teams) * teams;            // whole waves reach the ballots
    for (int64_t i = (int64_t)blockIdx.x * (PBLOCK / TRI_TEAM) + threadIdx.x / TRI_TEAM; i < n_pad; i += teams) {
        const int64_t b0 = i < n ? row_ptr[i] : 0, b1 = i < n ? row_ptr[i + 1] : 0;
        const int64_t d = b1 - b0;
        const bool mine = i < n && d <= TRI_SMALL;
        const int di = mine ? (int)d : 0;
        int32_t j[TRI_SMALL / TRI_TEAM], dj[TRI_SMALL / TRI_TEAM];
#pragma unroll
        for (int u = 0; u < TRI_SMALL / TRI_TEAM; ++u) {
            const int q = u * TRI_TEAM + sub;
            j[u] = q < di ? col[b0 + q] : -1;
        }
#pragma unroll
        for (int u = 0; u < TRI_SMALL / TRI_TEAM; ++u) dj[u] = j[u] >= 0 ? deg[j[u]] : 0;
        int au = 0, ad = 0;
#pragma unroll
        for (int u = 0; u < TRI_SMALL / TRI_TEAM; ++u) {
            const bool up = j[u] >= 0 && (dj[u] > di || (dj[u] == di && j[u] > i));
            const bool down = j[u] >= 0 && !up;
            const unsigned long long mu = (__ballot(up) >> shift) & 0xffffull;
            const unsigned long long md = (__ballot(down) >> shift) & 0xffffull;
            if (up) dir[b0 + au + __popcll(mu & below)] = j[u];
            if (down) dir[b1 - 1 - ad - __popcll(md & below)] = j[u];
            au += __popcll(mu);
            ad += __popcll(md);
        }
        if (mine && sub == 0) place[i] = tri_place(b0, au);
    }
}

// Rows of up to TRI_SMALL entries, 16 lanes each; a lane per lower neighbour
// (whose row is no longer than b's).
__global__ __launch_bounds__(PBLOCK) void k_triangles_small(int64_t n, const int64_t *__restrict__ row_ptr,
                                                            const int32_t *__restrict__ dir,
                                                            const uint64_t *__restrict__ place,
                                                            unsigned long long *__restrict__ lam) {
    constexpr int TEAMS = PBLOCK / TRI_TEAM, SLOTS = 4 * TRI_SMALL, K = TRI_SMALL / TRI_TEAM;
    __shared__ int4 keys[TEAMS][SLOTS / 4];
    __shared__ unsigned int cnts[TEAMS][SLOTS];
    const int team = threadIdx.x / TRI_TEAM, lane = threadIdx.x % TRI_TEAM;
    int32_t *key = (int32_t *)keys[team];
    unsigned int *cnt = cnts[team];
    for (int s = lane; s < SLOTS; s += TRI_TEAM) {
        key[s] = TRI_EMPTY;
        cnt[s] = 0u;
    }
    // a team's lanes are lanes of one wave: fences order their LDS accesses
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int64_t b = (int64_t)blockIdx.x * TEAMS + team; b < n; b += (int64_t)gridDim.x * TEAMS) {
        const int64_t b0 = row_ptr[b], b1 = row_ptr[b + 1];
        const int up = tri_len(place[b]);
        if (b1 - b0 > TRI_SMALL || up == 0 || up == b1 - b0) continue;      // uniform over the team
        int32_t x[K];
        int slot[K];
#pragma unroll
        for (int u = 0; u < K; ++u) x[u] = u * TRI_TEAM + lane < up ? dir[b0 + u * TRI_TEAM + lane] : TRI_EMPTY;
#pragma unroll
        for (int u = 0; u < K; ++u) slot[u] = x[u] != TRI_EMPTY ? tri_put<SLOTS>(key, x[u]) : -1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        unsigned int own = 0;
        for (int64_t q = b0 + up + lane; q < b1; q += TRI_TEAM) {
            const int32_t a = dir[q];
            const uint64_t p = place[a];
            if (tri_len(p) < 2) continue;                            // N+(a) = {b}
            const unsigned int t = tri_walk<SLOTS>(dir, tri_start(p), tri_start(p) + tri_len(p), 1, key, cnt);
            if (t) atomicAdd(&lam[a], (unsigned long long)t);
            own += t;
        }
        for (int o = TRI_TEAM / 2; o >= 1; o >>= 1) own += __shfl_xor(own, o, WAVE);
        if (lane == 0 && own) atomicAdd(&lam[b], (unsigned long long)own);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < K; ++u)
            if (slot[u] >= 0) {
                if (cnt[slot[u]]) atomicAdd(&lam[x[u]], (unsigned long long)cnt[slot[u]]);
                key[slot[u]] = TRI_EMPTY;
                cnt[slot[u]] = 0u;
            }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

// Listed rows, a workgroup each, or TRI_SLICES (grid y) for the rows from TRI_HUB
// entries and TRI_WIDE_SLICES for the wide ones, each with every so many-th block of TB lower
// neighbours.
// Lower neighbours a are read 64 to a wave, then their rows walked
// with 4, 16 or 64 lanes each by length, TRI_U loads in flight per lane.  The table
// takes CAP entries of N+ at a time; unless WIDE, rows of more than TRI_WIDE are left out.
template <int TB, int CAP, int SLOTS, bool WIDE>
__global__ __launch_bounds__(TB) void k_triangles_rows(const int32_t *__restrict__ rows,
                                                           const unsigned int *__restrict__ count,
                                                           const int64_t *__restrict__ row_ptr,
                                                           const int32_t *__restrict__ dir,
                                                           const uint64_t *__restrict__ place,
                                                           unsigned long long *__restrict__ lam) {
    constexpr int K = CAP / TB;
    __shared__ int4 keys[SLOTS / 4];
    __shared__ unsigned int cnt[SLOTS];
    __shared__ unsigned long long wsum[TB / WAVE];
    __shared__ uint8_t sel[TB / WAVE][WAVE];
    __shared__ unsigned int hits[TB / WAVE][WAVE];
    int32_t *key = (int32_t *)keys;
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x >> 6;
    for (int s = threadIdx.x; s < SLOTS; s += TB) {
        key[s] = TRI_EMPTY;
        cnt[s] = 0u;
    }
    __syncthreads();
    const unsigned int nr = *count;
    for (unsigned int h = blockIdx.x; h < nr; h += gridDim.x) {
        const int64_t b = rows[h];
        const int64_t b0 = row_ptr[b], b1 = row_ptr[b + 1];
        const int up = tri_len(place[b]);
        const int64_t first = b0 + up + (int64_t)blockIdx.y * TB;
        if (up == 0 || first >= b1 || (!WIDE && up > TRI_WIDE)) continue; // uniform over the workgroup
        unsigned long long own = 0;
        for (int c0 = 0; c0 < up; c0 += CAP) {
            int32_t x[K];
            int slot[K];
#pragma unroll
            for (int u = 0; u < K; ++u) {
                const int q = c0 + u * TB + (int)threadIdx.x;
                x[u] = q < up ? dir[b0 + q] : TRI_EMPTY;
            }
#pragma unroll
            for (int u = 0; u < K; ++u) slot[u] = x[u] != TRI_EMPTY ? tri_put<SLOTS>(key, x[u]) : -1;
            __syncthreads();
            for (int64_t q0 = first + wv * WAVE; q0 < b1; q0 += (int64_t)gridDim.y * TB) {
                const bool have = q0 + lane < b1;
                const int32_t a = have ? dir[q0 + lane] : 0;
                const uint64_t p = have ? place[a] : 0;
                const int len = tri_len(p);
                const unsigned long long m4 = __ballot(len >= 2 && len <= 4 * TRI_U);
                const unsigned long long m16 = __ballot(len > 4 * TRI_U && len <= 16 * TRI_U);
                unsigned long long m64 = __ballot(len > 16 * TRI_U);
                // the lanes of either length in order, so that every round is full
                const int n4 = __popcll(m4), n16 = __popcll(m16);
                const unsigned long long below = (1ull << lane) - 1ull;
                if ((m4 >> lane) & 1) sel[wv][__popcll(m4 & below)] = (uint8_t)lane;
                if ((m16 >> lane) & 1) sel[wv][n4 + __popcll(m16 & below)] = (uint8_t)lane;
                hits[wv][lane] = 0u;                                 // of this lane's a
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                for (int r = 0; r < n4; r += 16) {
                    const int k = r + (lane >> 2), s = k < n4 ? sel[wv][k] : 0;
                    const int64_t e0 = tri_start(__shfl(p, s, WAVE));
                    const int l = __shfl(len, s, WAVE);
                    unsigned int t = tri_walk<SLOTS>(dir, e0 + (lane & 3), e0 + (k < n4 ? l : 0), 4, key, cnt);
                    t += __shfl_xor(t, 1, WAVE);
                    t += __shfl_xor(t, 2, WAVE);
                    if ((lane & 3) == 0 && k < n4) hits[wv][s] = t;
                }
                for (int r = 0; r < n16; r += 4) {
                    const int k = r + (lane >> 4), s = k < n16 ? sel[wv][n4 + k] : 0;
                    const int64_t e0 = tri_start(__shfl(p, s, WAVE));
                    const int l = __shfl(len, s, WAVE);
                    unsigned int t = tri_walk<SLOTS>(dir, e0 + (lane & 15), e0 + (k < n16 ? l : 0), 16, key, cnt);
                    for (int o = 8; o >= 1; o >>= 1) t += __shfl_xor(t, o, WAVE);
                    if ((lane & 15) == 0 && k < n16) hits[wv][s] = t;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                unsigned int mine = hits[wv][lane];
                while (m64) {
                    const int s = __ffsll((long long)m64) - 1;
                    m64 &= m64 - 1;
                    const int64_t e0 = tri_start(__shfl(p, s, WAVE));
                    const int n_e = __shfl(len, s, WAVE);
                    unsigned int t = tri_walk<SLOTS>(dir, e0 + lane, e0 + n_e, WAVE, key, cnt);
                    for (int o = WAVE / 2; o >= 1; o >>= 1) t += __shfl_xor(t, o, WAVE);
                    if (lane == s) mine = t;
                }
                if (mine) atomicAdd(&lam[a], (unsigned long long)mine);
                own += mine;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < K; ++u)
                if (slot[u] >= 0) {
                    if (cnt[slot[u]]) atomicAdd(&lam[x[u]], (unsigned long long)cnt[slot[u]]);
                    key[slot[u]] = TRI_EMPTY;
                    cnt[slot[u]] = 0u;
                }
            __syncthreads();
        }
        for (int o = WAVE / 2; o >= 1; o >>= 1) own += __shfl_xor(own, o, WAVE);
        if (lane == 0) wsum[wv] = own;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long tot = 0;
            for (int w = 0; w < TB / WAVE; ++w) tot += wsum[w];
            if (tot) atomicAdd(&lam[b], tot);
        }
        // wsum is written again only after the next row's barriers
    }
}

// lambda_i and c_i; per-block partial sums of c_i over d_i > 1 (and their
// count), in a fixed order for the host to finish.
__global__ void k_clustering(int64_t n, const int64_t *__restrict__ row_ptr, const unsigned long long *__restrict__ lam,
                             int64_t *__restrict__ lambda, double *__restrict__ c, double *__restrict__ part_sum,
                             unsigned long long *__restrict__ part_cnt) {
    __shared__ double ssum[PBLOCK];
    __shared__ unsigned long long scnt[PBLOCK];
    double s = 0.0;
    unsigned long long k = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t l = (int64_t)lam[i];
        const int64_t d = row_ptr[i + 1] - row_ptr[i];
        double ci = 0.0;
        if (d > 1) {
            ci = (double)l / ((double)d * (double)(d - 1) / 2.0);
            s += ci;
            ++k;
        }
        if (lambda) lambda[i] = l;
        if (c) c[i] = ci;
    }
    ssum[threadIdx.x] = s;
    scnt[threadIdx.x] = k;
    __syncthreads();
    for (int o = PBLOCK / 2; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) {
            ssum[threadIdx.x] += ssum[threadIdx.x + o];
            scnt[threadIdx.x] += scnt[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part_sum[blockIdx.x] = ssum[0];
        part_cnt[blockIdx.x] = scnt[0];
    }
}

// ----------------------------------------------------------- components --

// Every vertex starts under the smaller of itself and its first neighbour (the
// smallest one: rows are ascending), a plain store per vertex.  In a
// connected power-law graph stored by degree that already hangs most
// vertices under vertex 0, two or three steps up.  Where neighbours are stored near one another
// (meshes row by row, banded orders) it makes chains as long as the band is narrow, so
// a workgroup first follows the parents inside its HOOK_ROWS vertices in LDS, by
// doubling, until they lie outside or are roots.
constexpr int HOOK_TB = 1024, HOOK_ROWS = 4096;

__global__ __launch_bounds__(HOOK_TB) void k_hook_first(int64_t n, const int64_t *__restrict__ row_ptr,
                                                        const int32_t *__restrict__ col,
                                                        int32_t *__restrict__ parent) {
    constexpr int K = HOOK_ROWS / HOOK_TB;
    __shared__ int32_t par[HOOK_ROWS];
    const int64_t base = (int64_t)blockIdx.x * HOOK_ROWS;
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const int k = u * HOOK_TB + (int)threadIdx.x;
        const int64_t i = base + k;
        int32_t p = (int32_t)i;
        if (i < n) {
            const int64_t b = row_ptr[i];
            if (row_ptr[i + 1] > b) p = min(p, col[b]);
        }
        par[k] = p;
    }
    // any value read is an ancestor, whichever thread wrote it last
    auto at = [&](int k) { return __hip_atomic_load(&par[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    int moved;
    do {
        __syncthreads();
        moved = 0;
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const int k = u * HOOK_TB + (int)threadIdx.x;
            const int32_t p = at(k);
            if (p < base || p == base + k) continue;
            const int32_t q = at((int)(p - base));
            if (q != p) {
                __hip_atomic_store(&par[k], q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                moved = 1;
            }
        }
    } while (__syncthreads_or(moved));
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const int k = u * HOOK_TB + (int)threadIdx.x;
        if (base + k < n) parent[base + k] = at(k);
    }
}

// Parent of x as this workgroup may see it: a load that the vector L1 and the
// XCD's L2 serve, so that the many lookups of one popular root stay on the
// chip (the same loads with device scope go to the memory side, where a
// million reads of one address are answered one after another).  It can be
// an older value: that is still a vertex of the same tree, smaller than x.
__device__ __forceinline__ int32_t uf_seen(const int32_t *parent, int32_t x) {
    return __hip_atomic_load(&parent[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Root of x, halving the path on the way: x is pointed at its grandparent
// with atomicMin.  Ids decrease along every path, so the smaller of two
// ancestors is the one nearer the root: a halving never moves a vertex away
// from its root, whatever other halvings or final writes it races with.
// The first UF_NEAR steps read cached values; a longer path (a chain of
// vertices) is followed with device scope, where it sees the other
// threads' halvings.  Vertex 0 is a root whatever happens.  The answer can be
// a vertex that has been joined since; joins confirm it (uf_union).
constexpr int UF_NEAR = 8;

__device__ __forceinline__ int32_t uf_root(int32_t *parent, int32_t x) {
    for (int t = 0; t < UF_NEAR; ++t) {
        const int32_t px = uf_seen(parent, x);
        if (px == x || px == 0) return px;
        x = px;
    }
    int32_t px = __hip_atomic_load(&parent[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while (px != x && px != 0) {
        const int32_t ppx = __hip_atomic_load(&parent[px], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ppx != px) atomicMin(&parent[x], ppx);
        x = px;
        px = ppx;
    }
    return px;
}

// Join the trees of a and b: the larger root goes under the smaller.  The
// compare-and-swap succeeds only on a vertex that is a root at that moment
// (the smaller vertex may be an inner one of its tree: the larger root then
// hangs below it); a failed one returns the vertex the larger was joined to,
// which is smaller, and the lookup goes on from there, so the loop ends.
__device__ __forceinline__ void uf_union(int32_t *parent, int32_t a, int32_t b) {
    for (;;) {
        a = uf_root(parent, a);
        b = uf_root(parent, b);
        if (a == b) return;
        if (a > b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t was = atomicCAS(&parent[b], b, a);
        if (was == b) return;
        b = was;
    }
}

// Every vertex points at its root (atomicMin: the root is the smallest
// ancestor, so a late halving by another thread cannot replace it).  Between
// the joins the root may be out of date, which is harmless; after the last
// join's kernel it is the tree's.
// A wave whose parents are all one vertex looks its root up once.
__global__ __launch_bounds__(PBLOCK) void k_flatten(int64_t n, int32_t *__restrict__ parent) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x - lane); base < n; base += step) {
        const int64_t i = base + lane;
        const int32_t p = i < n ? uf_seen(parent, (int32_t)i) : 0;
        const bool go = p != 0 && p != (int32_t)i;
        const unsigned long long want = __ballot(go);
        if (!want) continue;
        const int lead = __ffsll((long long)want) - 1;
        const bool one = __all(!go || p == __shfl(p, lead, WAVE));
        int32_t r = p;
        if (one ? lane == lead : go) r = uf_root(parent, p);
        if (one) r = __shfl(r, lead, WAVE);
        if (go && r != p) atomicMin(&parent[i], r);
    }
}

// Joins in two passes (the sampling idea of Afforest, Sutton et al., 2018)
// after k_hook_first: the first UF_ROOT entries of every vertex that hooked
// nowhere, then all entries of the rows whose root is not 0 at that moment.
// A skipped row's vertex is joined to 0, and any edge from it to a vertex
// outside 0's tree is taken from that vertex's own row, which is not skipped,
// so every component is found.  Only the roots join in the first pass, each
// mostly moving itself: had every vertex of a hub's tree joined its own
// second entry, all of them would have tried the same compare-and-swap on the
// hub (n = 2^20, m = 16M by degree: 1.57 ms of it).
constexpr int64_t UF_ROOT = 4;

__global__ void k_union_roots(int64_t n, const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ col,
                              int32_t *__restrict__ parent) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        if (i == 0 || uf_seen(parent, (int32_t)i) != (int32_t)i) continue;
        const int64_t b = row_ptr[i], e = min(row_ptr[i + 1], b + UF_ROOT);
        for (int64_t p = b; p < e; ++p) uf_union(parent, (int32_t)i, col[p]);
    }
}

// All entries of the remaining rows (an entry joined before finds its two
// roots equal): a wave finds the rows of its 64 that do not hang under 0; rows of up to
// UF_LANE entries are walked by their own lanes, longer ones by all of the wave's.
constexpr int64_t UF_LANE = 4;

__global__ __launch_bounds__(PBLOCK) void k_union_rest(int64_t n, const int64_t *__restrict__ row_ptr,
                                                       const int32_t *__restrict__ col, int32_t *__restrict__ parent) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t nw = (int64_t)gridDim.x * (PBLOCK / WAVE);
    for (int64_t base = ((int64_t)blockIdx.x * (PBLOCK / WAVE) + (threadIdx.x >> 6)) * WAVE; base < n;
         base += nw * WAVE) {
        const int64_t mine = base + lane;
        int64_t b = 0, e = 0;
        if (mine < n && uf_seen(parent, (int32_t)mine) != 0) {
            b = row_ptr[mine];
            e = row_ptr[mine + 1];
        }
        const bool small = e - b <= UF_LANE;
        if (small)
            for (int64_t p = b; p < e; ++p) uf_union(parent, (int32_t)mine, col[p]);
        unsigned long long todo = __ballot(!small);
        while (todo) {
            const int t = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            const int64_t i = base + t, b0 = shfl(b, t), b1 = shfl(e, t);
            if (shfl(uf_seen(parent, (int32_t)i), t) == 0) continue;      // joined to 0 meanwhile
            for (int64_t p = b0 + lane; p < b1; p += WAVE) uf_union(parent, (int32_t)i, col[p]);
        }
    }
}

__global__ void k_count_roots(int64_t n, const int32_t *__restrict__ parent, unsigned long long *__restrict__ cnt) {
    unsigned long long k = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        k += parent[i] == (int32_t)i ? 1 : 0;
    for (int o = WAVE / 2; o >= 1; o >>= 1) k += __shfl_xor(k, o, WAVE);
    if ((threadIdx.x & (WAVE - 1)) == 0 && k) atomicAdd(cnt, k);
}

// Grouping of the components for the relaxation's per-component centring:
// sort keys (the component's smallest vertex; isolated vertices last).
__global__ void k_comp_keys(int64_t n, const int64_t *__restrict__ row_ptr, const int32_t *__restrict__ parent,
                            uint32_t *__restrict__ key, uint32_t *__restrict__ val) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        key[i] = row_ptr[i + 1] > row_ptr[i] ? (uint32_t)parent[i] : (uint32_t)n;   // isolated: n, sorted last
        val[i] = (uint32_t)i;
    }
}

// head[p] = 1 where sorted position p starts a component.
__global__ void k_comp_heads(int64_t n, const uint32_t *__restrict__ key, uint32_t *__restrict__ head) {
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x)
        head[p] = (key[p] != (uint32_t)n && (p == 0 || key[p] != key[p - 1])) ? 1u : 0u;
}

// comp_of, members and the component starts from the sorted order and the
// exclusive scan of the heads; the last live position closes the last
// component.
__global__ void k_comp_fill(int64_t n, const uint32_t *__restrict__ key, const uint32_t *__restrict__ val,
                            const uint32_t *__restrict__ head, const uint32_t *__restrict__ before,
                            int32_t *__restrict__ comp_of, int32_t *__restrict__ members,
                            int64_t *__restrict__ comp_start) {
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = (int32_t)val[p];
        if (key[p] == (uint32_t)n) {
            comp_of[v] = -1;
            continue;
        }
        const int64_t c = (int64_t)before[p] + head[p] - 1;
        comp_of[v] = (int32_t)c;
        members[p] = v;
        if (head[p]) comp_start[c] = p;
        if (p + 1 == n || key[p + 1] == (uint32_t)n) comp_start[c + 1] = p + 1;
    }
}

// Chunks of COMP_CHUNK members per component (the entry after the last is 0,
// so an exclusive scan ends with the total).
__global__ void k_comp_chunks(int64_t nc, const int64_t *__restrict__ comp_start, int64_t *__restrict__ cnt) {
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c <= nc; c += (int64_t)gridDim.x * blockDim.x)
        cnt[c] = c < nc ? (comp_start[c + 1] - comp_start[c] + COMP_CHUNK - 1) / COMP_CHUNK : 0;
}

// ------------------------------------------------------------- spearman --

// Twice the mean rank of every score, from the sorted scores: a run of equal
// scores at sorted positions [a, b) holds ranks a+1 .. b, mean (a + 1 + b) / 2.
template <typename K>
__global__ void k_mean_ranks(int64_t n, const K *__restrict__ sorted, const uint32_t *__restrict__ idx,
                             int64_t *__restrict__ rank2) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
        const K v = sorted[t];
        int64_t a = t, b = t + 1;
        // run bounds by binary search over the sorted scores
        int64_t lo = 0, hi = t;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (sorted[mid] < v) lo = mid + 1;
            else hi = mid;
        }
        a = lo;
        lo = t + 1;
        hi = n;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (sorted[mid] <= v) lo = mid + 1;
            else hi = mid;
        }
        b = lo;
        rank2[idx[t]] = a + 1 + b;
    }
}

// Per-block sums of (2 p_i)^2 in a fixed order (exact while below 2^53 per term).
__global__ void k_rank_diff2(int64_t n, const int64_t *__restrict__ rx2, const int64_t *__restrict__ ry2,
                             double *__restrict__ part) {
    __shared__ double s[PBLOCK];
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double d = (double)(rx2[i] - ry2[i]);
        acc += d * d;
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int o = PBLOCK / 2; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = s[0];
}

// ------------------------------------------------------------- layouts --

struct SubLayout {
    uint32_t *k32, *new_id;   // [m]
    uint32_t *pos;            // [2m] kept entries before each stored entry
    void *temp;
    size_t temp_bytes;
};

static size_t sub_layout(const ad_graph *g, void *ws, size_t ws_bytes, SubLayout *L) {
    Carver c(ws, ws_bytes);
    const size_t m = (size_t)std::max<int64_t>(1, g->m);
    SubLayout l;
    l.k32 = c.take<uint32_t>(m);
    l.new_id = c.take<uint32_t>(m);
    l.pos = c.take<uint32_t>(2 * m);
    size_t t1 = 0, t2 = 0;
    if (rocprim::exclusive_scan(nullptr, t1, (uint32_t *)nullptr, (uint32_t *)nullptr, 0u, m,
                                rocprim::plus<uint32_t>()) != hipSuccess)
        t1 = 0;
    if (rocprim::exclusive_scan(nullptr, t2, entry_kept(nullptr, nullptr), (uint32_t *)nullptr, 0u, 2 * m,
                                rocprim::plus<uint32_t>()) != hipSuccess)
        t2 = 0;
    l.temp_bytes = std::max(t1, t2);
    l.temp = c.take<char>(l.temp_bytes);
    if (L) *L = l;
    return c.ok() ? c.used : 0;
}

struct PropLayout {
    unsigned long long *lam;      // [n]
    unsigned int *flags;          // [4]: rows per list of long rows
    int32_t *tri_rows;            // [2][n]: the long rows
    int32_t *tri_wide;            // [m / (TRI_WIDE + 1) + 1]: rows with more than TRI_WIDE upper neighbours
    int32_t *deg;                 // [n]
    int32_t *dir;                 // [2m]: rows, upper neighbours first
    uint64_t *place;              // [n]: upper neighbours' places in dir
    unsigned long long *roots;    // [1]
    double *part_sum;             // [PREDUCE_BLOCKS]
    unsigned long long *part_cnt; // [PREDUCE_BLOCKS]
    int32_t *parent;              // [n] when the caller passes no comp array
};

static size_t prop_layout(const ad_graph *g, void *ws, size_t ws_bytes, PropLayout *L) {
    Carver c(ws, ws_bytes);
    const size_t m = (size_t)std::max<int64_t>(1, g->m), n = (size_t)std::max<int64_t>(1, g->n);
    PropLayout l;
    l.lam = c.take<unsigned long long>(n);
    l.flags = c.take<unsigned int>(4);
    l.tri_rows = c.take<int32_t>(2 * n);
    l.tri_wide = c.take<int32_t>(m / (TRI_WIDE + 1) + 1);
    l.deg = c.take<int32_t>(n);
    l.dir = c.take<int32_t>(2 * m);
    l.place = c.take<uint64_t>(n);
    l.roots = c.take<unsigned long long>(1);
    l.part_sum = c.take<double>(PREDUCE_BLOCKS);
    l.part_cnt = c.take<unsigned long long>(PREDUCE_BLOCKS);
    l.parent = c.take<int32_t>(n);
    if (L) *L = l;
    return c.ok() ? c.used : 0;
}

// Connected components by union-find: every vertex starts under its smallest
// neighbour (k_hook_first), the other entries (i, j) join the trees of i and j
// (k_union_roots, k_union_rest for the rows not yet under 0), hanging the
// larger root under the smaller with a compare-and-swap, then every vertex
// is pointed at its root.  A parent is always smaller than its child, so the
// trees have no cycles, every root search ends, and each component's root is
// its smallest vertex whatever the order of the joins.  No host round trips.
// Bound by the dependent parent lookups.  n = 2^20, m = 16M stored by degree:
// 2.3 ms with the first two entries of every row joined by compare-and-swap
// and every lookup at device scope (2.1 ms of it one address, the hub's),
// 0.035 ms here (six launches).  A component build, so / here, and with the chains left to
// k_flatten: 2,048 x 2,048 mesh row by row 3.63 / 0.49 (0.65) ms, path of 2^22 vertices in order
// 8 to 11 / 0.53 (16.3), 2^19 pairs 0.34 / 0.29 (their rows walked by whole waves: 0.37).
ad_status label_components(const ad_graph *g, int32_t *parent, hipStream_t stream) {
    const int64_t n = g->n;
    hipLaunchKernelGGL(k_hook_first, dim3((unsigned)std::max<int64_t>(1, ceil_div(n, HOOK_ROWS))), dim3(HOOK_TB), 0, stream, n,
                       g->row_ptr, g->col, parent);
    AD_LAUNCH_CHECK("k_hook_first");
    if (g->m > 0) {
        hipLaunchKernelGGL(k_flatten, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, parent);
        AD_LAUNCH_CHECK("k_flatten");
        hipLaunchKernelGGL(k_union_roots, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, g->row_ptr, g->col, parent);
        AD_LAUNCH_CHECK("k_union_roots");
        hipLaunchKernelGGL(k_flatten, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, parent);
        AD_LAUNCH_CHECK("k_flatten");
        hipLaunchKernelGGL(k_union_rest, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(4096, ceil_div(n, PBLOCK)))),
                           dim3(PBLOCK), 0, stream, n, g->row_ptr, g->col, parent);
        AD_LAUNCH_CHECK("k_union_rest");
        hipLaunchKernelGGL(k_flatten, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, parent);
        AD_LAUNCH_CHECK("k_flatten");
    }
    return AD_OK;
}

struct CompLayout {
    int32_t *parent;              // [n]
    uint32_t *key0, *key1, *val0, *val1, *head, *before;   // [n]
    int64_t *cnt;                 // [n + 1]
    void *temp;
    size_t temp_bytes;
};

static size_t comp_layout(int64_t n, void *ws, size_t ws_bytes, CompLayout *L) {
    Carver c(ws, ws_bytes);
    const size_t nn = (size_t)std::max<int64_t>(1, n);
    CompLayout l;
    l.parent = c.take<int32_t>(nn);
    l.key0 = c.take<uint32_t>(nn);
    l.key1 = c.take<uint32_t>(nn);
    l.val0 = c.take<uint32_t>(nn);
    l.val1 = c.take<uint32_t>(nn);
    l.head = c.take<uint32_t>(nn);
    l.before = c.take<uint32_t>(nn);
    l.cnt = c.take<int64_t>(nn + 1);
    size_t t0 = 0, t1 = 0, t2 = 0;
    if (rocprim::radix_sort_pairs(nullptr, t0, (uint32_t *)nullptr, (uint32_t *)nullptr, (uint32_t *)nullptr,
                                  (uint32_t *)nullptr, nn) != hipSuccess)
        t0 = 0;
    if (rocprim::exclusive_scan(nullptr, t1, (uint32_t *)nullptr, (uint32_t *)nullptr, 0u, nn,
                                rocprim::plus<uint32_t>()) != hipSuccess)
        t1 = 0;
    if (rocprim::exclusive_scan(nullptr, t2, (int64_t *)nullptr, (int64_t *)nullptr, (int64_t)0, nn + 1,
                                rocprim::plus<int64_t>()) != hipSuccess)
        t2 = 0;
    l.temp_bytes = std::max(t0, std::max(t1, t2));
    l.temp = c.take<char>(l.temp_bytes);
    if (L) *L = l;
    return c.ok() ? c.used : 0;
}

struct RankLayout {
    double *keys1;                // [n] sorted scores
    uint32_t *idx1;               // [n] and whose they are
    int64_t *rx2, *ry2;           // [n]
    double *part;                 // [PREDUCE_BLOCKS]
    void *temp;
    size_t temp_bytes;
};

static size_t rank_layout(int64_t n, void *ws, size_t ws_bytes, RankLayout *L) {
    Carver c(ws, ws_bytes);
    const size_t nn = (size_t)std::max<int64_t>(1, n);
    RankLayout l;
    l.keys1 = c.take<double>(nn);
    l.idx1 = c.take<uint32_t>(nn);
    l.rx2 = c.take<int64_t>(nn);
    l.ry2 = c.take<int64_t>(nn);
    l.part = c.take<double>(PREDUCE_BLOCKS);
    size_t t = 0;
    if (rocprim::radix_sort_pairs(nullptr, t, (const double *)nullptr, (double *)nullptr,
                                  rocprim::counting_iterator<uint32_t>(0), (uint32_t *)nullptr, nn) != hipSuccess)
        t = 0;
    size_t t32 = 0;
    if (rocprim::radix_sort_pairs(nullptr, t32, (const uint32_t *)nullptr, (uint32_t *)nullptr,
                                  rocprim::counting_iterator<uint32_t>(0), (uint32_t *)nullptr, nn) == hipSuccess)
        t = std::max(t, t32);
    l.temp_bytes = t;
    l.temp = c.take<char>(t);
    if (L) *L = l;
    return c.ok() ? c.used : 0;
}

#define AD_RP(call)                                                         \
    do {                                                                    \
        hipError_t e_ = (call);                                             \
        if (e_ != hipSuccess) return fail(AD_ERR_HIP, std::string("rocPRIM: ") + hipGetErrorString(e_)); \
    } while (0)

static ad_status check_ws(void *ws, size_t need, size_t ws_bytes) {
    if (!ws) return fail(AD_ERR_INVALID_ARG, "workspace is NULL");
    if (((uintptr_t)ws & 255) != 0) return fail(AD_ERR_WORKSPACE, "workspace not 256-byte aligned");
    if (need == 0 || ws_bytes < need) return fail(AD_ERR_WORKSPACE, "workspace too small");
    return AD_OK;
}

}  // namespace ad

using namespace ad;

extern "C" size_t ad_subgraph_workspace_size(const ad_graph *g) {
    if (check_graph_args(g) != AD_OK) return 0;
    return sub_layout(g, nullptr, 0, nullptr);
}

extern "C" ad_status ad_subgraph(const ad_graph *g, const uint8_t *keep, int64_t *sub_row_ptr, int32_t *sub_col,
                                 float *sub_w, int32_t *sub_eid, int32_t *orig_edge, int64_t *m_sub_host, void *ws,
                                 size_t ws_bytes, hipStream_t stream) {
    ad_status s = check_graph_args(g);
    if (s != AD_OK) return s;
    if (g->m > 0 && !keep) return fail(AD_ERR_INVALID_ARG, "keep is NULL");
    if (!sub_row_ptr || !m_sub_host) return fail(AD_ERR_INVALID_ARG, "sub_row_ptr or m_sub_host is NULL");
    if (g->m > 0 && (!sub_col || !sub_eid)) return fail(AD_ERR_INVALID_ARG, "sub_col or sub_eid is NULL");
    if (g->m >= ((int64_t)1 << 31)) return fail(AD_ERR_UNSUPPORTED, "more than 2^31 - 1 edges");
    s = check_ws(ws, sub_layout(g, nullptr, 0, nullptr), ws_bytes);
    if (s != AD_OK) return s;
    SubLayout L;
    if (sub_layout(g, ws, ws_bytes, &L) == 0) return fail(AD_ERR_WORKSPACE, "workspace too small");
    TraceScope trace("k_subgraph", stream);
    const int64_t n = g->n, m = g->m;
    uint32_t last[2] = {0, 0};
    if (m > 0) {
        hipLaunchKernelGGL(k_keep_u32, dim3(pgrid(m)), dim3(PBLOCK), 0, stream, m, keep, L.k32);
        AD_LAUNCH_CHECK("k_keep_u32");
        size_t tb = L.temp_bytes;
        AD_RP(rocprim::exclusive_scan(L.temp, tb, L.k32, L.new_id, 0u, (size_t)m, rocprim::plus<uint32_t>(), stream));
        AD_HIP(hipMemcpyAsync(&last[0], L.new_id + (m - 1), sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
        AD_HIP(hipMemcpyAsync(&last[1], L.k32 + (m - 1), sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    }
    if (m > 0) {
        size_t tb = L.temp_bytes;
        AD_RP(rocprim::exclusive_scan(L.temp, tb, entry_kept(keep, g->eid), L.pos, 0u, (size_t)(2 * m),
                                      rocprim::plus<uint32_t>(), stream));
    }
    hipLaunchKernelGGL(k_sub_rows, dim3(pgrid(n + 1)), dim3(PBLOCK), 0, stream, n, 2 * m, g->row_ptr, g->eid, keep,
                       L.pos, sub_row_ptr);
    AD_LAUNCH_CHECK("k_sub_rows");
    if (m > 0) {
        hipLaunchKernelGGL(k_compact_entries, dim3(pgrid(2 * m)), dim3(PBLOCK), 0, stream, 2 * m, g->col, g->w,
                           g->eid, keep, L.new_id, L.pos, sub_col, g->w ? sub_w : nullptr, sub_eid, orig_edge);
        AD_LAUNCH_CHECK("k_compact_entries");
    }
    AD_HIP(hipStreamSynchronize(stream));
    *m_sub_host = (int64_t)last[0] + (int64_t)last[1];
    return AD_OK;
}

extern "C" size_t ad_graph_properties_workspace_size(const ad_graph *g) {
    if (check_graph_args(g) != AD_OK) return 0;
    return prop_layout(g, nullptr, 0, nullptr);
}

extern "C" ad_status ad_graph_properties(const ad_graph *g, int64_t *lambda, double *c, int32_t *comp,
                                         double *summary_host, void *ws, size_t ws_bytes, hipStream_t stream) {
    ad_status s = check_graph_args(g);
    if (s != AD_OK) return s;
    if (!summary_host) return fail(AD_ERR_INVALID_ARG, "summary_host is NULL");
    if (g->m >= ((int64_t)1 << 31)) return fail(AD_ERR_UNSUPPORTED, "more than 2^31 - 1 edges");
    s = check_ws(ws, prop_layout(g, nullptr, 0, nullptr), ws_bytes);
    if (s != AD_OK) return s;
    PropLayout L;
    if (prop_layout(g, ws, ws_bytes, &L) == 0) return fail(AD_ERR_WORKSPACE, "workspace too small");
    TraceScope trace("k_properties", stream);
    const int64_t n = g->n;
    summary_host[0] = 0.0;
    summary_host[1] = 0.0;
    if (n == 0) return AD_OK;
    // triangles and clustering
    s = fill_u64(L.lam, 0, n, stream);
    if (s != AD_OK) return s;
    s = fill_i32((int32_t *)L.flags, 0, 4, stream);
    if (s != AD_OK) return s;
    if (g->m > 0) {
        hipLaunchKernelGGL(k_triangles_lists, dim3((unsigned)ceil_div(n, TRI_LIST_B)), dim3(TRI_LIST_B), 0, stream, n,
                           g->row_ptr, L.deg, L.tri_rows, L.flags);
        AD_LAUNCH_CHECK("k_triangles_lists");
        const unsigned teams = (unsigned)std::min<int64_t>(4096, ceil_div(n, PBLOCK / TRI_TEAM));
        hipLaunchKernelGGL(k_triangles_orient, dim3(teams), dim3(PBLOCK), 0, stream, n, g->row_ptr, g->col, L.deg,
                           L.tri_rows, L.flags, L.dir, L.place, L.tri_wide);
        AD_LAUNCH_CHECK("k_triangles_orient");
        // a listed row has more than TRI_HUB (TRI_SMALL) of the 2m entries
        const int64_t hubs = 2 * g->m / (TRI_HUB + 1), longs = 2 * g->m / (TRI_SMALL + 1);
        // a wide row has TRI_WIDE + 1 upper neighbours, each of at least as long a row
        if (g->m >= (int64_t)(TRI_WIDE + 1) * (TRI_WIDE + 2) / 2)
            hipLaunchKernelGGL((k_triangles_rows<TRI_WIDE_B, TRI_WIDE_CAP, 2 * TRI_WIDE_CAP, true>), dim3(256, TRI_WIDE_SLICES),
                               dim3(TRI_WIDE_B), 0, stream, L.tri_wide, L.flags + 2, g->row_ptr, L.dir, L.place, L.lam);
        if (hubs > 0)
            hipLaunchKernelGGL((k_triangles_rows<PBLOCK, TRI_CAP, 4 * TRI_CAP, false>),
                               dim3((unsigned)std::min<int64_t>(512, hubs), TRI_SLICES), dim3(PBLOCK), 0, stream,
                               L.tri_rows + n, L.flags + 1, g->row_ptr, L.dir, L.place, L.lam);
        if (longs > 0)
            hipLaunchKernelGGL((k_triangles_rows<PBLOCK, TRI_CAP, 4 * TRI_CAP, false>),
                               dim3((unsigned)std::min<int64_t>(4096, longs), 1), dim3(PBLOCK), 0, stream, L.tri_rows,
                               L.flags, g->row_ptr, L.dir, L.place, L.lam);
        AD_LAUNCH_CHECK("k_triangles_rows");
        hipLaunchKernelGGL(k_triangles_small, dim3(teams), dim3(PBLOCK), 0, stream, n, g->row_ptr, L.dir, L.place,
                           L.lam);
        AD_LAUNCH_CHECK("k_triangles_small");
    }
    hipLaunchKernelGGL(k_clustering, dim3(PREDUCE_BLOCKS), dim3(PBLOCK), 0, stream, n, g->row_ptr, L.lam, lambda, c,
                       L.part_sum, L.part_cnt);
    AD_LAUNCH_CHECK("k_clustering");
    // components by union-find, in a fixed number of launches
    int32_t *parent = comp ? comp : L.parent;
    s = label_components(g, parent, stream);
    if (s != AD_OK) return s;
    s = fill_u64(L.roots, 0, 1, stream);
    if (s != AD_OK) return s;
    hipLaunchKernelGGL(k_count_roots, dim3(std::min<unsigned>(256, pgrid(n))), dim3(PBLOCK), 0, stream, n, parent,
                       L.roots);
    AD_LAUNCH_CHECK("k_count_roots");
    double psum[PREDUCE_BLOCKS];
    unsigned long long pcnt[PREDUCE_BLOCKS], roots = 0;
    AD_HIP(hipMemcpyAsync(psum, L.part_sum, sizeof(psum), hipMemcpyDeviceToHost, stream));
    AD_HIP(hipMemcpyAsync(pcnt, L.part_cnt, sizeof(pcnt), hipMemcpyDeviceToHost, stream));
    AD_HIP(hipMemcpyAsync(&roots, L.roots, sizeof(roots), hipMemcpyDeviceToHost, stream));
    AD_HIP(hipStreamSynchronize(stream));
    double sum = 0.0;
    unsigned long long cnt = 0;
    for (int b = 0; b < PREDUCE_BLOCKS; ++b) {
        sum += psum[b];
        cnt += pcnt[b];
    }
    summary_host[0] = cnt ? sum / (double)cnt : 0.0;
    summary_host[1] = (double)roots;
    return AD_OK;
}

extern "C" size_t ad_components_workspace_size(const ad_graph *g) {
    if (check_graph_args(g) != AD_OK || g->n >= ((int64_t)1 << 31)) return 0;
    return comp_layout(g->n, nullptr, 0, nullptr);
}

extern "C" ad_status ad_components_build(const ad_graph *g, int32_t *comp_of, int32_t *members, int64_t *comp_start,
                                         int64_t *chunk_start, int64_t *n_comp_host, int64_t *n_chunks_host,
                                         void *ws, size_t ws_bytes, hipStream_t stream) {
    ad_status s = check_graph_args(g);
    if (s != AD_OK) return s;
    if (!n_comp_host || !n_chunks_host) return fail(AD_ERR_INVALID_ARG, "n_comp_host or n_chunks_host is NULL");
    if (!comp_start || !chunk_start) return fail(AD_ERR_INVALID_ARG, "comp_start or chunk_start is NULL");
    if (g->n > 0 && (!comp_of || !members)) return fail(AD_ERR_INVALID_ARG, "comp_of or members is NULL");
    if (g->n >= ((int64_t)1 << 31)) return fail(AD_ERR_UNSUPPORTED, "n must be below 2^31");
    s = check_ws(ws, comp_layout(g->n, nullptr, 0, nullptr), ws_bytes);
    if (s != AD_OK) return s;
    CompLayout L;
    if (comp_layout(g->n, ws, ws_bytes, &L) == 0) return fail(AD_ERR_WORKSPACE, "workspace too small");
    TraceScope trace("k_components", stream);
    const int64_t n = g->n;
    *n_comp_host = 0;
    *n_chunks_host = 0;
    int64_t zero[2] = {0, 0};
    if (n == 0) {
        AD_HIP(hipMemcpyAsync(comp_start, zero, sizeof(int64_t), hipMemcpyHostToDevice, stream));
        AD_HIP(hipMemcpyAsync(chunk_start, zero, sizeof(int64_t), hipMemcpyHostToDevice, stream));
        AD_HIP(hipStreamSynchronize(stream));
        return AD_OK;
    }
    s = label_components(g, L.parent, stream);
    if (s != AD_OK) return s;
    hipLaunchKernelGGL(k_comp_keys, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, g->row_ptr, L.parent, L.key0, L.val0);
    AD_LAUNCH_CHECK("k_comp_keys");
    size_t tb = L.temp_bytes;
    // keys are at most n (< 2^31): only their low bit_width(n) bits are sorted
    int key_bits = 1;
    while (key_bits < 32 && ((uint64_t)n >> key_bits) != 0) ++key_bits;
    AD_RP(rocprim::radix_sort_pairs(L.temp, tb, L.key0, L.key1, L.val0, L.val1, (size_t)n, 0, key_bits, stream));
    hipLaunchKernelGGL(k_comp_heads, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, L.key1, L.head);
    AD_LAUNCH_CHECK("k_comp_heads");
    tb = L.temp_bytes;
    AD_RP(rocprim::exclusive_scan(L.temp, tb, L.head, L.before, 0u, (size_t)n, rocprim::plus<uint32_t>(), stream));
    uint32_t last[2] = {0, 0};
    AD_HIP(hipMemcpyAsync(&last[0], L.before + (n - 1), sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    AD_HIP(hipMemcpyAsync(&last[1], L.head + (n - 1), sizeof(uint32_t), hipMemcpyDeviceToHost, stream));
    AD_HIP(hipStreamSynchronize(stream));
    const int64_t nc = (int64_t)last[0] + (int64_t)last[1];
    if (nc == 0) {
        hipLaunchKernelGGL(k_comp_fill, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, L.key1, L.val1, L.head, L.before,
                           comp_of, members, comp_start);
        AD_LAUNCH_CHECK("k_comp_fill");
        AD_HIP(hipMemcpyAsync(comp_start, zero, sizeof(int64_t), hipMemcpyHostToDevice, stream));
        AD_HIP(hipMemcpyAsync(chunk_start, zero, sizeof(int64_t), hipMemcpyHostToDevice, stream));
        AD_HIP(hipStreamSynchronize(stream));
        return AD_OK;
    }
    hipLaunchKernelGGL(k_comp_fill, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, L.key1, L.val1, L.head, L.before,
                       comp_of, members, comp_start);
    AD_LAUNCH_CHECK("k_comp_fill");
    hipLaunchKernelGGL(k_comp_chunks, dim3(pgrid(nc + 1)), dim3(PBLOCK), 0, stream, nc, comp_start, L.cnt);
    AD_LAUNCH_CHECK("k_comp_chunks");
    tb = L.temp_bytes;
    AD_RP(rocprim::exclusive_scan(L.temp, tb, L.cnt, chunk_start, (int64_t)0, (size_t)(nc + 1),
                                  rocprim::plus<int64_t>(), stream));
    int64_t nch = 0;
    AD_HIP(hipMemcpyAsync(&nch, chunk_start + nc, sizeof(int64_t), hipMemcpyDeviceToHost, stream));
    AD_HIP(hipStreamSynchronize(stream));
    *n_comp_host = nc;
    *n_chunks_host = nch;
    return AD_OK;
}

extern "C" size_t ad_spearman_workspace_size(int64_t n) {
    if (n < 0 || n >= ((int64_t)1 << 31)) return 0;
    return rank_layout(n, nullptr, 0, nullptr);
}

// Spearman's formula for scores of `bits` bits: doubles, or whole numbers as
// uint32_t, whose sort moves 8 bytes per score instead of 12 (the degrees of
// ad_compare_properties).  The scores are read where they are and the index array
// is an iterator: two passes over n less per score.
template <typename K>
static ad_status spearman_impl(int64_t n, const K *x, const K *y, unsigned bits, double *rho_host, void *ws,
                               size_t ws_bytes, hipStream_t stream) {
    if (n < 0) return fail(AD_ERR_INVALID_ARG, "negative n");
    if (n >= ((int64_t)1 << 31)) return fail(AD_ERR_UNSUPPORTED, "n must be below 2^31");
    if (n > 0 && (!x || !y)) return fail(AD_ERR_INVALID_ARG, "x or y is NULL");
    if (!rho_host) return fail(AD_ERR_INVALID_ARG, "rho_host is NULL");
    ad_status s = check_ws(ws, rank_layout(n, nullptr, 0, nullptr), ws_bytes);
    if (s != AD_OK) return s;
    RankLayout L;
    if (rank_layout(n, ws, ws_bytes, &L) == 0) return fail(AD_ERR_WORKSPACE, "workspace too small");
    *rho_host = 0.0;
    if (n < 2) return AD_OK;
    TraceScope trace("k_spearman", stream);
    const K *src[2] = {x, y};
    K *sorted = reinterpret_cast<K *>(L.keys1);
    int64_t *dst[2] = {L.rx2, L.ry2};
    for (int v = 0; v < 2; ++v) {
        size_t tb = L.temp_bytes;
        AD_RP(rocprim::radix_sort_pairs(L.temp, tb, src[v], sorted, rocprim::counting_iterator<uint32_t>(0), L.idx1,
                                        (size_t)n, 0, bits, stream));
        hipLaunchKernelGGL(k_mean_ranks<K>, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, sorted, L.idx1, dst[v]);
        AD_LAUNCH_CHECK("k_mean_ranks");
    }
    hipLaunchKernelGGL(k_rank_diff2, dim3(PREDUCE_BLOCKS), dim3(PBLOCK), 0, stream, n, L.rx2, L.ry2, L.part);
    AD_LAUNCH_CHECK("k_rank_diff2");
    double part[PREDUCE_BLOCKS];
    AD_HIP(hipMemcpyAsync(part, L.part, sizeof(part), hipMemcpyDeviceToHost, stream));
    AD_HIP(hipStreamSynchronize(stream));
    double sum4 = 0.0;    // sum of (2 p_i)^2
    for (int b = 0; b < PREDUCE_BLOCKS; ++b) sum4 += part[b];
    const double dn = (double)n;
    *rho_host = 1.0 - 6.0 * (sum4 / 4.0) / (dn * (dn * dn - 1.0));
    return AD_OK;
}

extern "C" ad_status ad_spearman(int64_t n, const double *x, const double *y, double *rho_host, void *ws,
                                 size_t ws_bytes, hipStream_t stream) {
    return spearman_impl<double>(n, x, y, 8 * (unsigned)sizeof(double), rho_host, ws, ws_bytes, stream);
}

// ------------------------------------------------------------ comparison --

namespace ad {

// Degree of every vertex (the score Spearman's formula ranks).
__global__ void k_degrees(int64_t n, const int64_t *__restrict__ row_ptr, uint32_t *__restrict__ deg) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        deg[i] = (uint32_t)(row_ptr[i + 1] - row_ptr[i]);
}

struct CmpLayout {
    int64_t *sub_row_ptr;
    int32_t *sub_col, *sub_eid;
    double *c_o, *c_s;
    uint32_t *deg_o, *deg_s;
    void *ws;                 // the largest of the subgraph, properties and Spearman workspaces
    size_t ws_bytes;
};

static size_t cmp_layout(const ad_graph *g, void *ws, size_t ws_bytes, CmpLayout *L) {
    Carver c(ws, ws_bytes);
    const size_t n = (size_t)std::max<int64_t>(1, g->n), nnz = (size_t)std::max<int64_t>(1, 2 * g->m);
    CmpLayout l;
    l.sub_row_ptr = c.take<int64_t>(n + 1);
    l.sub_col = c.take<int32_t>(nnz);
    l.sub_eid = c.take<int32_t>(nnz);
    l.c_o = c.take<double>(n);
    l.c_s = c.take<double>(n);
    l.deg_o = c.take<uint32_t>(n);
    l.deg_s = c.take<uint32_t>(n);
    ad_graph gu = *g;
    gu.w = nullptr;
    l.ws_bytes = std::max(sub_layout(&gu, nullptr, 0, nullptr),
                          std::max(prop_layout(&gu, nullptr, 0, nullptr), rank_layout(g->n, nullptr, 0, nullptr)));
    l.ws = c.take<char>(l.ws_bytes);
    if (L) *L = l;
    return c.ok() ? c.used : 0;
}

}  // namespace ad

extern "C" size_t ad_compare_properties_workspace_size(const ad_graph *g) {
    if (check_graph_args(g) != AD_OK || g->n >= ((int64_t)1 << 31) || g->m >= ((int64_t)1 << 31)) return 0;
    return cmp_layout(g, nullptr, 0, nullptr);
}

extern "C" ad_status ad_compare_properties(const ad_graph *g, const uint8_t *keep, double *out_host, void *ws,
                                           size_t ws_bytes, hipStream_t stream) {
    ad_status s = check_graph_args(g);
    if (s != AD_OK) return s;
    if (!out_host) return fail(AD_ERR_INVALID_ARG, "out_host is NULL");
    if (g->m > 0 && !keep) return fail(AD_ERR_INVALID_ARG, "keep is NULL");
    if (g->n >= ((int64_t)1 << 31) || g->m >= ((int64_t)1 << 31))
        return fail(AD_ERR_UNSUPPORTED, "n and m must be below 2^31");
    s = check_ws(ws, cmp_layout(g, nullptr, 0, nullptr), ws_bytes);
    if (s != AD_OK) return s;
    CmpLayout L;
    if (cmp_layout(g, ws, ws_bytes, &L) == 0) return fail(AD_ERR_WORKSPACE, "workspace too small");
    for (int q = 0; q < AD_CMP_FIELDS; ++q) out_host[q] = 0.0;
    const int64_t n = g->n;
    ad_graph go = *g;             // the properties read the structure only
    go.w = nullptr;
    go.col_orig = nullptr;
    int64_t ms = 0;
    s = ad_subgraph(&go, keep, L.sub_row_ptr, L.sub_col, nullptr, L.sub_eid, nullptr, &ms, L.ws, L.ws_bytes, stream);
    if (s != AD_OK) return s;
    ad_graph gs = go;
    gs.m = ms;
    gs.row_ptr = L.sub_row_ptr;
    gs.col = L.sub_col;
    gs.eid = L.sub_eid;
    double sum_o[2] = {0.0, 0.0}, sum_s[2] = {0.0, 0.0};
    s = ad_graph_properties(&go, nullptr, L.c_o, nullptr, sum_o, L.ws, L.ws_bytes, stream);
    if (s != AD_OK) return s;
    s = ad_graph_properties(&gs, nullptr, L.c_s, nullptr, sum_s, L.ws, L.ws_bytes, stream);
    if (s != AD_OK) return s;
    double rho_deg = 0.0, rho_c = 0.0;
    if (n > 0) {
        hipLaunchKernelGGL(k_degrees, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, go.row_ptr, L.deg_o);
        AD_LAUNCH_CHECK("k_degrees");
        hipLaunchKernelGGL(k_degrees, dim3(pgrid(n)), dim3(PBLOCK), 0, stream, n, gs.row_ptr, L.deg_s);
        AD_LAUNCH_CHECK("k_degrees");
        unsigned bits = 1;                   // of a degree, at most 2m < 2^32
        while (bits < 32 && ((uint64_t)(2 * g->m) >> bits) != 0) ++bits;
        s = spearman_impl<uint32_t>(n, L.deg_o, L.deg_s, bits, &rho_deg, L.ws, L.ws_bytes, stream);
        if (s != AD_OK) return s;
        s = ad_spearman(n, L.c_o, L.c_s, &rho_c, L.ws, L.ws_bytes, stream);
        if (s != AD_OK) return s;
    }
    out_host[0] = (double)ms;
    out_host[1] = sum_o[0];
    out_host[2] = sum_s[0];
    out_host[3] = sum_o[1];
    out_host[4] = sum_s[1];
    out_host[5] = sum_o[1] > 0.0 ? sum_s[1] / sum_o[1] : 0.0;
    out_host[6] = rho_deg;
    out_host[7] = rho_c;
    return AD_OK;
}
