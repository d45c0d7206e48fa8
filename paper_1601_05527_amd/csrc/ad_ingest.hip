// Ingest: an undirected edge list into the symmetric CSR that every other
// call reads (the graph model of Section 2: undirected, no self-loops, no
// repeated pairs), optionally with the vertices stored by decreasing degree.
//
// Readings (shared with the oracle, which is written separately): (u, v) and
// (v, u) name the same edge; self-loops are dropped; repeated pairs become
// one edge whose weight is the exact sum of the listed weights rounded once
// to single precision (listed weights must be finite and positive, as the
// graph model requires); edge ids enumerate the edges
// in (smaller endpoint, larger endpoint) order, the CSR order of their upper
// entries; rows list neighbours in ascending order; the decreasing-degree
// order breaks ties by listed id, and orig_id names the listed vertex.  The
// reverse Cuthill-McKee order: components by increasing smallest id, each
// searched breadth first from its vertex of least (degree, id), the
// neighbours of a dequeued vertex queued by increasing (degree, id), the
// whole order reversed.
//
// The pipeline: canonical pair keys of 2 log2(n) bits, a radix sort (rocPRIM) of
// (key, weight), a scan of the run heads (edge ids), and
// the exact weight sum of every run (a short run by its wave's lanes together, longer ones by
// a wave or a workgroup each); for
// the degree order a stable sort of the vertices by degree and a second pair sort
// under the new labels (for reverse Cuthill-McKee, the graph placed under
// the listed ids, its components, and a level-by-level search with two
// sorts per level, then the same relabelling); then per-row counts from the run lengths of the
// sorted endpoints (no atomics, so hub vertices cost nothing extra), their
// scans and the placement of the upper entries (edge order) and of the
// lower entries (a stable sort of the edges by larger endpoint).
#include "ad_internal.h"

#include <cstring>    // before rocPRIM: its host code calls memset

#include <rocprim/rocprim.hpp>

#include <algorithm>
#include <cfloat>
#include <cstdint>

namespace ad {

constexpr int IBLOCK = 256;
static unsigned bits_for(int64_t n) {
    unsigned b = 1;
    while (b < 32 && ((int64_t)1 << b) < n) ++b;
    return b;
}

// Pair keys hold both ids in 2b bits, b = bits_for(n), smaller id above: the
// radix sorts take a pass per 8 bits, 140 us for 16M keys with weights (n = 2^20:
// five passes; 64-bit keys with list indices took eight and a gather of the
// weights after them: 16M pairs stored by degree, with their components, 6.0 ms;
// 4.4 ms here).
// All ones, the pair of the largest id with itself, stands for no pair and sorts last.
struct PairCode {
    unsigned b;
    unsigned long long none;
    explicit PairCode(int64_t n) : b(bits_for(n)), none((1ull << (2 * b)) - 1) {}
};
__device__ __forceinline__ unsigned long long pair_key(PairCode c, uint64_t lo, uint64_t hi) { return (lo << c.b) | hi; }
__device__ __forceinline__ int32_t pair_lo(PairCode c, unsigned long long k) { return (int32_t)(k >> c.b); }
__device__ __forceinline__ int32_t pair_hi(PairCode c, unsigned long long k) {
    return (int32_t)(k & ((1ull << c.b) - 1));
}

// Key of every listed pair, none for self-loops; endpoints out
// of [0, n) raise the error flag (and sort last).
__global__ void k_pair_keys(int64_t m_in, int64_t n, PairCode code, const int32_t *__restrict__ u,
                            const int32_t *__restrict__ v, const float *__restrict__ w,
                            unsigned long long *__restrict__ key, unsigned int *__restrict__ err) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < m_in; q += (int64_t)gridDim.x * blockDim.x) {
        const int64_t a = u[q], b = v[q];
        unsigned long long k = code.none;
        if (w && !(w[q] > 0.0f && w[q] <= FLT_MAX)) atomicOr(err, 2u);
        if (a < 0 || a >= n || b < 0 || b >= n) {
            atomicOr(err, 1u);
        } else if (a != b) {
            k = pair_key(code, (uint64_t)(a < b ? a : b), (uint64_t)(a < b ? b : a));
        }
        key[q] = k;
    }
}

// 1 at the first entry of every run of equal pair keys, as an iterator for the scan.
struct RunHead {
    const unsigned long long *key;
    unsigned long long none;
    __device__ __host__ uint32_t operator()(int64_t q) const {
        return (key[q] != none && (q == 0 || key[q] != key[q - 1])) ? 1u : 0u;
    }
};
using RunHeadIt = rocprim::transform_iterator<rocprim::counting_iterator<int64_t>, RunHead, uint32_t>;
static RunHeadIt run_heads(const unsigned long long *key, unsigned long long none) {
    return RunHeadIt(rocprim::counting_iterator<int64_t>(0), RunHead{key, none});
}

// Counts as 64-bit numbers, 0 from index n on.
struct CountAt {
    const uint32_t *cnt;
    int64_t n;
    __device__ __host__ uint64_t operator()(int64_t i) const { return i < n ? (uint64_t)cnt[i] : 0ull; }
};
using CountIt = rocprim::transform_iterator<rocprim::counting_iterator<int64_t>, CountAt, uint64_t>;
static CountIt counts_of(const uint32_t *cnt, int64_t n) {
    return CountIt(rocprim::counting_iterator<int64_t>(0), CountAt{cnt, n});
}

// Merged weights: the exact sum of a run's listed weights, rounded once to
// single precision (to nearest, ties to even), so no order of additions
// matters and a run can be summed by many lanes.  A positive finite float
// x is mant * 2^(shift - 149) with mant < 2^24 and 0 <= shift <= 253.  When
// every value of a run lies within 53 bits of one another (the bit span of
// the set plus the bits its count adds), every partial sum is exact in
// double and the double sum, rounded to float, is the answer; otherwise the
// run is summed as an integer count of 2^-149 in XDIG base-2^32 digits with
// deferred carries.
constexpr uint32_t MERGE_SHORT = 16;     // runs up to this length are summed by the wave's lanes together,
constexpr uint32_t MERGE_WAVE = 4096;    // up to this one by a wave each, longer ones by a workgroup each
constexpr int MERGE_TB = 1024;           // threads of a long run's workgroup
constexpr int XDIG = 11;                 // 352 bits: 2^31 floats below 2^277 units each

__device__ __forceinline__ void f32_split(float x, uint32_t &mant, int &shift) {
    const uint32_t b = __float_as_uint(x);
    const uint32_t ex = (b >> 23) & 0xffu, fr = b & 0x7fffffu;
    mant = ex ? (fr | 0x800000u) : fr;
    shift = ex ? (int)ex - 1 : 0;
}

__device__ __forceinline__ int ceil_log2_u32(uint32_t c) { return c <= 1 ? 0 : 32 - __clz((int)(c - 1)); }

// Digits hold values below 2^63 for fewer than 2^31 added floats.
__device__ __forceinline__ void digits_add(unsigned long long (&acc)[XDIG], float x) {
    uint32_t mant;
    int shift;
    f32_split(x, mant, shift);
    const int k = shift >> 5;
    const unsigned long long add = (unsigned long long)mant << (shift & 31);
    const unsigned long long lo = add & 0xffffffffull, hi = add >> 32;
#pragma unroll
    for (int d = 0; d < XDIG; ++d) {
        acc[d] += (d == k) ? lo : 0ull;
        acc[d] += (d == k + 1) ? hi : 0ull;
    }
}

// The float nearest to acc * 2^-149 (ties to even; +inf past the range).
__device__ float digits_round(const unsigned long long (&acc)[XDIG]) {
    uint32_t dg[XDIG];
    unsigned long long carry = 0;
#pragma unroll
    for (int d = 0; d < XDIG; ++d) {
        const unsigned long long t = acc[d] + carry;
        dg[d] = (uint32_t)t;
        carry = t >> 32;
    }
    int top = -1;
#pragma unroll
    for (int d = XDIG - 1; d >= 0; --d)
        if (top < 0 && dg[d] != 0u) top = 32 * d + 31 - __clz((int)dg[d]);
    if (top < 0) return 0.0f;
    if (top <= 23) return ldexpf((float)dg[0], -149);       // below 2^24 units: exact
    // bits [top - 24, top] from the digits k .. k + 2, and whether any bit below is set
    const int low = top - 24, k = low >> 5, o = low & 31;
    uint32_t d0 = 0, d1 = 0, d2 = 0;
    bool sticky = false;
#pragma unroll
    for (int d = 0; d < XDIG; ++d) {
        d0 = (d == k) ? dg[d] : d0;
        d1 = (d == k + 1) ? dg[d] : d1;
        d2 = (d == k + 2) ? dg[d] : d2;
        sticky |= (d < k) && dg[d] != 0u;
    }
    sticky |= o != 0 && (d0 & ((1u << o) - 1u)) != 0u;
    unsigned long long win = ((unsigned long long)d1 << 32) | d0;
    if (o) win = (win >> o) | ((unsigned long long)d2 << (64 - o));
    uint32_t mant = (uint32_t)(win >> 1) & 0xffffffu;
    const bool rnd = (win & 1ull) != 0ull;
    if (rnd && (sticky || (mant & 1u))) {
        ++mant;
        if (mant == (1u << 24)) {
            mant >>= 1;
            ++top;
        }
    }
    if (top - 149 > 127) return __int_as_float(0x7f800000);
    return ldexpf((float)mant, top - 23 - 149);
}

// One thread per sorted pair; the first of a run writes the edge's endpoints and, for
// a short run, its weight (w: the weights in the keys' order), which the wave's lanes
// sum together.  Longer runs get bounds and go to lists for k_merge_long and
// k_merge_big, the first by way of LDS (a reservation per wave, on one address, was
// most of the 570 us that merging a coarse graph's 16M pairs in runs of all
// lengths took; 200 us here).  total: the edges.
constexpr int MERGE_STAGE = 1024;        // staged long runs
constexpr int MERGE_ROUNDS = 32;         // steps between flushes: at most IBLOCK / (MERGE_SHORT + 1) + 1 start in each
static_assert(MERGE_ROUNDS * (IBLOCK / ((int)MERGE_SHORT + 1) + 2) <= MERGE_STAGE, "the stage holds every round's runs");

__global__ __launch_bounds__(IBLOCK) void k_merge_runs(int64_t count, PairCode code, const unsigned long long *__restrict__ key,
                             const uint32_t *__restrict__ edge_of, const float *__restrict__ w,
                             int32_t *__restrict__ ea, int32_t *__restrict__ eb, float *__restrict__ ew,
                             uint2 *__restrict__ bounds, uint32_t *__restrict__ long_list,
                             unsigned int *__restrict__ long_count, uint32_t *__restrict__ big_list,
                             unsigned int *__restrict__ big_count, unsigned int *__restrict__ total) {
    // the loop bound is uniform per wave (blocks are whole waves), so every
    // lane reaches the wave-wide append
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t n_pad = ceil_div_dev(count, stride) * stride;
    const int lane = threadIdx.x & (WAVE - 1);
    __shared__ uint32_t stage[MERGE_STAGE];
    __shared__ unsigned int n_stage, base_s;
    if (threadIdx.x == 0) n_stage = 0u;
    __syncthreads();
    auto flush = [&] {                   // by the whole workgroup
        __syncthreads();
        const unsigned int ns = n_stage;
        if (threadIdx.x == 0 && ns) base_s = atomicAdd(long_count, ns);
        __syncthreads();
        for (unsigned int i = threadIdx.x; i < ns; i += IBLOCK) long_list[base_s + i] = stage[i];
        __syncthreads();
        if (threadIdx.x == 0) n_stage = 0u;
        __syncthreads();
    };
    int round = 0;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n_pad; q += stride) {
        bool defer = false, big = false;
        uint32_t e = 0;
        const unsigned long long k = q < count ? key[q] : code.none;
        const bool first = k != code.none && (q == 0 || key[q - 1] != k);
        if (q == count - 1) *total = edge_of[q] + (first ? 1u : 0u);
        if (first) {
            e = edge_of[q];
            ea[e] = pair_lo(code, k);
            eb[e] = pair_hi(code, k);
        }
        // the run's end: the wave's next run, or for the last run of the wave a
        // search by all its lanes (64 keys on, then 64 probes at a time)
        const int64_t base = q - lane;
        const unsigned long long starts = __ballot(q >= count || q == 0 || key[q - 1] != k);
        const unsigned long long heads = __ballot(first);
        const unsigned long long after = lane == WAVE - 1 ? 0ull : starts >> (lane + 1);
        const int stop = after ? lane + __ffsll((long long)after) : WAVE;   // first lane past this one's run
        int64_t end = base + stop;
        const int tail = heads ? 63 - __clzll((long long)heads) : -1;    // its run passes the wave's end unless `after`
        if (w && tail >= 0 && (tail == WAVE - 1 || !(starts >> (tail + 1)))) {
            const unsigned long long kt = __shfl(k, tail, WAVE);
            int64_t at = base + WAVE;                                    // key[at - 1] == kt throughout
            unsigned long long past = __ballot(at + lane >= count || key[min(at + lane, count - 1)] != kt);
            if (past) {
                at += __ffsll((long long)past) - 1;
            } else {
                at += WAVE;
                int64_t top = count;                                     // the end is at most top
                while (at < top) {
                    const int64_t step = ceil_div_dev(top - at, WAVE), p = at + lane * step;
                    past = __ballot(p >= top || key[p] != kt);
                    if (past & 1ull) break;
                    const int f = past ? __ffsll((long long)past) - 1 : WAVE;
                    top = min(top, at + f * step);
                    at += (f - 1) * step + 1;
                }
            }
            if (lane == tail) end = at;
        }
        // span and sum of every short run at its first lane: its lanes' values by
        // doubling, and the lanes past the wave's end for the last one
        float x = 0.0f;
        int lo = 1 << 20, hi = -1;
        double sum = 0.0;
        if (w) {
            uint32_t mant;
            int shift;
            if (q < count) {
                x = w[q];
                f32_split(x, mant, shift);
                lo = shift;
                hi = shift + 24;
                sum = (double)x;
            }
            static_assert(MERGE_SHORT == 16, "four doublings and 16 lanes cover a short run");
#pragma unroll
            for (int o = 1; o < (int)MERGE_SHORT; o <<= 1) {
                const int lo_o = __shfl_down(lo, o, WAVE), hi_o = __shfl_down(hi, o, WAVE);
                const double sum_o = __shfl_down(sum, o, WAVE);
                if (lane + o < stop) {
                    lo = min(lo, lo_o);
                    hi = max(hi, hi_o);
                    sum += sum_o;
                }
            }
            const int64_t tail_q = base + tail, tail_end = tail >= 0 ? __shfl(end, tail, WAVE) : 0;
            if (tail >= 0 && tail_end > base + WAVE && tail_end - tail_q <= (int64_t)MERGE_SHORT) {
                int lo2 = 1 << 20, hi2 = -1;
                double sum2 = 0.0;
                if (base + WAVE + lane < tail_end) {
                    const float y = w[base + WAVE + lane];
                    f32_split(y, mant, shift);
                    lo2 = shift;
                    hi2 = shift + 24;
                    sum2 = (double)y;
                }
#pragma unroll
                for (int o = (int)MERGE_SHORT / 2; o >= 1; o >>= 1) {
                    lo2 = min(lo2, __shfl_xor(lo2, o, WAVE));
                    hi2 = max(hi2, __shfl_xor(hi2, o, WAVE));
                    sum2 += __shfl_xor(sum2, o, WAVE);
                }
                lo2 = __shfl(lo2, 0, WAVE);
                hi2 = __shfl(hi2, 0, WAVE);
                sum2 = __shfl(sum2, 0, WAVE);
                if (lane == tail) {
                    lo = min(lo, lo2);
                    hi = max(hi, hi2);
                    sum += sum2;
                }
            }
        }
        if (first && w) {
            const uint32_t len = (uint32_t)(end - q);
            if (len == 1) {
                ew[e] = x;
            } else if (len <= MERGE_SHORT) {
                if (hi + ceil_log2_u32(len) - lo <= 53) {
                    ew[e] = (float)sum;
                } else {
                    unsigned long long acc[XDIG] = {};
                    for (int64_t r = q; r < end; ++r) digits_add(acc, w[r]);
                    ew[e] = digits_round(acc);
                }
            } else {
                bounds[e] = make_uint2((uint32_t)q, (uint32_t)end);
                defer = true;
                big = len > MERGE_WAVE;
            }
        }
        if (defer && !big) stage[atomicAdd(&n_stage, 1u)] = e;
        if (__any(big)) {
            const unsigned int bt = wave_append(big, big_count);
            if (big) big_list[bt] = e;
        }
        if (++round == MERGE_ROUNDS) {   // uniform: every thread takes as many steps
            flush();
            round = 0;
        }
    }
    flush();
}

// One wave per run of MERGE_SHORT < length <= MERGE_WAVE: every lane sums
// its share (double partial sums when the whole run spans at most 53 bits,
// digits otherwise), then the wave combines them; both are exact, so the
// order does not matter.
constexpr int MERGE_LOADS = 4;           // weights each lane loads per step

__global__ __launch_bounds__(IBLOCK) void k_merge_long(const unsigned int *__restrict__ long_count,
                                                       const uint32_t *__restrict__ long_list,
                                                       const uint2 *__restrict__ bounds,
                                                       const float *__restrict__ w, float *__restrict__ ew) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int64_t nw = (int64_t)gridDim.x * (IBLOCK / WAVE);
    const int64_t count = *long_count;
    for (int64_t q = (int64_t)blockIdx.x * (IBLOCK / WAVE) + (threadIdx.x >> 6); q < count; q += nw) {
        const uint32_t e = long_list[q];
        const uint2 b = bounds[e];
        int lo = 1 << 20, hi = -1;
        double sum = 0.0;
        for (uint32_t base = b.x; base < b.y; base += WAVE * MERGE_LOADS) {
            float x[MERGE_LOADS];
#pragma unroll
            for (int t = 0; t < MERGE_LOADS; ++t) {
                const uint32_t r = base + (uint32_t)(t * WAVE + lane);
                x[t] = r < b.y ? w[r] : 0.0f;
            }
#pragma unroll
            for (int t = 0; t < MERGE_LOADS; ++t) {
                if (x[t] == 0.0f) continue;                  // past the run's end
                uint32_t mant;
                int shift;
                f32_split(x[t], mant, shift);
                lo = min(lo, shift);
                hi = max(hi, shift + 24);
                sum += (double)x[t];
            }
        }
        for (int o = WAVE / 2; o >= 1; o >>= 1) {
            lo = min(lo, __shfl_xor(lo, o, WAVE));
            hi = max(hi, __shfl_xor(hi, o, WAVE));
            sum += __shfl_xor(sum, o, WAVE);
        }
        if (hi + ceil_log2_u32(b.y - b.x) - lo <= 53) {
            if (lane == 0) ew[e] = (float)sum;
            continue;
        }
        unsigned long long acc[XDIG] = {};
        for (uint32_t r = b.x + (uint32_t)lane; r < b.y; r += WAVE) digits_add(acc, w[r]);
#pragma unroll
        for (int d = 0; d < XDIG; ++d)
            for (int o = WAVE / 2; o >= 1; o >>= 1) acc[d] += __shfl_xor(acc[d], o, WAVE);
        if (lane == 0) ew[e] = digits_round(acc);
    }
}

// One workgroup of MERGE_TB threads per run longer than MERGE_WAVE: digits
// always (exact at any length), MERGE_LOADS weights per thread in flight.
__global__ __launch_bounds__(MERGE_TB) void k_merge_big(const unsigned int *__restrict__ big_count,
                                                        const uint32_t *__restrict__ big_list,
                                                        const uint2 *__restrict__ bounds,
                                                        const float *__restrict__ w, float *__restrict__ ew) {
    __shared__ unsigned long long part[MERGE_TB / WAVE][XDIG];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x >> 6;
    const unsigned int count = *big_count;
    for (unsigned int q = blockIdx.x; q < count; q += gridDim.x) {
        const uint32_t e = big_list[q];
        const uint2 b = bounds[e];
        unsigned long long acc[XDIG] = {};
        for (uint32_t base = b.x; base < b.y; base += MERGE_TB * MERGE_LOADS) {
            float x[MERGE_LOADS];
#pragma unroll
            for (int t = 0; t < MERGE_LOADS; ++t) {
                const uint32_t r = base + (uint32_t)(t * MERGE_TB) + threadIdx.x;
                x[t] = r < b.y ? w[r] : 0.0f;
            }
#pragma unroll
            for (int t = 0; t < MERGE_LOADS; ++t) digits_add(acc, x[t]);     // a zero adds nothing
        }
#pragma unroll
        for (int d = 0; d < XDIG; ++d) {
            for (int o = WAVE / 2; o >= 1; o >>= 1) acc[d] += __shfl_xor(acc[d], o, WAVE);
            if (lane == 0) part[wv][d] = acc[d];
        }
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int d = 0; d < XDIG; ++d) {
                unsigned long long t = 0;
                for (int k = 0; k < MERGE_TB / WAVE; ++k) t += part[k][d];
                acc[d] = t;
            }
            ew[e] = digits_round(acc);
        }
        __syncthreads();
    }
}

// Run ends of a sorted key array: start[k] = first position, cnt[k] = end
// (both zero beforehand); k_count_finish turns them into counts.
__global__ void k_count_marks(int64_t m, const int32_t *__restrict__ keys, uint32_t *__restrict__ start,
                              uint32_t *__restrict__ cnt) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m; t += (int64_t)gridDim.x * blockDim.x) {
        const int32_t k = keys[t];
        if (t == 0 || keys[t - 1] != k) start[k] = (uint32_t)t;
        if (t + 1 == m || keys[t + 1] != k) cnt[k] = (uint32_t)(t + 1);
    }
}

// cnt[i] -= start[i]; deg[i] = cnt[i] + other[i] when deg is given.
__global__ void k_count_finish(int64_t n, const uint32_t *__restrict__ start, uint32_t *__restrict__ cnt,
                               const uint32_t *__restrict__ other, uint32_t *__restrict__ deg) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t c = cnt[i] - start[i];
        cnt[i] = c;
        if (deg) deg[i] = c + other[i];
    }
}

__global__ void k_degree_max(int64_t n, const uint32_t *__restrict__ deg, unsigned int *__restrict__ dmax) {
    unsigned int mx = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        mx = max(mx, deg[i]);
    for (int o = WAVE / 2; o >= 1; o >>= 1) mx = max(mx, (unsigned int)__shfl_xor((int)mx, o, WAVE));
    if ((threadIdx.x & (WAVE - 1)) == 0) atomicMax(dmax, mx);
}

// Storage-order key of vertex i: decreasing degree; the stable sort keeps equal
// ones by increasing listed id.  top: the largest key.
__global__ void k_vertex_keys(int64_t n, const uint32_t *__restrict__ deg, uint32_t top,
                              uint32_t *__restrict__ vkey) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        vkey[i] = top - deg[i];
}

__global__ void k_new_ids(int64_t n, const uint32_t *__restrict__ vid_sorted, uint32_t *__restrict__ new_of,
                          const int32_t *__restrict__ orig_in, int32_t *__restrict__ orig_out) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t i = vid_sorted[r];
        new_of[i] = (uint32_t)r;
        orig_out[r] = orig_in ? orig_in[i] : (int32_t)i;
    }
}

__global__ void k_orig_identity(int64_t n, const int32_t *__restrict__ orig_in, int32_t *__restrict__ orig_out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        orig_out[i] = orig_in ? orig_in[i] : (int32_t)i;
}

// Edge keys under the new labels (no repeats remain).
__global__ void k_relabel_keys(int64_t m, PairCode code, const int32_t *__restrict__ ea,
                               const int32_t *__restrict__ eb, const uint32_t *__restrict__ new_of,
                               unsigned long long *__restrict__ key) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t x = new_of[ea[e]], y = new_of[eb[e]];
        key[e] = pair_key(code, x < y ? x : y, x < y ? y : x);
    }
}

__global__ void k_unpack_edges(int64_t m, PairCode code, const unsigned long long *__restrict__ key,
                               int32_t *__restrict__ ea, int32_t *__restrict__ eb) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        ea[e] = pair_lo(code, key[e]);
        eb[e] = pair_hi(code, key[e]);
    }
}

// Upper entry of edge e = (a, b): after row a's lower entries, at e's place
// among the edges that start at a (edge ids are in (a, b) order).
__global__ void k_place_upper(int64_t m, const int32_t *__restrict__ ea, const int32_t *__restrict__ eb,
                              const float *__restrict__ ew, const int64_t *__restrict__ row_ptr,
                              const uint32_t *__restrict__ lower_cnt, const uint64_t *__restrict__ upper_start,
                              int32_t *__restrict__ col, float *__restrict__ w_out, int32_t *__restrict__ eid) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += (int64_t)gridDim.x * blockDim.x) {
        const int32_t a = ea[e];
        const int64_t pos = row_ptr[a] + lower_cnt[a] + (e - (int64_t)upper_start[a]);
        col[pos] = eb[e];
        eid[pos] = (int32_t)e;
        if (w_out) w_out[pos] = ew[e];
    }
}

// Lower entry of edge e = (a, b), from the edges sorted by b (stably, so by a
// within each b): at its place among the edges that end at b.
__global__ void k_place_lower(int64_t m, const uint32_t *__restrict__ b_sorted, const uint32_t *__restrict__ e_sorted,
                              const int32_t *__restrict__ ea, const float *__restrict__ ew,
                              const int64_t *__restrict__ row_ptr, const uint64_t *__restrict__ lower_start,
                              int32_t *__restrict__ col, float *__restrict__ w_out, int32_t *__restrict__ eid) {
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m; t += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t b = b_sorted[t], e = e_sorted[t];
        const int64_t pos = row_ptr[b] + (t - (int64_t)lower_start[b]);
        col[pos] = ea[e];
        eid[pos] = (int32_t)e;
        if (w_out) w_out[pos] = ew[e];
    }
}

// Zeroes four arrays of n.
__global__ void k_zero_counts(int64_t n, uint32_t *__restrict__ a, uint32_t *__restrict__ b, uint32_t *__restrict__ c,
                              uint32_t *__restrict__ d) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = b[i] = c[i] = d[i] = 0u;
}

// ------------------------------------------------ reverse Cuthill-McKee --
// The order of the oracle's reading, built level by level: a breadth-first
// search visits a level in queue order, and each vertex of the next level
// is queued by its first-visited neighbour in the level, its siblings in
// increasing (degree, id) order, so the next level is the set of unplaced
// neighbours ordered by (smallest place among their placed neighbours,
// degree, id).  Every component is searched at once, each in its own range
// of places (components in increasing order of their smallest id, each
// starting at its vertex of least (degree, id)).
constexpr uint32_t RC_UNSET = 0xffffffffu;

// Sizes and starts of the components.  A workgroup takes a contiguous range of vertices
// and gathers the share of its first vertex's component, mostly the giant one, in
// LDS: two atomics on one address for every vertex took 11.9 ms at n = 2^20 (16M pairs
// into this order 25.9 ms; 10.4 so).
constexpr unsigned RC_BLOCKS = 512;

__global__ __launch_bounds__(IBLOCK) void k_rc_init(int64_t n, const int64_t *__restrict__ row_ptr,
                                                    const int32_t *__restrict__ root, uint32_t *__restrict__ size,
                                                    unsigned long long *__restrict__ start,
                                                    uint32_t *__restrict__ pos, uint32_t *__restrict__ par) {
    __shared__ uint32_t cnt[IBLOCK / WAVE];
    __shared__ unsigned long long low[IBLOCK / WAVE];
    const int64_t per = ceil_div_dev(n, (int64_t)gridDim.x);
    const int64_t i0 = (int64_t)blockIdx.x * per, i1 = min(n, i0 + per);
    if (i0 >= i1) return;                                            // uniform over the workgroup
    const int32_t own = root[i0];
    uint32_t c = 0;
    unsigned long long mn = ~0ull;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += IBLOCK) {
        const int32_t r = root[i];
        const unsigned long long d = (unsigned long long)(row_ptr[i + 1] - row_ptr[i]);
        const unsigned long long code = (d << 32) | (unsigned long long)i;
        if (r == own) {
            ++c;
            mn = min(mn, code);
        } else {
            atomicAdd(&size[r], 1u);
            atomicMin(&start[r], code);
        }
        pos[i] = RC_UNSET;
        par[i] = RC_UNSET;
    }
    for (int o = WAVE / 2; o >= 1; o >>= 1) {
        c += __shfl_xor(c, o, WAVE);
        mn = min(mn, (unsigned long long)__shfl_xor(mn, o, WAVE));
    }
    if ((threadIdx.x & (WAVE - 1)) == 0) {
        cnt[threadIdx.x / WAVE] = c;
        low[threadIdx.x / WAVE] = mn;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < IBLOCK / WAVE; ++w) {
            c += cnt[w];
            mn = min(mn, low[w]);
        }
        atomicAdd(&size[own], c);
        atomicMin(&start[own], mn);
    }
}

// Each component's start takes the component's first place and joins the
// first frontier.
__global__ void k_rc_seed(int64_t n, const uint32_t *__restrict__ size, const uint32_t *__restrict__ off,
                          const unsigned long long *__restrict__ start, uint32_t *__restrict__ pos,
                          uint32_t *__restrict__ fill, uint32_t *__restrict__ front, unsigned int *__restrict__ cnt) {
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (int64_t)gridDim.x * blockDim.x) {
        if (size[r] == 0) continue;
        const uint32_t v = (uint32_t)(start[r] & 0xffffffffull);
        pos[v] = off[r];
        fill[r] = off[r] + 1u;
        front[atomicAdd(&cnt[0], 1u)] = v;
    }
}

// One wave per frontier vertex: every unplaced neighbour keeps the smallest
// place among its frontier neighbours; the first to reach it lists it.
__global__ void k_rc_expand(unsigned int nf, const uint32_t *__restrict__ front, const int64_t *__restrict__ row_ptr,
                            const int32_t *__restrict__ col, const uint32_t *__restrict__ pos,
                            uint32_t *__restrict__ par, uint32_t *__restrict__ cand, unsigned int *__restrict__ ncand) {
    const int lane = threadIdx.x & (WAVE - 1);
    const unsigned int nw = gridDim.x * (IBLOCK / WAVE);
    for (unsigned int f = blockIdx.x * (IBLOCK / WAVE) + (threadIdx.x >> 6); f < nf; f += nw) {
        const uint32_t v = front[f];
        const uint32_t pv = pos[v];
        const int64_t b1 = row_ptr[v + 1];
        for (int64_t p = row_ptr[v] + lane; p < b1; p += WAVE) {
            const int32_t u = col[p];
            if (pos[u] != RC_UNSET) continue;
            if (atomicMin(&par[u], pv) == RC_UNSET) cand[atomicAdd(ncand, 1u)] = (uint32_t)u;
        }
    }
}

// Sort key of a candidate: (smallest neighbour place, degree); its id breaks
// ties through the stable sort of candidates already in id order.
__global__ void k_rc_keys(unsigned int nc, const uint32_t *__restrict__ cand, const uint32_t *__restrict__ par,
                          const int64_t *__restrict__ row_ptr, unsigned long long *__restrict__ key) {
    for (unsigned int i = blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += gridDim.x * blockDim.x) {
        const uint32_t u = cand[i];
        key[i] = ((unsigned long long)par[u] << 32) | (unsigned long long)(row_ptr[u + 1] - row_ptr[u]);
    }
}

// A component's candidates are contiguous in the sorted level (their
// parents' places lie in the component's range): first index of each run,
// the places, then the component's next free place.
__global__ void k_rc_first(unsigned int nc, const uint32_t *__restrict__ vert, const int32_t *__restrict__ root,
                           uint32_t *__restrict__ first) {
    for (unsigned int i = blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += gridDim.x * blockDim.x) {
        const int32_t r = root[vert[i]];
        if (i == 0 || root[vert[i - 1]] != r) first[r] = i;
    }
}

__global__ void k_rc_place(unsigned int nc, const uint32_t *__restrict__ vert, const int32_t *__restrict__ root,
                           const uint32_t *__restrict__ first, const uint32_t *__restrict__ fill,
                           uint32_t *__restrict__ pos) {
    for (unsigned int i = blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += gridDim.x * blockDim.x) {
        const uint32_t u = vert[i];
        const int32_t r = root[u];
        pos[u] = fill[r] + (i - first[r]);
    }
}

__global__ void k_rc_advance(unsigned int nc, const uint32_t *__restrict__ vert, const int32_t *__restrict__ root,
                             const uint32_t *__restrict__ first, uint32_t *__restrict__ fill) {
    for (unsigned int i = blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += gridDim.x * blockDim.x) {
        const int32_t r = root[vert[i]];
        if (i + 1 == nc || root[vert[i + 1]] != r) fill[r] += i - first[r] + 1u;
    }
}

// Reversed: the vertex at Cuthill-McKee place q is stored as n - 1 - q.
__global__ void k_rc_order(int64_t n, const uint32_t *__restrict__ pos, uint32_t *__restrict__ vid_sorted) {
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t)gridDim.x * blockDim.x)
        vid_sorted[n - 1 - (int64_t)pos[v]] = (uint32_t)v;
}

constexpr int INGEST_FLAGS = 5;

struct IngestLayout {
    unsigned long long *key0, *key1;     // [m_in] pair keys (sort double buffer)
    uint32_t *list;                      // [m_in] long runs
    uint32_t *b_sorted;                  // [m_in] larger endpoints, sorted
    uint32_t *edge_of;                   // [m_in] edge of a sorted pair; edges by larger endpoint
    float *w_sorted;                     // [m_in] weights in the order of the sorted pairs
    int32_t *ea, *eb;                    // [m_in] edges (a < b)
    float *ew, *ew2;                     // [m_in]
    uint32_t *deg, *lower_cnt, *upper_cnt, *new_of;   // [n]
    uint64_t *lower_start, *upper_start; // [n]
    uint32_t *vkey0, *vkey1;             // [n]
    uint32_t *vid0, *vid1;               // [n]
    unsigned int *flags;                 // [INGEST_FLAGS]: error bits, d_max, runs for a workgroup, runs for a wave, edges
    // reverse Cuthill-McKee order ([n] each)
    int32_t *rc_root;                    // component of every vertex (its smallest id)
    uint32_t *rc_pos;                    // place in the Cuthill-McKee order (RC_UNSET before)
    uint32_t *rc_par;                    // smallest place among a candidate's placed neighbours
    uint32_t *rc_size, *rc_off, *rc_fill, *rc_first;  // per component root: size, first place, next place,
                                                      // first index in the sorted candidates
    unsigned long long *rc_start;        // per component root: (degree << 32 | id) of its start
    uint32_t *rc_front, *rc_cand, *rc_cand2, *rc_vert;
    unsigned long long *rc_key0, *rc_key1;
    unsigned int *rc_cnt;                // [2]: frontier size, candidates
    void *temp;                          // rocPRIM temporary storage
    size_t temp_bytes;
};

// Largest temporary storage any of the pipeline's rocPRIM calls asks for (0
// when a query fails; the launch then reports the error).
static size_t rocprim_temp_bytes(int64_t m_in, int64_t n) {
    size_t need = 0, t = 0;
    hipError_t e = hipSuccess;
    const size_t mm = (size_t)std::max<int64_t>(1, m_in), nn = (size_t)std::max<int64_t>(1, n);
    const rocprim::counting_iterator<uint32_t> ids(0);
    e = rocprim::radix_sort_pairs(nullptr, t, (unsigned long long *)nullptr, (unsigned long long *)nullptr,
                                  (const float *)nullptr, (float *)nullptr, mm, 0, 64);
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::radix_sort_keys(nullptr, t, (unsigned long long *)nullptr, (unsigned long long *)nullptr, mm, 0, 64);
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::radix_sort_pairs(nullptr, t, (unsigned long long *)nullptr, (unsigned long long *)nullptr,
                                  (uint32_t *)nullptr, (uint32_t *)nullptr, nn, 0, 64);
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::radix_sort_pairs(nullptr, t, (const uint32_t *)nullptr, (uint32_t *)nullptr, ids, (uint32_t *)nullptr,
                                  mm, 0, 32);
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::radix_sort_keys(nullptr, t, (const uint32_t *)nullptr, (uint32_t *)nullptr, mm, 0, 32);
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::radix_sort_pairs(nullptr, t, (const uint32_t *)nullptr, (uint32_t *)nullptr, ids, (uint32_t *)nullptr,
                                  nn, 0, 32);
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::exclusive_scan(nullptr, t, run_heads(nullptr, 0), (uint32_t *)nullptr, 0u, mm,
                                rocprim::plus<uint32_t>());
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::exclusive_scan(nullptr, t, counts_of(nullptr, 0), (uint64_t *)nullptr, (uint64_t)0, nn + 1,
                                rocprim::plus<uint64_t>());
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::exclusive_scan(nullptr, t, (uint32_t *)nullptr, (uint32_t *)nullptr, 0u, nn,
                                rocprim::plus<uint32_t>());
    need = std::max(need, e == hipSuccess ? t : 0);
    e = rocprim::radix_sort_keys(nullptr, t, (uint32_t *)nullptr, (uint32_t *)nullptr, nn, 0, 32);
    need = std::max(need, e == hipSuccess ? t : 0);
    return need;
}

static size_t ingest_layout(int64_t n, int64_t m_in, void *ws, size_t ws_bytes, IngestLayout *L) {
    Carver c(ws, ws_bytes);
    const size_t mm = (size_t)std::max<int64_t>(1, m_in), nn = (size_t)std::max<int64_t>(1, n) + 1;
    IngestLayout l;
    l.key0 = c.take<unsigned long long>(mm);
    l.key1 = c.take<unsigned long long>(mm);
    l.list = c.take<uint32_t>(mm);
    l.b_sorted = c.take<uint32_t>(mm);
    l.edge_of = c.take<uint32_t>(mm);
    l.w_sorted = c.take<float>(mm);
    l.ea = c.take<int32_t>(mm);
    l.eb = c.take<int32_t>(mm);
    l.ew = c.take<float>(mm);
    l.ew2 = c.take<float>(mm);
    l.deg = c.take<uint32_t>(nn);
    l.lower_cnt = c.take<uint32_t>(nn);
    l.upper_cnt = c.take<uint32_t>(nn);
    l.new_of = c.take<uint32_t>(nn);
    l.lower_start = c.take<uint64_t>(nn);
    l.upper_start = c.take<uint64_t>(nn);
    l.vkey0 = c.take<uint32_t>(nn);
    l.vkey1 = c.take<uint32_t>(nn);
    l.vid0 = c.take<uint32_t>(nn);
    l.vid1 = c.take<uint32_t>(nn);
    l.flags = c.take<unsigned int>(INGEST_FLAGS);
    l.rc_root = c.take<int32_t>(nn);
    l.rc_pos = c.take<uint32_t>(nn);
    l.rc_par = c.take<uint32_t>(nn);
    l.rc_size = c.take<uint32_t>(nn);
    l.rc_off = c.take<uint32_t>(nn);
    l.rc_fill = c.take<uint32_t>(nn);
    l.rc_first = c.take<uint32_t>(nn);
    l.rc_start = c.take<unsigned long long>(nn);
    l.rc_front = c.take<uint32_t>(nn);
    l.rc_cand = c.take<uint32_t>(nn);
    l.rc_cand2 = c.take<uint32_t>(nn);
    l.rc_vert = c.take<uint32_t>(nn);
    l.rc_key0 = c.take<unsigned long long>(nn);
    l.rc_key1 = c.take<unsigned long long>(nn);
    l.rc_cnt = c.take<unsigned int>(2);
    l.temp_bytes = rocprim_temp_bytes(m_in, n);
    l.temp = c.take<char>(l.temp_bytes);
    if (L) *L = l;
    return c.ok() ? c.used : 0;
}

static unsigned igrid(int64_t count) { return grid_for(std::max<int64_t>(1, count), IBLOCK); }

#define AD_RP(call)                                                         \
    do {                                                                    \
        hipError_t e_ = (call);                                             \
        if (e_ != hipSuccess) return fail(AD_ERR_HIP, std::string("rocPRIM: ") + hipGetErrorString(e_)); \
    } while (0)

// Degrees of the m edges (ea < eb, sorted by (ea, eb)) without atomics:
// upper_cnt from the runs of ea, lower_cnt from the runs of the sorted eb
// (left in b_sorted; with_edges: the edge ids, stably sorted by eb, in edge_of for
// the lower placement), deg = upper + lower.  deg, upper_cnt, lower_cnt: [n];
// vid0 / vid1 serve as scratch.
static ad_status edge_counts(int64_t n, int64_t m, const int32_t *ea, const int32_t *eb, bool with_edges,
                             const IngestLayout &L, hipStream_t st) {
    hipLaunchKernelGGL(k_zero_counts, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.upper_cnt, L.lower_cnt, L.vid0, L.vid1);
    AD_LAUNCH_CHECK("k_zero_counts");
    hipLaunchKernelGGL(k_count_marks, dim3(igrid(m)), dim3(IBLOCK), 0, st, m, ea, L.vid0, L.upper_cnt);
    AD_LAUNCH_CHECK("k_count_marks");
    size_t tb = L.temp_bytes;
    const uint32_t *b = (const uint32_t *)eb;
    if (with_edges)
        AD_RP(rocprim::radix_sort_pairs(L.temp, tb, b, L.b_sorted, rocprim::counting_iterator<uint32_t>(0), L.edge_of,
                                        (size_t)m, 0, bits_for(n), st));
    else
        AD_RP(rocprim::radix_sort_keys(L.temp, tb, b, L.b_sorted, (size_t)m, 0, bits_for(n), st));
    hipLaunchKernelGGL(k_count_marks, dim3(igrid(m)), dim3(IBLOCK), 0, st, m, (const int32_t *)L.b_sorted, L.vid1,
                       L.lower_cnt);
    AD_LAUNCH_CHECK("k_count_marks");
    hipLaunchKernelGGL(k_count_finish, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.vid0, L.upper_cnt,
                       (const uint32_t *)nullptr, (uint32_t *)nullptr);
    AD_LAUNCH_CHECK("k_count_finish");
    hipLaunchKernelGGL(k_count_finish, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.vid1, L.lower_cnt, L.upper_cnt,
                       L.deg);
    AD_LAUNCH_CHECK("k_count_finish");
    return AD_OK;
}

// The edges (ea < eb, sorted by (ea, eb); weights ew or NULL) as the
// symmetric CSR: per-row counts (upper_cnt: edges whose smaller endpoint is
// the row, lower_cnt: larger), the edges sorted by larger endpoint
// (b_sorted / edge_of), the degrees and their maximum (flags[1]), row_ptr, then
// the upper entries in edge order and the lower ones.  w_out NULL: no weights.
static ad_status place_csr(int64_t n, int64_t m, const int32_t *ea, const int32_t *eb, const float *ew,
                           int64_t *row_ptr, int32_t *col, float *w_out, int32_t *eid, const IngestLayout &L,
                           hipStream_t st) {
    ad_status s;
    if (n > 0) {
        if (m > 0) {
            s = edge_counts(n, m, ea, eb, true, L, st);
            if (s != AD_OK) return s;
        } else {
            hipLaunchKernelGGL(k_zero_counts, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.upper_cnt, L.lower_cnt, L.deg,
                               L.vid0);
            AD_LAUNCH_CHECK("k_zero_counts");
        }
        hipLaunchKernelGGL(k_degree_max, dim3(std::min<unsigned>(256, igrid(n))), dim3(IBLOCK), 0, st, n, L.deg,
                           L.flags + 1);
        AD_LAUNCH_CHECK("k_degree_max");
    }
    // row_ptr = exclusive scan of the degrees over n + 1 entries (the last one 0)
    size_t tb = L.temp_bytes;
    AD_RP(rocprim::exclusive_scan(L.temp, tb, counts_of(L.deg, n), (uint64_t *)row_ptr, (uint64_t)0, (size_t)n + 1,
                                  rocprim::plus<uint64_t>(), st));
    if (m > 0) {
        tb = L.temp_bytes;
        AD_RP(rocprim::exclusive_scan(L.temp, tb, counts_of(L.upper_cnt, n), L.upper_start, (uint64_t)0, (size_t)n,
                                      rocprim::plus<uint64_t>(), st));
        tb = L.temp_bytes;
        AD_RP(rocprim::exclusive_scan(L.temp, tb, counts_of(L.lower_cnt, n), L.lower_start, (uint64_t)0, (size_t)n,
                                      rocprim::plus<uint64_t>(), st));
        hipLaunchKernelGGL(k_place_upper, dim3(igrid(m)), dim3(IBLOCK), 0, st, m, ea, eb, ew, row_ptr, L.lower_cnt,
                           L.upper_start, col, w_out, eid);
        AD_LAUNCH_CHECK("k_place_upper");
        // lower entries from the edges sorted (stably) by their larger endpoint
        hipLaunchKernelGGL(k_place_lower, dim3(igrid(m)), dim3(IBLOCK), 0, st, m, L.b_sorted, L.edge_of, ea, ew, row_ptr,
                           L.lower_start, col, w_out, eid);
        AD_LAUNCH_CHECK("k_place_lower");
    }
    return AD_OK;
}

// Relabel the edges by new_of and number them again in (smaller, larger)
// order: ea, eb rewritten, the weights (when given) permuted into ew2.
static ad_status relabel_edges(int64_t n, int64_t m, const int32_t *ea, const int32_t *eb, const float *ew,
                               const IngestLayout &L, hipStream_t st) {
    if (m <= 0) return AD_OK;
    const PairCode code(n);
    hipLaunchKernelGGL(k_relabel_keys, dim3(igrid(m)), dim3(IBLOCK), 0, st, m, code, ea, eb, L.new_of, L.key0);
    AD_LAUNCH_CHECK("k_relabel_keys");
    size_t tb = L.temp_bytes;
    if (ew)
        AD_RP(rocprim::radix_sort_pairs(L.temp, tb, L.key0, L.key1, ew, L.ew2, (size_t)m, 0, 2 * code.b, st));
    else
        AD_RP(rocprim::radix_sort_keys(L.temp, tb, L.key0, L.key1, (size_t)m, 0, 2 * code.b, st));
    hipLaunchKernelGGL(k_unpack_edges, dim3(igrid(m)), dim3(IBLOCK), 0, st, m, code, L.key1, L.ea, L.eb);
    AD_LAUNCH_CHECK("k_unpack_edges");
    return AD_OK;
}

// Reverse Cuthill-McKee order of the CSR (n vertices, m edges): vid_sorted[r]
// is the vertex stored at r.  One host read-back per level of the search.
static ad_status rcm_order(int64_t n, int64_t m, const int64_t *row_ptr, const int32_t *col, const int32_t *eid,
                           const IngestLayout &L, uint32_t *vid_sorted, hipStream_t st) {
    ad_graph g{};
    g.n = n;
    g.m = m;
    g.row_ptr = row_ptr;
    g.col = m > 0 ? col : nullptr;
    g.eid = m > 0 ? eid : nullptr;
    ad_status s = label_components(&g, L.rc_root, st);
    if (s != AD_OK) return s;
    s = fill_i32((int32_t *)L.rc_size, 0, n, st);
    if (s != AD_OK) return s;
    s = fill_u64(L.rc_start, ~0ull, n, st);
    if (s != AD_OK) return s;
    s = fill_i32((int32_t *)L.rc_cnt, 0, 2, st);
    if (s != AD_OK) return s;
    hipLaunchKernelGGL(k_rc_init, dim3(std::min<unsigned>(RC_BLOCKS, igrid(n))), dim3(IBLOCK), 0, st, n, row_ptr, L.rc_root, L.rc_size, L.rc_start,
                       L.rc_pos, L.rc_par);
    AD_LAUNCH_CHECK("k_rc_init");
    size_t tb = L.temp_bytes;
    AD_RP(rocprim::exclusive_scan(L.temp, tb, L.rc_size, L.rc_off, 0u, (size_t)n, rocprim::plus<uint32_t>(), st));
    hipLaunchKernelGGL(k_rc_seed, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.rc_size, L.rc_off, L.rc_start, L.rc_pos,
                       L.rc_fill, L.rc_front, L.rc_cnt);
    AD_LAUNCH_CHECK("k_rc_seed");
    unsigned int nf = 0;
    AD_HIP(hipMemcpyAsync(&nf, L.rc_cnt, sizeof(nf), hipMemcpyDeviceToHost, st));
    AD_HIP(hipStreamSynchronize(st));
    uint32_t *front = L.rc_front, *next = L.rc_vert;
    const unsigned wgrid = (unsigned)std::max<int64_t>(1, std::min<int64_t>(4096, ceil_div(n, IBLOCK / WAVE)));
    int64_t placed = nf;
    while (nf > 0 && placed < n) {
        s = fill_i32((int32_t *)L.rc_cnt + 1, 0, 1, st);
        if (s != AD_OK) return s;
        hipLaunchKernelGGL(k_rc_expand, dim3(wgrid), dim3(IBLOCK), 0, st, nf, front, row_ptr, col, L.rc_pos, L.rc_par,
                           L.rc_cand, L.rc_cnt + 1);
        AD_LAUNCH_CHECK("k_rc_expand");
        unsigned int nc = 0;
        AD_HIP(hipMemcpyAsync(&nc, L.rc_cnt + 1, sizeof(nc), hipMemcpyDeviceToHost, st));
        AD_HIP(hipStreamSynchronize(st));
        if (nc == 0) break;
        if ((int64_t)nc > n - placed) return fail(AD_ERR_INTERNAL, "search listed a vertex twice");
        // candidates by id, then stably by (parent place, degree)
        tb = L.temp_bytes;
        AD_RP(rocprim::radix_sort_keys(L.temp, tb, L.rc_cand, L.rc_cand2, (size_t)nc, 0, bits_for(n), st));
        hipLaunchKernelGGL(k_rc_keys, dim3(igrid(nc)), dim3(IBLOCK), 0, st, nc, L.rc_cand2, L.rc_par, row_ptr,
                           L.rc_key0);
        AD_LAUNCH_CHECK("k_rc_keys");
        tb = L.temp_bytes;
        AD_RP(rocprim::radix_sort_pairs(L.temp, tb, L.rc_key0, L.rc_key1, L.rc_cand2, next, (size_t)nc, 0, 64, st));
        hipLaunchKernelGGL(k_rc_first, dim3(igrid(nc)), dim3(IBLOCK), 0, st, nc, next, L.rc_root, L.rc_first);
        AD_LAUNCH_CHECK("k_rc_first");
        hipLaunchKernelGGL(k_rc_place, dim3(igrid(nc)), dim3(IBLOCK), 0, st, nc, next, L.rc_root, L.rc_first,
                           L.rc_fill, L.rc_pos);
        AD_LAUNCH_CHECK("k_rc_place");
        hipLaunchKernelGGL(k_rc_advance, dim3(igrid(nc)), dim3(IBLOCK), 0, st, nc, next, L.rc_root, L.rc_first,
                           L.rc_fill);
        AD_LAUNCH_CHECK("k_rc_advance");
        std::swap(front, next);
        nf = nc;
        placed += nc;
    }
    if (placed != n) return fail(AD_ERR_INTERNAL, "search did not place every vertex");
    hipLaunchKernelGGL(k_rc_order, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.rc_pos, vid_sorted);
    AD_LAUNCH_CHECK("k_rc_order");
    return AD_OK;
}

static ad_status ingest_impl(int64_t n, int64_t m_in, const int32_t *u, const int32_t *v, const float *w,
                             const int32_t *orig_in, int32_t order, int64_t *row_ptr, int32_t *col, float *w_out,
                             int32_t *eid, int32_t *orig_out, int64_t *m_host, int32_t *d_max_host,
                             int64_t *n_dropped_host, const IngestLayout &L, hipStream_t st) {
    TraceScope trace("k_ingest", st);
    ad_status s = fill_i32((int32_t *)L.flags, 0, INGEST_FLAGS, st);
    if (s != AD_OK) return s;
    int64_t m = 0;
    if (m_in > 0) {
        const PairCode code(n);
        hipLaunchKernelGGL(k_pair_keys, dim3(igrid(m_in)), dim3(IBLOCK), 0, st, m_in, n, code, u, v, w, L.key0,
                           L.flags);
        AD_LAUNCH_CHECK("k_pair_keys");
        size_t tb = L.temp_bytes;
        if (w)
            AD_RP(rocprim::radix_sort_pairs(L.temp, tb, L.key0, L.key1, w, L.w_sorted, (size_t)m_in, 0, 2 * code.b, st));
        else
            AD_RP(rocprim::radix_sort_keys(L.temp, tb, L.key0, L.key1, (size_t)m_in, 0, 2 * code.b, st));
        tb = L.temp_bytes;
        AD_RP(rocprim::exclusive_scan(L.temp, tb, run_heads(L.key1, code.none), L.edge_of, 0u, (size_t)m_in,
                                      rocprim::plus<uint32_t>(), st));
        // long runs' bounds in key0 and the list of a workgroup's runs in ew2 (both free here)
        uint2 *bounds = reinterpret_cast<uint2 *>(L.key0);
        uint32_t *big_list = reinterpret_cast<uint32_t *>(L.ew2);
        const float *ws = w ? L.w_sorted : nullptr;
        hipLaunchKernelGGL(k_merge_runs, dim3(std::min<unsigned>(2048, igrid(m_in))), dim3(IBLOCK), 0, st, m_in, code, L.key1, L.edge_of, ws,
                           L.ea, L.eb, L.ew, bounds, L.list, L.flags + 3, big_list, L.flags + 2, L.flags + 4);
        AD_LAUNCH_CHECK("k_merge_runs");
        if (w) {
            hipLaunchKernelGGL(k_merge_long, dim3(1024), dim3(IBLOCK), 0, st, L.flags + 3, L.list, bounds, ws, L.ew);
            AD_LAUNCH_CHECK("k_merge_long");
            hipLaunchKernelGGL(k_merge_big, dim3(1024), dim3(MERGE_TB), 0, st, L.flags + 2, big_list, bounds, ws, L.ew);
            AD_LAUNCH_CHECK("k_merge_big");
        }
        unsigned int hflags[INGEST_FLAGS];
        AD_HIP(hipMemcpyAsync(hflags, L.flags, sizeof(hflags), hipMemcpyDeviceToHost, st));
        AD_HIP(hipStreamSynchronize(st));
        if (hflags[0] & 1u) return fail(AD_ERR_GRAPH, "edge list names a vertex outside [0, n)");
        if (hflags[0] & 2u) return fail(AD_ERR_GRAPH, "a listed weight is not finite and positive");
        m = (int64_t)hflags[4];
    }
    const int32_t *ea = L.ea, *eb = L.eb;
    const float *ew = L.ew;
    if (order == 1 && n > 0) {
        s = fill_i32((int32_t *)L.deg, 0, n, st);
        if (s != AD_OK) return s;
        if (m > 0) {
            // degrees before relabelling: run lengths of the sorted smaller and larger endpoints
            s = edge_counts(n, m, ea, eb, false, L, st);
            if (s != AD_OK) return s;
        }
        // degrees are below n, so the keys fill bits_for(n) bits
        const unsigned b = bits_for(n);
        hipLaunchKernelGGL(k_vertex_keys, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.deg, (uint32_t)((1ull << b) - 1),
                           L.vkey0);
        AD_LAUNCH_CHECK("k_vertex_keys");
        size_t tb = L.temp_bytes;
        AD_RP(rocprim::radix_sort_pairs(L.temp, tb, (const uint32_t *)L.vkey0, L.vkey1,
                                        rocprim::counting_iterator<uint32_t>(0), L.vid1, (size_t)n, 0, b, st));
        hipLaunchKernelGGL(k_new_ids, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.vid1, L.new_of, orig_in, orig_out);
        AD_LAUNCH_CHECK("k_new_ids");
        s = relabel_edges(n, m, ea, eb, w ? ew : nullptr, L, st);
        if (s != AD_OK) return s;
        if (m > 0) ew = L.ew2;
    } else if (order == 2 && n > 0) {
        // the graph under the listed ids (in the outputs, rewritten below) for the search
        s = place_csr(n, m, ea, eb, nullptr, row_ptr, col, nullptr, eid, L, st);
        if (s != AD_OK) return s;
        s = rcm_order(n, m, row_ptr, col, eid, L, L.vid1, st);
        if (s != AD_OK) return s;
        hipLaunchKernelGGL(k_new_ids, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, L.vid1, L.new_of, orig_in, orig_out);
        AD_LAUNCH_CHECK("k_new_ids");
        s = relabel_edges(n, m, ea, eb, w ? ew : nullptr, L, st);
        if (s != AD_OK) return s;
        if (m > 0) ew = L.ew2;
    } else if (n > 0) {
        hipLaunchKernelGGL(k_orig_identity, dim3(igrid(n)), dim3(IBLOCK), 0, st, n, orig_in, orig_out);
        AD_LAUNCH_CHECK("k_orig_identity");
    }
    s = place_csr(n, m, ea, eb, w ? ew : nullptr, row_ptr, col, w ? w_out : nullptr, eid, L, st);
    if (s != AD_OK) return s;
    unsigned int dmax = 0;
    if (n > 0) AD_HIP(hipMemcpyAsync(&dmax, L.flags + 1, sizeof(unsigned int), hipMemcpyDeviceToHost, st));
    AD_HIP(hipStreamSynchronize(st));
    *m_host = m;
    if (d_max_host) *d_max_host = (int32_t)dmax;
    if (n_dropped_host) *n_dropped_host = m_in - m;
    return AD_OK;
}

}  // namespace ad

using namespace ad;

extern "C" size_t ad_ingest_workspace_size(int64_t n, int64_t m_in) {
    if (n < 0 || m_in < 0 || n >= ((int64_t)1 << 31) || m_in >= ((int64_t)1 << 31)) return 0;
    return ingest_layout(n, m_in, nullptr, 0, nullptr);
}

extern "C" ad_status ad_ingest(int64_t n, int64_t m_in, const int32_t *u, const int32_t *v, const float *w,
                               const int32_t *orig_id, int32_t order, int64_t *row_ptr, int32_t *col, float *w_out,
                               int32_t *eid, int32_t *orig_id_out, int64_t *m_host, int32_t *d_max_host,
                               int64_t *n_dropped_host, void *ws, size_t ws_bytes, hipStream_t stream) {
    if (n < 0 || m_in < 0) return fail(AD_ERR_INVALID_ARG, "negative n or edge count");
    if (n >= ((int64_t)1 << 31) || m_in >= ((int64_t)1 << 31))
        return fail(AD_ERR_UNSUPPORTED, "n and the edge count must be below 2^31");
    if (order < 0 || order > 2)
        return fail(AD_ERR_INVALID_ARG, "order must be 0 (as listed), 1 (by degree) or 2 (reverse Cuthill-McKee)");
    if (m_in > 0 && (!u || !v)) return fail(AD_ERR_INVALID_ARG, "u or v is NULL");
    if (!row_ptr || !m_host) return fail(AD_ERR_INVALID_ARG, "row_ptr or m_host is NULL");
    if (m_in > 0 && (!col || !eid)) return fail(AD_ERR_INVALID_ARG, "col or eid is NULL");
    if (n > 0 && !orig_id_out) return fail(AD_ERR_INVALID_ARG, "orig_id_out is NULL");
    if (w && m_in > 0 && !w_out) return fail(AD_ERR_INVALID_ARG, "w_out is NULL for a weighted list");
    if (!ws) return fail(AD_ERR_INVALID_ARG, "workspace is NULL");
    if (((uintptr_t)ws & 255) != 0) return fail(AD_ERR_WORKSPACE, "workspace not 256-byte aligned");
    IngestLayout L;
    if (ingest_layout(n, m_in, ws, ws_bytes, &L) == 0) return fail(AD_ERR_WORKSPACE, "workspace too small");
    return ingest_impl(n, m_in, u, v, w, orig_id, order, row_ptr, col, w_out, eid, orig_id_out, m_host, d_max_host,
                       n_dropped_host, L, stream);
}
