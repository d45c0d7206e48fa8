// ad_backward.hip -- reverse-mode derivative of L(rho) with respect to the
// edge weights, through the distance, the rescale and the k JOR sweeps of
// Algorithm 1 (FP32).
//
// Forward recap (per vector r; x^(t) below is the relaxation's own value,
// the stored one plus its component's shift, which no sweep changes):
//   x^(t)_i = (1-omega) x^(t-1)_i + omega y^(t)_i,  y^(t)_i = sum_j w_ij x^(t-1)_j / s_i,
//   xhat_i  = (x^(k)_i - m) / (M - m) - 1/2   (m, M: min and max over live rows),
//   rho_e   = sqrt(sum_r (xhat_i - xhat_j)^2).
// Adjoint:
//   xhatbar_i = sum_{e=(i,j)} gbar_e (xhat_i - xhat_j) / rho_e      (0 when rho_e = 0)
//   lambda^(k)_i = xhatbar_i / (M-m), plus
//     sum_i xhatbar_i (x_i - M) / (M-m)^2 at the first row attaining m and
//    -sum_i xhatbar_i (x_i - m) / (M-m)^2 at the first row attaining M;
//   for t = k..1, with w_ij in row i's formula:
//     g_ij += omega * sum_r lambda^(t)_i (x^(t-1)_j - y^(t)_i) / s_i
//     lambda^(t-1) = (1-omega) lambda^(t) + omega W (lambda^(t) / s)
//   dL/dw_e = g_ij + g_ji.
// x^(t-1) for every t comes from the checkpoints: each segment of
// ckpt_every sweeps is recomputed with the forward sweep kernel and launch
// shape, so the recomputed values equal the forward ones bit for bit.
#include "ad_internal.h"

#include <math.h>

#include <algorithm>

namespace ad {

constexpr int BB = 256;
constexpr int PART_ROWS = 256;           // rows per workgroup of k_adj_rescale (1,024: too few workgroups
                                         // in flight, 39 us at n = 2^18, R = 8; 256: 15 us)

static int lanes_for(double avg) {
    int lpr = 1;
    while (lpr < 64 && lpr < avg) lpr <<= 1;
    return lpr;
}

// xhatbar from grad_rho: one lane per stored entry, LPR lanes per row.  rho
// is recomputed in the forward distance kernel's order: VEC values per chunk
// summed in order, chunks combined by a pairwise tree when their count is a
// power of two, else in order -- so it equals the forward value bit for bit.
template <int RB, int VEC>
__global__ __launch_bounds__(BB) void k_adj_dist(int64_t n, const int64_t *__restrict__ row_ptr,
                                                 const int32_t *__restrict__ col,
                                                 const int32_t *__restrict__ eid,
                                                 const float *__restrict__ x, const double *__restrict__ minmax,
                                                 const float *__restrict__ grad_rho, float *__restrict__ xbh,
                                                 int R, int LPR) {
    __shared__ float inv_l[64];
    if (threadIdx.x < R) {
        double lo = minmax[threadIdx.x], hi = minmax[R + threadIdx.x];
        inv_l[threadIdx.x] = (hi > lo) ? (float)(1.0 / (hi - lo)) : 0.f;
    }
    __syncthreads();
    const int64_t row = (int64_t)blockIdx.x * (BB / LPR) + threadIdx.x / LPR;
    const int lane = threadIdx.x % LPR;
    float acc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) acc[r] = 0.f;
    if (row < n) {
        const int64_t beg = row_ptr[row], end = row_ptr[row + 1];
        const float *xi = x + row * R;
        for (int64_t p = beg + lane; p < end; p += LPR) {
            const float *xj = x + (int64_t)col[p] * R;
            float d[RB];
#pragma unroll
            for (int r = 0; r < RB; ++r) d[r] = r < R ? (xi[r] - xj[r]) * inv_l[r] : 0.f;
            constexpr int NC = RB / VEC;
            const int C = R / VEC;
            float part[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                float a = 0.f;
#pragma unroll
                for (int q = 0; q < VEC; ++q) a = fmaf(d[c * VEC + q], d[c * VEC + q], a);
                part[c] = a;
            }
            float ss;
            if ((C & (C - 1)) == 0) {
#pragma unroll
                for (int off = 1; off < NC; off <<= 1) {
#pragma unroll
                    for (int c = 0; c + off < NC; c += 2 * off)
                        if (off < C) part[c] += part[c + off];
                }
                ss = part[0];
            } else {
                ss = part[0];
#pragma unroll
                for (int c = 1; c < NC; ++c)
                    if (c < C) ss += part[c];
            }
            const float rho = sqrtf(ss);
            if (rho > 0.f) {
                const float c = grad_rho[eid[p]] / rho;
#pragma unroll
                for (int r = 0; r < RB; ++r) acc[r] = fmaf(c, d[r], acc[r]);
            }
        }
    }
    for (int off = LPR >> 1; off >= 1; off >>= 1) {
#pragma unroll
        for (int r = 0; r < RB; ++r) acc[r] += shfl_down(acc[r], off);
    }
    if (row < n && lane == 0) {
#pragma unroll
        for (int r = 0; r < RB; ++r)
            if (r < R) xbh[row * R + r] = acc[r];
    }
}

// First live row attaining the min and the max of each vector (values with
// their shift added back exactly as ad_relax's min / max pass adds it).
__global__ void k_adj_argminmax(int64_t n, int R, const int64_t *__restrict__ row_ptr,
                                const float *__restrict__ x, const double *__restrict__ shift,
                                const int32_t *__restrict__ comp_of, const double *__restrict__ minmax,
                                unsigned long long *__restrict__ arg) {
    const int64_t total = n * R;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = idx / R;
        const int r = (int)(idx - i * R);
        if (row_ptr[i + 1] == row_ptr[i]) continue;
        bool zero;
        const double *sh = row_shift(shift, comp_of, i, 0, R, zero);
        const double v = (double)x[idx] + (zero ? 0.0 : sh[r]);
        if (v == minmax[r]) atomicMin(&arg[r], (unsigned long long)i);
        if (v == minmax[R + r]) atomicMin(&arg[R + r], (unsigned long long)i);
    }
}

// lambda = xhatbar / (M - m) on live rows; partial sums for the min/max terms.
__global__ __launch_bounds__(BB) void k_adj_rescale(int64_t n, int R, const int64_t *__restrict__ row_ptr,
                                                   const float *__restrict__ x, const double *__restrict__ shift,
                                                   const int32_t *__restrict__ comp_of,
                                                   const double *__restrict__ minmax,
                                                   const float *__restrict__ xbh, float *__restrict__ lam,
                                                   double *__restrict__ part) {
    __shared__ double a_l[BB];
    __shared__ double b_l[BB];
    const int t = threadIdx.x;
    const int stride = BB / R;
    const int r = t % R;
    const int row_off = t / R;
    const double lo = minmax[r], hi = minmax[R + r];
    const double D = hi - lo;
    const double inv = D > 0 ? 1.0 / D : 0.0;
    double a = 0.0, b = 0.0;
    const int64_t r0 = (int64_t)blockIdx.x * PART_ROWS;
    const int64_t r1 = min(n, r0 + PART_ROWS);
    if (row_off < stride) {
        for (int64_t i = r0 + row_off; i < r1; i += stride) {
            const bool live = row_ptr[i + 1] > row_ptr[i];
            const double xb = live ? (double)xbh[i * R + r] : 0.0;
            lam[i * R + r] = (float)(xb * inv);
            bool zero;
            const double *sh = row_shift(shift, comp_of, i, 0, R, zero);
            const double xv = (double)x[i * R + r] + (zero ? 0.0 : sh[r]);
            a += xb * (xv - hi) * inv * inv;
            b -= xb * (xv - lo) * inv * inv;
        }
    }
    a_l[t] = a;
    b_l[t] = b;
    __syncthreads();
    if (t < R) {
        double sa = 0.0, sb = 0.0;
        for (int q = t; q < stride * R; q += R) {
            sa += a_l[q];
            sb += b_l[q];
        }
        part[(int64_t)blockIdx.x * 2 * R + t] = sa;
        part[(int64_t)blockIdx.x * 2 * R + R + t] = sb;
    }
}

// The rows attaining min and max, a wave per vector (a thread per vector read
// 256 workgroups' sums one after another: 64 us; 8 us).
__global__ __launch_bounds__(WAVE) void k_adj_corner(int R, int64_t nblocks, const double *__restrict__ part,
                                                     const unsigned long long *__restrict__ arg,
                                                     const double *__restrict__ minmax, float *__restrict__ lam) {
    const int r = blockIdx.x;
    if (!(minmax[R + r] > minmax[r])) return;
    double sa = 0.0, sb = 0.0;
    for (int64_t b = threadIdx.x; b < nblocks; b += WAVE) {
        sa += part[b * 2 * R + r];
        sb += part[b * 2 * R + R + r];
    }
    for (int o = WAVE / 2; o >= 1; o >>= 1) {
        sa += __shfl_xor(sa, o, WAVE);
        sb += __shfl_xor(sb, o, WAVE);
    }
    if (threadIdx.x != 0) return;
    const unsigned long long imin = arg[r], imax = arg[R + r];
    // one wave per vector: the two updates of column r never race
    lam[imin * R + r] = (float)((double)lam[imin * R + r] + sa);
    lam[imax * R + r] = (float)((double)lam[imax * R + r] + sb);
}

// mu = lambda / s of the first reverse step.
__global__ void k_adj_scale_rows(int64_t n, int R, const float *__restrict__ a, const float *__restrict__ s,
                                 float *__restrict__ out) {
    const int64_t total = n * R;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x)
        out[idx] = a[idx] * s[idx / R];
}

// One reverse step, a row per group of CP * S lanes (CP: a power of two not below the
// C = R / VEC lanes that hold a row of R values; S slots share the row's entries):
//   y_i = sum_j w_ij x_j / s_i,  W_i = sum_j w_ij mu_j
//   g_p += omega / s_i * lambda_i . (x_j - y_i) for every entry p = (i, j)
//   lambda'_i = (1 - omega) lambda_i + omega W_i,  mu'_i = lambda'_i / s_i
// Both gathers of a row are issued together and the gathered x_j kept for g
// where the row fits ADJ_U entries per slot; longer rows gather x_j twice.  Rows
// beyond hub_d are listed, and the first hub_blocks workgroups take one each.
// Bound by the gathers.  As five launches (two sweeps, the gradient with a third
// gather, two passes over n x R for the scale and the sum) a step took
// 52 us at n = 2^18, m = 526K, R = 8 and a gradient through 20 sweeps 1.68 ms;
// 19.4 us and 0.95 ms here.
constexpr int ADJ_U = 4;                 // entries per slot and chunk

template <int VEC>
struct AdjRow {
    int64_t beg, end;
    float is;
    int off, slot, step;          // of R values, of entries
    bool on;                      // this lane holds values
};

// Entries p, p + step, ... of one chunk: x_j (and mu_j into am).
template <int VEC, bool SUMS>
__device__ __forceinline__ void adj_gather(const AdjRow<VEC> &a, int64_t p, const int32_t *__restrict__ col,
                                           const float *__restrict__ w, const float *__restrict__ x,
                                           const float *__restrict__ mu, int R, float (&xv)[ADJ_U][VEC],
                                           float (&ay)[VEC], float (&am)[VEC]) {
    int32_t jj[ADJ_U];
    float ww[ADJ_U];
#pragma unroll
    for (int u = 0; u < ADJ_U; ++u) {
        const int64_t q = p + (int64_t)u * a.step;
        const bool ok = a.on && q < a.end;
        jj[u] = ok ? col[q] : -1;
        if (SUMS) ww[u] = ok ? (w ? w[q] : 1.f) : 0.f;
    }
    float mv[ADJ_U][VEC];
#pragma unroll
    for (int u = 0; u < ADJ_U; ++u) {
#pragma unroll
        for (int q = 0; q < VEC; ++q) {
            xv[u][q] = 0.f;
            if (SUMS) mv[u][q] = 0.f;
        }
        if (jj[u] >= 0) {
            load_vec<VEC>(x + (int64_t)jj[u] * R + a.off, xv[u]);
            if (SUMS) load_vec<VEC>(mu + (int64_t)jj[u] * R + a.off, mv[u]);
        }
    }
    if (SUMS) {
#pragma unroll
        for (int u = 0; u < ADJ_U; ++u) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                ay[q] = fmaf(ww[u], xv[u][q], ay[q]);
                am[q] = fmaf(ww[u], mv[u][q], am[q]);
            }
        }
    }
}

template <int VEC>
__device__ __forceinline__ void adj_grad(const AdjRow<VEC> &a, int64_t p, int CP, float sc, const float (&li)[VEC],
                                         const float (&y)[VEC], const float (&xv)[ADJ_U][VEC], float *__restrict__ g) {
    float dot[ADJ_U];
#pragma unroll
    for (int u = 0; u < ADJ_U; ++u) {
        dot[u] = 0.f;
#pragma unroll
        for (int q = 0; q < VEC; ++q) dot[u] = fmaf(li[q], xv[u][q] - y[q], dot[u]);     // li is 0 off the row
    }
    for (int o = 1; o < CP; o <<= 1) {
#pragma unroll
        for (int u = 0; u < ADJ_U; ++u) dot[u] += __shfl_xor(dot[u], o, WAVE);
    }
#pragma unroll
    for (int u = 0; u < ADJ_U; ++u) {
        const int64_t q = p + (int64_t)u * a.step;
        if (a.off == 0 && q < a.end) g[q] = fmaf(sc, dot[u], g[q]);
    }
}

template <int VEC>
__global__ __launch_bounds__(BB) void k_adj_step(int64_t n, const int64_t *__restrict__ row_ptr,
                                                 const int32_t *__restrict__ col, const float *__restrict__ w,
                                                 const float *__restrict__ inv_s, float omega,
                                                 const float *__restrict__ x, const float *__restrict__ lam,
                                                 const float *__restrict__ mu, float *__restrict__ g,
                                                 float *__restrict__ lam_out, float *__restrict__ mu_out, int R,
                                                 int CP, int S, int64_t hub_d, const int32_t *__restrict__ hubs,
                                                 const unsigned int *__restrict__ hub_count, unsigned int hub_blocks,
                                                 int64_t row_blocks) {
    constexpr int NW = BB / WAVE;
    __shared__ float part[NW][WAVE][2 * VEC];
    const int c = threadIdx.x % CP;
    AdjRow<VEC> a;
    a.off = c * VEC;
    a.on = a.off < R;
    const bool hub = blockIdx.x < hub_blocks;
    // the workgroup's listed rows, or its blocks of BB / (CP * S) rows
    const int64_t items = hub ? (int64_t)*hub_count : row_blocks;
    const unsigned int stride = hub ? hub_blocks : gridDim.x - hub_blocks;
    for (int64_t h = hub ? blockIdx.x : blockIdx.x - hub_blocks; h < items; h += stride) {
        int64_t row;
        if (hub) {
            row = hubs[h];
            a.slot = threadIdx.x / CP;
            a.step = BB / CP;
        } else {
            const int group = CP * S;
            row = h * (BB / group) + threadIdx.x / group;
            a.slot = (threadIdx.x % group) / CP;
            a.step = S;
            if (row >= n) continue;                                  // uniform over the group
        }
        a.beg = row_ptr[row];
        a.end = row_ptr[row + 1];
        if (!hub && a.end - a.beg > hub_d) continue;                 // uniform over the group
        a.is = inv_s[row];
        float li[VEC], ay[VEC], am[VEC], xv[ADJ_U][VEC];
#pragma unroll
        for (int q = 0; q < VEC; ++q) li[q] = ay[q] = am[q] = 0.f;
        if (a.on) load_vec<VEC>(lam + row * R + a.off, li);
        const int64_t chunk = (int64_t)ADJ_U * a.step;
        for (int64_t p = a.beg + a.slot; p < a.end; p += chunk)
            adj_gather<VEC, true>(a, p, col, w, x, mu, R, xv, ay, am);
        // the slots' sums, over the wave's slots and then over the workgroup's waves
        const int span = hub ? WAVE : CP * S;
        for (int o = CP; o < span; o <<= 1) {
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                ay[q] += __shfl_xor(ay[q], o, WAVE);
                am[q] += __shfl_xor(am[q], o, WAVE);
            }
        }
        if (hub) {
            const int wv = threadIdx.x / WAVE;
            if ((int)(threadIdx.x % WAVE) < CP) {
#pragma unroll
                for (int q = 0; q < VEC; ++q) {
                    part[wv][c][q] = ay[q];
                    part[wv][c][VEC + q] = am[q];
                }
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                ay[q] = am[q] = 0.f;
                for (int v = 0; v < NW; ++v) {
                    ay[q] += part[v][c][q];
                    am[q] += part[v][c][VEC + q];
                }
            }
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < VEC; ++q) ay[q] *= a.is;
        const float sc = omega * a.is;
        if (a.end - a.beg <= chunk) {
            if (a.beg + a.slot < a.end) adj_grad<VEC>(a, a.beg + a.slot, CP, sc, li, ay, xv, g);
        } else {
            for (int64_t p = a.beg + a.slot; p < a.end; p += chunk) {
                adj_gather<VEC, false>(a, p, col, w, x, mu, R, xv, ay, am);
                adj_grad<VEC>(a, p, CP, sc, li, ay, xv, g);
            }
        }
        if (a.slot == 0 && a.on) {
            float nl[VEC], nm[VEC];
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                nl[q] = fmaf(omega, am[q], (1.f - omega) * li[q]);
                nm[q] = nl[q] * a.is;
            }
            store_vec<VEC>(lam_out + row * R + a.off, nl);
            store_vec<VEC>(mu_out + row * R + a.off, nm);
        }
    }
}

__global__ void k_edge_to_entries(int64_t nnz, const int32_t *__restrict__ eid, const float *__restrict__ we,
                                  float *__restrict__ out) {
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz;
         p += (int64_t)gridDim.x * blockDim.x)
        out[p] = we[eid[p]];
}

__global__ void k_adj_fold(int64_t nnz, const int32_t *__restrict__ eid, const float *__restrict__ g,
                           float *__restrict__ grad_w) {
    // two addends per edge onto a zeroed slot: the result does not depend on order
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < nnz;
         p += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&grad_w[eid[p]], g[p]);
}

struct BwdLayout {
    float *inv_s, *sdeg;
    SweepPlan plan;
    float *xbh, *lam, *lam2, *mu, *mu2, *seg, *g;
    double *part;
    unsigned long long *arg;
};

static size_t bwd_layout(const ad_graph *g, const ad_relax_opts *o, void *ws, size_t ws_bytes, BwdLayout *L) {
    Carver c(ws, ws_bytes);
    const int64_t n = std::max<int64_t>(1, g->n);
    const int64_t nnz = std::max<int64_t>(1, 2 * g->m);
    const size_t nR = (size_t)n * o->R;
    const int64_t nb = std::max<int64_t>(1, ceil_div(g->n, PART_ROWS));
    BwdLayout l;
    l.inv_s = c.take<float>(n);
    l.sdeg = c.take<float>(n);
    sweep_plan_carve(c, n, ceil_div(n, PLAN_TILE), l.plan);
    l.xbh = c.take<float>(nR);
    l.lam = c.take<float>(nR);
    l.lam2 = c.take<float>(nR);
    l.mu = c.take<float>(nR);
    l.mu2 = c.take<float>(nR);
    l.seg = c.take<float>(nR * (size_t)std::max(1, o->ckpt_every));
    l.g = c.take<float>(nnz);
    l.part = c.take<double>(nb * 2 * o->R);
    l.arg = c.take<unsigned long long>(2 * o->R);
    if (L) *L = l;
    return c.ok() ? c.used : 0;
}

template <int RB>
static ad_status launch_rb(const ad_graph *g, const ad_relax_opts *o, const float *x_k, const double *minmax,
                           const float *grad_rho, const BwdLayout &L, int lpr, hipStream_t st) {
    const unsigned nb = (unsigned)ceil_div(g->n, BB / lpr);
    const int R = o->R;
    // the forward distance kernel's vector width for FP32
    const int vec = R % 4 == 0 ? 4 : (R % 2 == 0 ? 2 : 1);
    if (vec == 4)
        hipLaunchKernelGGL((k_adj_dist<RB, 4>), dim3(nb), dim3(BB), 0, st, g->n, g->row_ptr, g->col, g->eid, x_k,
                           minmax, grad_rho, L.xbh, R, lpr);
    else if (vec == 2)
        hipLaunchKernelGGL((k_adj_dist<RB, 2>), dim3(nb), dim3(BB), 0, st, g->n, g->row_ptr, g->col, g->eid, x_k,
                           minmax, grad_rho, L.xbh, R, lpr);
    else
        hipLaunchKernelGGL((k_adj_dist<RB, 1>), dim3(nb), dim3(BB), 0, st, g->n, g->row_ptr, g->col, g->eid, x_k,
                           minmax, grad_rho, L.xbh, R, lpr);
    AD_LAUNCH_CHECK("k_adj_dist");
    return AD_OK;
}

// Workgroups for rows, each with several blocks of them on larger graphs: 64 lanes to
// every row of a graph of 2^26 would be 2^32 threads, more than a launch takes.
constexpr int64_t STEP_BLOCKS = (int64_t)1 << 16;

template <int VEC>
static ad_status launch_step(const ad_graph *g, const BwdLayout &L, const SweepPlan &plan, float omega,
                             const float *xprev, const float *lam, const float *mu, float *lam_out, float *mu_out,
                             int R, hipStream_t st) {
    int cp = 1;
    while (cp * VEC < R) cp *= 2;
    // slots: a chunk holds 1.5 times the average row, so that most rows need one.  Average
    // 4, R = 8, entries per slot x slots: 4 x 2 19.4 us a step, 4 x 1 21.4, 2 x 2 22.1,
    // 2 x 4 25.1, 8 x 1 22.7, 8 x 2 32.1.  One count for all rows also serves skewed
    // degrees (a gradient with the former sweeps, lanes planned per 64 rows / here: power law of
    // average 32, n = 2^16, R = 8 3.75 / 1.50 ms, n = 2^20 25.4 / 15.2, 10 sweeps; R-MAT 2^17 17.4 / 4.4)
    const double avg = 2.0 * (double)g->m / (double)g->n;
    int slots = 1;
    while (2 * cp * slots <= WAVE && 2 * slots * ADJ_U < 3 * avg) slots *= 2;
    // a listed row has more than hub_d of the 2m entries
    const unsigned hub_blocks = (unsigned)std::min<int64_t>(512, 2 * g->m / (plan.sh.hub_d + 1));
    const int64_t blocks = ceil_div(g->n, BB / (cp * slots));
    const unsigned grid = hub_blocks + (unsigned)std::min<int64_t>(STEP_BLOCKS, blocks);
    hipLaunchKernelGGL((k_adj_step<VEC>), dim3(grid), dim3(BB), 0, st, g->n, g->row_ptr,
                       g->col, g->w, L.inv_s, omega, xprev, lam, mu, L.g, lam_out, mu_out, R, cp, slots,
                       plan.sh.hub_d, plan.hub_list, plan.hub_count, hub_blocks, blocks);
    AD_LAUNCH_CHECK("k_adj_step");
    return AD_OK;
}

}  // namespace ad

using namespace ad;

extern "C" ad_status ad_edge_to_entries(const ad_graph *g, const float *w_edge, float *w_entries,
                                        hipStream_t stream) {
    ad_status s = check_graph_args(g);
    if (s != AD_OK) return s;
    if (g->m == 0) return AD_OK;
    if (!w_edge || !w_entries) return fail(AD_ERR_INVALID_ARG, "w_edge or w_entries is NULL");
    const int64_t nnz = 2 * g->m;
    hipLaunchKernelGGL(k_edge_to_entries, dim3(grid_for(nnz, BB)), dim3(BB), 0, stream, nnz, g->eid, w_edge,
                       w_entries);
    AD_LAUNCH_CHECK("k_edge_to_entries");
    return AD_OK;
}

extern "C" size_t ad_relax_backward_workspace_size(const ad_graph *g, const ad_relax_opts *o) {
    if (check_graph_args(g) != AD_OK || !o || o->R < 1 || o->R > 64 || o->ckpt_every < 1) return 0;
    return bwd_layout(g, o, nullptr, 0, nullptr);
}

extern "C" ad_status ad_relax_backward(const ad_graph *g, const ad_relax_opts *o, const void *ckpt,
                                       const void *x_k, const double *minmax, const double *shift,
                                       const float *grad_rho, float *grad_w, void *ws, size_t ws_bytes,
                                       hipStream_t stream) {
    ad_status s = check_graph_args(g);
    if (s != AD_OK) return s;
    if (!o) return fail(AD_ERR_INVALID_ARG, "opts is NULL");
    if (o->R < 1 || o->R > 64) return fail(AD_ERR_INVALID_ARG, "R must be in [1, 64]");
    if (o->k < 0) return fail(AD_ERR_INVALID_ARG, "k must be >= 0");
    if (!(o->omega > 0.0 && o->omega <= 1.0)) return fail(AD_ERR_INVALID_ARG, "omega must be in (0, 1]");
    if (o->store != AD_F32) return fail(AD_ERR_UNSUPPORTED, "the adjoint needs FP32 storage");
    if (o->fp64_tail != 0) return fail(AD_ERR_UNSUPPORTED, "the adjoint needs fp64_tail == 0");
    if (o->ckpt_every < 1) return fail(AD_ERR_INVALID_ARG, "the adjoint needs ckpt_every >= 1");
    if (g->m > 0 && (!x_k || !minmax || !shift || !grad_rho || !grad_w))
        return fail(AD_ERR_INVALID_ARG, "x_k, minmax, shift, grad_rho or grad_w is NULL");
    if (o->comp && o->comp->n_comp > 0 && !o->comp->comp_of)
        return fail(AD_ERR_INVALID_ARG, "component arrays are NULL");
    const int32_t *comp_of = o->comp ? o->comp->comp_of : nullptr;
    if (o->k > 0 && g->m > 0 && !ckpt) return fail(AD_ERR_INVALID_ARG, "ckpt is NULL");
    if (!ws) return fail(AD_ERR_INVALID_ARG, "workspace is NULL");
    if (((uintptr_t)ws & 255) != 0) return fail(AD_ERR_WORKSPACE, "workspace not 256-byte aligned");
    BwdLayout L;
    if (bwd_layout(g, o, ws, ws_bytes, &L) == 0) return fail(AD_ERR_WORKSPACE, "workspace too small");
    if (g->m == 0) return AD_OK;

    const int R = o->R;
    const int64_t n = g->n, nnz = 2 * g->m;
    const size_t nR = (size_t)n * R;
    const double avg = (double)nnz / (double)n;
    const int lpr = lanes_for(avg);
    const float omega = (float)o->omega;
    const float *xk = (const float *)x_k;

    SweepPlan plan = L.plan;
    plan.sh = sweep_shape(R, sizeof(float), o->rows_per_wave, o->hub_degree);
    s = sweep_plan_build(g, plan, true, Segs(), stream);
    if (s != AD_OK) return s;
    s = weighted_degree_f32(g, L.inv_s, L.sdeg, plan, stream);
    if (s != AD_OK) return s;
    s = fill_i32((int32_t *)L.g, 0, nnz, stream);
    if (s != AD_OK) return s;
    s = fill_i32((int32_t *)grad_w, 0, g->m, stream);
    if (s != AD_OK) return s;

    // distance adjoint
    if (R <= 8) s = launch_rb<8>(g, o, xk, minmax, grad_rho, L, lpr, stream);
    else if (R <= 16) s = launch_rb<16>(g, o, xk, minmax, grad_rho, L, lpr, stream);
    else if (R <= 32) s = launch_rb<32>(g, o, xk, minmax, grad_rho, L, lpr, stream);
    else s = launch_rb<64>(g, o, xk, minmax, grad_rho, L, lpr, stream);
    if (s != AD_OK) return s;

    // rescale adjoint
    s = fill_u64(L.arg, ~0ull, 2 * R, stream);
    if (s != AD_OK) return s;
    hipLaunchKernelGGL(k_adj_argminmax, dim3(grid_for((int64_t)nR, BB)), dim3(BB), 0, stream, n, R, g->row_ptr,
                       xk, shift, comp_of, minmax, L.arg);
    AD_LAUNCH_CHECK("k_adj_argminmax");
    const int64_t nb = std::max<int64_t>(1, ceil_div(n, PART_ROWS));
    hipLaunchKernelGGL(k_adj_rescale, dim3((unsigned)nb), dim3(BB), 0, stream, n, R, g->row_ptr, xk, shift,
                       comp_of, minmax, L.xbh, L.lam, L.part);
    AD_LAUNCH_CHECK("k_adj_rescale");
    hipLaunchKernelGGL(k_adj_corner, dim3((unsigned)R), dim3(WAVE), 0, stream, R, nb, L.part, L.arg, minmax, L.lam);
    AD_LAUNCH_CHECK("k_adj_corner");

    // reverse sweeps, one checkpoint segment at a time
    const int c = o->ckpt_every;
    const int nseg = ad_relax_num_checkpoints(o);
    float *lam = L.lam, *lam_next = L.lam2, *mu = L.mu, *mu_next = L.mu2;
    hipLaunchKernelGGL(k_adj_scale_rows, dim3(grid_for((int64_t)nR, BB)), dim3(BB), 0, stream, n, R, lam, L.inv_s, mu);
    AD_LAUNCH_CHECK("k_adj_scale_rows");
    for (int q = nseg - 1; q >= 0; --q) {
        const int t0 = q * c;
        const int t1 = std::min(o->k, (q + 1) * c);
        const float *base = (const float *)ckpt + (size_t)q * nR;
        // seg[u] = x^(t0 + u), u = 0 .. t1 - t0 - 1
        for (int u = 1; u < t1 - t0; ++u) {
            const float *src = u == 1 ? base : L.seg + (size_t)(u - 1) * nR;
            s = sweep_f32(g, L.inv_s, omega, src, L.seg + (size_t)u * nR, R, plan, stream);
            if (s != AD_OK) return s;
        }
        for (int t = t1; t > t0; --t) {
            const int u = t - 1 - t0;
            const float *xprev = u == 0 ? base : L.seg + (size_t)u * nR;
            if (plan.sh.vec == 4)
                s = launch_step<4>(g, L, plan, omega, xprev, lam, mu, lam_next, mu_next, R, stream);
            else if (plan.sh.vec == 2)
                s = launch_step<2>(g, L, plan, omega, xprev, lam, mu, lam_next, mu_next, R, stream);
            else
                s = launch_step<1>(g, L, plan, omega, xprev, lam, mu, lam_next, mu_next, R, stream);
            if (s != AD_OK) return s;
            std::swap(mu, mu_next);
            std::swap(lam, lam_next);
        }
    }
    hipLaunchKernelGGL(k_adj_fold, dim3(grid_for(nnz, BB)), dim3(BB), 0, stream, nnz, g->eid, L.g, grad_w);
    AD_LAUNCH_CHECK("k_adj_fold");
    return AD_OK;
}
