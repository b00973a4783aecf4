// Backward pass of the fused attention call for the degree-1 filter (the paper states the forward pass only,
// Algorithm 1; training and conservative forces F = -dE/dpos need its derivative).  As in the forward pass nothing
// per pair is written to memory: the pair quantities are recomputed from positions, q, k, v and two per-atom
// softmax statistics, and every atom's gradients are accumulated by the workgroup that owns the atom (no atomics,
// deterministic).  The message is linear in the pair vector for this filter, m_ij = sum_mu (r_ij)_mu G_mu v_j with
// the three axis operators G_mu = D(R_mu)^T P D(R_mu) of the tile kernel, which gives, per head, with g = dL/d out:
//     u_mu   = <g_i, G_mu v_j>                     w = sum_mu r_mu u_mu = <g_i, m_ij>
//     P_ij   = exp(s_ij - lse_i)                   alpha_ij = P_ij phi(d)
//     ds_ij  = P_ij (phi w - D_i),  D_i = <g_i, out_i>         (softmax with the gate outside, Eq. attn)
//     dq_i  += tau ds_ij k_j          dk_j += tau ds_ij q_i          dv_j += alpha_ij sum_mu r_mu G_mu^T g_i
//     dL/dr_ij = sum_heads [ alpha_ij u + (ds_ij b'(d) + P_ij w phi'(d)) r/d ],   dpos_j += dL/dr_ij,  dpos_i -= dL/dr_ij
// Three kernels, one workgroup per atom with one thread per channel: the softmax statistics (lse, D), the sums an
// atom owns as a target (dq, its share of dpos), and the sums it owns as a source (dk, dv, its share of dpos).  The
// last one walks the atom's own neighbours, which are exactly the targets that see it: the relation is symmetric
// (also under periodic boundaries, with opposite images), which is why a neighbour cap is not supported here.
#include <limits.h>

#include "e2f_axis_pattern.h"
#include "e2f_device.h"

namespace {

constexpr int BCAP = 128;   // neighbours per batch of the list
constexpr int WP_BINS = 32;  // row length of the per-atom path-weight partials ((L_max + 1)^2 <= 25 used)
constexpr int WB_PER_THREAD = 8;   // radial basis functions per thread of a head in the dWb sums: B <= 8 * C/H

struct BwdParams {
    E2fCellsView cv;
    const float4* spos;   // sorted positions (folded on periodic axes), w = atom index
    const float* q;       // [N][L+1][C] sorted order
    const float* k;
    const void* v;        // [N][n][C] sorted order, feature dtype
    const float* G;       // [3][25][25] axis operators
    const float* Wb;      // [H][B]
    const float* out;     // forward result, caller's order
    const float* gout;    // dL/d out, caller's order
    float* lse;           // [N][H] sorted order: log of the softmax normaliser, reference included
    float* Dn;            // [N][H] sorted order: <g_i, out_i> per head
    float* gpos;          // [N][3] caller's order
    float* gq;            // [N][L+1][C] caller's order
    float* gk;
    float* gv;            // [N][n][C] caller's order
    // gradients of the attention's own weights (null unless asked for): per-atom partial sums, reduced afterwards
    const float* Gu;      // [3][25][25] axis operators with unit path weights
    float* pWb;           // [N][H][B]
    float* pwp;           // [N][WP_BINS], bin li * (L_max + 1) + lo
    // TL instances (the crowded tiles that the tile kernels of e2f_bwd_tile.hip leave out) read the tile layouts
    // instead of q, k, v, lse and Dn: q rows scaled by tau log2 e and k rows in binary16, value blocks, statistics
    // in base-2 units
    const uint16_t *q16, *k16, *v4;
    float2* stat4;            // [group of 4 slots][H][4] (lse, D)
    const int4* lists_hdr;    // per tile of 16 slots: x < 0 marks a crowded tile
    int C, H, B, Ch;
    float tau, rc2, cutoff, rbf_step, rbf_gamma;
};

constexpr float LOG2E = 1.44269504088896341f, LN2 = 0.69314718055994531f;

// Operand access in the plain layouts or (TL) in the layouts of the tile kernels (heads of 16 channels).
template <int L, bool TL>
__device__ __forceinline__ float load_q(const BwdParams& P, int t, int l, int c) {
    if constexpr (TL) {
        constexpr int DKP = ((L + 1) * 16 + 31) / 32 * 32;
        return (float)__builtin_bit_cast(_Float16, P.q16[((size_t)t * P.H + (c >> 4)) * DKP + l * 16 + (c & 15)]);
    } else {
        return P.q[((size_t)t * (L + 1) + l) * P.C + c];
    }
}
template <int L, bool TL>
__device__ __forceinline__ float load_k(const BwdParams& P, int j, int l, int c) {
    if constexpr (TL) {
        constexpr int DKP = ((L + 1) * 16 + 31) / 32 * 32;
        return (float)__builtin_bit_cast(_Float16, P.k16[e2f::k16_offset(j, P.H, c >> 4, DKP, l * 16 + (c & 15))]);
    } else {
        return P.k[((size_t)j * (L + 1) + l) * P.C + c];
    }
}
template <int L, typename VT, bool TL>
__device__ __forceinline__ float load_v(const BwdParams& P, int j, int x, int c) {
    constexpr int n = (L + 1) * (L + 1);
    if constexpr (TL)
        return e2f::bf16_bits_to_float(P.v4[((size_t)(j >> 2) * P.H + (c >> 4)) * n * 64 + e2f::v4_offset(n, x, c & 15) + (j & 3)]);
    else
        return e2f::load_as_float<VT>((const VT*)P.v + ((size_t)j * n + x) * P.C + c);
}
// Softmax weight P_ij from the dot product of the layout's q and k rows, the bias (natural units) and the statistic.
template <bool TL>
__device__ __forceinline__ float pair_prob(const BwdParams& P, float dot, float bias, float lse) {
    if constexpr (TL) return exp2f(dot + bias * LOG2E - lse);
    else return __expf(dot * P.tau + bias - lse);
}
template <bool TL>
__device__ __forceinline__ float load_lse(const BwdParams& P, int t, int head) {
    if constexpr (TL) return P.stat4[((size_t)(t >> 2) * P.H + head) * 4 + (t & 3)].x;
    else return P.lse[(size_t)t * P.H + head];
}
template <bool TL>
__device__ __forceinline__ float load_Dn(const BwdParams& P, int t, int head) {
    if constexpr (TL) return P.stat4[((size_t)(t >> 2) * P.H + head) * 4 + (t & 3)].y;
    else return P.Dn[(size_t)t * P.H + head];
}

// Sum over the Ch threads of a head (Ch a power of two <= 64, heads aligned inside a wave).
__device__ __forceinline__ float head_sum(float x, int Ch) {
    float one[1] = {x};
    e2f::group_sums(one, Ch);
    return one[0];
}
// Whether the rows of a batch's next pair are requested before the current pair is worked on (both sets in registers).
// One pair after the other, each waiting for its rows and for four sums over the head's lanes through the LDS unit, and the
// stencil's runs in scratch memory, took 218 and 205 us for the two sides of 2 240 atoms, L = 2, 128 fp32 channels (936
// us the training step); with the sums in the additions, the rows ahead and the runs in LDS the step takes 263 us less.
// At L = 3 and 4 the second set does not fit the registers.
template <int L>
constexpr bool ROWS_AHEAD = L <= 2;

// The neighbours of slot t in batches: wave 0 walks the 18 stencil runs and packs (slot, image position) of the
// atoms inside the cutoff into LDS; every thread of the workgroup then reads the batch.
// The workgroup then evaluates what depends on the distance alone, once per pair instead of once per channel:
// s_rad[e] = (phi, dphi/dd, d, -) and s_bias[e * H + h] = (b_h(d), db_h/dd).
__device__ __forceinline__ int next_batch(const BwdParams& P, const e2f::RunList& runs, int& base, int t, const float4& pi, int* s_list,
                                          float4* s_pos, float4* s_rad, float2* s_bias, int* s_ctl) {
    __syncthreads();   // the previous batch has been consumed
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int cnt = 0;
        const int total = runs.total();
        while (base < total && cnt + 64 <= BCAP) {
            bool ok = false;
            int j = 0;
            float4 pj = pi;
            if (base + lane < total) {
                int run;
                runs.candidate(base + lane, run, j);
                const float4 sh = runs.sh[run];
                pj = P.spos[j];
                pj.x += sh.x;
                pj.y += sh.y;
                pj.z += sh.z;
                ok = j != t && e2f::is_neighbor(e2f::dist2_exact(pi.x, pi.y, pi.z, pj.x, pj.y, pj.z), P.rc2);
            }
            const unsigned long long mask = __ballot(ok);
            const int at = cnt + __popcll(mask & ((1ull << lane) - 1ull));
            if (ok) {
                s_list[at] = j;
                s_pos[at] = pj;
            }
            cnt += __popcll(mask);
            base += 64;
        }
        if (lane == 0) {
            s_ctl[0] = cnt;
            s_ctl[1] = base >= total ? 1 : 0;
        }
    }
    __syncthreads();
    const int cnt = s_ctl[0];
    // what depends on the distance alone, spread over the whole workgroup: one (pair, head) item per thread and step
    for (int it = threadIdx.x; it < cnt * P.H; it += blockDim.x) {
        const int e = it / P.H, hh = it % P.H;
        const float4 pj = s_pos[e];
        const float rx = pj.x - pi.x, ry = pj.y - pi.y, rz = pj.z - pi.z;
        const float d = sqrtf(rx * rx + ry * ry + rz * rz);
        if (hh == 0) {
            const float arg = 3.14159265358979f * d / P.cutoff;   // in [0, pi]
            s_rad[e] = make_float4(0.5f * (1.0f + __cosf(arg)), -0.5f * 3.14159265358979f / P.cutoff * __sinf(arg), d, 0.0f);
        }
        float b = 0.0f, db = 0.0f;
        for (int i = 0; i < P.B; ++i) {
            const float x = d - (float)i * P.rbf_step;
            const float g = P.Wb[hh * P.B + i] * __expf(-P.rbf_gamma * x * x);
            b += g;
            db += -2.0f * P.rbf_gamma * x * g;
        }
        s_bias[it] = make_float2(b, db);
    }
    __syncthreads();
    return cnt;
}

// Node-level products with the axis operators, once per atom: T[mu] = G_mu^T a (TRANSPOSE) or G_mu a.
template <int L, bool TRANSPOSE>
__device__ __forceinline__ void axis_apply(const float (&a)[(L + 1) * (L + 1)], const float* s_G,
                                           float (&T)[3][(L + 1) * (L + 1)]) {
    constexpr int n = (L + 1) * (L + 1);
#pragma unroll
    for (int mu = 0; mu < 3; ++mu) {
#pragma unroll
        for (int x = 0; x < n; ++x) T[mu][x] = 0.0f;
#pragma unroll
        for (int xo = 0; xo < n; ++xo)
#pragma unroll
            for (int xi = 0; xi < n; ++xi)
                if ((E2F_AXIS_NZ[mu][xo] >> xi) & 1u) {
                    const float gv = s_G[(mu * E2F_MAX_N + xo) * E2F_MAX_N + xi];
                    if (TRANSPOSE) T[mu][xi] += gv * a[xo];
                    else T[mu][xo] += gv * a[xi];
                }
    }
}

// ---- softmax statistics: lse_i = log sum_j exp(s_ij) and D_i = <g_i, out_i>, per head
template <int L, bool TL>
__global__ __launch_bounds__(256) void k_bwd_stats(BwdParams P) {
    constexpr int n = (L + 1) * (L + 1);
    __shared__ int s_list[BCAP];
    __shared__ float4 s_pos[BCAP], s_rad[BCAP];
    extern __shared__ float2 s_bias[];   // [BCAP][H]
    __shared__ int s_ctl[2];
    const int t = e2f::xcd_remap(blockIdx.x, P.cv.N), C = P.C;
    if (t < 0) return;
    if (TL && P.lists_hdr[t >> 4].x >= 0) return;   // (whole workgroup) the tile kernels own this atom
    const bool live = (int)threadIdx.x < C;        // workgroups have at least one full wave: the list walk needs it
    const int c = live ? threadIdx.x : 0, head = c / P.Ch;
    const int a = P.cv.perm[t];
    const float4 pi = P.spos[t];
    float qv[L + 1];
#pragma unroll
    for (int l = 0; l <= L; ++l) qv[l] = load_q<L, TL>(P, t, l, c);
    float dsum = 0.0f;
    for (int x = 0; x < n; ++x) dsum += P.gout[((size_t)a * n + x) * C + c] * P.out[((size_t)a * n + x) * C + c];
    dsum = head_sum(dsum, P.Ch);
    float m = -INFINITY, z = 0.0f;
    __shared__ e2f::RunList s_run;
    if (threadIdx.x < 64) e2f::fill_runs(s_run, P.cv, t, threadIdx.x);
    int walked = 0;   // (next_batch opens with the barrier that the runs need)
    while (true) {
        const int cnt = next_batch(P, s_run, walked, t, pi, s_list, s_pos, s_rad, s_bias, s_ctl);
        constexpr int PG = 4;   // pairs whose rows are requested and summed together; the last ones repeat, not counted
        for (int e0 = 0; e0 < cnt; e0 += PG) {
          float dots[PG];
#pragma unroll
          for (int u = 0; u < PG; ++u) {
            const int j = s_list[min(e0 + u, cnt - 1)];
            dots[u] = 0.0f;
#pragma unroll
            for (int l = 0; l <= L; ++l) dots[u] += qv[l] * load_k<L, TL>(P, j, l, c);
          }
          e2f::group_sums(dots, P.Ch);
#pragma unroll
          for (int u = 0; u < PG; ++u) {
            const int e = e0 + u;
            if (e >= cnt) break;
            const float dot = dots[u];
            if constexpr (TL) {   // base-2 units, as the tile kernels keep them
                const float s = dot + s_bias[e * P.H + head].x * LOG2E;
                const float mn = fmaxf(m, s);
                z = z * exp2f(m - mn) + exp2f(s - mn);
                m = mn;
            } else {
                const float s = dot * P.tau + s_bias[e * P.H + head].x;
                const float mn = fmaxf(m, s);
                z = z * __expf(m - mn) + __expf(s - mn);
                m = mn;
            }
          }
        }
        if (s_ctl[1]) break;
    }
    if (live && c % P.Ch == 0) {
        if constexpr (TL) {
            P.stat4[((size_t)(t >> 2) * P.H + head) * 4 + (t & 3)] = make_float2(z > 0.0f ? m + log2f(z) : 0.0f, dsum);
        } else {
            P.lse[(size_t)t * P.H + head] = z > 0.0f ? m + logf(z) : 0.0f;
            P.Dn[(size_t)t * P.H + head] = dsum;
        }
    }
}

// Degree of component x (index l*l + l + m).
__host__ __device__ constexpr int degree_of(int x) { return x >= 16 ? 4 : x >= 9 ? 3 : x >= 4 ? 2 : x >= 1 ? 1 : 0; }

// ---- what an atom owns as a target i: dq_i and -sum_j dL/dr_ij; with WGRAD also its partial sums of
//   dL/dWb[h][b] = sum_j ds_ij,h exp(-gamma (d_ij - mu_b)^2)
template <int L, typename VT, bool WGRAD, bool TL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_bwd_target(BwdParams P) {
    constexpr int n = (L + 1) * (L + 1);
    __shared__ int s_list[BCAP];
    __shared__ float4 s_pos[BCAP], s_rad[BCAP];
    extern __shared__ float2 s_bias[];   // [BCAP][H]
    __shared__ int s_ctl[2];
    __shared__ float s_G[3 * E2F_MAX_N * E2F_MAX_N];
    __shared__ float s_gp[E2F_MAX_H][3];
    const int t = e2f::xcd_remap(blockIdx.x, P.cv.N), C = P.C;
    if (t < 0) return;
    if (TL && P.lists_hdr[t >> 4].x >= 0) return;   // (whole workgroup) the tile kernels own this atom
    const bool live = (int)threadIdx.x < C;        // workgroups have at least one full wave: the list walk needs it
    const int c = live ? threadIdx.x : 0, head = c / P.Ch;
    const int a = P.cv.perm[t];
    for (int i = threadIdx.x; i < 3 * E2F_MAX_N * E2F_MAX_N; i += blockDim.x) s_G[i] = P.G[i];
    const float4 pi = P.spos[t];
    float qv[L + 1], dq[L + 1], g[n];
#pragma unroll
    for (int l = 0; l <= L; ++l) {
        qv[l] = load_q<L, TL>(P, t, l, c);
        dq[l] = 0.0f;
    }
#pragma unroll
    for (int x = 0; x < n; ++x) g[x] = P.gout[((size_t)a * n + x) * C + c];
    const float lse = load_lse<TL>(P, t, head), Dn = load_Dn<TL>(P, t, head);
    float gx = 0.0f, gy = 0.0f, gz = 0.0f;   // sum_j dL/dr_ij of this head
    __shared__ e2f::RunList s_run;
    if (threadIdx.x < 64) e2f::fill_runs(s_run, P.cv, t, threadIdx.x);
    int walked = 0;   // (next_batch opens with the barrier that the runs need)
    __syncthreads();
    float gt[3][n];   // G_mu^T g_i: u_mu = <g_i, G_mu v_j> = <gt_mu, v_j>
    axis_apply<L, true>(g, s_G, gt);
    float accWb[WGRAD ? WB_PER_THREAD : 1];
    if (WGRAD) {
#pragma unroll
        for (int i = 0; i < WB_PER_THREAD; ++i) accWb[i] = 0.0f;
    }
    while (true) {
        const int cnt = next_batch(P, s_run, walked, t, pi, s_list, s_pos, s_rad, s_bias, s_ctl);
        constexpr bool AHEAD = ROWS_AHEAD<L>;
        float kn[L + 1], vn[n];   // the rows of the pair to come
        auto request = [&](int e) {
            const int j = s_list[e];
#pragma unroll
            for (int l = 0; l <= L; ++l) kn[l] = load_k<L, TL>(P, j, l, c);
#pragma unroll
            for (int x = 0; x < n; ++x) vn[x] = load_v<L, VT, TL>(P, j, x, c);
        };
        if (AHEAD && cnt > 0) request(0);
        for (int e = 0; e < cnt; ++e) {
            if (!AHEAD) request(e);
            const float4 pj = s_pos[e];
            const float rx = pj.x - pi.x, ry = pj.y - pi.y, rz = pj.z - pi.z;
            const float4 rad = s_rad[e];
            const float2 bb = s_bias[e * P.H + head];
            float kv[L + 1], u[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // the three u_mu, then q k
#pragma unroll
            for (int l = 0; l <= L; ++l) {
                kv[l] = kn[l];
                u[3] += qv[l] * kv[l];
            }
#pragma unroll
            for (int x = 0; x < n; ++x) {
                u[0] += gt[0][x] * vn[x];
                u[1] += gt[1][x] * vn[x];
                u[2] += gt[2][x] * vn[x];
            }
            if (AHEAD) request(min(e + 1, cnt - 1));
            e2f::group_sums(u, P.Ch);
            const float p = pair_prob<TL>(P, u[3], bb.x, lse);
            const float phi = rad.x, dphi = rad.y;
            const float wsum = rx * u[0] + ry * u[1] + rz * u[2];
            const float ds = p * (phi * wsum - Dn);
            const float alpha = p * phi;
            const float dd = (ds * bb.y + p * wsum * dphi) / rad.z;
#pragma unroll
            for (int l = 0; l <= L; ++l) dq[l] += P.tau * ds * kv[l];
            if (WGRAD) {   // the head's threads share its basis functions: thread ci takes b = ci, ci + Ch, ...
#pragma unroll
                for (int i = 0; i < WB_PER_THREAD; ++i) {
                    const int b = c % P.Ch + i * P.Ch;
                    const float xb = rad.z - (float)b * P.rbf_step;
                    if (b < P.B) accWb[i] += ds * __expf(-P.rbf_gamma * xb * xb);
                }
            }
            gx += alpha * u[0] + dd * rx;
            gy += alpha * u[1] + dd * ry;
            gz += alpha * u[2] + dd * rz;
        }
        if (s_ctl[1]) break;
    }
    if (live) {
#pragma unroll
        for (int l = 0; l <= L; ++l) P.gq[((size_t)a * (L + 1) + l) * C + c] = dq[l];
    }
    if (live && c % P.Ch == 0) {
        s_gp[head][0] = gx;
        s_gp[head][1] = gy;
        s_gp[head][2] = gz;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int c = threadIdx.x;
        float s = 0.0f;
        for (int hh = 0; hh < P.H; ++hh) s += s_gp[hh][c];
        P.gpos[(size_t)a * 3 + c] = -s;
    }
    if (WGRAD) {
        if (live) {
#pragma unroll
            for (int i = 0; i < WB_PER_THREAD; ++i) {
                const int b = c % P.Ch + i * P.Ch;
                if (b < P.B) P.pWb[((size_t)a * P.H + head) * P.B + b] = accWb[i];
            }
        }
    }
}

// Sum of the per-atom partials, one workgroup per output element, in a fixed order.
__global__ __launch_bounds__(256) void k_reduce_partials(const float* __restrict__ part, int N, int stride, int M,
                                                         float* __restrict__ out) {
    __shared__ float s_acc[256];
    const int m = blockIdx.x;
    float s = 0.0f;
    for (int a = threadIdx.x; a < N; a += 256) s += part[(size_t)a * stride + m];
    s_acc[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) s_acc[threadIdx.x] += s_acc[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0 && m < M) out[m] = s_acc[0];
}

// ---- what an atom owns as a source j: dk_j, dv_j and +sum_i dL/dr_ij (added to the target kernel's share); with
// WGRAD also its partial sums of the path-weight gradient.  The message is linear in the path weights,
// G_mu[xo][xi] = w_path[li(xi)][lo(xo)] Gu_mu[xo][xi] with the unit-weight operators Gu, so with the sums
// Y_mu = sum_i alpha_ij r_mu g_i that this kernel forms anyway
//   dL/dw_path[li][lo] = sum_j sum_mu sum_{xo in lo, xi in li} Y_mu[xo] Gu_mu[xo][xi] v_j[xi].
template <int L, typename VT, bool WGRAD, bool TL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_bwd_source(BwdParams P) {
    constexpr int n = (L + 1) * (L + 1);
    __shared__ int s_list[BCAP];
    __shared__ float4 s_pos[BCAP], s_rad[BCAP];
    extern __shared__ float2 s_bias[];   // [BCAP][H]
    __shared__ int s_ctl[2];
    __shared__ float s_G[3 * E2F_MAX_N * E2F_MAX_N];
    __shared__ float s_gp[E2F_MAX_H][3];
    const int t = e2f::xcd_remap(blockIdx.x, P.cv.N), C = P.C;
    if (t < 0) return;
    if (TL && P.lists_hdr[t >> 4].x >= 0) return;   // (whole workgroup) the tile kernels own this atom
    const bool live = (int)threadIdx.x < C;        // workgroups have at least one full wave: the list walk needs it
    const int c = live ? threadIdx.x : 0, head = c / P.Ch;
    const int a = P.cv.perm[t];
    for (int i = threadIdx.x; i < 3 * E2F_MAX_N * E2F_MAX_N; i += blockDim.x) s_G[i] = P.G[i];
    const float4 pj = P.spos[t];   // this atom is the source j of every pair below
    float kv[L + 1], dk[L + 1], vj[n], Y[3][n];
#pragma unroll
    for (int l = 0; l <= L; ++l) {
        kv[l] = load_k<L, TL>(P, t, l, c);
        dk[l] = 0.0f;
    }
#pragma unroll
    for (int x = 0; x < n; ++x) {
        vj[x] = load_v<L, VT, TL>(P, t, x, c);
        Y[0][x] = Y[1][x] = Y[2][x] = 0.0f;
    }
    float gx = 0.0f, gy = 0.0f, gz = 0.0f;   // sum_i dL/dr_ij of this head
    __shared__ e2f::RunList s_run;
    if (threadIdx.x < 64) e2f::fill_runs(s_run, P.cv, t, threadIdx.x);
    int walked = 0;   // (next_batch opens with the barrier that the runs need)
    __syncthreads();
    float Gv[3][n];   // G_mu v_j: u_mu = <g_i, G_mu v_j>
    axis_apply<L, false>(vj, s_G, Gv);
    while (true) {
        const int cnt = next_batch(P, s_run, walked, t, pj, s_list, s_pos, s_rad, s_bias, s_ctl);
        constexpr bool AHEAD = ROWS_AHEAD<L>;
        float qn[L + 1], gn[n], lse_n = 0.0f, Dn_n = 0.0f;   // the rows and statistics of the pair to come
        auto request = [&](int e) {
            const int i = s_list[e], ai = __float_as_int(s_pos[e].w);
#pragma unroll
            for (int l = 0; l <= L; ++l) qn[l] = load_q<L, TL>(P, i, l, c);
#pragma unroll
            for (int x = 0; x < n; ++x) gn[x] = P.gout[((size_t)ai * n + x) * C + c];
            lse_n = load_lse<TL>(P, i, head);
            Dn_n = load_Dn<TL>(P, i, head);
        };
        if (AHEAD && cnt > 0) request(0);
        for (int e = 0; e < cnt; ++e) {
            if (!AHEAD) request(e);
            const float4 pim = s_pos[e];       // the target, seen from j at its image
            const float rx = pj.x - pim.x, ry = pj.y - pim.y, rz = pj.z - pim.z;   // r_ij = pos_j - pos_i
            const float4 rad = s_rad[e];
            const float2 bb = s_bias[e * P.H + head];
            float qv[L + 1], g[n], u[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // the three u_mu, then q k
#pragma unroll
            for (int l = 0; l <= L; ++l) {
                qv[l] = qn[l];
                u[3] += qv[l] * kv[l];
            }
#pragma unroll
            for (int x = 0; x < n; ++x) {
                g[x] = gn[x];
                u[0] += Gv[0][x] * g[x];
                u[1] += Gv[1][x] * g[x];
                u[2] += Gv[2][x] * g[x];
            }
            const float lse = lse_n, Dn = Dn_n;
            if (AHEAD) request(min(e + 1, cnt - 1));
            e2f::group_sums(u, P.Ch);
            const float p = pair_prob<TL>(P, u[3], bb.x, lse);
            const float phi = rad.x, dphi = rad.y;
            const float wsum = rx * u[0] + ry * u[1] + rz * u[2];
            const float ds = p * (phi * wsum - Dn);
            const float alpha = p * phi;
            const float dd = (ds * bb.y + p * wsum * dphi) / rad.z;
#pragma unroll
            for (int l = 0; l <= L; ++l) dk[l] += (TL ? LN2 : P.tau) * ds * qv[l];   // (TL: the q rows carry tau log2 e)
            const float ax = alpha * rx, ay = alpha * ry, az = alpha * rz;
#pragma unroll
            for (int x = 0; x < n; ++x) {
                Y[0][x] += ax * g[x];
                Y[1][x] += ay * g[x];
                Y[2][x] += az * g[x];
            }
            gx += alpha * u[0] + dd * rx;
            gy += alpha * u[1] + dd * ry;
            gz += alpha * u[2] + dd * rz;
        }
        if (s_ctl[1]) break;
    }
    if (live) {
#pragma unroll
        for (int l = 0; l <= L; ++l) P.gk[((size_t)a * (L + 1) + l) * C + c] = dk[l];
    }
    // dv_j = sum_mu G_mu^T Y_mu
    float dv[n];
#pragma unroll
    for (int x = 0; x < n; ++x) dv[x] = 0.0f;
#pragma unroll
    for (int mu = 0; mu < 3; ++mu)
#pragma unroll
        for (int xo = 0; xo < n; ++xo)
#pragma unroll
            for (int xi = 0; xi < n; ++xi)
                if ((E2F_AXIS_NZ[mu][xo] >> xi) & 1u) dv[xi] += s_G[(mu * E2F_MAX_N + xo) * E2F_MAX_N + xi] * Y[mu][xo];
    if (live) {
#pragma unroll
        for (int x = 0; x < n; ++x) P.gv[((size_t)a * n + x) * C + c] = dv[x];
    }
    if (live && c % P.Ch == 0) {
        s_gp[head][0] = gx;
        s_gp[head][1] = gy;
        s_gp[head][2] = gz;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int c = threadIdx.x;
        float s = 0.0f;
        for (int hh = 0; hh < P.H; ++hh) s += s_gp[hh][c];
        P.gpos[(size_t)a * 3 + c] += s;   // the target kernel wrote this atom's other share before
    }
    if (WGRAD) {
        // bins per thread, then summed over the channels in a fixed order
        __syncthreads();
        for (int i = threadIdx.x; i < 3 * E2F_MAX_N * E2F_MAX_N; i += blockDim.x) s_G[i] = P.Gu[i];
        __syncthreads();
        float bins[(L + 1) * (L + 1)], vr[n];   // (the value row is read again: keeping it through the loop costs registers)
#pragma unroll
        for (int i = 0; i < (L + 1) * (L + 1); ++i) bins[i] = 0.0f;
#pragma unroll
        for (int x = 0; x < n; ++x) vr[x] = load_v<L, VT, TL>(P, t, x, c);
#pragma unroll
        for (int mu = 0; mu < 3; ++mu)
#pragma unroll
            for (int xo = 0; xo < n; ++xo)
#pragma unroll
                for (int xi = 0; xi < n; ++xi)
                    if ((E2F_AXIS_NZ[mu][xo] >> xi) & 1u)
                        bins[degree_of(xi) * (L + 1) + degree_of(xo)] +=
                            Y[mu][xo] * s_G[(mu * E2F_MAX_N + xo) * E2F_MAX_N + xi] * vr[xi];
        float* s_red = reinterpret_cast<float*>(s_bias);   // [(L+1)^2][C]: the list batches are done
        if (live) {
#pragma unroll
            for (int i = 0; i < (L + 1) * (L + 1); ++i) s_red[i * C + c] = bins[i];
        }
        __syncthreads();
        if ((int)threadIdx.x < WP_BINS) {
            float s = 0.0f;
            if ((int)threadIdx.x < (L + 1) * (L + 1))
                for (int cc = 0; cc < C; ++cc) s += s_red[threadIdx.x * C + cc];
            P.pwp[(size_t)a * WP_BINS + threadIdx.x] = s;
        }
    }
}

template <int L, typename VT>
void launch_LV(const BwdParams& P, hipStream_t st) {
    const int N = P.cv.N, C = P.C < 64 ? 64 : P.C;
    const size_t shm = (size_t)BCAP * P.H * sizeof(float2);
    // with weight gradients the same bytes later hold the [(L+1)^2][C] channel sums of the path-weight bins
    const size_t shm_w = shm > (size_t)(L + 1) * (L + 1) * P.C * 4 ? shm : (size_t)(L + 1) * (L + 1) * P.C * 4;
    k_bwd_stats<L, false><<<e2f::xcd_grid(N), C, shm, st>>>(P);
    if (P.pWb) {
        k_bwd_target<L, VT, true, false><<<e2f::xcd_grid(N), C, shm, st>>>(P);
        k_bwd_source<L, VT, true, false><<<e2f::xcd_grid(N), C, shm_w, st>>>(P);
    } else {
        k_bwd_target<L, VT, false, false><<<e2f::xcd_grid(N), C, shm, st>>>(P);
        k_bwd_source<L, VT, false, false><<<e2f::xcd_grid(N), C, shm, st>>>(P);
    }
}

// The per-atom kernels over the tile layouts, for the atoms of crowded tiles only (every other workgroup leaves at
// once).  `what` 0: the statistics, which the tile kernels of the other tiles read too; 1: the pair kernels.
template <int L>
void launch_crowded(const BwdParams& P, int what, hipStream_t st) {
    const int N = P.cv.N, C = P.C < 64 ? 64 : P.C;
    const size_t shm = (size_t)BCAP * P.H * sizeof(float2);
    const size_t shm_w = shm > (size_t)(L + 1) * (L + 1) * P.C * 4 ? shm : (size_t)(L + 1) * (L + 1) * P.C * 4;
    if (what == 0) {
        k_bwd_stats<L, true><<<e2f::xcd_grid(N), C, shm, st>>>(P);
    } else if (P.pWb) {   // with the per-atom partial sums of the weight gradients
        k_bwd_target<L, uint16_t, true, true><<<e2f::xcd_grid(N), C, shm, st>>>(P);
        k_bwd_source<L, uint16_t, true, true><<<e2f::xcd_grid(N), C, shm_w, st>>>(P);
    } else {
        k_bwd_target<L, uint16_t, false, true><<<e2f::xcd_grid(N), C, shm, st>>>(P);
        k_bwd_source<L, uint16_t, false, true><<<e2f::xcd_grid(N), C, shm, st>>>(P);
    }
}

template <int L>
void launch_L(const e2f_ctx* ctx, const BwdParams& P, hipStream_t st) {
    if (ctx->cfg.feat_dtype == E2F_BF16) launch_LV<L, uint16_t>(P, st);
    else launch_LV<L, float>(P, st);
}

}  // namespace

bool e2f_backward_supported(const e2f_ctx* ctx) {
    const int Ch = ctx->Ch;
    return ctx->cfg.lf == 1 && ctx->cfg.L_max >= 1 && Ch <= 64 && (Ch & (Ch - 1)) == 0 && ctx->cfg.C <= 256;
}

e2f_status e2f_launch_backward(const e2f_ctx* ctx, const E2fCellsView& cv, const e2f_weights* w, const E2fAttnWs& ws,
                               const E2fBwdWs& bw, const float* out, const float* grad_out, float* grad_pos,
                               float* grad_q, float* grad_k, float* grad_v, const void* h, float* grad_h,
                               float* grad_Wb, float* grad_w_path, float* grad_W, const E2fBwdTileWs* tw,
                               hipStream_t st, bool lists_ready) {
    if (cv.N == 0) return E2F_OK;
    const bool wgrad = grad_Wb || grad_w_path;
    if (wgrad && ctx->cfg.B > WB_PER_THREAD * ctx->Ch) return E2F_ERR_UNSUPPORTED;
    if (tw && wgrad && !e2f_backward_tile_weight_gradients_supported(ctx)) return E2F_ERR_INVALID_ARG;
    BwdParams P;
    P.cv = cv;
    P.spos = ws.spos; P.q = ws.q; P.k = ws.k; P.v = ws.v; P.G = tw ? ws.G : bw.G; P.Wb = w->Wb;
    P.out = out; P.gout = grad_out; P.lse = bw.lse; P.Dn = bw.Dn;
    P.gpos = grad_pos; P.gq = grad_q; P.gk = grad_k; P.gv = grad_v;
    P.q16 = ws.q16; P.k16 = ws.k16; P.v4 = ws.v4;
    P.stat4 = tw ? reinterpret_cast<float2*>(tw->stat4) : nullptr;
    P.lists_hdr = ws.lists_hdr;
    P.C = ctx->cfg.C; P.H = ctx->cfg.H; P.B = ctx->cfg.B; P.Ch = ctx->Ch;
    P.tau = ctx->tau; P.rc2 = ctx->rc2; P.cutoff = ctx->cfg.cutoff; P.rbf_step = ctx->rbf_step; P.rbf_gamma = ctx->rbf_gamma;
    P.Gu = nullptr; P.pWb = nullptr; P.pwp = nullptr;
    e2f_status rc;
    // the axis operators that no earlier launch has left: those of the per-atom kernels without a tile form, and those
    // with unit path weights (full form for the per-atom kernels, packed for the tile kernels)
    if ((wgrad || !tw) && (rc = e2f_launch_axis_operators(ctx, w->w_path, tw ? nullptr : bw.G, wgrad ? bw.Gu : nullptr,
                                                          wgrad && tw ? tw->Gu : nullptr, st)) != E2F_OK)
        return rc;
    if (wgrad) {
        P.Gu = bw.Gu; P.pWb = bw.pWb; P.pwp = bw.pwp;
    }
    if (tw) {
        // pair work on the matrix cores, tile by tile; the atoms of crowded tiles (lists that do not fit) go through
        // the per-atom kernels, which read the same layouts and statistics
        if (!lists_ready && (rc = e2f_launch_tile_lists(ctx, cv, ws, st)) != E2F_OK) return rc;
        auto crowded = [&](int what) {
            switch (ctx->cfg.L_max) {
                case 1: launch_crowded<1>(P, what, st); break;
                case 2: launch_crowded<2>(P, what, st); break;
                case 3: launch_crowded<3>(P, what, st); break;
                default: launch_crowded<4>(P, what, st); break;
            }
        };
        crowded(0);
        if ((rc = e2f_launch_backward_tile(ctx, cv, ws, *tw, out, grad_out, grad_pos, grad_q, grad_k, grad_v, wgrad, st)) != E2F_OK)
            return rc;
        crowded(1);
        if (wgrad && (rc = e2f_launch_backward_tile_wsum(ctx, cv, ws, *tw, bw.pWb, bw.pwp, grad_Wb, grad_w_path, st)) != E2F_OK)
            return rc;
    }
    if (!tw) switch (ctx->cfg.L_max) {
        case 1: launch_L<1>(ctx, P, st); break;
        case 2: launch_L<2>(ctx, P, st); break;
        case 3: launch_L<3>(ctx, P, st); break;
        case 4: launch_L<4>(ctx, P, st); break;
        default: return E2F_ERR_UNSUPPORTED;
    }
    if (wgrad && !tw) {
        const int L1 = ctx->cfg.L_max + 1, HB = ctx->cfg.H * ctx->cfg.B;
        if (grad_Wb) k_reduce_partials<<<HB, 256, 0, st>>>(bw.pWb, cv.N, HB, HB, grad_Wb);
        if (grad_w_path) k_reduce_partials<<<L1 * L1, 256, 0, st>>>(bw.pwp, cv.N, WP_BINS, L1 * L1, grad_w_path);
    }
    if (grad_h || grad_W) {
        rc = e2f_launch_backward_maps(ctx, cv.N, w, h, grad_q, grad_k, grad_v, grad_h, grad_W, bw, st);
        if (rc != E2F_OK) return rc;
    }
    E2F_HIP_CHECK(hipGetLastError());
    return E2F_OK;
}
