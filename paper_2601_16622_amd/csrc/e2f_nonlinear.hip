// Fused on-the-fly attention with the non-linear pair feature in the logit (App. "Role of Non-linearity",
// Eqs. app-nonlin-fea and app-nonlin-alpha).  The reading built here: with Y^(l) the real harmonics of the unit pair
// vector, Q = W_Q1 h_i (the target's first query projection, all components) and V = W_V h_j,
//     a[l][c] = sum_m Q[l,m,c] Y^(l)_m ,   b[l][c] = sum_m V[l,m,c] Y^(l)_m          (invariants, degree by degree)
//     Fea     = sigma(a || b),  sigma(x) = x / (1 + e^-x)
//     s_ij,h  = tau sum_{l, c in h} q_i[l][c] k_j[l][c] (sigma(a[l][c]) + sigma(b[l][c])) + b_h(d_ij)
// and everything after the logit as in Algorithm 1 (softmax over the neighbours, gate outside, EAAS message).
//
// One workgroup per target atom, one thread per channel (one or more waves; every wave walks the stencil and reads the
// pair geometry that the first lanes of each wave build, identically), like the ALU form of the fused call.  The
// harmonics of the pair direction cost nothing extra: R_ij takes the pair direction to +z, so Y^(l)(r/|r|) is the
// m = 0 row of the block D^(l)(R_ij) that the message needs anyway.  The value row of a neighbour is read once and
// serves the feature and the message; the softmax is online per pair (Algorithm 1 as printed).
#include <limits.h>
#include <stdlib.h>

#include "e2f_tile_shared.h"

namespace {

struct NlParams {
    E2fCellsView cv;
    const float4* spos;
    const float* q;
    const float* k;
    const void* v;
    const void* q1;   // [N][n][C] sorted order, same type as v: W_Q1 h
    const float* cw;
    const float* Wb;
    float* out;
    int C, H, B, Ch;
    float tau, rc2, cutoff, rbf_step, rbf_gamma;
};

constexpr int PB = 16;    // pairs per chunk
constexpr int CAP = 192;  // capacity of the neighbour list in LDS
constexpr int RUN_SHIFT = 26;   // a list entry is slot | run << 26; the launcher checks N < 2^26

__device__ __forceinline__ float silu(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

template <int L, int LF, typename VT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_fused_nonlinear(NlParams P) {
    constexpr int CPL = 1;
    constexpr int n = (L + 1) * (L + 1);
    constexpr int DS = e2f::d_offset(L + 1);
    constexpr int DSP = (DS + 3) & ~3;
    __shared__ int s_list[CAP];
    __shared__ __attribute__((aligned(16))) float s_D[PB * DSP];
    __shared__ float s_bias[PB * E2F_MAX_H];
    __shared__ float s_wgt[PB];

    const int t = e2f::xcd_remap(blockIdx.x, P.cv.N), lane = threadIdx.x & 63;
    if (t < 0) return;  // padding block of the XCD map (whole workgroup)
    const int C = P.C, H = P.H;
    const bool active = (int)threadIdx.x < C;
    const int c0 = active ? threadIdx.x : 0;  // idle lanes shadow channel 0's loads and store nothing
    const int head = c0 / P.Ch;
    const int lanes_per_head = P.Ch;
    const float4 pi = P.spos[t];

    float q[L + 1][CPL];
#pragma unroll
    for (int l = 0; l <= L; ++l)
#pragma unroll
        for (int u = 0; u < CPL; ++u) q[l][u] = P.q[((size_t)t * (L + 1) + l) * C + c0 + u];
    // the target's query components: in LDS (component-major), not in registers, where they would sit beside the
    // accumulators, the value row and its rotated copy
    extern __shared__ float s_q1[];   // [n][threads]
    const int nthreads = blockDim.x;
#pragma unroll
    for (int x = 0; x < n; ++x)
        s_q1[x * nthreads + threadIdx.x] = e2f::load_as_float((const VT*)P.q1 + ((size_t)t * n + x) * C + c0);

    float A[n][CPL];
#pragma unroll
    for (int x = 0; x < n; ++x)
#pragma unroll
        for (int u = 0; u < CPL; ++u) A[x][u] = 0.0f;
    float mu = -INFINITY, z = 0.0f;

    __shared__ e2f::RunList s_run;   // (serves open boundaries too: the extra runs are empty, the translations zero)
    if (threadIdx.x < 64) e2f::fill_runs(s_run, P.cv, t, lane);
    __syncthreads();
    const int total = s_run.total();
    int base = 0;
    while (true) {
        // ---- fill the list
        int cnt = 0;
        while (base < total && cnt + 64 <= CAP) {
            bool ok = false;
            int j = 0, run = 0;
            if (base + lane < total) {
                s_run.candidate(base + lane, run, j);
                const float4 pj = P.spos[j], sh = s_run.sh[run];
                const float d2 = e2f::dist2_exact(pi.x, pi.y, pi.z, pj.x + sh.x, pj.y + sh.y, pj.z + sh.z);
                ok = j != t && e2f::is_neighbor(d2, P.rc2);
            }
            const unsigned long long mask = __ballot(ok);
            if (ok) s_list[cnt + __popcll(mask & ((1ull << lane) - 1ull))] = j | (run << RUN_SHIFT);
            cnt += __popcll(mask);
            base += 64;
        }
        __syncthreads();
        // ---- consume it
        for (int p0 = 0; p0 < cnt; p0 += PB) {
            const int np = min(PB, cnt - p0);
            if (lane < np) {
                const int e = s_list[p0 + lane], j = e & ((1 << RUN_SHIFT) - 1), run = e >> RUN_SHIFT;
                const float4 pj = P.spos[j], sh = s_run.sh[run];
                const float dx = (pj.x + sh.x) - pi.x, dy = (pj.y + sh.y) - pi.y;
                const float dz = (pj.z + sh.z) - pi.z;
                const float d = sqrtf(dx * dx + dy * dy + dz * dz);
                e2f::align_D<L>(dx, dy, dz, d, s_D + lane * DSP);   // also for LF = 0: the feature needs Y
                for (int hh = 0; hh < H; ++hh) {
                    float acc = 0.0f;
                    for (int b = 0; b < P.B; ++b) acc += P.Wb[hh * P.B + b] * e2f::radial_basis(d, b, P.rbf_step, P.rbf_gamma);
                    s_bias[lane * E2F_MAX_H + hh] = acc;
                }
                s_wgt[lane] = e2f::radial_gate(d, P.cutoff) * e2f::pow_lf<LF>(d);
            }
            __syncthreads();
#pragma unroll 1
            for (int p = 0; p < np; ++p) {
                const int j = s_list[p0 + p] & ((1 << RUN_SHIFT) - 1);
                const VT* vj = (const VT*)P.v + (size_t)j * n * C + c0;
                const float* kj = P.k + (size_t)j * (L + 1) * C + c0;
                const float* Dp = s_D + p * DSP;
                float vin[n][CPL];
#pragma unroll
                for (int x = 0; x < n; ++x)
#pragma unroll
                    for (int u = 0; u < CPL; ++u) vin[x][u] = e2f::load_as_float(vj + x * C + u);
                // logit with the pair feature: Y^(l)_m = D^(l)[m = 0][m]
                float dot = 0.0f;
#pragma unroll
                for (int l = 0; l <= L; ++l) {
                    float a[CPL], b[CPL];
#pragma unroll
                    for (int u = 0; u < CPL; ++u) a[u] = b[u] = 0.0f;
#pragma unroll
                    for (int m = 0; m < 2 * l + 1; ++m) {
                        const float y = Dp[e2f::d_offset(l) + l * (2 * l + 1) + m];
#pragma unroll
                        for (int u = 0; u < CPL; ++u) {
                            a[u] += s_q1[(l * l + m) * nthreads + threadIdx.x] * y;
                            b[u] += vin[l * l + m][u] * y;
                        }
                    }
#pragma unroll
                    for (int u = 0; u < CPL; ++u) dot += q[l][u] * kj[l * C + u] * (silu(a[u]) + silu(b[u]));
                }
                for (int off = 1; off < lanes_per_head; off <<= 1) dot += __shfl_xor(dot, off);
                const float s = dot * P.tau + s_bias[p * E2F_MAX_H + head];
                // the recurrences of Algorithm 1
                const float mu_new = fmaxf(mu, s);
                const float scale = __expf(mu - mu_new);   // 0 for the first neighbour (mu = -inf)
                const float pe = __expf(s - mu_new);
                z = z * scale + pe;
#pragma unroll
                for (int x = 0; x < n; ++x)
#pragma unroll
                    for (int u = 0; u < CPL; ++u) A[x][u] *= scale;
                mu = mu_new;
                e2f::eaas_accumulate<L, LF, CPL>(vin, Dp, P.cw, pe * s_wgt[p], A);
            }
            __syncthreads();
        }
        if (base >= total) break;
    }

    if (active) {
        const float inv = z > 0.0f ? 1.0f / z : 0.0f;
        float* o = P.out + (size_t)P.cv.perm[t] * n * C + c0;
#pragma unroll
        for (int x = 0; x < n; ++x)
#pragma unroll
            for (int u = 0; u < CPL; ++u) o[x * C + u] = A[x][u] * inv;
    }
}

// ---- degree-1 filter, bf16 features, heads of 16 channels: one wave per (target, head) on the matrix cores.
//
// Vector work and waits: a pair costs every channel 2 (L + 1) sigma's, each an exponential and a reciprocal at a quarter of the
// rate, and the products around them (vector ALUs active 51 % of the SIMD cycles), and a wave waits 44 % of its cycles, mostly
// for the rows of the pairs it is about to use.  What the kernel above spends beside that goes to the matrix cores:
//   a       the target's feature is a product over its own rows, [pairs] x (2l+1) times (2l+1) x [channels] per degree
//   message linear in the pair vector, so T_mu += w_ij (r_ij)_mu v_j, three rows against the value rows, and the axis
//           operators G_mu = D(R_mu)^T P D(R_mu) once per target in place of two rotations per pair
// Neither loses bits: the 32-bit operand (harmonics, weights) is cut into three 8-bit significands that lie side by side
// along the product's unused rows (3 axes x 3 parts of 16) or its unused depth (3 x (2l+1) <= 27 of 32); the other
// operand is bf16 in memory.  A wave takes 16 pairs at a time, lane = (channel, 4 pairs).
// Value rows as k_nonlinear_rows leaves them, so that a lane fetches 8 components of its channel with one 16-byte load.
// Measured at 4 000 atoms, L = 4, 128 channels, 60 neighbours: whole call 1 250 us with the kernel above (1 084 in it), 571
// with this one; 256 registers, two waves per SIMD, the value rows of one group of 16 pairs in flight.
typedef short s16x4 __attribute__((ext_vector_type(4)));
constexpr int HB = 64;          // pairs per batch of geometry
constexpr int HLIST = 512;      // neighbours listed before they are consumed (a pass of the list adds up to 256)

// Harmonics of degree l of the pair direction: the m = 0 row of the block D^(l) of the aligning rotation, times `scale`.
template <int l>
__device__ __forceinline__ void harmonics(float ct, float st, float cp, float sp, float scale, float (&Y)[2 * l + 1]) {
    constexpr int nl = 2 * l + 1;
    float ck[E2F_MAX_L + 1], sk[E2F_MAX_L + 1], cm[E2F_MAX_L + 1], sm[E2F_MAX_L + 1], dl[nl * nl];
    ck[0] = cm[0] = 1.0f;
    sk[0] = sm[0] = 0.0f;
#pragma unroll
    for (int k = 1; k <= l; ++k) {
        ck[k] = ck[k - 1] * ct - sk[k - 1] * st;
        sk[k] = sk[k - 1] * ct + ck[k - 1] * st;
        cm[k] = cm[k - 1] * cp - sm[k - 1] * sp;
        sm[k] = sm[k - 1] * cp + cm[k - 1] * sp;
    }
    e2f::delta_align<l>(ck, sk, dl);
    Y[l] = dl[l * nl + l] * scale;
#pragma unroll
    for (int m = 1; m <= l; ++m) {
        Y[l + m] = dl[l * nl + l + m] * cm[m] * scale;
        Y[l - m] = dl[l * nl + l + m] * sm[m] * scale;
    }
}

// x = part 0 + part 1 + part 2 exactly, 8 significant bits each: the upper halves of the three words
__device__ __forceinline__ void split3(float x, uint32_t (&p)[3]) {
    p[0] = __float_as_uint(x);
    const float r1 = x - __uint_as_float(p[0] & 0xffff0000u);
    p[1] = __float_as_uint(r1);
    p[2] = __float_as_uint(r1 - __uint_as_float(p[1] & 0xffff0000u));
}
__device__ __forceinline__ uint32_t high_halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
__device__ __forceinline__ uint32_t low_halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x05040100u); }

// Degree l of a pair's geometry into LDS: the harmonics [component][pair], and their parts as a row of the product's
// left operand, depth index part * (2l + 1) + m.
template <int l>
__device__ __forceinline__ void store_degree(float ct, float st, float cp, float sp, int lane, float* s_Y, uint16_t* s_A) {
    constexpr int nl = 2 * l + 1;
    float Y[nl];
    harmonics<l>(ct, st, cp, sp, -1.44269504088896341f, Y);
    uint32_t part[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) part[k] = 0u;
#pragma unroll
    for (int m = 0; m < nl; ++m) {
        s_Y[(l * l - 1 + m) * HB + lane] = Y[m];
        uint32_t p[3];
        split3(Y[m], p);
#pragma unroll
        for (int s = 0; s < 3; ++s) part[s * nl + m] = p[s];
    }
    u32x4* row = reinterpret_cast<u32x4*>(s_A + ((l - 1) * HB + lane) * 32);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        u32x4 w;
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = high_halves(part[8 * q + 2 * i], part[8 * q + 2 * i + 1]);
        row[q] = w;
    }
}

// sigma from y = -x log2 e, without the factor -ln 2
__device__ __forceinline__ float sigma_scaled(float y) { return y * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(y)); }

template <int L>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_nonlinear_heads(NlParams P, const float* w_path,
                                                                                                    AxisTable tab) {
    constexpr int n = (L + 1) * (L + 1), ND = (n + 1) / 2, OCT = n / 8, REM = n % 8;
    static_assert(REM == 0 || REM == 1 || REM == 4, "the tail of a value row is a 2-byte or an 8-byte load");
    static_assert(L >= 1 && L <= 4, "a wave per degree, and a degree-1 filter needs one");
    __shared__ int s_list[HLIST];
    __shared__ int s_wcnt[4];
    __shared__ e2f::RunList s_run;
    __shared__ __attribute__((aligned(16))) int s_slot[HB];
    __shared__ __attribute__((aligned(16))) float s_Y[(n - 1) * HB];
    __shared__ __attribute__((aligned(16))) uint16_t s_A[L * HB * 32];
    __shared__ __attribute__((aligned(16))) float s_bias[4 * HB], s_wr[4 * HB];   // s_wr: gate times the pair vector, then zeros
    __shared__ float s_G[AXIS_NNZ];

    int t, hg;
    if (!tile_xcd_remap(blockIdx.x, P.cv.N, e2f::XCD_CHUNK, (P.H + 3) / 4, t, hg)) return;   // whole workgroup
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, tn = lane & 15, g = lane >> 4;
    const int C = P.C, H = P.H, head = hg * 4 + wave;
    const bool have = head < H;   // (whole wave) a head for this wave; without one it still shares the list and geometry
    const int hd = have ? head : 0, c0 = hd * 16 + tn;
    const float4 pi = P.spos[t];
    if (wave == 0) e2f::fill_runs(s_run, P.cv, t, lane);
    if (tid < AXIS_NNZ) s_G[tid] = axis_entry(tab, w_path, L, tid);
    s_wr[3 * HB + lane] = 0.0f;
    // the head's invariant query (times -tau: base-2 logits from sigma's without their -ln 2), and the target's rows of
    // W_Q1 h as right operands, repeated for the three parts of the harmonics
    float q[L + 1];
#pragma unroll
    for (int l = 0; l <= L; ++l) q[l] = P.q[((size_t)t * (L + 1) + l) * C + c0] * -P.tau;
    const uint16_t* q1 = (const uint16_t*)P.q1 + (size_t)t * n * C + c0;
    u32x4 bq[L];
#pragma unroll
    for (int l = 1; l <= L; ++l) {
        const int nl = 2 * l + 1;
        uint32_t u[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int k = 8 * g + i;
            const uint32_t val = q1[(size_t)(l * l + k % nl) * C];
            u[i] = k < 3 * nl ? val : 0u;
        }
        bq[l - 1] = (u32x4){u[0] | (u[1] << 16), u[2] | (u[3] << 16), u[4] | (u[5] << 16), u[6] | (u[7] << 16)};
    }
    const float a0 = sigma_scaled(e2f::bf16_bits_to_float(q1[0]) * -1.44269504088896341f);
    // this lane's row of the weights: axis tn & 3, part tn >> 2
    const uint32_t cut1 = tn >= 4 ? 0xffff0000u : 0u, cut2 = tn >= 8 ? 0xffff0000u : 0u;
    const float* wrow = s_wr + (tn >= 12 ? 3 : tn & 3) * HB;

    f32x4 T[n];
#pragma unroll
    for (int x = 0; x < n; ++x) T[x] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m = -1.0e30f, z = 0.0f;   // reference of the softmax (finite), moved when a logit exceeds it by M_STEP

    __syncthreads();
    const int total = s_run.total();
    int base = 0;
    while (base < total) {
        // ---- list: one candidate of the 27 cells per thread, kept ones in order
        int cnt = 0;
        while (base < total && cnt + 256 <= HLIST) {
            const int c = base + tid;
            bool ok = false;
            int j = 0, run = 0;
            if (c < total) {
                s_run.candidate(c, run, j);
                const float4 pj = P.spos[j], sh = s_run.sh[run];
                const float d2 = e2f::dist2_exact(pi.x, pi.y, pi.z, pj.x + sh.x, pj.y + sh.y, pj.z + sh.z);
                ok = j != t && e2f::is_neighbor(d2, P.rc2);
            }
            const unsigned long long mask = __ballot(ok);
            if (lane == 0) s_wcnt[wave] = __popcll(mask);
            __syncthreads();
            int off = cnt;
            for (int w = 0; w < 4; ++w) {
                off += w < wave ? s_wcnt[w] : 0;
                cnt += s_wcnt[w];
            }
            if (ok) s_list[off + __popcll(mask & ((1ull << lane) - 1ull))] = j | (run << RUN_SHIFT);
            base += 256;
            __syncthreads();
        }
        // ---- consume it, a batch of 64 pairs at a time
        for (int p0 = 0; p0 < cnt; p0 += HB) {
            const int np = min(HB, cnt - p0);
            {   // geometry: lane = pair, wave = degree and head; what lies behind the last pair repeats it with weight 0
                const int e = s_list[p0 + min(lane, np - 1)], j = e & ((1 << RUN_SHIFT) - 1);
                const float4 pj = P.spos[j], sh = s_run.sh[e >> RUN_SHIFT];
                const float dx = (pj.x + sh.x) - pi.x, dy = (pj.y + sh.y) - pi.y, dz = (pj.z + sh.z) - pi.z;
                const float d = sqrtf(dx * dx + dy * dy + dz * dz);
                const float inv = __builtin_amdgcn_rcpf(d), rho = __builtin_amdgcn_sqrtf(dx * dx + dy * dy);
                const float ct = dz * inv, st = rho * inv, ir = __builtin_amdgcn_rcpf(rho);
                const float cp = rho > 0.0f ? dx * ir : 1.0f, sp = rho > 0.0f ? dy * ir : 0.0f;
                const bool real = lane < np;
                if (wave == 0) {
                    store_degree<1>(ct, st, cp, sp, lane, s_Y, s_A);
                    const float gate = real ? e2f::radial_gate(d, P.cutoff) : 0.0f;
                    s_slot[lane] = j;
                    s_wr[lane] = gate * dx;
                    s_wr[HB + lane] = gate * dy;
                    s_wr[2 * HB + lane] = gate * dz;
                }
                if constexpr (L >= 2)
                    if (wave == 1) store_degree<2>(ct, st, cp, sp, lane, s_Y, s_A);
                if constexpr (L >= 3)
                    if (wave == 2) store_degree<3>(ct, st, cp, sp, lane, s_Y, s_A);
                if constexpr (L >= 4)
                    if (wave == 3) store_degree<4>(ct, st, cp, sp, lane, s_Y, s_A);
                float acc = 0.0f;
                for (int b = 0; b < P.B; ++b) acc += P.Wb[hd * P.B + b] * e2f::radial_basis(d, b, P.rbf_step, P.rbf_gamma);
                s_bias[wave * HB + lane] = real ? acc * 1.44269504088896341f : -INFINITY;
            }
            __syncthreads();
            if (have) {
#pragma unroll 1
                for (int p = 0; p < np; p += 16) {
                    const int at = p + 4 * g;   // this lane's four pairs
                    const int4 j4 = *reinterpret_cast<const int4*>(s_slot + at);
                    const int js[4] = {j4.x, j4.y, j4.z, j4.w};
                    uint32_t V[4][ND];
                    float kk[4][L + 1];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const uint16_t* vj = (const uint16_t*)P.v + ((size_t)js[r] * H + hd) * (n * 16);
#pragma unroll
                        for (int o = 0; o < OCT; ++o) {
                            const u32x4 w = *reinterpret_cast<const u32x4*>(vj + o * 128 + tn * 8);
#pragma unroll
                            for (int i = 0; i < 4; ++i) V[r][4 * o + i] = w[i];
                        }
                        if constexpr (REM == 4) {
                            const u32x2 w = *reinterpret_cast<const u32x2*>(vj + OCT * 128 + tn * 4);
                            V[r][4 * OCT] = w[0];
                            V[r][4 * OCT + 1] = w[1];
                        }
                        if constexpr (REM == 1) V[r][4 * OCT] = vj[OCT * 128 + tn];
#pragma unroll
                        for (int l = 0; l <= L; ++l) kk[r][l] = P.k[((size_t)js[r] * (L + 1) + l) * C + c0];
                    }
                    f32x4 dot;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float b = __uint_as_float(V[r][0] << 16) * -1.44269504088896341f;
                        dot[r] = q[0] * kk[r][0] * (a0 + sigma_scaled(b));
                    }
#pragma unroll
                    for (int l = 1; l <= L; ++l) {
                        const u32x4 ya = *reinterpret_cast<const u32x4*>(s_A + ((l - 1) * HB + p + tn) * 32 + 8 * g);
                        const f32x4 a = mfma(__builtin_bit_cast(bf16x8, ya), __builtin_bit_cast(bf16x8, bq[l - 1]),
                                             (f32x4){0.f, 0.f, 0.f, 0.f});
                        f32x4 b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int mm = 0; mm < 2 * l + 1; ++mm) {
                            const int x = l * l + mm;
                            const f32x4 y = *reinterpret_cast<const f32x4*>(s_Y + (x - 1) * HB + at);
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                b[r] += __uint_as_float((x & 1) ? V[r][x >> 1] & 0xffff0000u : V[r][x >> 1] << 16) * y[r];
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r) dot[r] += q[l] * kk[r][l] * (sigma_scaled(a[r]) + sigma_scaled(b[r]));
                    }
                    const f32x4 bias = *reinterpret_cast<const f32x4*>(s_bias + wave * HB + at);
                    float s[4], top;
#pragma unroll
                    for (int r = 0; r < 4; ++r) s[r] = dot[r];
                    e2f::group_sums(s, 16);
#pragma unroll
                    for (int r = 0; r < 4; ++r) s[r] += bias[r];
                    top = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
                    top = fmaxf(top, __shfl_xor(top, 16));
                    top = fmaxf(top, __shfl_xor(top, 32));
                    if (__any(top > m + M_STEP)) {   // (the same in every lane)
                        const float f = __builtin_amdgcn_exp2f(m - top);   // 0 for the first neighbours
                        z *= f;
#pragma unroll
                        for (int x = 0; x < n; ++x) T[x] *= f;
                        m = top;
                    }
                    const f32x4 wr = *reinterpret_cast<const f32x4*>(wrow + at);
                    uint32_t w[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float pe = __builtin_amdgcn_exp2f(s[r] - m);
                        z += pe;
                        const float w0 = pe * wr[r], w1 = w0 - __uint_as_float(__float_as_uint(w0) & cut1);
                        w[r] = __float_as_uint(w1 - __uint_as_float(__float_as_uint(w1) & cut2));
                    }
                    const s16x4 wa = __builtin_bit_cast(s16x4, (u32x2){high_halves(w[0], w[1]), high_halves(w[2], w[3])});
#pragma unroll
                    for (int x = 0; x < n; ++x) {
                        const u32x2 vb = (x & 1) ? (u32x2){high_halves(V[0][x >> 1], V[1][x >> 1]), high_halves(V[2][x >> 1], V[3][x >> 1])}
                                                 : (u32x2){low_halves(V[0][x >> 1], V[1][x >> 1]), low_halves(V[2][x >> 1], V[3][x >> 1])};
                        T[x] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wa, __builtin_bit_cast(s16x4, vb), T[x], 0, 0, 0);
                    }
                }
            }
            __syncthreads();   // the next batch or list overwrites what this one read
        }
    }

    if (have) {
        // lane (g, channel) holds part g of T_mu in element mu: the operators on the parts, then the sum over the parts
        z += __shfl_xor(z, 16);
        z += __shfl_xor(z, 32);
        const float inv = z > 0.0f ? 1.0f / z : 0.0f;
        float* o = P.out + (size_t)P.cv.perm[t] * n * C + c0;
#pragma unroll
        for (int xo = 0; xo < n; ++xo) {
            float v = 0.0f;
#pragma unroll
            for (int mu = 0; mu < 3; ++mu)
#pragma unroll
                for (int xi = 0; xi < n; ++xi)
                    if ((E2F_AXIS_NZ[mu][xo] >> xi) & 1u) v += s_G[AXIS_INDEX.v[mu][xo][xi]] * T[xi][mu];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (g == (xo & 3)) o[xo * C] = v * inv;
        }
    }
}

// Value rows from the plain layout [component][channel] into the one that k_nonlinear_heads reads, in place: per head n * 16
// bf16 in blocks of eight components, [16 channels][8], then the n % 8 components left over as [16 channels][n % 8].  A
// workgroup reads its slot's row whole before it writes it.
template <int L>
__global__ __launch_bounds__(256) void k_nonlinear_rows(uint16_t* v, int C) {
    constexpr int n = (L + 1) * (L + 1), OCT = n / 8, REM = n % 8;
    extern __shared__ __attribute__((aligned(16))) uint16_t s_row[];
    uint16_t* row = v + (size_t)blockIdx.x * n * C;
    for (int i = threadIdx.x; i < n * C / 8; i += 256)
        reinterpret_cast<u32x4*>(s_row)[i] = reinterpret_cast<const u32x4*>(row)[i];
    __syncthreads();
    if constexpr (OCT > 0)
        for (int i = threadIdx.x; i < C * OCT; i += 256) {   // (head, block, channel)
            const int ch = i & 15, head = (i >> 4) / OCT, o = (i >> 4) % OCT;
            const uint16_t* src = s_row + 8 * o * C + head * 16 + ch;
            u32x4 w;
#pragma unroll
            for (int u = 0; u < 4; ++u) w[u] = src[2 * u * C] | ((uint32_t)src[(2 * u + 1) * C] << 16);
            *reinterpret_cast<u32x4*>(row + head * (n * 16) + o * 128 + ch * 8) = w;
        }
    if constexpr (REM > 0)
        for (int i = threadIdx.x; i < C; i += 256)
#pragma unroll
            for (int u = 0; u < REM; ++u)
                row[(i >> 4) * (n * 16) + OCT * 128 + (i & 15) * REM + u] = s_row[(8 * OCT + u) * C + i];
}

template <int L>
void launch_heads(const e2f_ctx* ctx, const NlParams& P, const float* w_path, hipStream_t st) {
    k_nonlinear_rows<L><<<P.cv.N, 256, (size_t)ctx->n * P.C * 2, st>>>((uint16_t*)P.v, P.C);
    k_nonlinear_heads<L><<<tile_grid(P.cv.N, e2f::XCD_CHUNK, (P.H + 3) / 4), 256, 0, st>>>(P, w_path, axis_table(ctx));
}

template <int L, int LF>
bool launch_dtype(const e2f_ctx* ctx, const NlParams& P, hipStream_t st) {
    const int grid = e2f::xcd_grid(P.cv.N), threads = (P.C + 63) / 64 * 64;
    const size_t shm = (size_t)(L + 1) * (L + 1) * threads * sizeof(float);
    if (ctx->cfg.feat_dtype == E2F_BF16)
        k_fused_nonlinear<L, LF, uint16_t><<<grid, threads, shm, st>>>(P);
    else
        k_fused_nonlinear<L, LF, float><<<grid, threads, shm, st>>>(P);
    return true;
}

template <int L>
bool launch_lf(const e2f_ctx* ctx, const NlParams& P, hipStream_t st) {
    switch (ctx->cfg.lf) {
        case 0: return launch_dtype<L, 0>(ctx, P, st);
        case 1: return launch_dtype<L, 1>(ctx, P, st);
        case 2: return launch_dtype<L, 2>(ctx, P, st);
    }
    return false;
}

}  // namespace

// A head's channels sit in one wave (the logit is reduced by a butterfly over them); at most four waves per target.
bool e2f_nonlinear_supported(const e2f_ctx* ctx) {
    const int Ch = ctx->Ch;
    return ctx->cfg.C <= 256 && Ch <= 64 && (Ch & (Ch - 1)) == 0;
}

// bf16 features in heads of 16 channels under a degree-1 filter take the matrix-core kernel (one wave per head; the
// parts of a product's operands fill its 16 columns and rows only there).  It wants 16-byte aligned value rows, which
// whole heads of 32 (L_max + 1)^2 bytes are.  Everything else: one thread per channel.
static bool nonlinear_on_matrix_cores(const e2f_ctx* ctx) {
    return ctx->cfg.feat_dtype == E2F_BF16 && ctx->Ch == 16 && ctx->cfg.lf == 1 && ctx->cfg.L_max >= 1;
}

e2f_status e2f_launch_fused_nonlinear(const e2f_ctx* ctx, const E2fCellsView& cv, const e2f_weights* w,
                                      const E2fAttnWs& ws, const void* q1, float* out, hipStream_t st) {
    if (cv.N == 0) return E2F_OK;
    if (cv.N >= (1 << 26)) return E2F_ERR_UNSUPPORTED;   // list entries carry the run in their top bits
    NlParams P;
    P.cv = cv;
    P.spos = ws.spos; P.q = ws.q; P.k = ws.k; P.v = ws.v; P.q1 = q1; P.cw = ws.cw; P.Wb = w->Wb; P.out = out;
    P.C = ctx->cfg.C; P.H = ctx->cfg.H; P.B = ctx->cfg.B; P.Ch = ctx->Ch;
    P.tau = ctx->tau; P.rc2 = ctx->rc2; P.cutoff = ctx->cfg.cutoff; P.rbf_step = ctx->rbf_step; P.rbf_gamma = ctx->rbf_gamma;
    if (nonlinear_on_matrix_cores(ctx)) {
        switch (ctx->cfg.L_max) {
            case 1: launch_heads<1>(ctx, P, w->w_path, st); break;
            case 2: launch_heads<2>(ctx, P, w->w_path, st); break;
            case 3: launch_heads<3>(ctx, P, w->w_path, st); break;
            case 4: launch_heads<4>(ctx, P, w->w_path, st); break;
        }
        E2F_HIP_CHECK(hipGetLastError());
        return E2F_OK;
    }
    bool ok = false;
    switch (ctx->cfg.L_max) {
        case 0: ok = launch_lf<0>(ctx, P, st); break;
        case 1: ok = launch_lf<1>(ctx, P, st); break;
        case 2: ok = launch_lf<2>(ctx, P, st); break;
        case 3: ok = launch_lf<3>(ctx, P, st); break;
        case 4: ok = launch_lf<4>(ctx, P, st); break;
    }
    if (!ok) return E2F_ERR_UNSUPPORTED;
    E2F_HIP_CHECK(hipGetLastError());
    return E2F_OK;
}
