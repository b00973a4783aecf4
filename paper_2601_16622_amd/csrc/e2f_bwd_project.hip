// Backward pass through the l-wise linear maps: dL/dh and the gradients of the five projection matrices from dL/dq,
// dL/dk, dL/dv (all in the caller's atom order).  With p_k = W_k x for a row x = h[atom][l, m], the invariants
// q[l] = sum_m p_0 p_1, k[l] = sum_m p_2 p_3 and v = p_4 (Eq. qk) give the row factors
//     t = (dq[l] p_1, dq[l] p_0, dk[l] p_3, dk[l] p_2, dv[l, m])
// and from them  dx = sum_k W_k^T t_k  and  dW_k = sum over rows of t_k (x) x.
//
// A degree's rows (atoms x orders) are one long list of N (2l+1) rows, cut into units of equal size, so that both
// kernels are matrix products over row tiles on the matrix cores, for bf16 features (16-bit operands, fp32 sums) and
// fp32 features (binary32 operands) alike.  Neither kernel stores the row factors: the weight-gradient kernel forms them again from h
// (two fifths of its matrix work), where writing and reading five fp32 rows per row of h took 100 us of a training step at 4 000
// atoms and 128 channels.
#include <type_traits>

#include "e2f_device.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {   // round to nearest even
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){a, b}, bf16x2));
}

// Four 32-bit factors as bf16 operands.  PARTS = 1: rounded.  PARTS = 3: cut into three parts of 8 significant bits, which
// together are the factor (infinities and NaN sit in the first part alone, so that the sum over the parts keeps them).
template <int PARTS>
__device__ __forceinline__ void split_bf16(f32x4 t, u32x2 (&part)[PARTS]) {
    if constexpr (PARTS == 1) {
        part[0] = (u32x2){pack_bf16(t[0], t[1]), pack_bf16(t[2], t[3])};
    } else {
#pragma unroll
        for (int p = 0; p < PARTS; ++p) {
            const u32x4 b = __builtin_bit_cast(u32x4, t);
            part[p] = (u32x2){__builtin_amdgcn_perm(b[1], b[0], 0x07060302u), __builtin_amdgcn_perm(b[3], b[2], 0x07060302u)};
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const float r = t[x] - __uint_as_float(b[x] & 0xffff0000u);
                t[x] = r == r ? r : 0.0f;
            }
        }
    }
}
// Parts of a row factor as an operand.  fp32 features: one, the factor itself.  bf16 features: at 256 channels three, the
// whole 32 bits; up to 128 channels one for dL/dh (the counterpart of the forward pass rounding the projected values
// to bf16: 1.6e-3 of the norm of dL/dh, where three leave the rounding of the sums) and two for the weights' gradients.
template <typename T, int CP>
constexpr int H_PARTS = sizeof(T) == 2 && CP > 128 ? 3 : 1;
template <typename T, int CP>
constexpr int W_PARTS = sizeof(T) == 4 ? 1 : CP > 128 ? 3 : 2;

// The matrix operands of a feature type.  A fragment is 16 bytes of one row per lane: EPF elements of the contraction
// index.  Which index an element stands for is free as long as both operands agree; a half-wave (32-row tiles) or a
// quarter-wave (16-row tiles) takes the next EPF elements of the row, so that a lane's load is contiguous.
template <typename T>
struct Mat;
template <>
struct Mat<uint16_t> {
    static constexpr int EPF = 8;
    static __device__ __forceinline__ f32x16 mma32(u32x4 a, u32x4 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
    static __device__ __forceinline__ f32x4 mma16(u32x4 a, u32x4 b, f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <>
struct Mat<float> {
    static constexpr int EPF = 4;
    static __device__ __forceinline__ f32x16 mma32(u32x4 a, u32x4 b, f32x16 c) {
        const f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
#pragma unroll
        for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[s], fb[s], c, 0, 0, 0);
        return c;
    }
    static __device__ __forceinline__ f32x4 mma16(u32x4 a, u32x4 b, f32x4 c) {
        const f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
#pragma unroll
        for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[s], fb[s], c, 0, 0, 0);
        return c;
    }
};

template <typename T>
struct MapWeights {
    const T* W[5];   // WQ1, WQ2, WK1, WK2, WV: [L+1][C out][C in]
};

// WT[k][l][ci][co] = W_k[l][co][ci], so that the transposed products of bf16 features read their weights by rows too (a
// fragment is eight of them); one workgroup per (k, l, 16 x 16 tile).
// FRAG: the elements of a map and degree in the order in which k_bwd_rows takes them, block [32 rows][16 columns] by block, a
// block as the 64 lanes' eight elements one behind the other: a fragment is then 1 KB in one piece, where by rows it is 32
// pieces of 32 bytes, each in a cache line of its own.
template <bool FRAG>
__global__ __launch_bounds__(256) void k_transpose_weights(MapWeights<uint16_t> mw, int L1, int C, uint16_t* __restrict__ WT) {
    __shared__ uint16_t s[16][17];
    const int tiles = C / 16, t = blockIdx.x % (tiles * tiles), kl = blockIdx.x / (tiles * tiles);
    const int k = kl / L1, l = kl % L1, tr = t / tiles, tc = t % tiles;
    const uint16_t* W = k == 0 ? mw.W[0] : k == 1 ? mw.W[1] : k == 2 ? mw.W[2] : k == 3 ? mw.W[3] : mw.W[4];
    const int r = threadIdx.x >> 4, c = threadIdx.x & 15;
    s[r][c] = W[((size_t)l * C + 16 * tr + r) * C + 16 * tc + c];
    __syncthreads();
    uint16_t* out = WT + ((size_t)k * L1 + l) * C * C;
    if constexpr (FRAG) {   // row 16 tc + r', columns 16 tr ..: thread -> (half of the columns, row, column)
        const int hf = threadIdx.x >> 7, rr = (threadIdx.x >> 3) & 15, x = threadIdx.x & 7;
        out[(((size_t)(tc >> 1) * tiles + tr) * 64 + hf * 32 + (tc & 1) * 16 + rr) * 8 + x] = s[8 * hf + x][rr];
    } else {
        out[(size_t)(16 * tc + r) * C + 16 * tr + c] = s[c][r];
    }
}

// Workgroups [first[d], first[d + 1]) own the rows of degree L - d, the degree with the most rows first.
struct DegreeMap {
    int first[E2F_MAX_L + 2];
};

// ---- dL/dh.  A workgroup owns 32 RT rows of one degree and all channels: the rows x stay in LDS, and for each of the
// five maps the factors t_k = (dq or dk) (W x) go through LDS as H_PARTS more operands of the same shape.  Wave w owns 32 output channels of the first
// product, written with the channels as rows, so that a lane holds four consecutive channels of its row (16-byte loads of
// dq and dk, 8- or 16-byte stores to LDS), and the same 32 input channels of the second one, written with the data rows as
// rows, so that a store of the result covers whole 128-byte lines.  The weights are read once per workgroup, by
// fragments straight into registers, eight of them (one chunk) ahead of the products: they stay in the L2s (five 128-channel
// degrees are 0.8 MB, 1.5 with the transposes that bf16 features read), and no channel count is too wide for the registers.
// Bound: fp32 by the matrix cores (nine products, 6 GFLOP at 2 240 atoms, L = 2, 128 channels: 38 us at the fp32 peak), bf16 by
// the fp32 rows of dv and dh (0.13 GB at 4 000 atoms, L = 4, 128 channels: 25 us at the rate of a copy).  Measured, with the
// one-thread-per-channel kernel on the vector ALUs in brackets: fp32 2 240 atoms L = 2 x 128: 75 us (442); bf16 3 840 atoms L = 4
// x 256: 271 us (2 818 at 4 000; one bf16 a factor would take less, at the loss stated at H_PARTS).  Up to 128 bf16 channels it
// has the smaller calls, see k_bwd_rows_stationary.
// CP: channels padded up to a multiple of 32 (PAD: C < CP; the missing ones read as zero).
template <typename T, int CP, int RT, bool PAD>
__global__ __launch_bounds__(2 * CP) __attribute__((amdgpu_waves_per_eu(2))) void k_bwd_rows(
    const T* __restrict__ h, MapWeights<T> mw, const T* __restrict__ WT, const float* __restrict__ gq,
    const float* __restrict__ gk, const float* __restrict__ gv, float* __restrict__ gh, int L, int C_, int N,
    DegreeMap map) {
    constexpr int EPF = Mat<T>::EPF, ROWS = 32 * RT, THREADS = 2 * CP, PARTS = H_PARTS<T, CP>;
    constexpr int ROW = CP + EPF;              // LDS row pitch: 16 bytes of padding against bank conflicts
    constexpr int NF = CP / (2 * EPF);         // fragments of a whole contraction
    constexpr int CF = NF < 8 ? NF : 8;        // fragments per chunk
    constexpr int CPS = NF / CF;               // chunks per product
    static_assert(NF % CF == 0, "whole chunks");
    __shared__ __attribute__((aligned(16))) T s_X[ROWS * ROW], s_T[PARTS * ROWS * ROW];
    __shared__ __attribute__((aligned(16))) int s_row[ROWS];   // row -> atom * n + component
    __shared__ int s_inv[ROWS];                                // row -> atom * (L + 1) + degree
    const int C = PAD ? C_ : CP;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, i = lane & 31, hf = lane >> 5;
    const int n = (L + 1) * (L + 1);
    int d = 0;
    while (d < L && (int)blockIdx.x >= map.first[d + 1]) ++d;
    const int l = L - d, nl = 2 * l + 1;
    const int rows = N * nl, r0 = ((int)blockIdx.x - map.first[d]) * ROWS;
    for (int x = tid; x < ROWS; x += THREADS) {
        const int r = min(r0 + x, rows - 1), atom = r / nl;   // the rows after the last repeat it and are not stored
        s_row[x] = atom * n + l * l + (r - atom * nl);
        s_inv[x] = atom * (L + 1) + l;
    }
    __syncthreads();
    // stage 2k + 0 .. of the sequence below: second product of map 4, then first and second product of maps 0 .. 3
    const size_t wl = (size_t)l * C * C, kstride = (size_t)(L + 1) * C * C;
    u32x4 buf[2][CF];
    auto load_chunk = [&](int q, u32x4 (&dst)[CF]) {   // q: chunk of the whole sequence
        const int st = q / CPS, c = q % CPS;
        // stage 0: map 4 transposed; stage 1 + 2k: the map whose product enters t_k (1, 0, 3, 2); stage 2 + 2k: map k transposed
        const int kt = st == 0 ? 4 : (st - 2) / 2, row = 32 * w + i;
        const bool transposed = !(st & 1);
        const T* base = !transposed ? mw.W[((st - 1) / 2) ^ 1] + wl : EPF == 8 ? WT + kt * kstride + wl : mw.W[kt] + wl;
        if (EPF == 8 && transposed) {   // in the order of the fragments (k_transpose_weights; bf16 features come in whole 32 channels)
#pragma unroll
            for (int f = 0; f < CF; ++f) dst[f] = *reinterpret_cast<const u32x4*>(base + ((size_t)(w * NF + c * CF + f) * 64 + lane) * 8);
            return;
        }
#pragma unroll
        for (int f = 0; f < CF; ++f) {
            const int col = (c * CF + f) * 2 * EPF + EPF * hf;
            if (EPF == 4 && transposed) {   // fp32: the four elements one by one, 32 lanes side by side, no copy needed
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    dst[f][x] = (!PAD || (row < C && col < C)) ? __float_as_uint((float)base[(size_t)(col + x) * C + row]) : 0u;
                continue;
            }
            dst[f] = (!PAD || (row < C && col < C)) ? *reinterpret_cast<const u32x4*>(base + (size_t)row * C + col) : (u32x4){0u, 0u, 0u, 0u};
        }
    };
    auto store_factor = [&](int at, f32x4 t) {   // four channels of a row
        if constexpr (EPF == 8) {
            u32x2 part[PARTS];
            split_bf16<PARTS>(t, part);
#pragma unroll
            for (int p = 0; p < PARTS; ++p) *reinterpret_cast<u32x2*>(s_T + p * ROWS * ROW + at) = part[p];
        } else {
            *reinterpret_cast<f32x4*>(s_T + at) = t;
        }
    };
    load_chunk(0, buf[0]);
    {   // x and dv of the unit's rows
        constexpr int PX = ROWS * CP / EPF / THREADS;   // 16-byte pieces of x per thread
#pragma unroll
        for (int j = 0; j < PX; ++j) {
            const int e = tid + THREADS * j, rr = e / (CP / EPF), c = EPF * (e % (CP / EPF));
            *reinterpret_cast<u32x4*>(s_X + rr * ROW + c) =
                (!PAD || c < C) ? *reinterpret_cast<const u32x4*>(h + (size_t)s_row[rr] * C + c) : (u32x4){0u, 0u, 0u, 0u};
        }
        constexpr int PV = ROWS * CP / 4 / THREADS;     // 16-byte pieces of dv per thread
#pragma unroll
        for (int j = 0; j < PV; ++j) {
            const int e = tid + THREADS * j, rr = e / (CP / 4), c = 4 * (e % (CP / 4));
            const f32x4 v = (!PAD || c < C) ? *reinterpret_cast<const e2f::f32x4_unaligned*>(gv + (size_t)s_row[rr] * C + c) : (f32x4){0.f, 0.f, 0.f, 0.f};
            store_factor(rr * ROW + c, v);
        }
    }
    f32x16 dx[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) dx[rt] = (f32x16)(0.0f);
    __syncthreads();
    auto frag = [&](const T* s, int rt, int f) {
        return *reinterpret_cast<const u32x4*>(s + (32 * rt + i) * ROW + 2 * EPF * f + EPF * hf);
    };
    // The fragments of rows are read from LDS while those before them are multiplied (left to itself the compiler reads one, waits
    // for it and multiplies: 345 us at 3 840 atoms, L = 4, 256 bf16 channels, where this takes 325, and 271 with the transposes in order).
    u32x4 fr[2][PARTS][RT];
    auto get = [&](const T* src, int parts, int f) {
#pragma unroll
        for (int p = 0; p < PARTS; ++p)
            if (p < parts)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) fr[f & 1][p][rt] = frag(src + p * ROWS * ROW, rt, f);
    };
#pragma unroll
    for (int st = 0; st < 9; ++st) {
        if (st == 0 || !(st & 1)) {   // dx[row][channel 32 w + i] += sum over co of t[row][co] W[co][ci]
            get(s_T, PARTS, 0);
#pragma unroll
            for (int c = 0; c < CPS; ++c) {
                const int q = st * CPS + c;
                if (q + 1 < 9 * CPS) load_chunk(q + 1, buf[(q + 1) & 1]);
#pragma unroll
                for (int f = 0; f < CF; ++f) {
                    const int at = c * CF + f;
                    if (at + 1 < NF) get(s_T, PARTS, at + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int p = 0; p < PARTS; ++p)
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) dx[rt] = Mat<T>::mma32(fr[at & 1][p][rt], buf[q & 1][f], dx[rt]);
                }
            }
        } else {   // p[channel][row] of the map, then t
            f32x16 p[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) p[rt] = (f32x16)(0.0f);
            get(s_X, 1, 0);
#pragma unroll
            for (int c = 0; c < CPS; ++c) {
                const int q = st * CPS + c;
                if (q + 1 < 9 * CPS) load_chunk(q + 1, buf[(q + 1) & 1]);
#pragma unroll
                for (int f = 0; f < CF; ++f) {
                    const int at = c * CF + f;
                    if (at + 1 < NF) get(s_X, 1, at + 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) p[rt] = Mat<T>::mma32(buf[q & 1][f], fr[at & 1][0][rt], p[rt]);
                }
            }
            const float* g = st < 4 ? gq : gk;   // stages 1, 3: dq; 5, 7: dk
            __syncthreads();   // the factors of the map before have been read
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const float* grow = g + (size_t)s_inv[32 * rt + i] * C + 32 * w + 4 * hf;
                const int at = (32 * rt + i) * ROW + 32 * w + 4 * hf;
#pragma unroll
                for (int j = 0; j < 4; ++j) {   // channels 32 w + 8 j + 4 hf + 0 .. 3
                    const f32x4 gg = (!PAD || 32 * w + 8 * j < C) ? *reinterpret_cast<const e2f::f32x4_unaligned*>(grow + 8 * j) : (f32x4){0.f, 0.f, 0.f, 0.f};
                    const f32x4 t = {gg[0] * p[rt][4 * j], gg[1] * p[rt][4 * j + 1], gg[2] * p[rt][4 * j + 2], gg[3] * p[rt][4 * j + 3]};
                    store_factor(at + 8 * j, t);
                }
            }
            __syncthreads();
        }
    }
    const int ci = 32 * w + i;
    if (PAD && ci >= C) return;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int rr = 32 * rt + 8 * j + 4 * hf;
            const int4 at = *reinterpret_cast<const int4*>(s_row + rr);
            const int ats[4] = {at.x, at.y, at.z, at.w};
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r0 + rr + r < rows) gh[(size_t)ats[r] * C + ci] = dx[rt][4 * j + r];
        }
}

// ---- dL/dh for many rows, bf16 features and up to 128 channels: the weights stay.  A workgroup owns one degree and
// a few consecutive tiles of 16 atoms and walks their (tile, order) slabs with one load of its weights, in registers;
// wave ct owns output channels 16 ct .. 16 ct + 15 of the forward products and the same input channels of the transposed
// ones.  Both products are written with the channels as rows and the atoms as columns, (W x)^T = W X^T and
// dX^T = sum_k W_k^T T_k^T, so that the weights are the A operand, a lane ends up with four consecutive channels
// of one atom (16-byte loads of dq, dk, dv and 16-byte stores of the result) and the row factors t_k cross the waves
// through LDS as [atom][channel] rows, rounded to bf16 as in k_bwd_rows.  The feature rows of a slab are fetched once per
// workgroup and shared through LDS as well.
// It takes a call from STATIONARY_WORK row elements on: a load of the weights is shared by more rows the more rows there are, and
// below that its workgroups do not fill the chip.  Measured, us, this kernel / k_bwd_rows: 128 channels, L = 4: 500 atoms 35 / 17,
// 1 000 37 / 24, 1 311 (the line) 37 / 31, 1 500 37 / 31.5, 2 000 38 / 40, 3 000 40 / 50, 4 000 51 / 70, 6 000 68 / 99, 9 000 101 / 134; L = 2:
// 3 640 (the line) 35 / 30, 5 000 36 / 32, 7 000 38 / 42; L = 1: 8 192 (the line) 32 / 25, 12 000 33 / 33; 64 channels, L = 3: 2 000 18.3 / 13.1,
// 4 000 19.0 / 18.9, 5 000 20 / 22, 9 000 28 / 43; L = 2: 5 000 17.9 / 16.0, 7 282 (the line) 18.6 / 20.1; 32 channels, L = 4: 5 243 (the line)
// 15.8 / 14.2, 9 000 19.3 / 20.0; L = 1: 20 000 14 / 11, 40 000 17 / 18.  The line was drawn where the two met before k_bwd_rows read its
// fragments a step ahead; at 64 channels they still meet there, at 128 from the line up to 6 million elements k_bwd_rows is
// ahead by up to 7 us of a call of some 250.
constexpr long long STATIONARY_WORK = 1ll << 22;
constexpr int SLABS_MIN = 18, SLABS_MAX = 36;   // slabs a workgroup walks with one load of its weights
// Workgroups [first[d], first[d + 1]) own degree L - d (the highest degree, with the most slabs per tile, first) and
// tiles[d] consecutive tiles of 16 atoms each, so that every workgroup walks about the same number of slabs.
struct SlabMap {
    int first[E2F_MAX_L + 2];
    int tiles[E2F_MAX_L + 1];
};

template <int C>
__global__ __launch_bounds__(64 * (C / 16)) void k_bwd_rows_stationary(
    const uint16_t* __restrict__ h, MapWeights<uint16_t> mw, const uint16_t* __restrict__ WT, const float* __restrict__ gq,
    const float* __restrict__ gk, const float* __restrict__ gv, float* __restrict__ gh, int L, int N, SlabMap map) {
    constexpr int NS = C / 32, ROW = C + 8;   // LDS rows of 16 atoms, 16 bytes of padding against bank conflicts
    constexpr int PD = 3;                     // slabs in flight from memory
    // Two buffers each, used in turn.  In one pass of the loop a wave runs the second stage of slab s (reads s_T[s & 1]),
    // the first stage of slab s + 1 (reads s_X[(s + 1) & 1], writes s_T[(s + 1) & 1]) and stores the feature rows of
    // slab s + 2 (s_X[s & 1]): the two stages of consecutive slabs overlap inside a wave and one barrier per slab is enough.
    __shared__ __attribute__((aligned(16))) uint16_t s_T[2][5][16][ROW];
    __shared__ __attribute__((aligned(16))) uint16_t s_X[2][16][ROW];
    // (the wave's index through readfirstlane, so that the compiler knows it to be the same in all lanes)
    const int tid = threadIdx.x, ct = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, i = lane & 15, g = lane >> 4;
    const int n_tiles = (N + 15) / 16, n = (L + 1) * (L + 1);
    int d = 0;
    while (d < L && (int)blockIdx.x >= map.first[d + 1]) ++d;
    const int l = L - d, nl = 2 * l + 1;
    const int tile0 = ((int)blockIdx.x - map.first[d]) * map.tiles[d];
    const int n_slabs = (min(n_tiles, tile0 + map.tiles[d]) - tile0) * nl;   // slab s: tile tile0 + s / nl, order s % nl
    if (n_slabs <= 0) return;
    const int ch0 = 16 * ct + 4 * g;   // the four channels this lane holds of its atom
    auto frag = [](const uint16_t* p) { return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p)); };
    bf16x8 W1[4][NS], W2[5][NS];
    {
        const size_t row = ((size_t)l * C + 16 * ct + i) * C + 8 * g;
        const size_t lstride = (size_t)(L + 1) * C * C;
#pragma unroll
        for (int S = 0; S < NS; ++S) {
            W1[0][S] = frag(mw.W[0] + row + 32 * S);
            W1[1][S] = frag(mw.W[1] + row + 32 * S);
            W1[2][S] = frag(mw.W[2] + row + 32 * S);
            W1[3][S] = frag(mw.W[3] + row + 32 * S);
#pragma unroll
            for (int k = 0; k < 5; ++k) W2[k][S] = frag(WT + k * lstride + row + 32 * S);
        }
    }
    // What is read of a slab.  The feature rows of its 16 atoms, shared by the waves: thread tid fetches four channels
    // (xa, xc) of one row, which reach the waves through s_X.  dv for the lane's own atom and channels.  Both are
    // requested PD slabs before their use, in rings of registers indexed at compile time; dq and dk of a tile (lane's
    // atom and channels again) are requested when the tile before it starts.
    const int xa = tid / (C / 4), xc = 4 * (tid % (C / 4));
    // the four places where the sequence of slabs is walked (requests of x and of dv, first stage, second stage)
    // each keep (first atom of the tile, order); a cursor stays on the last slab once it gets there
    struct Cursor {
        int a0, m;
    };
    const int a_last = (tile0 + n_slabs / nl - 1) * 16;
    auto advance = [&](Cursor& c) {
        if (c.m + 1 < nl) {
            ++c.m;
        } else if (c.a0 < a_last) {
            c.m = 0;
            c.a0 += 16;
        }
    };
    Cursor cx = {tile0 * 16, 0}, cv = cx, cf = cx, co = cx;
    auto fetch_x = [&]() {
        const u32x2 v = *reinterpret_cast<const u32x2*>(h + ((size_t)min(cx.a0 + xa, N - 1) * n + l * l + cx.m) * C + xc);
        advance(cx);
        return v;
    };
    auto fetch_dv = [&]() {
        const f32x4 v = *reinterpret_cast<const e2f::f32x4_unaligned*>(gv + ((size_t)min(cv.a0 + i, N - 1) * n + l * l + cv.m) * C + ch0);
        advance(cv);
        return v;
    };
    auto fetch_dqk = [&](int a0, f32x4& dq, f32x4& dk) {
        const size_t at = ((size_t)min(a0 + i, N - 1) * (L + 1) + l) * C + ch0;
        dq = *reinterpret_cast<const e2f::f32x4_unaligned*>(gq + at);
        dk = *reinterpret_cast<const e2f::f32x4_unaligned*>(gk + at);
    };
    auto store_x = [&](int s, u32x2 v) { *reinterpret_cast<u32x2*>(&s_X[s & 1][xa][xc]) = v; };
    f32x4 dq, dk, dq_next, dk_next;
    // first stage of slab s: the four forward products of the slab's rows, then the five row factors
    // t = (dq (WQ2 x), dq (WQ1 x), dk (WK2 x), dk (WK1 x), dv), to LDS as bf16 (an absent atom's row is not stored at the end)
    auto factors = [&](int s, f32x4 dv) {
        if (cf.m == 0) {   // (uniform) a new tile
            dq = dq_next;
            dk = dk_next;
            fetch_dqk(cf.a0 + 16, dq_next, dk_next);
        }
        advance(cf);
        f32x4 p[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] = (f32x4){0.f, 0.f, 0.f, 0.f};
        bf16x8 X[NS];
#pragma unroll
        for (int S = 0; S < NS; ++S) X[S] = frag(&s_X[s & 1][i][32 * S + 8 * g]);
        __builtin_amdgcn_sched_barrier(0);   // (all requested before any is waited for; see second_stage)
#pragma unroll
        for (int S = 0; S < NS; ++S)
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W1[k][S], X[S], p[k], 0, 0, 0);
        // p[k][r] = (W_k x)[channel 16 ct + 4 g + r] of atom i
        f32x4 t[5];
        t[0] = dq * p[1];
        t[1] = dq * p[0];
        t[2] = dk * p[3];
        t[3] = dk * p[2];
        t[4] = dv;
        const int buf = s & 1;
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            *reinterpret_cast<u32x2*>(&s_T[buf][k][i][ch0]) = (u32x2){pack_bf16(t[k][0], t[k][1]), pack_bf16(t[k][2], t[k][3])};
        }
    };
    // ring slot of slab s: s % PD.  Before pass s of the loop the rings hold x of slabs s + 2 .. s + 4 and dv of
    // slabs s + 1 .. s + 3; s_X holds x of slabs s and s + 1 and s_T the factors of slab s.
    u32x2 xr[PD];
    f32x4 dvr[PD];
    fetch_dqk(tile0 * 16, dq_next, dk_next);
    store_x(0, fetch_x());
    store_x(1, fetch_x());
#pragma unroll
    for (int u = 0; u < PD; ++u) {
        xr[(u + 2) % PD] = fetch_x();
        dvr[u] = fetch_dv();
    }
    __syncthreads();
    factors(0, dvr[0]);
    dvr[0] = fetch_dv();
    __syncthreads();
    // One pass of the loop, for slab s = s0 + u with ring slots known at compile time.  (LAST: a pass of the last,
    // partial group, which checks whether its slab and the next exist.  The passes of the full groups have no such
    // branches: the compiler places its waits on the loads by the least number of memory instructions on any path
    // from a request to its use, and a path that skips passes would make it wait for requests one pass old.)
    auto pass = [&](int s, int u, bool LAST) __attribute__((always_inline)) {
        // The first stage of the next slab and the second stage of this one are independent.
        auto first_stage = [&]() {
            // the feature rows of slab s + 2 have arrived: into the buffer that slab s used
            store_x(s + 2, xr[(u + 2) % PD]);
            xr[(u + 2) % PD] = fetch_x();
            if (!LAST || s + 1 < n_slabs) factors(s + 1, dvr[(u + 1) % PD]);
            dvr[(u + 1) % PD] = fetch_dv();
        };
        auto second_stage = [&]() {
            const int buf = s & 1;
            // (two partial sums: one accumulator would chain all the matrix instructions one after the other)
            f32x4 dp[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
            // (the factors of a map are read from LDS while those of the map before are multiplied; left to itself the compiler
            // reads one operand, waits for it and multiplies, 20 times a slab)
            bf16x8 T[2][NS];
#pragma unroll
            for (int S = 0; S < NS; ++S) T[0][S] = frag(&s_T[buf][0][i][32 * S + 8 * g]);
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                if (k < 4)
#pragma unroll
                    for (int S = 0; S < NS; ++S) T[(k + 1) & 1][S] = frag(&s_T[buf][k + 1][i][32 * S + 8 * g]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int S = 0; S < NS; ++S) {
                    const int j = (k * NS + S) & 1;
                    dp[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W2[k][S], T[k & 1][S], dp[j], 0, 0, 0);
                }
            }
            const f32x4 dx = dp[0] + dp[1];
            // dx[r] = dL/dh[atom i][component][channel 16 ct + 4 g + r]
            const int atom = co.a0 + i;
            if (atom < N) *reinterpret_cast<e2f::f32x4_unaligned*>(gh + ((size_t)atom * n + l * l + co.m) * C + ch0) = dx;
            advance(co);
        };
        first_stage();
        second_stage();
        __syncthreads();
    };
    int s0 = 0;
    for (; s0 + PD < n_slabs; s0 += PD) {
#pragma unroll
        for (int u = 0; u < PD; ++u) pass(s0 + u, u, false);
    }
#pragma unroll
    for (int u = 0; u < PD; ++u)
        if (s0 + u < n_slabs) pass(s0 + u, u, true);   // (uniform)
}

// ---- dL/dW.  A workgroup owns a slice of a degree's rows, one of the five maps and 16 output channels per wave (up to
// eight waves), with all input channels; it walks its rows 64 at a time.  The rows x of a step are shared by the waves
// through LDS; a wave forms the products p of its own channels with the weights in registers, written with the data rows as
// rows, which leaves the factors t in the register layout that the second product wants as its A operand (contraction
// over the data rows), so they never leave the wave.  bf16 features: the factors as W_PARTS bf16, and a second copy of x turned in LDS, with the eight rows that a lane takes of one
// channel side by side.  fp32 features: the rows of x as they are (a lane takes one row of 16 channels per step of the
// fp32 instruction).  One map per workgroup: two (sharing dq or dk and the rows of x) take 200 registers, which
// leaves one workgroup per CU and a half-empty second round of them (bf16 98 us, fp32 154 us).
// Measured, the sum over the slices included, with the kernels that read stored factors in brackets: bf16 4 000 atoms L = 4 x 128:
// 75 us (195), fp32 2 240 atoms L = 2 x 128: 91 us (227).
constexpr int WSTEP = 64;   // rows per step

template <typename T, int CP, int NW, bool PAD>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(CP <= 128 ? 4 : 2))) void k_bwd_wgrad(
    const T* __restrict__ h, MapWeights<T> mw, const float* __restrict__ gq, const float* __restrict__ gk,
    const float* __restrict__ gv, int L, int C_, int N, int split, float* __restrict__ part) {
    constexpr int EPF = Mat<T>::EPF, THREADS = 64 * NW, PARTS = W_PARTS<T, CP>;
    constexpr bool BF = EPF == 8;
    constexpr int ROW = CP + EPF, TROW = WSTEP + 8;
    constexpr int NF = CP / (4 * EPF);      // fragments of a contraction over the channels
    constexpr int CT = CP / 16;             // tiles of input channels
    constexpr int UNITS = WSTEP / 4 * CP / 4 / THREADS;   // units of loading per thread: four rows x four channels
    static_assert(UNITS >= 1, "whole units");
    __shared__ __attribute__((aligned(16))) T s_X[WSTEP * ROW];
    __shared__ __attribute__((aligned(16))) T s_Xt[BF ? CP * TROW : 1];
    __shared__ int s_row[2 * WSTEP], s_inv[2 * WSTEP];   // two sets, used in turn
    const int C = PAD ? C_ : CP;
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, i = lane & 15, g = lane >> 4;
    const int n = (L + 1) * (L + 1), slice = blockIdx.x;
    int l = 0;   // degree l has split * (2l+1) slices
    while (split * (l + 1) * (l + 1) <= slice) ++l;
    const int nl = 2 * l + 1, rows = N * nl, slices = split * nl, mine = slice - split * l * l;
    const int steps = (rows + WSTEP - 1) / WSTEP;
    const int s_lo = (int)((long long)steps * mine / slices), s_hi = (int)((long long)steps * (mine + 1) / slices);
    const int k = blockIdx.y % 5, cb = blockIdx.y / 5;
    const int co0 = 16 * (cb * NW + w), co = co0 + i;   // this wave's and this lane's output channel
    const bool value = k == 4;                          // dv itself: no first product
    const float* gr = value ? gv : k < 2 ? gq : gk;
    u32x4 W[NF];
    if (!value) {   // the map whose product enters t_k: 1, 0, 3, 2
        const T* base = (k == 0 ? mw.W[1] : k == 1 ? mw.W[0] : k == 2 ? mw.W[3] : mw.W[2]) + (size_t)l * C * C + (size_t)co * C;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int col = 4 * EPF * f + EPF * g;
            W[f] = (!PAD || (co < C && col < C)) ? *reinterpret_cast<const u32x4*>(base + col) : (u32x4){0u, 0u, 0u, 0u};
        }
    }
    f32x4 acc[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    typedef typename std::conditional<BF, u32x2, u32x4>::type piece;   // four channels of a row
    piece xr[UNITS][4];
    f32x4 gn[WSTEP / 16];   // dq, dk or dv of the lane's channel: rows 16 S + 4 g + 0 .. 3 of the step fetched last
    auto table = [&](int s) {   // where the rows of step s are (factors beyond the last row: -1, read as zero)
        for (int x = tid; x < WSTEP; x += THREADS) {
            const int r = s * WSTEP + x, rc = min(r, rows - 1), atom = rc / nl, at = atom * n + l * l + (rc - atom * nl);
            s_row[(s & 1) * WSTEP + x] = at;
            s_inv[(s & 1) * WSTEP + x] = r < rows ? (value ? at : atom * (L + 1) + l) : -1;
        }
    };
    auto fetch_g = [&](int s, int S) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int at = s_inv[(s & 1) * WSTEP + 16 * S + 4 * g + r];
            gn[S][r] = (at >= 0 && (!PAD || co < C)) ? gr[(size_t)at * C + co] : 0.0f;
        }
    };
    auto fetch_x = [&](int s) {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int e = tid + THREADS * u, rq = e / (CP / 4), c = 4 * (e % (CP / 4));
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int at = s_row[(s & 1) * WSTEP + 4 * rq + j];
                xr[u][j] = (!PAD || c < C) ? *reinterpret_cast<const piece*>(h + (size_t)at * C + c) : (piece)(0u);
            }
        }
    };
    auto store_x = [&]() {
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            const int e = tid + THREADS * u, rq = e / (CP / 4), c = 4 * (e % (CP / 4));
#pragma unroll
            for (int j = 0; j < 4; ++j) *reinterpret_cast<piece*>(s_X + (4 * rq + j) * ROW + c) = xr[u][j];
            if constexpr (BF) {
                // rows 4 rq .. + 3 of four channels, turned.  Row 32 P + 16 S + 4 g + j of a step sits at position
                // 32 P + 8 g + 4 S + j of its channel: what quarter-wave g contracts over in one instruction.
                // (16-byte pieces permuted by channel, so that neither the turned stores nor the loads pile up in few banks)
                const int at = 8 * ((4 * (rq >> 3) + (rq & 3)) ^ ((c >> 2) & 7)) + 4 * ((rq >> 2) & 1);
                const u32x2 a = xr[u][0], b = xr[u][1], cc = xr[u][2], dd = xr[u][3];
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const uint32_t sel = (x & 1) ? 0x07060302u : 0x05040100u;   // upper or lower half of both words
                    const u32x2 v = {__builtin_amdgcn_perm(b[x >> 1], a[x >> 1], sel), __builtin_amdgcn_perm(dd[x >> 1], cc[x >> 1], sel)};
                    *reinterpret_cast<u32x2*>(s_Xt + (c + x) * TROW + at) = v;
                }
            }
        }
    };
    if (s_lo < s_hi) {
        table(s_lo);
        __syncthreads();
        fetch_x(s_lo);
#pragma unroll
        for (int S = 0; S < WSTEP / 16; ++S) fetch_g(s_lo, S);
    }
    for (int s = s_lo; s < s_hi; ++s) {
        __syncthreads();   // the rows of the step before have been read
        store_x();
        const int sn = min(s + 1, s_hi - 1);   // (the last step fetches itself once more: no branch around the requests)
        if (sn != s) table(sn);
        __syncthreads();
        fetch_x(sn);
        auto factors = [&](int S) {   // t[r]: row 16 S + 4 g + r, channel co
            const f32x4 gs = gn[S];
            fetch_g(sn, S);
            if (value) return gs;
            f32x4 p = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int f = 0; f < NF; ++f)
                p = Mat<T>::mma16(*reinterpret_cast<const u32x4*>(s_X + (16 * S + i) * ROW + 4 * EPF * f + EPF * g), W[f], p);
            return gs * p;
        };
        if constexpr (BF) {
#pragma unroll
            for (int P = 0; P < WSTEP / 32; ++P) {
                u32x4 part[PARTS];
#pragma unroll
                for (int S = 0; S < 2; ++S) {
                    const f32x4 t = factors(2 * P + S);
                    if constexpr (PARTS == 3) {
                        u32x2 p[3];
                        split_bf16<3>(t, p);
#pragma unroll
                        for (int u = 0; u < 3; ++u) {
                            part[u][2 * S] = p[u][0];
                            part[u][2 * S + 1] = p[u][1];
                        }
                    } else {
#pragma unroll
                        for (int x = 0; x < 2; ++x) {
                            const uint32_t v = pack_bf16(t[2 * x], t[2 * x + 1]);
                            part[0][2 * S + x] = v;
                            part[1][2 * S + x] = pack_bf16(t[2 * x] - __uint_as_float(v << 16), t[2 * x + 1] - __uint_as_float(v & 0xffff0000u));
                        }
                    }
                }
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    const u32x4 X = *reinterpret_cast<const u32x4*>(s_Xt + (16 * ct + i) * TROW + 8 * ((4 * P + g) ^ ((4 * ct + (i >> 2)) & 7)));
#pragma unroll
                    for (int u = 0; u < PARTS; ++u) acc[ct] = Mat<T>::mma16(part[u], X, acc[ct]);
                }
            }
        } else {
#pragma unroll
            for (int S = 0; S < WSTEP / 16; ++S) {
                const f32x4 t = factors(S);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[r], reinterpret_cast<const float*>(s_X)[(16 * S + 4 * g + r) * ROW + 16 * ct + i], acc[ct], 0, 0, 0);
            }
        }
    }
    // part[slice][k][co][ci]: lane (i, g) holds rows co = 4 g + r of column ci = i of every tile
    if (PAD && co0 >= C) return;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
        if (!PAD || 16 * ct < C)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[(((size_t)slice * 5 + k) * C + co0 + 4 * g + r) * C + 16 * ct + i] = acc[ct][r];
}

// out[k][l][co][ci] = sum over the slices of degree l, in a fixed order; a thread sums four neighbouring elements.
__global__ __launch_bounds__(64) void k_sum_slices(const float* __restrict__ part, int L, int C, int split, float* __restrict__ out) {
    const size_t CC = (size_t)C * C, M = (size_t)5 * (L + 1) * CC;
    const size_t e4 = 4 * ((size_t)blockIdx.x * 64 + threadIdx.x);
    if (e4 >= M) return;
    const int k = (int)(e4 / ((L + 1) * CC)), l = (int)((e4 / CC) % (L + 1));
    const float* p = part + ((size_t)split * l * l * 5 + k) * CC + e4 % CC;
    const int m = split * (2 * l + 1);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 8
    for (int c = 0; c < m; ++c) s += *reinterpret_cast<const f32x4*>(p + (size_t)c * 5 * CC);
    *reinterpret_cast<e2f::f32x4_unaligned*>(out + e4) = s;
}

template <typename T, int CP, int RT, bool PAD>
void launch_rows(const MapWeights<T>& mw, const T* WT, const T* h, const float* gq, const float* gk, const float* gv,
                 float* gh, int L, int C, int N, hipStream_t st) {
    DegreeMap map;
    map.first[0] = 0;
    for (int d = 0; d <= L; ++d) map.first[d + 1] = map.first[d] + (N * (2 * (L - d) + 1) + 32 * RT - 1) / (32 * RT);
    k_bwd_rows<T, CP, RT, PAD><<<map.first[L + 1], 2 * CP, 0, st>>>(h, mw, WT, gq, gk, gv, gh, L, C, N, map);
}

template <int C>
void launch_rows_stationary(const MapWeights<uint16_t>& mw, const uint16_t* WT, const uint16_t* h, const float* gq, const float* gk,
                            const float* gv, float* gh, int L, int N, hipStream_t st) {
    const int tiles = (N + 15) / 16;
    auto make = [&](int slabs, int& longest) {   // every workgroup about `slabs`, whatever its degree
        SlabMap map;
        map.first[0] = longest = 0;
        for (int d = 0; d <= L; ++d) {
            const int nl = 2 * (L - d) + 1;
            map.tiles[d] = (slabs + nl - 1) / nl;
            map.first[d + 1] = map.first[d] + (tiles + map.tiles[d] - 1) / map.tiles[d];
            if (map.tiles[d] * nl > longest) longest = map.tiles[d] * nl;
        }
        return map;
    };
    // Workgroups of about equal length run in whole rounds of what the chip holds (one, three or eight to a CU, by registers),
    // and a load of the weights costs about six slabs: the slabs per workgroup with the shortest sum of rounds.  (128 channels,
    // L = 4, always 18 / so: 3 840 atoms 75 / 53 us, 6 000 86 / 76, 9 973 157 / 127.)
    const int at_once = 256 * (C == 128 ? 1 : C == 64 ? 3 : 8);
    SlabMap map;
    long long best = -1;
    for (int slabs = SLABS_MIN; slabs <= SLABS_MAX; ++slabs) {
        int longest;
        const SlabMap m = make(slabs, longest);
        const long long cost = (long long)((m.first[L + 1] + at_once - 1) / at_once) * (longest + 6);
        if (best < 0 || cost < best) {
            best = cost;
            map = m;
        }
    }
    k_bwd_rows_stationary<C><<<map.first[L + 1], 64 * (C / 16), 0, st>>>(h, mw, WT, gq, gk, gv, gh, L, N, map);
}

template <typename T, int CP, bool PAD>
void launch_C(const MapWeights<T>& mw, T* WT, const T* h, const float* gq, const float* gk, const float* gv, float* gh,
              float* grad_W, float* part, int L, int C, int N, hipStream_t st) {
    if (gh) {
        const long long rows = (long long)N * (L + 1) * (L + 1);
        if constexpr (sizeof(T) == 2) {
            const int t16 = C / 16;
            if (CP <= 128 && rows * C >= STATIONARY_WORK) k_transpose_weights<false><<<5 * (L + 1) * t16 * t16, 256, 0, st>>>(mw, L + 1, C, WT);
            else k_transpose_weights<true><<<5 * (L + 1) * t16 * t16, 256, 0, st>>>(mw, L + 1, C, WT);
        }
        if constexpr (sizeof(T) == 2 && CP <= 128) {
            if (rows * C >= STATIONARY_WORK) launch_rows_stationary<CP>(mw, WT, h, gq, gk, gv, gh, L, N, st);
            else launch_rows<T, CP, 2, PAD>(mw, WT, h, gq, gk, gv, gh, L, C, N, st);
        } else {
            // 64 rows a workgroup while that leaves two workgroups per CU, else 32: the weights pass through every workgroup.  Measured,
            // us, 32 / 64 rows: 256 bf16 channels, L = 4, 300 atoms 35 / 43, 700 90 / 81, 1 311 (the line) 144 / 120, 4 000 380 / 300; fp32 256
            // channels, L = 4, 700 atoms 248 / 310, 1 311 392 / 449, 3 000 815 / 772; fp32 128 channels, L = 4, 500 to 1 300 atoms 1.0 to 1.08,
            // 1 600 117 / 128, 3 000 218 / 200, L = 2, 2 240 71 / 86, 3 641 (the line) 106 / 122, 6 000 155 / 162; fp32 64 channels, L = 2, 2 240
            // 27 / 41, 3 641 38 / 43, 6 000 53 / 52; 16 channels, L = 1, 9 000 17 / 28: bf16 would take 64 rows earlier, fp32 later.
            if (rows >= 512 * 64) launch_rows<T, CP, 2, PAD>(mw, WT, h, gq, gk, gv, gh, L, C, N, st);
            else launch_rows<T, CP, 1, PAD>(mw, WT, h, gq, gk, gv, gh, L, C, N, st);
        }
    }
    if (grad_W) {
        constexpr int NW = CP / 16 < 8 ? CP / 16 : 8;
        const int split = e2f_wgrad_split(L, C, N, sizeof(T) == 4);
        const dim3 grid(split * (L + 1) * (L + 1), 5 * (CP / 16 / NW));
        k_bwd_wgrad<T, CP, NW, PAD><<<grid, 64 * NW, 0, st>>>(h, mw, gq, gk, gv, L, C, N, split, part);
        const size_t M = (size_t)5 * (L + 1) * C * C;
        k_sum_slices<<<(unsigned)((M / 4 + 63) / 64), 64, 0, st>>>(part, L, C, split, grad_W);
    }
}

template <typename T>
e2f_status launch_T(const e2f_ctx* ctx, int N, const e2f_weights* w, const void* h, const float* gq, const float* gk,
                    const float* gv, float* gh, float* grad_W, const E2fBwdWs& bw, hipStream_t st) {
    const MapWeights<T> mw = {{(const T*)w->WQ1, (const T*)w->WQ2, (const T*)w->WK1, (const T*)w->WK2, (const T*)w->WV}};
    const int L = ctx->cfg.L_max, C = ctx->cfg.C;
    T* WT = reinterpret_cast<T*>(bw.wT);
#define E2F_C(CP, PAD) launch_C<T, CP, PAD>(mw, WT, (const T*)h, gq, gk, gv, gh, grad_W, bw.wpart, L, C, N, st)
    if constexpr (sizeof(T) == 4) {   // (bf16 features come in whole 32 channels)
        if (C == 16) E2F_C(32, true);
        if (C == 48) E2F_C(64, true);
    }
    switch (C) {
        case 16: case 48: break;
        case 32: E2F_C(32, false); break;
        case 64: E2F_C(64, false); break;
        case 128: E2F_C(128, false); break;
        case 256: E2F_C(256, false); break;
        default: return E2F_ERR_UNSUPPORTED;   // (192 channels: no head width that is a power of two)
    }
#undef E2F_C
    E2F_HIP_CHECK(hipGetLastError());
    return E2F_OK;
}

}  // namespace

e2f_status e2f_launch_backward_maps(const e2f_ctx* ctx, int N, const e2f_weights* w, const void* h, const float* grad_q,
                                    const float* grad_k, const float* grad_v, float* grad_h, float* grad_W,
                                    const E2fBwdWs& bw, hipStream_t st) {
    if (N == 0) return E2F_OK;
    return ctx->cfg.feat_dtype == E2F_BF16 ? launch_T<uint16_t>(ctx, N, w, h, grad_q, grad_k, grad_v, grad_h, grad_W, bw, st)
                                           : launch_T<float>(ctx, N, w, h, grad_q, grad_k, grad_v, grad_h, grad_W, bw, st);
}
