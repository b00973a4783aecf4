// GPU cell lists: per-segment bounding boxes, grids of edge >= cutoff, a deterministic counting sort of the
// atoms by (segment, cell, atom index), and the neighbour-set test kernels that walk the result.
#include <limits.h>

#include "e2f_device.h"

namespace {

__device__ __forceinline__ int float_to_ordered(float f) {
    int i = __float_as_int(f);
    return i >= 0 ? i : i ^ 0x7fffffff;
}
__device__ __forceinline__ float ordered_to_float(int i) { return __int_as_float(i >= 0 ? i : i ^ 0x7fffffff); }

__global__ void k_cells_init(int32_t* bbox, int S, int32_t* cell_start, int32_t* cell_fill, int max_cells) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < S * 6) bbox[i] = (i % 6 < 3) ? INT_MAX : INT_MIN;
    if (i <= max_cells) cell_start[i] = 0;
    if (i < max_cells) cell_fill[i] = 0;
}

// Boxes of a wave's segments: v comes as the lane's position twice and leaves, in the first lane of every run of lanes
// with the same `seg` (-1: no atom), as min x, y, z and max x, y, z of the run.  Returns whether this lane is the first of a run.
__device__ __forceinline__ bool run_boxes(int seg, int lane, float (&v)[6]) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const bool same = __shfl_down(seg, off) == seg && lane + off < 64;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const float o = __shfl_down(v[k], off);
            if (same) v[k] = k < 3 ? fminf(v[k], o) : fmaxf(v[k], o);
        }
    }
    const int before = __shfl_up(seg, 1);
    return seg >= 0 && (lane == 0 || before != seg);
}
__device__ __forceinline__ int segment_of(const int32_t* seg_offsets, int S, int a) {   // largest s with seg_offsets[s] <= a
    int lo = 0, hi = S;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (seg_offsets[mid] <= a) lo = mid; else hi = mid;
    }
    return lo;
}

// Segment of every atom (binary search in the offsets) and the segment bounding boxes.
__global__ void k_cells_bbox(const float* __restrict__ pos, const int32_t* __restrict__ seg_offsets, int N, int S,
                             int32_t* __restrict__ atom_seg, int32_t* __restrict__ bbox) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = a < N;
    int s = 0;
    float x = 0.f, y = 0.f, z = 0.f;
    if (live) {
        s = segment_of(seg_offsets, S, a);
        atom_seg[a] = s;
        x = pos[3 * a]; y = pos[3 * a + 1]; z = pos[3 * a + 2];
    }
    // One set of atomics per workgroup when all of it sits in one segment (the common case: few, large segments), else
    // one per wave and segment.  Atoms come segment by segment, so a segment's atoms are neighbouring lanes and six steps
    // reduce all of a wave's segments, each into its first lane.  (One set per atom of a mixed wave, 384 atomics on
    // a handful of addresses, took 66 to 70 us for 64 molecules of 10 to 60 atoms and 25 us for 16 of 150 to 350.)
    __shared__ float s_box[16][6];
    __shared__ int s_seg[16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n_waves = (blockDim.x + 63) >> 6;
    const int sl = live ? s : -1, s0 = __shfl(sl, 0);
    const bool uniform = __all(live && s == s0);
    float v[6] = {x, y, z, x, y, z};   // min x, y, z; max x, y, z
    const bool first = run_boxes(sl, lane, v);
    if (lane == 0) {
        s_seg[wave] = uniform ? s0 : -1;
#pragma unroll
        for (int k = 0; k < 6; ++k) s_box[wave][k] = v[k];
    }
    __syncthreads();
    bool block_uniform = s_seg[0] >= 0;
    for (int w = 1; w < n_waves; ++w) block_uniform = block_uniform && s_seg[w] == s_seg[0];
    auto publish = [&](int seg, int k, float val) {
        if (k < 3) atomicMin(&bbox[seg * 6 + k], float_to_ordered(val));
        else atomicMax(&bbox[seg * 6 + k], float_to_ordered(val));
    };
    if (block_uniform) {
        if (threadIdx.x < 6) {
            float val = s_box[0][threadIdx.x];
            for (int w = 1; w < n_waves; ++w) val = threadIdx.x < 3 ? fminf(val, s_box[w][threadIdx.x]) : fmaxf(val, s_box[w][threadIdx.x]);
            publish(s_seg[0], threadIdx.x, val);
        }
    } else if (first) {
#pragma unroll
        for (int k = 0; k < 6; ++k) publish(s, k, v[k]);
    }
}

// Grid of a segment of ns atoms with bounding box bb (ordered integers): the edge is doubled until the segment stays
// within its cell budget of 27 + 2 * atoms, so that the total never exceeds the workspace.  A periodic axis (box: lengths
// and their reciprocals, or null; length > 0) gets floor(length / edge) >= 3 cells that tile the box exactly, origin 0.
// Returns the number of cells; the first cell's id is left to the caller.
__device__ __forceinline__ int segment_grid(int ns, const int32_t* bb, float edge0, const float* __restrict__ box, E2fSegGrid& g) {
    int cells = 1;  // an empty segment keeps one empty cell
    const float lx = box ? box[0] : 0.0f, ly = box ? box[1] : 0.0f, lz = box ? box[2] : 0.0f;
    g.lx = lx; g.ly = ly; g.lz = lz;
    g.rx = box ? box[3] : 0.0f;
    g.ry = box ? box[4] : 0.0f;
    g.rz = box ? box[5] : 0.0f;
    if (ns > 0) {
        const float mnx = ordered_to_float(bb[0]), mny = ordered_to_float(bb[1]);
        const float mnz = ordered_to_float(bb[2]), mxx = ordered_to_float(bb[3]);
        const float mxy = ordered_to_float(bb[4]), mxz = ordered_to_float(bb[5]);
        const long long budget = 27ll + 2ll * ns;
        float edge = edge0;
        long long nx = 1, ny = 1, nz = 1;
        bool fits = false;
        auto cells_along = [&](float len, float extent) -> long long {
            const long long whole = (long long)floorf((len > 0.0f ? len : extent) / edge);
            return len > 0.0f ? (whole > 3 ? whole : 3) : whole + 1;   // (27 cells always fit the budget)
        };
        for (int it = 0; it < 200 && !fits; ++it) {  // bounded: edge overflows to inf long before
            nx = cells_along(lx, mxx - mnx);
            ny = cells_along(ly, mxy - mny);
            nz = cells_along(lz, mxz - mnz);
            fits = nx >= 1 && ny >= 1 && nz >= 1 && nx <= budget && ny <= budget && nz <= budget &&
                   nx * ny * nz <= budget;
            if (!fits) edge *= 2.0f;
        }
        if (!fits) {  // non-finite coordinates: one cell holds the whole segment
            nx = ny = nz = 1;
            edge = edge0;
        }
        g.ox = lx > 0.0f ? 0.0f : mnx;
        g.oy = ly > 0.0f ? 0.0f : mny;
        g.oz = lz > 0.0f ? 0.0f : mnz;
        g.ix = lx > 0.0f ? (float)nx / lx : 1.0f / edge;
        g.iy = ly > 0.0f ? (float)ny / ly : 1.0f / edge;
        g.iz = lz > 0.0f ? (float)nz / lz : 1.0f / edge;
        g.nx = (int)nx; g.ny = (int)ny; g.nz = (int)nz;
        cells = (int)(nx * ny * nz);
    }
    return cells;
}

// One block: grid of every segment, and an exclusive scan of the cell counts.
__global__ void k_cells_grid(const int32_t* __restrict__ bbox, const int32_t* __restrict__ seg_offsets, int S,
                             float edge0, const float* __restrict__ box, E2fSegGrid* __restrict__ grid) {
    __shared__ int s_part[1024];
    __shared__ int s_carry;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (int s0 = 0; s0 < S; s0 += blockDim.x) {
        const int s = s0 + threadIdx.x;
        int cells = 0;
        E2fSegGrid g = {0.f, 0.f, 0.f, 1.f, 1.f, 1.f, 1, 1, 1, 0, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (s < S) {
            const int ns = seg_offsets[s + 1] - seg_offsets[s];
            cells = segment_grid(ns, bbox + 6 * s, edge0, box ? box + 6 * s : nullptr, g);
        }
        // block-wide exclusive scan of `cells`
        s_part[threadIdx.x] = cells;
        __syncthreads();
        for (int off = 1; off < (int)blockDim.x; off <<= 1) {
            int v = (threadIdx.x >= (unsigned)off) ? s_part[threadIdx.x - off] : 0;
            __syncthreads();
            s_part[threadIdx.x] += v;
            __syncthreads();
        }
        const int incl = s_part[threadIdx.x];
        const int carry = s_carry;
        if (s < S) {
            g.base = carry + incl - cells;
            grid[s] = g;
        }
        __syncthreads();
        if (threadIdx.x == blockDim.x - 1) s_carry = carry + incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) grid[S].base = s_carry;   // cells in use: what the scan of the counts has to cover
}

// Cell of a position p, and its place in the order inside the cell.
__device__ __forceinline__ void cell_of(const float* p, const E2fSegGrid& g, int& c, int& sub) {
    const float fx = (e2f::fold_coord(p[0], g.lx, g.rx) - g.ox) * g.ix;
    const float fy = (e2f::fold_coord(p[1], g.ly, g.ry) - g.oy) * g.iy;
    const float fz = (e2f::fold_coord(p[2], g.lz, g.rz) - g.oz) * g.iz;
    int cx = (int)floorf(fx), cy = (int)floorf(fy), cz = (int)floorf(fz);
    cx = min(max(cx, 0), g.nx - 1); cy = min(max(cy, 0), g.ny - 1); cz = min(max(cz, 0), g.nz - 1);
    c = g.base + (cz * g.ny + cy) * g.nx + cx;
    // Order inside the cell: Morton index over 4x4x4 sub-cells, so that atoms that are consecutive in the sorted
    // order (the 16-atom target tiles and the 4-slot candidate groups of the attention kernels) are close in space.
    const int sx = min(max((int)((fx - (float)cx) * 4.0f), 0), 3), sy = min(max((int)((fy - (float)cy) * 4.0f), 0), 3);
    const int sz = min(max((int)((fz - (float)cz) * 4.0f), 0), 3);
    auto spread = [](int v) { return (v & 1) | ((v & 2) << 2); };   // bit 0 -> 0, bit 1 -> 3
    sub = spread(sx) | (spread(sy) << 1) | (spread(sz) << 2);
}

__global__ void k_cells_assign(const float* __restrict__ pos, const int32_t* __restrict__ atom_seg,
                               const E2fSegGrid* __restrict__ grid, int N, int32_t* __restrict__ atom_cell,
                               int32_t* __restrict__ atom_sub, int32_t* __restrict__ cell_count /* = cell_start + 1 */) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= N) return;
    int c, sub;
    cell_of(pos + 3 * a, grid[atom_seg[a]], c, sub);
    atom_cell[a] = c;
    atom_sub[a] = sub;
    atomicAdd(&cell_count[c], 1);
}

// One block: in-place inclusive scan of data[0..n) (data[0] is 0, data[c+1] the count of cell c), which turns
// the counts into first-slot offsets.  Every thread sums one contiguous chunk, the chunk sums are scanned across
// the block, and a second sweep writes the running totals.
__global__ void k_cells_scan(int32_t* __restrict__ data, const E2fSegGrid* __restrict__ grid, int S) {
    __shared__ int s_part[1024];
    const int n = grid[S].base + 1;   // cells in use + 1; the counts beyond are zero and never read
    const int chunk = (n + (int)blockDim.x - 1) / (int)blockDim.x;
    const int b = min((int)threadIdx.x * chunk, n), e = min(b + chunk, n);
    int sum = 0;
    for (int i = b; i < e; ++i) sum += data[i];
    s_part[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < (int)blockDim.x; off <<= 1) {
        const int v = (threadIdx.x >= (unsigned)off) ? s_part[threadIdx.x - off] : 0;
        __syncthreads();
        s_part[threadIdx.x] += v;
        __syncthreads();
    }
    int run = s_part[threadIdx.x] - sum;
    for (int i = b; i < e; ++i) {
        run += data[i];
        data[i] = run;
    }
}

__global__ void k_cells_scatter(const int32_t* __restrict__ atom_cell, const int32_t* __restrict__ cell_start, int N,
                                int32_t* __restrict__ cell_fill, int32_t* __restrict__ tmp_slot) {
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= N) return;
    const int c = atom_cell[a];
    tmp_slot[cell_start[c] + atomicAdd(&cell_fill[c], 1)] = a;
}

__device__ __forceinline__ void store_sinfo(int4* dst, int seg, int c, const E2fSegGrid& g) {
    const int local = c - g.base;
    dst[0] = make_int4(seg, local % g.nx, (local / g.nx) % g.ny, local / (g.nx * g.ny));
    dst[1] = make_int4(g.nx, g.ny, g.nz, g.base);
}

// The scatter above fills each cell in arrival order; ranking every atom among its cell mates by (sub-cell, atom
// index) makes the final order independent of that.
__global__ void k_cells_rank(const int32_t* __restrict__ tmp_slot, const int32_t* __restrict__ atom_cell,
                             const int32_t* __restrict__ atom_sub, const int32_t* __restrict__ atom_seg, const int32_t* __restrict__ cell_start, int N,
                             const E2fSegGrid* __restrict__ grid, int32_t* __restrict__ perm,
                             int32_t* __restrict__ scell, int32_t* __restrict__ sseg, int32_t* __restrict__ atom_slot,
                             int4* __restrict__ sinfo) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N) return;
    const int a = tmp_slot[t];
    const int c = atom_cell[a];
    const int b = cell_start[c], e = cell_start[c + 1];
    const int sa = atom_sub[a];
    int rank = 0;
    for (int u = b; u < e; ++u) {
        const int o = tmp_slot[u], so = atom_sub[o];
        rank += (so < sa || (so == sa && o < a)) ? 1 : 0;
    }
    perm[b + rank] = a;
    scell[b + rank] = c;
    sseg[b + rank] = atom_seg[a];
    atom_slot[a] = b + rank;
    store_sinfo(sinfo + 2 * (b + rank), atom_seg[a], c, grid[atom_seg[a]]);
}

// Inclusive scan over the 1024 threads of a workgroup (s: 16 ints, free again after the caller's next barrier).
__device__ __forceinline__ int block_scan(int v, int* s) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(v, off);
        if (lane >= off) v += o;
    }
    if (lane == 63) s[wave] = v;
    __syncthreads();
    for (int w = 0; w < wave; ++w) v += s[w];
    return v;
}

// The whole construction for a small call, in one workgroup and one launch: what the kernels above pass on through
// memory stays in LDS (boxes, grids, cell offsets, sort keys) and registers (an atom's cell).  The same functions in the
// same order, so the same lists.  The seven launches above are mostly launch: the call in us, seven launches / this, at 64
// atoms 25 / 13, 1 000 33 / 15, 2 240 in 64 molecules 28 / 17, 4 000 in 16 31 / 22, 4 096 38 / 23, 3 900 in 200 35 / 35, 1 500 in
// 700 26 / 27; everything in one cell, where the ranks cost most, 1 000 atoms 191 / 35, 4 096 702 / 379.  It ends where its
// room does, four atoms per thread in registers and 60 KB of LDS (51 at 4 000 atoms in 16 molecules), still ahead there.
constexpr int SMALL_N = 4096, SMALL_S = 1024, SMALL_PER = SMALL_N / 1024;
__global__ __launch_bounds__(1024) void k_cells_small(const float* __restrict__ pos, const int32_t* __restrict__ seg_offsets, int N,
                                                      int S, int max_cells, float edge0, const float* __restrict__ box,
                                                      E2fSegGrid* __restrict__ grid, int32_t* __restrict__ cell_start,
                                                      int32_t* __restrict__ perm, int32_t* __restrict__ scell,
                                                      int32_t* __restrict__ sseg, int32_t* __restrict__ atom_slot,
                                                      int4* __restrict__ sinfo) {
    extern __shared__ int s_mem[];
    int* s_bbox = s_mem;                                            // [S][6]
    int* s_off = s_bbox + 6 * S;                                    // [S + 1] segment offsets
    E2fSegGrid* s_grid = reinterpret_cast<E2fSegGrid*>(s_off + S + 1);   // [S]
    int* s_start = reinterpret_cast<int*>(s_grid + S);              // [max_cells + 1] counts, then offsets
    unsigned* s_key = reinterpret_cast<unsigned*>(s_start + max_cells + 1);   // [N]
    __shared__ int s_scan[2][16];
    __shared__ int s_cells;
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < 6 * S; i += 1024) s_bbox[i] = (i % 6 < 3) ? INT_MAX : INT_MIN;
    for (int i = tid; i <= S; i += 1024) s_off[i] = seg_offsets[i];
    for (int i = tid; i <= max_cells; i += 1024) s_start[i] = 0;
    __syncthreads();
    int seg[SMALL_PER], cell[SMALL_PER], sub[SMALL_PER], turn[SMALL_PER];
    float p[SMALL_PER][3];
#pragma unroll
    for (int k = 0; k < SMALL_PER; ++k) {
        const int a = tid + 1024 * k;
        seg[k] = -1;
        p[k][0] = p[k][1] = p[k][2] = 0.0f;
        if (a < N) {
            p[k][0] = pos[3 * a];
            p[k][1] = pos[3 * a + 1];
            p[k][2] = pos[3 * a + 2];
            seg[k] = segment_of(s_off, S, a);
        }
    }
#pragma unroll
    for (int k = 0; k < SMALL_PER; ++k) {
        float v[6] = {p[k][0], p[k][1], p[k][2], p[k][0], p[k][1], p[k][2]};
        if (run_boxes(seg[k], lane, v)) {
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                atomicMin(&s_bbox[6 * seg[k] + x], float_to_ordered(v[x]));
                atomicMax(&s_bbox[6 * seg[k] + 3 + x], float_to_ordered(v[3 + x]));
            }
        }
    }
    __syncthreads();
    {
        E2fSegGrid g = {0.f, 0.f, 0.f, 1.f, 1.f, 1.f, 1, 1, 1, 0, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        int cells = 0;
        if (tid < S) cells = segment_grid(s_off[tid + 1] - s_off[tid], s_bbox + 6 * tid, edge0, box ? box + 6 * tid : nullptr, g);
        const int end = block_scan(cells, s_scan[0]);
        if (tid < S) {
            g.base = end - cells;
            s_grid[tid] = g;
            grid[tid] = g;
        }
        if (tid == 1023) s_cells = end;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SMALL_PER; ++k)
        if (seg[k] >= 0) {
            cell_of(p[k], s_grid[seg[k]], cell[k], sub[k]);
            turn[k] = atomicAdd(&s_start[cell[k] + 1], 1);   // (any order: the ranks below do not depend on it)
        }
    __syncthreads();
    {
        const int n = s_cells + 1, chunk = (n + 1023) / 1024, b = min(tid * chunk, n), e = min(b + chunk, n);
        int sum = 0;
        for (int i = b; i < e; ++i) sum += s_start[i];
        int run = block_scan(sum, s_scan[1]) - sum;
        for (int i = b; i < e; ++i) {
            run += s_start[i];
            s_start[i] = run;
            cell_start[i] = run;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SMALL_PER; ++k)
        if (seg[k] >= 0) s_key[s_start[cell[k]] + turn[k]] = ((unsigned)sub[k] << 16) | (unsigned)(tid + 1024 * k);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < SMALL_PER; ++k)
        if (seg[k] >= 0) {
            const int a = tid + 1024 * k, b = s_start[cell[k]], e = s_start[cell[k] + 1];
            const unsigned key = ((unsigned)sub[k] << 16) | (unsigned)a;
            int slot = b;
#pragma unroll 4
            for (int u = b; u < e; ++u) slot += s_key[u] < key ? 1 : 0;
            perm[slot] = a;
            scell[slot] = cell[k];
            sseg[slot] = seg[k];
            atom_slot[a] = slot;
            store_sinfo(sinfo + 2 * slot, seg[k], cell[k], s_grid[seg[k]]);
        }
    if (tid == 0) grid[S].base = s_cells;
}

// One wave per target: walk the 27-cell stencil 64 candidates at a time.
// Position of an atom as the predicate sees it: folded into the segment's box on periodic axes.
template <bool PBC>
__device__ __forceinline__ void atom_position(const float* __restrict__ pos, int atom, const E2fSegGrid& g, float& x,
                                              float& y, float& z) {
    x = pos[3 * atom];
    y = pos[3 * atom + 1];
    z = pos[3 * atom + 2];
    if (PBC) {
        x = e2f::fold_coord(x, g.lx, g.rx);
        y = e2f::fold_coord(y, g.ly, g.ry);
        z = e2f::fold_coord(z, g.lz, g.rz);
    }
}

template <bool LIST, bool PBC>
__global__ __launch_bounds__(64) void k_neighbors(E2fCellsView cv, const float* __restrict__ pos, float rc2,
                                                  int32_t* __restrict__ degree, const int64_t* __restrict__ offsets,
                                                  int32_t* __restrict__ idx) {
    const int t = blockIdx.x, lane = threadIdx.x;
    const int ai = cv.perm[t];
    const E2fSegGrid g = cv.grid[cv.sseg[t]];
    float xi, yi, zi;
    atom_position<PBC>(pos, ai, g, xi, yi, zi);
    e2f::Stencil<PBC> st;
    st.init(cv, t);
    int cnt = 0;
    const int64_t out0 = LIST ? offsets[ai] : 0;
    for (int r = 0; r < e2f::Stencil<PBC>::NR; ++r)
        for (int base = st.lo[r]; base < st.hi[r]; base += 64) {
            const int j = base + lane;
            bool ok = false;
            int aj = 0;
            if (j < st.hi[r] && j != t) {
                aj = cv.perm[j];
                float xj, yj, zj;
                atom_position<PBC>(pos, aj, g, xj, yj, zj);
                ok = e2f::is_neighbor(e2f::dist2_exact(xi, yi, zi, xj + st.shift_x(r), yj + st.shift_y(r),
                                                       zj + st.shift_z(r)), rc2);
            }
            const unsigned long long mask = __ballot(ok);
            if (LIST && ok) idx[out0 + cnt + __popcll(mask & ((1ull << lane) - 1ull))] = aj;
            cnt += __popcll(mask);
        }
    if (!LIST && lane == 0) degree[ai] = cnt;
}

// Neighbour cap: one wave per target finds the K-th smallest key (bits of d^2, atom index) among the target's
// neighbours inside the cutoff.  Up to 256 neighbours: by counting.  More: by an 8-bit radix select over the 64-bit keys (a
// 256-bin histogram in LDS per digit; the keys are kept in LDS after one stencil walk, or, beyond 512 neighbours, the
// stencil is walked once per digit, so there is no limit on their number).  Then writes the threshold key and / or the
// table row of the selected atoms (in cell order, -1 padded).  Keys are unique, so exactly min(K, degree) atoms pass.
template <bool PBC>
__global__ __launch_bounds__(64) void k_select_neighbors(E2fCellsView cv, const float* __restrict__ pos, float rc2,
                                                         int K, uint32_t* __restrict__ cap_d2,
                                                         int32_t* __restrict__ cap_idx, int32_t* __restrict__ table,
                                                         int32_t* __restrict__ count) {
    __shared__ int s_hist[256];
    const int t = blockIdx.x, lane = threadIdx.x;
    const int ai = cv.perm[t];
    const E2fSegGrid g = cv.grid[cv.sseg[t]];
    float xi, yi, zi;
    atom_position<PBC>(pos, ai, g, xi, yi, zi);
    __shared__ e2f::RunList s_run;
    e2f::fill_runs(s_run, cv, t, lane);
    __syncthreads();
    const int candidates = s_run.total();
    // walk(f): f(ok, key, atom) for every candidate of this lane, all lanes in step
    auto walk = [&](auto&& f) {
        for (int base = 0; base < candidates; base += 64) {
            bool ok = false;
            int aj = 0;
            unsigned long long key = ~0ull;
            if (base + lane < candidates) {
                int run, j;
                s_run.candidate<e2f::Stencil<PBC>::NR>(base + lane, run, j);
                aj = cv.perm[j];
                float xj, yj, zj;
                atom_position<PBC>(pos, aj, g, xj, yj, zj);
                if constexpr (PBC) {
                    const float4 sh = s_run.sh[run];
                    xj += sh.x;
                    yj += sh.y;
                    zj += sh.z;
                }
                const float d2 = e2f::dist2_exact(xi, yi, zi, xj, yj, zj);
                ok = j != t && e2f::is_neighbor(d2, rc2);
                key = ((unsigned long long)__float_as_uint(d2) << 32) | (unsigned int)aj;
            }
            f(ok, key, aj);
        }
    };
    // first walk: count the neighbours and keep their keys in LDS while they fit (they do in any physical system)
    constexpr int KEEP = 512;
    __shared__ unsigned long long s_key[KEEP];
    int total = 0;
    walk([&](bool ok, unsigned long long key, int) {
        const unsigned long long mask = __ballot(ok);
        const int at = total + __popcll(mask & ((1ull << lane) - 1ull));
        if (ok && at < KEEP) s_key[at] = key;
        total += __popcll(mask);
    });
    __syncthreads();
    const bool in_lds = total <= KEEP;
    // keys(f): f(ok, key) over all neighbour keys, from LDS or by walking the stencil again
    auto keys = [&](auto&& f) {
        if (in_lds) {
            for (int base = 0; base < total; base += 64) {
                const bool ok = base + lane < total;
                f(ok, ok ? s_key[base + lane] : ~0ull);
            }
        } else {
            walk([&](bool ok, unsigned long long key, int) { f(ok, key); });
        }
    };
    unsigned long long thr = ~0ull;   // no cap needed: every neighbour passes
    if (total > K && total <= 256) {
        // the key with K - 1 smaller ones, counted against all of them (keys are unique): a pass over the list costs a
        // fraction of one digit of the radix select (capped forward at 50 000 atoms 1 308 -> 1 295 us)
        auto count_below = [&](auto parts) {   // 64 keys to a register
            constexpr int U = decltype(parts)::value;
            unsigned long long mine[U];
            int below[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                mine[u] = lane + 64 * u < total ? s_key[lane + 64 * u] : ~0ull;
                below[u] = 0;
            }
#pragma unroll 4
            for (int x = 0; x < total; ++x) {
                const unsigned long long key = s_key[x];
#pragma unroll
                for (int u = 0; u < U; ++u) below[u] += key < mine[u] ? 1 : 0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned long long mask = __ballot(lane + 64 * u < total && below[u] == K - 1);
                if (mask) thr = __shfl(mine[u], __builtin_ctzll(mask));
            }
        };
        if (total <= 64) count_below(std::integral_constant<int, 1>{});
        else if (total <= 128) count_below(std::integral_constant<int, 2>{});
        else count_below(std::integral_constant<int, 4>{});
    } else if (total > K) {
        unsigned long long prefix = 0ull;
        int want = K;   // rank (1-based) of the key looked for among the keys that share the prefix
        for (int shift = 56; shift >= 0; shift -= 8) {
            for (int b = lane; b < 256; b += 64) s_hist[b] = 0;
            __syncthreads();
            keys([&](bool ok, unsigned long long key) {
                const bool same = shift == 56 || (key >> (shift + 8)) == (prefix >> (shift + 8));
                if (ok && same) atomicAdd(&s_hist[(int)((key >> shift) & 255ull)], 1);
            });
            __syncthreads();
            // lane l owns bins 4l..4l+3; find the bin where the running count reaches `want`
            const int h0 = s_hist[4 * lane], h1 = s_hist[4 * lane + 1], h2 = s_hist[4 * lane + 2], h3 = s_hist[4 * lane + 3];
            int incl = h0 + h1 + h2 + h3;
            for (int off = 1; off < 64; off <<= 1) {
                const int v = __shfl_up(incl, off);
                if (lane >= off) incl += v;
            }
            const int before = incl - (h0 + h1 + h2 + h3);
            const bool mine = before < want && want <= incl;
            int bin = 0, below = 0;
            if (mine) {
                int c = before;
                if (want <= c + h0) { bin = 4 * lane; below = c; }
                else if (want <= c + h0 + h1) { bin = 4 * lane + 1; below = c + h0; }
                else if (want <= c + h0 + h1 + h2) { bin = 4 * lane + 2; below = c + h0 + h1; }
                else { bin = 4 * lane + 3; below = c + h0 + h1 + h2; }
            }
            const int src = __ffsll((long long)__ballot(mine)) - 1;   // exactly one lane
            bin = __shfl(bin, src);
            below = __shfl(below, src);
            prefix |= (unsigned long long)bin << shift;
            want -= below;
            __syncthreads();
        }
        thr = prefix;
    }
    if (lane == 0) {
        if (cap_d2) cap_d2[t] = (uint32_t)(thr >> 32);
        if (cap_idx) cap_idx[t] = (thr == ~0ull) ? INT_MAX : (int32_t)(thr & 0xffffffffull);
        if (count) count[ai] = total < K ? total : K;
    }
    if (table) {
        int32_t* row = table + (size_t)ai * K;
        int n_out = 0;
        walk([&](bool ok, unsigned long long key, int aj) {
            const bool take = ok && key <= thr;
            const unsigned long long mask = __ballot(take);
            if (take) row[n_out + __popcll(mask & ((1ull << lane) - 1ull))] = aj;
            n_out += __popcll(mask);
        });
        for (int x = n_out + lane; x < K; x += 64) row[x] = -1;
    }
}

}  // namespace

e2f_status e2f_launch_build_cells(const e2f_ctx* ctx, e2f_cells* c, const float* pos, const int32_t* seg_offsets,
                                  hipStream_t st) {
    const int N = c->view.N, S = c->view.S;
    if (N == 0) return E2F_OK;
    const int tb = 256;
    int32_t* cell_start = const_cast<int32_t*>(c->view.cell_start);
    const float edge = e2f_cell_edge(ctx->cfg.cutoff);
    const size_t small_lds = ((size_t)6 * S + S + 1 + c->max_cells + 1 + N) * 4 + (size_t)S * sizeof(E2fSegGrid);
    if (N <= SMALL_N && S <= SMALL_S && small_lds <= 60 * 1024) {
        k_cells_small<<<1, 1024, small_lds, st>>>(pos, seg_offsets, N, S, c->max_cells, edge, c->view.periodic ? c->box : nullptr,
                                                 const_cast<E2fSegGrid*>(c->view.grid), cell_start, const_cast<int32_t*>(c->view.perm),
                                                 const_cast<int32_t*>(c->view.scell), const_cast<int32_t*>(c->view.sseg),
                                                 const_cast<int32_t*>(c->view.atom_slot), const_cast<int4*>(c->view.sinfo));
        E2F_HIP_CHECK(hipGetLastError());
        return E2F_OK;
    }
    const int n_init = c->max_cells + 1 > S * 6 ? c->max_cells + 1 : S * 6;
    k_cells_init<<<(n_init + tb - 1) / tb, tb, 0, st>>>(c->bbox, S, cell_start, c->cell_fill, c->max_cells);
    k_cells_bbox<<<(N + 1023) / 1024, 1024, 0, st>>>(pos, seg_offsets, N, S, c->atom_seg, c->bbox);
    // edge a hair above the cutoff: the binary32 predicate can accept a pair whose exact |dx| exceeds the
    // cutoff by rounding, and cell coordinates carry rounding of their own
    k_cells_grid<<<1, 1024, 0, st>>>(c->bbox, seg_offsets, S, edge, c->view.periodic ? c->box : nullptr, const_cast<E2fSegGrid*>(c->view.grid));
    k_cells_assign<<<(N + tb - 1) / tb, tb, 0, st>>>(pos, c->atom_seg, c->view.grid, N, c->atom_cell, c->atom_sub, cell_start + 1);
    k_cells_scan<<<1, 1024, 0, st>>>(cell_start, c->view.grid, S);
    k_cells_scatter<<<(N + tb - 1) / tb, tb, 0, st>>>(c->atom_cell, cell_start, N, c->cell_fill, c->tmp_slot);
    k_cells_rank<<<(N + tb - 1) / tb, tb, 0, st>>>(c->tmp_slot, c->atom_cell, c->atom_sub, c->atom_seg, cell_start, N,
                                                  c->view.grid, const_cast<int32_t*>(c->view.perm),
                                                  const_cast<int32_t*>(c->view.scell),
                                                  const_cast<int32_t*>(c->view.sseg),
                                                  const_cast<int32_t*>(c->view.atom_slot),
                                                  const_cast<int4*>(c->view.sinfo));
    E2F_HIP_CHECK(hipGetLastError());
    return E2F_OK;
}

e2f_status e2f_launch_count_neighbors(const e2f_ctx* ctx, const E2fCellsView& cv, const float* pos, int32_t* degree,
                                      hipStream_t st) {
    if (cv.N == 0) return E2F_OK;
    if (cv.periodic) k_neighbors<false, true><<<cv.N, 64, 0, st>>>(cv, pos, ctx->rc2, degree, nullptr, nullptr);
    else k_neighbors<false, false><<<cv.N, 64, 0, st>>>(cv, pos, ctx->rc2, degree, nullptr, nullptr);
    E2F_HIP_CHECK(hipGetLastError());
    return E2F_OK;
}

e2f_status e2f_launch_list_neighbors(const e2f_ctx* ctx, const E2fCellsView& cv, const float* pos,
                                     const int64_t* offsets, int32_t* idx, hipStream_t st) {
    if (cv.N == 0) return E2F_OK;
    if (cv.periodic) k_neighbors<true, true><<<cv.N, 64, 0, st>>>(cv, pos, ctx->rc2, nullptr, offsets, idx);
    else k_neighbors<true, false><<<cv.N, 64, 0, st>>>(cv, pos, ctx->rc2, nullptr, offsets, idx);
    E2F_HIP_CHECK(hipGetLastError());
    return E2F_OK;
}

e2f_status e2f_launch_select_neighbors(const e2f_ctx* ctx, const E2fCellsView& cv, const float* pos, int32_t K,
                                       uint32_t* cap_d2, int32_t* cap_idx, int32_t* table, int32_t* count,
                                       hipStream_t st) {
    if (cv.N == 0) return E2F_OK;
    if (cv.periodic) k_select_neighbors<true><<<cv.N, 64, 0, st>>>(cv, pos, ctx->rc2, K, cap_d2, cap_idx, table, count);
    else k_select_neighbors<false><<<cv.N, 64, 0, st>>>(cv, pos, ctx->rc2, K, cap_d2, cap_idx, table, count);
    E2F_HIP_CHECK(hipGetLastError());
    return E2F_OK;
}
