// HIP kernels of the SPFD library for gfx950 (CDNA4, wave64).
//
// Paper: Sec. II (Eqs. (1), (3)), Sec. III.A (unknowns only in conducting
// voxels), Sec. III.F (voxel-averaged field).  The multigrid method replaces
// the paper's closed-library algebraic multigrid; see engine.hip.
#include <math.h>

#include "kernels.h"
#include <hip/hip_fp16.h>

namespace spfd {

// ============================================================================
// shared per-workgroup operator state
// ============================================================================

// Label-form operator, phase 1: stage the brick's 9x9x9 conductivity tile in
// LDS (two voxels per thread; the sigma table has 256 entries, zero beyond the
// labels in use, and is read through the cache).  A barrier must follow.
template <typename T>
__device__ __forceinline__ void stage_tile(const OpArgs<T> &op, int b, T *tile)
{
    const uint8_t *tl = op.tiles + (long long)b * TILE_BYTES;
    const int i0 = threadIdx.x, i1 = threadIdx.x + NT;
    const int l0 = tl[i0];
    const int l1 = i1 < TILE_VOX ? tl[i1] : 0;
    const T *table = op.models ? op.table + op.models[b * NBR + NTAB] : op.table;
    const T s0 = table[l0], s1 = table[l1];
    tile[i0] = s0;
    if (i1 < TILE_VOX) tile[i1] = s1;
}

// weights of node t (after stage_tile and a barrier for the label form)
template <typename T>
__device__ __forceinline__ void op_weights(const OpArgs<T> &op, const T *tile, long long base, int t, int tx, int ty,
                                           int tz, const long long I[6], T W[6])
{
    if (op.w)
        stored_weights(op.w, op.stride, base, t, I, W);
    else
        tile_weights(tile, tx, ty, tz, op.geo4, W);
}

template <typename T>
__device__ __forceinline__ void op_stage(const OpArgs<T> &op, int b, T *tile)
{
    if (!op.w) {
        stage_tile(op, b, tile);
        __syncthreads();
    }
}

// ============================================================================
// setup kernels
// ============================================================================

// Mark the finest-level bricks that contain a node of a conducting voxel and validate labels / conductivities
// (err: 1 = label out of table, 2 = bad sigma).  A thread takes 16 consecutive voxels (one 16-byte load of labels
// where the array is aligned), and stores the flags of the few bricks they touch where these read as unmarked: one
// voxel per thread with eight stores each was bound by the stores (250x150x900 voxels: 107 us; this form 21 us).
// Conductivities per voxel are read by the wave, 64 consecutive ones at a time, and each thread takes its 16 bits from
// the ballots: 16 FP64 loads of a thread's own run lie 128 B from the next lane's (the same body: 433 us so, one voxel per
// thread 107, this form 67; 16 packed models, 0.8 GB: 1,573, 176 and 173 us, 4.6 TB/s).
constexpr int FLAG_V = 16;

template <bool VOX>
__global__ __launch_bounds__(256) void k_brick_flags(const uint8_t *__restrict__ labels,
                                                     const double *__restrict__ table, int nlab,
                                                     const double *__restrict__ sig_vox, Grid g, uint8_t *flags,
                                                     int *err)
{
    // per label: 0 air, 1 conductor, 2 not in the table
    __shared__ uint8_t kind[256];
    if (!VOX) {
        kind[threadIdx.x] = (int)threadIdx.x < nlab ? table[threadIdx.x] > 0.0 : 2;
        __syncthreads();
    }
    const long long nvox = (long long)g.nx * g.ny * g.nz;
    const bool wide = !VOX && ((uintptr_t)labels & 15) == 0;
    const int lane = threadIdx.x & 63;
    // w0: first voxel of the wave
    for (long long w0 = ((long long)blockIdx.x * 256 + (threadIdx.x & ~63)) * FLAG_V; w0 < nvox;
         w0 += (long long)gridDim.x * 256 * FLAG_V) {
        const long long v0 = w0 + lane * FLAG_V;
        uint32_t q[4] = {0u, 0u, 0u, 0u};
        uint32_t pos = 0u;   // bit u: voxel v0 + u conducts
        if (VOX) {
            double sg[FLAG_V];
            unsigned long long bits = 0ull;   // the ballot that holds the thread's voxels
#pragma unroll
            for (int u = 0; u < FLAG_V; ++u) {
                const long long v = w0 + 64 * u + lane;
                sg[u] = sig_vox[v < nvox ? v : nvox - 1];
            }
#pragma unroll
            for (int u = 0; u < FLAG_V; ++u) {
                const bool bad = !(sg[u] >= 0.0) || !isfinite(sg[u]);
                if (bad) *err = 2;
                const unsigned long long m = __ballot(!bad && sg[u] > 0.0 && w0 + 64 * u + lane < nvox);
                if (lane >> 2 == u) bits = m;
            }
            pos = (uint32_t)(bits >> (FLAG_V * (lane & 3))) & 0xffffu;
        }
        if (v0 >= nvox) continue;
        const int n = nvox - v0 < FLAG_V ? (int)(nvox - v0) : FLAG_V;
        if (!VOX) {
            if (wide && n == FLAG_V) {
                const uint4 w = *(const uint4 *)(labels + v0);
                q[0] = w.x;
                q[1] = w.y;
                q[2] = w.z;
                q[3] = w.w;
            } else {
#pragma unroll
                for (int u = 0; u < FLAG_V; ++u) q[u / 4] |= (uint32_t)labels[u < n ? v0 + u : v0] << (8 * (u % 4));
            }
#pragma unroll
            for (int u = 0; u < FLAG_V; ++u) {
                const int k = kind[(q[u / 4] >> (8 * (u % 4))) & 255u];
                if (u < n && k == 2) *err = 1;
                if (u < n && k == 1) pos |= 1u << u;
            }
        }
        if (pos == 0u) continue;
        int i, j, k;
        if (nvox <= 0x7fffffffLL) {
            const unsigned v = (unsigned)v0, r = v / (unsigned)g.nx;
            i = (int)(v - r * (unsigned)g.nx);
            k = (int)(r / (unsigned)g.ny);
            j = (int)(r - (unsigned)k * (unsigned)g.ny);
        } else {
            const long long r = v0 / g.nx;
            i = (int)(v0 - r * g.nx);
            k = (int)(r / g.ny);
            j = (int)(r - (long long)k * g.ny);
        }
        // row by row: the nodes that conducting voxels touch, eight to a brick
        for (int left = n; left > 0;) {
            const int len = left < g.nx - i ? left : g.nx - i;
            const uint32_t p = pos & ((1u << len) - 1u);
            int bi = i >> 3;
            for (uint32_t m = (p | p << 1) << (i & 7); m != 0u; m >>= 8, ++bi)
                if (m & 255u)
                    for (int bk = k >> 3; bk <= (k + 1) >> 3; ++bk)
                        for (int bj = j >> 3; bj <= (j + 1) >> 3; ++bj) {
                            uint8_t *f = flags + bi + (long long)g.Gx * (bj + (long long)g.Gy * bk);
                            if (*f == 0) *f = 1;
                        }
            pos >>= len;
            left -= len;
            i = 0;
            if (++j == g.ny) {
                j = 0;
                ++k;
            }
        }
    }
}

__global__ void k_w16(const float *w, long long n, float inv, uint16_t *h)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        h[i] = __half_as_ushort(__float2half_rn(w[i] * inv));
}
hipError_t launch_w16(const float *w, long long n, float inv, uint16_t *h, hipStream_t s)
{
    SPFD_LAUNCH(k_w16, dim3(1024), dim3(256), 0, s, w, n, inv, h);
    return hipGetLastError();
}

hipError_t launch_brick_flags(const uint8_t *labels, const double *table, int nlab, const double *sig_vox,
                              const Grid &g, uint8_t *flags, int *err, hipStream_t s)
{
    const long long nvox = (long long)g.nx * g.ny * g.nz;
    long long blocks = (nvox + 256 * FLAG_V - 1) / (256 * FLAG_V);
    if (blocks > 65536) blocks = 65536;
    if (sig_vox)
        SPFD_LAUNCH(k_brick_flags<true>, dim3((unsigned)blocks), dim3(256), 0, s, labels, table, nlab, sig_vox, g,
                    flags, err);
    else
        SPFD_LAUNCH(k_brick_flags<false>, dim3((unsigned)blocks), dim3(256), 0, s, labels, table, nlab, sig_vox, g,
                    flags, err);
    return hipGetLastError();
}

// flags of level l from those of level l - 1 (l > 0), and the active bricks of each workgroup's cells
__global__ __launch_bounds__(TOPO_WG) void k_topo_flags(TopoLevel L, TopoLevel fine, int first)
{
    __shared__ int count[TOPO_WG / 64];
    const int i = blockIdx.x * TOPO_WG + threadIdx.x;
    int f = 0;
    if (i < L.cells) {
        if (first) {
            f = L.flags[i];
        } else {
            const int x = 2 * (i % L.G[0]), y = 2 * (i / L.G[0] % L.G[1]), z = 2 * (i / L.G[0] / L.G[1]);
            for (int k = 0; k < 8; ++k) {
                const int cx = x + (k & 1), cy = y + (k >> 1 & 1), cz = z + (k >> 2);
                if (cx < fine.G[0] && cy < fine.G[1] && cz < fine.G[2])
                    f |= fine.flags[cx + fine.G[0] * (cy + fine.G[1] * cz)];
            }
            L.flags[i] = (uint8_t)f;
        }
    }
    const unsigned long long m = __ballot(f != 0);
    if ((threadIdx.x & 63) == 0) count[threadIdx.x >> 6] = __popcll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        int sum = 0;
        for (int k = 0; k < TOPO_WG / 64; ++k) sum += count[k];
        L.part[blockIdx.x] = sum;
    }
}

// slots and coordinates of one level per launch row
__global__ __launch_bounds__(TOPO_WG) void k_topo_slots(TopoLevels t)
{
    __shared__ int count[TOPO_WG / 64];
    const TopoLevel &L = t.lv[blockIdx.y];
    if ((int)blockIdx.x * TOPO_WG >= L.cells) return;
    const int i = blockIdx.x * TOPO_WG + threadIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const bool on = i < L.cells && L.flags[i] != 0;
    const unsigned long long m = __ballot(on);
    if (lane == 0) count[wv] = __popcll(m);
    __syncthreads();
    int slot = L.part[blockIdx.x] + __popcll(m & ((1ull << lane) - 1ull));
    for (int k = 0; k < wv; ++k) slot += count[k];
    if (i >= L.cells) return;
    L.slot_of[i] = on ? slot : -1;
    if (on) L.coord[slot] = make_int4(i % L.G[0], i / L.G[0] % L.G[1], i / L.G[0] / L.G[1], 0);
}

// the six neighbours of every brick and the coarse brick that holds it (slots are complete)
__global__ __launch_bounds__(TOPO_WG) void k_topo_nbr(TopoLevels t)
{
    const int l = blockIdx.y;
    const TopoLevel &L = t.lv[l];
    const int b = blockIdx.x * TOPO_WG + threadIdx.x;
    if (b >= L.nb) return;
    const int4 c = L.coord[b];
    auto look = [&](int x, int y, int z) {
        return x < 0 || y < 0 || z < 0 || x >= L.G[0] || y >= L.G[1] || z >= L.G[2]
                   ? -1
                   : L.slot_of[x + L.G[0] * (y + L.G[1] * z)];
    };
    int *nbr = L.nbr + (long long)b * NBR;
    nbr[NTAB] = nbr[NTAB + 1] = 0;
    nbr[NMX] = look(c.x - 1, c.y, c.z);
    nbr[NPX] = look(c.x + 1, c.y, c.z);
    nbr[NMY] = look(c.x, c.y - 1, c.z);
    nbr[NPY] = look(c.x, c.y + 1, c.z);
    nbr[NMZ] = look(c.x, c.y, c.z - 1);
    nbr[NPZ] = look(c.x, c.y, c.z + 1);
    if (L.parent_slot) {
        const TopoLevel &C = t.lv[l + 1];
        L.parent_slot[b] = C.slot_of[(c.x >> 1) + C.G[0] * ((c.y >> 1) + C.G[1] * (c.z >> 1))];
    }
}

hipError_t launch_topo_count(const TopoLevels &t, int *nb, hipStream_t s)
{
    if (t.n < 1 || t.n > MAX_LEVELS) return hipErrorInvalidValue;
    for (int l = 0; l < t.n; ++l) {
        const TopoLevel &L = t.lv[l];
        const int wg = (L.cells + TOPO_WG - 1) / TOPO_WG;
        SPFD_LAUNCH(k_topo_flags, dim3(wg), dim3(TOPO_WG), 0, s, L, t.lv[l > 0 ? l - 1 : 0], l == 0);
        HIP_RETURN_IF(hipGetLastError());
        HIP_RETURN_IF(scan_small(L.part, wg, nb + l, s));
    }
    return hipSuccess;
}

hipError_t launch_topo_fill(const TopoLevels &t, hipStream_t s)
{
    if (t.n < 1 || t.n > MAX_LEVELS || t.lv[t.n - 1].parent_slot) return hipErrorInvalidValue;
    int cells = 0, nb = 0;
    for (int l = 0; l < t.n; ++l) {
        cells = t.lv[l].cells > cells ? t.lv[l].cells : cells;
        nb = t.lv[l].nb > nb ? t.lv[l].nb : nb;
    }
    if (nb <= 0) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_topo_slots, dim3((cells + TOPO_WG - 1) / TOPO_WG, t.n), dim3(TOPO_WG), 0, s, t);
    SPFD_LAUNCH(k_topo_nbr, dim3((nb + TOPO_WG - 1) / TOPO_WG, t.n), dim3(TOPO_WG), 0, s, t);
    return hipGetLastError();
}

// Masks of one brick from the eight waves' node layers, and its unknowns counted into the level's statistics
__device__ __forceinline__ void brick_masks(bool unknown, int b, unsigned long long *__restrict__ cmask,
                                            LevelStat *stat, unsigned long long nm[8])
{
    const int t = threadIdx.x;
    const unsigned long long m = __ballot(unknown);
    if ((t & 63) == 0) nm[t >> 6] = m;
    __syncthreads();
    if (t == 0) {
        unsigned long long any = 0ull;
        unsigned count = 0;
        for (int k = 0; k < 8; ++k) {
            any |= nm[k];
            count += (unsigned)__popcll(nm[k]);
        }
        cmask[b] = any;
        if (count) atomicAdd(&stat[b % LEVEL_STATS].count, count);
    }
}

// The finest level, one workgroup per brick: stored conductances M_e (Eq. (3): mean sigma of the 4 voxels sharing
// the edge times dual area / length) of the edges to +x, +y, +z (FP32 too with a conductivity per voxel), label
// tiles (label form: voxels (8 bx - 1 + a, 8 by - 1 + b, 8 bz - 1 + c), a, b, c in 0..8; outside = air (0)), inverse
// diagonals, the node columns with unknowns, bit masks of the conducting edges and of the unknowns for the
// components, and the number of unknowns.  All of it follows from the 9x9x9 voxels, staged in LDS once; as six
// kernels, of which four read the stored weights again, this was 0.54 ms at 8.9 M unknowns; in one it is 95 us, bound
// by the bytes it writes.
template <bool VOX>
__global__ __launch_bounds__(NT) void k_finest_setup(const uint8_t *__restrict__ labels,
                                                     const double *__restrict__ table,
                                                     const double *__restrict__ sig_vox, Grid g, double gx, double gy,
                                                     double gz, const int4 *__restrict__ coord, long long stride,
                                                     FinestSetup out)
{
    __shared__ double tile[TILE_VOX + 7];
    __shared__ unsigned long long nm[8];
    const int b = blockIdx.x, t = threadIdx.x;
    const int4 c = coord[b];
#pragma unroll
    for (int idx = t; idx < TILE_BYTES; idx += NT) {
        uint8_t lab = 0;
        double sg = 0.0;
        if (idx < TILE_VOX) {
            const int i = c.x * 8 - 1 + idx % 9, j = c.y * 8 - 1 + (idx / 9) % 9, k = c.z * 8 - 1 + idx / 81;
            if (i >= 0 && j >= 0 && k >= 0 && i < g.nx && j < g.ny && k < g.nz) {
                const long long v = i + (long long)g.nx * (j + (long long)g.ny * k);
                if (!VOX || out.tiles) lab = labels[v];
                sg = VOX ? sig_vox[v] : table[lab];
            }
            tile[idx] = sg;
        }
        if (!VOX || out.tiles) out.tiles[(long long)b * TILE_BYTES + idx] = lab;
    }
    __syncthreads();
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    double W[6];
    const double geo4[3] = {gx, gy, gz};
    tile_weights(tile, tx, ty, tz, geo4, W);
    const long long n = (long long)b * BS + t;
    out.w64[n] = W[NPX];
    out.w64[stride + n] = W[NPY];
    out.w64[2 * stride + n] = W[NPZ];
    if (VOX && out.w32) {
        out.w32[n] = (float)W[NPX];
        out.w32[stride + n] = (float)W[NPY];
        out.w32[2 * stride + n] = (float)W[NPZ];
    }
    double D;
    {
        // the sum of the rounded weights, as every reader of the stored ones forms it (no products fused into it)
#pragma clang fp contract(off)
        D = ((((W[0] + W[1]) + W[2]) + W[3]) + W[4]) + W[5];
    }
    const double v = D > 0.0 ? 1.0 / D : 0.0;
    if (out.dinv64) out.dinv64[n] = v;
    if (out.dinv32) out.dinv32[n] = (float)v;
    const unsigned long long ex = __ballot(W[NPX] > 0.0), ey = __ballot(W[NPY] > 0.0), ez = __ballot(W[NPZ] > 0.0);
    brick_masks(D > 0.0, b, out.cmask, out.stat, nm);
    if ((t & 63) == 0) {
        unsigned long long *e = out.emask + (long long)b * EMASK + tz;
        e[0] = ex;
        e[8] = ey;
        e[16] = ez;
        e[24] = nm[tz];
    }
}

hipError_t launch_finest_setup(const uint8_t *labels, const double *table, const double *sig_vox, const Grid &g,
                               const double geo4[3], const int4 *coord, int nb, const FinestSetup &out, hipStream_t s)
{
    if (nb <= 0) return hipSuccess;
    if (!out.tiles && !(sig_vox && out.w32)) return hipErrorInvalidValue;
    if (sig_vox)
        SPFD_LAUNCH(k_finest_setup<true>, dim3(nb), dim3(NT), 0, s, labels, table, sig_vox, g, geo4[0], geo4[1],
                    geo4[2], coord, (long long)nb * BS, out);
    else
        SPFD_LAUNCH(k_finest_setup<false>, dim3(nb), dim3(NT), 0, s, labels, table, sig_vox, g, geo4[0], geo4[1],
                    geo4[2], coord, (long long)nb * BS, out);
    return hipGetLastError();
}

// A coarse structured level from its stored weights: inverse diagonals (0 where the diagonal vanishes), the node
// columns with unknowns, the number of unknowns, and the largest and smallest positive FP32 weight
__global__ __launch_bounds__(NT) void k_struct_setup(const double *__restrict__ w, const float *__restrict__ w32,
                                                     long long stride, Topo topo, double *__restrict__ d64,
                                                     float *__restrict__ d32, unsigned long long *__restrict__ cmask,
                                                     LevelStat *stat)
{
    __shared__ unsigned long long nm[8];
    __shared__ float smax[8], smin[8];
    const int b = blockIdx.x, t = threadIdx.x;
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    int nb[6];
    brick_nbrs(topo.nbr, b, nb);
    const long long base = (long long)b * BS;
    long long I[6];
    nbr_index(base, t, tx, ty, tz, nb, I);
    double W[6];
    stored_weights(w, stride, base, t, I, W);
    float m = 0.0f, mp = INFINITY;
    for (int d = 0; d < 3; ++d) {
        const float v = w32[d * stride + base + t];
        m = fmaxf(m, v);
        if (v > 0.0f) mp = fminf(mp, v);
    }
    const double D = diag_of(W);
    const double v = D > 0.0 ? 1.0 / D : 0.0;
    if (d64) d64[base + t] = v;
    if (d32) d32[base + t] = (float)v;
    for (int off = 32; off > 0; off >>= 1) {
        m = fmaxf(m, __shfl_down(m, off, 64));
        mp = fminf(mp, __shfl_down(mp, off, 64));
    }
    if ((t & 63) == 0) {
        smax[tz] = m;
        smin[tz] = mp;
    }
    brick_masks(D > 0.0, b, cmask, stat, nm);   // (its barrier also orders smax and smin)
    if (t == 0) {
        for (int k = 0; k < 8; ++k) {
            m = fmaxf(m, smax[k]);
            mp = fminf(mp, smin[k]);
        }
        // non-negative floats order like their bit patterns; the smallest as a largest of the complements
        atomicMax(&stat[b % LEVEL_STATS].wmax, __float_as_uint(m));
        atomicMax(&stat[b % LEVEL_STATS].wmin_not, ~__float_as_uint(mp));
    }
}

hipError_t launch_struct_setup(const double *w64, const float *w32, long long stride, Topo topo, double *d64,
                               float *d32, unsigned long long *cmask, LevelStat *stat, hipStream_t s)
{
    if (topo.nb <= 0) return hipSuccess;
    SPFD_LAUNCH(k_struct_setup, dim3(topo.nb), dim3(NT), 0, s, w64, w32, stride, Topo{topo.nb, topo.nbr}, d64, d32,
                cmask, stat);
    return hipGetLastError();
}

// Galerkin coarse operator for piecewise-constant aggregation of 2x2x2 nodes:
// the coarse conductance between aggregates I and I+e_d is the sum of the four
// fine conductances that cross their interface (fine edges from the fine
// nodes 2I+1 along d).  P^T A P of a graph Laplacian is again one.
__device__ __forceinline__ double fine_w(const double *wf, long long fstride, const int *slot_of, int fGx, int fGy,
                                         int fGz, int fNx, int fNy, int fNz, int fi, int fj, int fk, int d)
{
    if (fi >= fNx || fj >= fNy || fk >= fNz) return 0.0;
    const int bi = fi >> 3, bj = fj >> 3, bk = fk >> 3;
    if (bi >= fGx || bj >= fGy || bk >= fGz) return 0.0;
    const int sl = slot_of[bi + fGx * (bj + fGy * bk)];
    if (sl < 0) return 0.0;
    return wf[d * fstride + (long long)sl * BS + (fi & 7) + 8 * (fj & 7) + 64 * (fk & 7)];
}

__global__ void k_galerkin(const double *__restrict__ wf, long long fstride, const int *__restrict__ slot_of,
                           int fGx, int fGy, int fGz, int fNx, int fNy, int fNz, const int4 *__restrict__ ccoord,
                           double *wc64, float *wc32, long long cstride)
{
    const int b = blockIdx.x, t = threadIdx.x;
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    const int4 c = ccoord[b];
    const int I = c.x * 8 + tx, J = c.y * 8 + ty, K = c.z * 8 + tz;
    double s[3];
    s[0] = ((fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I + 1, 2 * J, 2 * K, 0) +
             fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I + 1, 2 * J + 1, 2 * K, 0)) +
            fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I + 1, 2 * J, 2 * K + 1, 0)) +
           fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I + 1, 2 * J + 1, 2 * K + 1, 0);
    s[1] = ((fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I, 2 * J + 1, 2 * K, 1) +
             fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I + 1, 2 * J + 1, 2 * K, 1)) +
            fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I, 2 * J + 1, 2 * K + 1, 1)) +
           fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I + 1, 2 * J + 1, 2 * K + 1, 1);
    s[2] = ((fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I, 2 * J, 2 * K + 1, 2) +
             fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I + 1, 2 * J, 2 * K + 1, 2)) +
            fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I, 2 * J + 1, 2 * K + 1, 2)) +
           fine_w(wf, fstride, slot_of, fGx, fGy, fGz, fNx, fNy, fNz, 2 * I + 1, 2 * J + 1, 2 * K + 1, 2);
    const long long n = (long long)b * BS + t;
    for (int d = 0; d < 3; ++d) {
        wc64[d * cstride + n] = s[d];
        wc32[d * cstride + n] = (float)s[d];
    }
}

hipError_t launch_galerkin(const double *wf, long long fstride, const int *f_slot_of, int fGx, int fGy, int fGz,
                           int fNx, int fNy, int fNz, const int4 *ccoord, int cnb, double *wc64, float *wc32,
                           long long cstride, hipStream_t s)
{
    if (cnb <= 0) return hipSuccess;
    SPFD_LAUNCH(k_galerkin, dim3(cnb), dim3(NT), 0, s, wf, fstride, f_slot_of, fGx, fGy, fGz, fNx, fNy, fNz,
                       ccoord, wc64, wc32, cstride);
    return hipGetLastError();
}

// ---------------------------------------------------------------- connected components
// Union-find over the nodes with D > 0 (hook the larger root under the smaller
// with compare-and-swap, path halving on the way).  Loads and stores of the
// parent array go through L2 (agent scope) so that every lane sees the hooks.
__device__ __forceinline__ int pload(const int *p, int i)
{
    return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int pfind(int *p, int x)
{
    int px = pload(p, x);
    while (px != x) {
        const int ppx = pload(p, px);
        if (ppx != px) __hip_atomic_store(p + x, ppx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = px;
        px = ppx;
    }
    return x;
}

__device__ __forceinline__ void punite(int *p, int a, int b)
{
    while (true) {
        a = pfind(p, a);
        b = pfind(p, b);
        if (a == b) return;
        if (a > b) { const int t = a; a = b; b = t; }
        int expected = b;
        if (__hip_atomic_compare_exchange_strong(p + b, &expected, a, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return;
    }
}

// union-find in LDS over the conducting edges inside one brick
__device__ __forceinline__ int lfind(int *p, int x)
{
    int px = __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (px != x) {
        x = px;
        px = __hip_atomic_load(p + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    return x;
}

__device__ __forceinline__ void lunite(int *p, int a, int b)
{
    while (true) {
        a = lfind(p, a);
        b = lfind(p, b);
        if (a == b) return;
        if (a > b) { const int t = a; a = b; b = t; }
        int expected = b;
        if (__hip_atomic_compare_exchange_strong(p + b, &expected, a, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_WORKGROUP))
            return;
    }
}

// Components in two stages: first inside each brick (LDS, workgroup atomics),
// storing every node's brick-local root as its parent; then, after the kernel
// boundary, across the brick faces only (global union-find), so the
// device-wide atomics see short chains.
// Edges and unknowns come from the finest level's bit masks, 256 B per brick, not from its 12 KB of weights.  An
// edge that closes a square of conducting edges with the edge before it (x, or for z also y) joins nothing new: its
// union is left out, and a brick of one tissue takes 63 + 448 unions along rows instead of 1344.
__global__ void k_cc_local(const unsigned long long *__restrict__ emask, int *parent)
{
    __shared__ int lp[BS];
    const int b = blockIdx.x, t = threadIdx.x;
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    const long long base = (long long)b * BS;
    const unsigned long long *e = emask + (long long)b * EMASK + tz;
    const int lane = t & 63;
    const unsigned long long mx = e[0], my = e[8], mz = e[16], mn = e[24];
    const unsigned long long ux = tz < 7 ? e[1] : 0ull, uy = tz < 7 ? e[9] : 0ull;   // the layer above
    // left: bits of x edges that end at a node (the edge from its -x neighbour inside the brick), and so on
    const unsigned long long no_x0 = 0xfefefefefefefefeull;
    const unsigned long long in_x = (mx << 1) & no_x0, in_ux = (ux << 1) & no_x0;
    const unsigned long long in_y = my << 8, in_uy = uy << 8;
    // rows (along x) are joined by the row's own start: no unions at all
    const bool node = (mn >> lane) & 1ull;
    int start = tx;
    {
        const unsigned row = (unsigned)(in_x >> (8 * ty)) & 255u;   // bit x: joined to x - 1
        while (start > 0 && ((row >> start) & 1u)) --start;
    }
    lp[t] = node ? t - tx + start : -1;
    __syncthreads();
    // y edges: left out where the edge at x - 1 and the x edges of both rows close the square
    const unsigned long long sq_y = (my << 1) & no_x0 & in_x & (in_x >> 8);
    const unsigned long long sq_z = ((mz << 1) & no_x0 & in_x & in_ux) | ((mz << 8) & in_y & in_uy);
    if (ty < 7 && ((my & ~sq_y) >> lane) & 1ull) lunite(lp, t, t + 8);
    if (tz < 7 && ((mz & ~sq_z) >> lane) & 1ull) lunite(lp, t, t + 64);
    __syncthreads();
    parent[base + t] = node ? (int)base + lfind(lp, t) : -1;
}

// Unions across the three plus faces of a brick, one wave per brick (a lane per face node): the time is the chains
// of dependent loads, so what counts is how many bricks are in flight.  Most face edges join the same pair of
// brick-local components as the face edge next to them: a face node whose (own parent, neighbour's parent) pair
// equals that of the previous node on the face skips its union (same sets, already joined or about to be).
// (8.9 M unknowns, components of each brick and unions: 271 + 324 us with a workgroup per brick and every edge
// united, now 76 + 250 us, beside the coarsening.)
__global__ __launch_bounds__(256) void k_cc_union(const unsigned long long *__restrict__ emask, Topo topo, int *parent)
{
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (b >= topo.nb) return;
    const unsigned long long *e = emask + (long long)b * EMASK;
    const int lo = lane & 7, hi = lane >> 3;
    const int base = b * BS;
    int me[3], other[3], pm[3], po[3];
    bool edge[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int nbk = topo.nbr[b * NBR + (d == 0 ? NPX : d == 1 ? NPY : NPZ)];
        // face nodes in the order of their two other axes
        const int t = d == 0 ? 7 + 8 * lo + 64 * hi : d == 1 ? lo + 56 + 64 * hi : lane + 448;
        const unsigned long long word = e[8 * d + (d == 2 ? 7 : hi)];
        edge[d] = nbk >= 0 && ((word >> (t & 63)) & 1ull);
        me[d] = base + t;
        other[d] = nbk * BS + t - (d == 0 ? 7 : d == 1 ? 56 : 448);
        pm[d] = edge[d] ? pload(parent, me[d]) : -1;
        po[d] = edge[d] ? pload(parent, other[d]) : -1;
    }
    // previous node on the face: one step along its first axis, else its second
    const int prev = lo > 0 ? lane - 1 : hi > 0 ? lane - 8 : 0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int lm = __shfl(pm[d], prev, 64), lq = __shfl(po[d], prev, 64);
        const bool same = lane > 0 && lm == pm[d] && lq == po[d];
        if (edge[d] && !same) punite(parent, me[d], other[d]);
    }
}

__global__ void k_cc_flatten(int *parent, long long n, int *flag)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        int r = -1;
        if (pload(parent, (int)i) >= 0) r = pfind(parent, (int)i);
        flag[i] = (r == (int)i) ? 1 : 0;
    }
}

__global__ void k_cc_store_root(int *parent, long long n)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const int p = pload(parent, (int)i);
        if (p >= 0) parent[i] = pfind(parent, (int)i);
    }
}

// exclusive scan of int flags in three passes (block sums, one-block scan of
// the sums, offsets); SCAN_CHUNK elements per block
constexpr int SCAN_CHUNK = 2048;

__global__ void k_scan_blocks(const int *in, long long n, int *out, int *bsum)
{
    __shared__ int s[NT];
    const long long off = (long long)blockIdx.x * SCAN_CHUNK;
    const int t = threadIdx.x;
    int v[4], tot = 0;
    for (int q = 0; q < 4; ++q) {
        const long long i = off + t * 4 + q;
        v[q] = i < n ? in[i] : 0;
        tot += v[q];
    }
    s[t] = tot;
    __syncthreads();
    for (int d = 1; d < NT; d <<= 1) {
        const int add = t >= d ? s[t - d] : 0;
        __syncthreads();
        s[t] += add;
        __syncthreads();
    }
    int run = s[t] - tot;
    for (int q = 0; q < 4; ++q) {
        const long long i = off + t * 4 + q;
        if (i < n) out[i] = run;
        run += v[q];
    }
    if (t == NT - 1) bsum[blockIdx.x] = s[t];
}

// exclusive sums of v[0..n) in place, one workgroup: each thread a run of consecutive values, 64 sums per wave
__global__ __launch_bounds__(1024) void k_scan_sums(int *v, int n, int *total)
{
    __shared__ int wsum[16];
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int per = (n + 1023) / 1024, i0 = t * per, i1 = min(i0 + per, n);
    int sum = 0;
    for (int i = i0; i < i1; ++i) sum += v[i];
    int incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(incl, off, 64);
        if (lane >= off) incl += u;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int run = incl - sum;
    for (int k = 0; k < wv; ++k) run += wsum[k];
    if (total && t == 1023) *total = run + sum;
    for (int i = i0; i < i1; ++i) {
        const int u = v[i];
        v[i] = run;
        run += u;
    }
}

hipError_t scan_small(int *v, int n, int *total, hipStream_t s)
{
    if (n <= 0) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_scan_sums, dim3(1), dim3(1024), 0, s, v, n, total);
    return hipGetLastError();
}

__global__ void k_scan_add(int *out, long long n, const int *bsum)
{
    const long long off = (long long)blockIdx.x * SCAN_CHUNK;
    const int add = bsum[blockIdx.x];
    for (int q = threadIdx.x; q < SCAN_CHUNK; q += blockDim.x) {
        const long long i = off + q;
        if (i < n) out[i] += add;
    }
}

static hipError_t scan_exclusive(const int *in, long long n, int *out, int *bsum, int *total, hipStream_t s)
{
    const long long nblk = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    if (nblk <= 0) return hipSuccess;
    SPFD_LAUNCH(k_scan_blocks, dim3((unsigned)nblk), dim3(NT), 0, s, in, n, out, bsum);
    HIP_RETURN_IF(scan_small(bsum, (int)nblk, total, s));
    SPFD_LAUNCH(k_scan_add, dim3((unsigned)nblk), dim3(NT), 0, s, out, n, bsum);
    return hipGetLastError();
}

// one workgroup where each of its threads takes at most 16 values (its loads are 16 apart), else three launches
hipError_t scan_ints(int *v, int n, int *tmp, hipStream_t s)
{
    if (n <= 16 * 1024) return scan_small(v, n, nullptr, s);
    return scan_exclusive(v, n, v, tmp, nullptr, s);
}

__global__ void k_cc_assign(const int *__restrict__ parent, const int *__restrict__ idx, long long n, int *comp)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const int p = parent[i];
        comp[i] = p >= 0 ? idx[p] : -1;
    }
}

// scan_tmp needs (n/2048 + 1) ints
hipError_t launch_components(const unsigned long long *emask, Topo topo, int *parent, int *flag, int *idx,
                             int *scan_tmp, int *comp, int *ncomp_dev, hipStream_t s)
{
    const int nb = topo.nb;
    const long long n = (long long)nb * BS;
    if (nb <= 0) return hipSuccess;
    SPFD_LAUNCH(k_cc_local, dim3(nb), dim3(NT), 0, s, emask, parent);
    SPFD_LAUNCH(k_cc_union, dim3((nb + 3) / 4), dim3(256), 0, s, emask, topo, parent);
    const unsigned gb = (unsigned)((n + 255) / 256 > 65536 ? 65536 : (n + 255) / 256);
    SPFD_LAUNCH(k_cc_store_root, dim3(gb), dim3(256), 0, s, parent, n);
    SPFD_LAUNCH(k_cc_flatten, dim3(gb), dim3(256), 0, s, parent, n, flag);
    hipError_t e = scan_exclusive(flag, n, idx, scan_tmp, ncomp_dev, s);
    if (e != hipSuccess) return e;
    SPFD_LAUNCH(k_cc_assign, dim3(gb), dim3(256), 0, s, parent, idx, n, comp);
    return hipGetLastError();
}

__global__ void k_comp_counts(const int *__restrict__ comp, long long n, int *counts)
{
    // the first 16 component ids are counted in LDS, one global atomic per block and id
    __shared__ int local[16];
    if (threadIdx.x < 16) local[threadIdx.x] = 0;
    __syncthreads();
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const int c = comp[i];
        if (c >= 16) atomicAdd(counts + c, 1);
        else if (c >= 0) atomicAdd(local + c, 1);
    }
    __syncthreads();
    if (threadIdx.x < 16 && local[threadIdx.x]) atomicAdd(counts + threadIdx.x, local[threadIdx.x]);
}

hipError_t launch_comp_counts(const int *comp, long long n, int *counts, hipStream_t s)
{
    const unsigned gb = (unsigned)((n + 255) / 256 > 4096 ? 4096 : (n + 255) / 256);
    if (n <= 0) return hipSuccess;
    SPFD_LAUNCH(k_comp_counts, dim3(gb), dim3(256), 0, s, comp, n, counts);
    return hipGetLastError();
}

// ---------------------------------------------------------------- coarsest level
// Enumerate the unknowns (D > 0) of the coarsest level in node order, one
// workgroup; adj[dof][6] = neighbour unknowns or -1.
__global__ __launch_bounds__(1024) void k_coarse_enum(const double *__restrict__ w, long long stride, Topo topo, int *dof_of_node,
                              int *node_of_dof, int *adj, int *ndof, int maxdof)
{
    __shared__ int count[16];
    const int t = threadIdx.x;
    const long long n = (long long)topo.nb * BS;
    int carry = 0;
    for (long long base = 0; base < n; base += 1024) {
        const long long i = base + t;
        bool isdof = false;
        if (i < n) {
            const int b = (int)(i / BS), tt = (int)(i % BS);
            int tx, ty, tz;
            brick_xyz(tt, tx, ty, tz);
            double W[6];
            long long I[6];
            nbr_index((long long)b * BS, tt, tx, ty, tz, topo.nbr + b * NBR, I);
            stored_weights(w, stride, (long long)b * BS, tt, I, W);
            isdof = diag_of(W) > 0.0;
        }
        int total;
        const int id = carry + flags_before(isdof, count, &total);
        if (i < n) {
            dof_of_node[i] = isdof ? id : -1;
            if (isdof && id < maxdof) node_of_dof[id] = (int)i;
        }
        carry += total;
    }
    if (t == 0) *ndof = carry;
    __syncthreads();
    // adjacency among unknowns (only meaningful when ndof <= maxdof)
    const int nd = carry < maxdof ? carry : maxdof;
    for (int q = t; q < nd; q += blockDim.x) {
        const int i = node_of_dof[q];
        const int b = i / BS, tt = i % BS;
        int tx, ty, tz;
        brick_xyz(tt, tx, ty, tz);
        const int *nb = topo.nbr + b * NBR;
        int m[6];
        m[NMX] = tx > 0 ? i - 1 : (nb[NMX] >= 0 ? nb[NMX] * BS + tt + 7 : -1);
        m[NPX] = tx < 7 ? i + 1 : (nb[NPX] >= 0 ? nb[NPX] * BS + tt - 7 : -1);
        m[NMY] = ty > 0 ? i - 8 : (nb[NMY] >= 0 ? nb[NMY] * BS + tt + 56 : -1);
        m[NPY] = ty < 7 ? i + 8 : (nb[NPY] >= 0 ? nb[NPY] * BS + tt - 56 : -1);
        m[NMZ] = tz > 0 ? i - 64 : (nb[NMZ] >= 0 ? nb[NMZ] * BS + tt + 448 : -1);
        m[NPZ] = tz < 7 ? i + 64 : (nb[NPZ] >= 0 ? nb[NPZ] * BS + tt - 448 : -1);
        double W[6];
        long long I[6];
        nbr_index((long long)b * BS, tt, tx, ty, tz, nb, I);
        stored_weights(w, stride, (long long)b * BS, tt, I, W);
        for (int k = 0; k < 6; ++k) adj[q * 6 + k] = (m[k] >= 0 && W[k] > 0.0) ? dof_of_node[m[k]] : -1;
    }
}

hipError_t launch_coarse_setup(const double *w64, long long stride, Topo topo, int *dof_of_node, int *node_of_dof,
                               int *adj, int *ndof_dev, int maxdof, hipStream_t s)
{
    SPFD_LAUNCH(k_coarse_enum, dim3(1), dim3(1024), 0, s, w64, stride, topo, dof_of_node, node_of_dof, adj,
                       ndof_dev, maxdof);
    return hipGetLastError();
}

// Dense matrix of the coarsest structured level over its unknowns (row-major n x n), one wave per row.
__global__ __launch_bounds__(256) void k_coarse_assemble_brick(const double *__restrict__ w, long long stride, Topo topo,
                                                               const int *__restrict__ node_of_dof,
                                                               const int *__restrict__ adj, int n, double *A)
{
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (q >= n) return;
    const int i = node_of_dof[q];
    const int b = i / BS, tt = i % BS;
    int tx, ty, tz;
    brick_xyz(tt, tx, ty, tz);
    double W[6];
    long long I[6];
    nbr_index((long long)b * BS, tt, tx, ty, tz, topo.nbr + b * NBR, I);
    stored_weights(w, stride, (long long)b * BS, tt, I, W);
    int m[6];
    double d = 0.0;
    for (int k = 0; k < 6; ++k) {
        m[k] = adj[q * 6 + k];
        if (m[k] >= 0) d += W[k];
    }
    for (int c = lane; c < n; c += 64) {
        double v = c == q ? d : 0.0;
        for (int k = 0; k < 6; ++k)
            if (m[k] == c) v -= W[k];
        A[(long long)q * n + c] = v;
    }
}

// Make the coarsest matrix definite: A += sum over its connected components c
// of (mean diagonal of c / |c|) 1_c 1_c^T.  For right sides with zero sum per
// component the inverse of the result applies the pseudo-inverse and returns
// the solution with zero sum per component.  Three kernels: the sparsity
// pattern as adjacency lists (one wave per row, many workgroups), the
// components by union-find in LDS and their diagonal sums (one workgroup), the
// rank-one updates (many workgroups).  The inverse follows (kernels_dense.hip).
constexpr int CMAXADJ = 64;

struct CoarseWork {
    int *comp, *csize, *deg, *adj;  // labels, component sizes, row degree (-1: dense row), [n][CMAXADJ]
    double *cdiag;                  // diagonal sum per component (indexed by the component's label)
};

__host__ __device__ inline CoarseWork coarse_work(int n, int *work)
{
    CoarseWork w;
    w.comp = work;
    w.csize = work + n;
    w.cdiag = (double *)(work + 2 * n + ((2 * n) & 1));
    w.deg = work + 4 * n + 2;
    w.adj = w.deg + n;
    return w;
}

__global__ __launch_bounds__(256) void k_creg_pattern(int n, const double *__restrict__ A, int *work)
{
    const CoarseWork w = coarse_work(n, work);
    const int lane = threadIdx.x & 63;
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (q >= n) return;
    if (lane == 0) {
        w.comp[q] = q;
        w.csize[q] = 0;
    }
    int d = 0;
    for (int m0 = 0; m0 < n; m0 += 64) {
        const int m = m0 + lane;
        const bool nz = m < n && m != q && A[(long long)q * n + m] != 0.0;
        const unsigned long long bal = __ballot(nz);
        const int pos = d + __popcll(bal & ((1ull << lane) - 1ull));
        if (nz && d >= 0 && pos < CMAXADJ) w.adj[(long long)q * CMAXADJ + pos] = m;
        if (d >= 0) d += __popcll(bal);
        if (d > CMAXADJ) d = -1;
    }
    if (lane == 0) w.deg[q] = d;
}

// One thread per unknown (n <= 1024): union-find in LDS over the row's neighbours, the first CREG_NB of them in
// registers; the smallest unknown labels its component.  (641 unknowns: rounds of minimum labels in global memory, and
// one thread adding up the diagonals, 103 us; the rounds in LDS, and a read under the comparison, 50
// us; this form 25 us.)
constexpr int CREG_NB = 16;

__global__ __launch_bounds__(1024) void k_creg_components(int n, const double *__restrict__ A, int *work)
{
    const CoarseWork w = coarse_work(n, work);
    const int q = threadIdx.x;
    const bool in = q < n;
    __shared__ int label[1024], size[1024];
    __shared__ double sdiag[1024];
    int nb[CREG_NB];
    const int d = in ? w.deg[q] : 0;   // -1: a row with more than CMAXADJ nonzeros
#pragma unroll
    for (int k = 0; k < CREG_NB; ++k) nb[k] = k < d ? w.adj[(long long)q * CMAXADJ + k] : q;
    sdiag[q] = in ? A[(long long)q * n + q] : 0.0;
    label[q] = q;
    size[q] = 0;
    __syncthreads();
    if (in) {
        for (int k = 0; k < CREG_NB; ++k)
            if (nb[k] > q) lunite(label, q, nb[k]);
        for (int k = CREG_NB; k < d; ++k) {
            const int m = w.adj[(long long)q * CMAXADJ + k];
            if (m > q) lunite(label, q, m);
        }
        if (d < 0)   // (its neighbours of smaller index may have it in a list or not)
            for (int m = 0; m < n; ++m)
                if (m != q && A[(long long)q * n + m] != 0.0) lunite(label, q, m);
    }
    __syncthreads();
    const int root = in ? lfind(label, q) : q;
    __syncthreads();
    label[q] = root;
    __syncthreads();
    if (in) {
        w.comp[q] = label[q];
        atomicAdd(size + label[q], 1);
    }
    __syncthreads();
    if (!in) return;
    w.csize[q] = size[q];
    // diagonal sum of each component, in the order of the unknowns, by the unknown that gives it its label
    double sum = 0.0;
    if (label[q] == q) {
        for (int m0 = 0; m0 < 1024 && m0 < n; m0 += 16) {   // (labels from n on are their own)
            double v[16];
            int l[16];
#pragma unroll
            for (int m = 0; m < 16; ++m) {   // all read before any is used: a read under the comparison waits for it
                v[m] = sdiag[m0 + m];
                l[m] = label[m0 + m];
            }
#pragma unroll
            for (int m = 0; m < 16; ++m) sum += l[m] == q ? v[m] : 0.0;
        }
    }
    w.cdiag[q] = sum;
}

__global__ __launch_bounds__(256) void k_creg_update(int n, double *A, const int *work)
{
    const CoarseWork w = coarse_work(n, const_cast<int *>(work));
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < (long long)n * n;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(e / n), j = (int)(e % n);
        const int c = w.comp[i];
        if (w.comp[j] == c) {
            const double sz = (double)w.csize[c];
            A[e] += (w.cdiag[c] / sz) / sz;
        }
    }
}

hipError_t launch_coarse_assemble_brick(const double *w64, long long stride, Topo topo, const int *node_of_dof,
                                        const int *adj, int n, double *A, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    SPFD_LAUNCH(k_coarse_assemble_brick, dim3((n + 3) / 4), dim3(256), 0, s, w64, stride, topo, node_of_dof, adj, n, A);
    return hipGetLastError();
}

size_t coarse_factor_work_ints(int n) { return (size_t)(5 + CMAXADJ) * n + 8; }

hipError_t launch_coarse_factor(int n, double *A, int *work, double *dwork, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n > 1024) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_creg_pattern, dim3((n + 3) / 4), dim3(256), 0, s, n, A, work);
    SPFD_LAUNCH(k_creg_components, dim3(1), dim3(1024), 0, s, n, A, work);
    const long long nn = (long long)n * n;
    SPFD_LAUNCH(k_creg_update, dim3((unsigned)((nn + 255) / 256 > 4096 ? 4096 : (nn + 255) / 256)), dim3(256), 0, s,
                n, A, work);
    HIP_RETURN_IF(hipGetLastError());
    return launch_dense_inverse(n, A, dwork, s);
}

// ============================================================================
// solve kernels
// ============================================================================

template <typename T>
__global__ void k_fill(T *x, long long n, T v)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        x[i] = v;
}

template <typename T>
hipError_t launch_fill(T *x, long long n, T v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const unsigned gb = (unsigned)((n + 255) / 256 > 65536 ? 65536 : (n + 255) / 256);
    SPFD_LAUNCH(k_fill<T>, dim3(gb), dim3(256), 0, s, x, n, v);
    return hipGetLastError();
}
template hipError_t launch_fill<double>(double *, long long, double, hipStream_t);
template hipError_t launch_fill<float>(float *, long long, float, hipStream_t);
template hipError_t launch_fill<int>(int *, long long, int, hipStream_t);

// start of a solve: keeps ||b||^2 from the right-side kernel, arms the stop test
__global__ void k_scal_init(Scal *sc, double tol, int use_x0)
{
    (void)use_x0;
    sc += blockIdx.x;
    if (threadIdx.x == 0) {
        const double bb = sc->bb;
        sc->rz = 0.0; sc->pq = 0.0; sc->alpha = 0.0; sc->beta = 0.0; sc->zq = 0.0;
        sc->rr = bb;
        sc->tol2 = tol * tol * bb;
        sc->done = bb > 0.0 ? 0 : 1;
        sc->iters = 0; sc->status = 0; sc->hcount = 0; sc->happlied = 0; sc->stamp = 0; sc->rzn = 0.0;
    }
}

hipError_t launch_scal_init(Scal *sc, double tol, int use_x0, int nbatch, hipStream_t s)
{
    SPFD_LAUNCH(k_scal_init, dim3(nbatch), dim3(64), 0, s, sc, tol, use_x0);
    return hipGetLastError();
}

// ---------------------------------------------------------------- reductions
// Every reduction is two-stage and deterministic: each brick workgroup stores
// its partial sum with a plain store, and after the kernel boundary one
// workgroup (k_finish) sums the partials in a fixed order and updates the
// scalars of the solve.  No grid-wide fence is needed inside a kernel.

__device__ __forceinline__ double block_sum_any(double v, double *lds)
{
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) lds[wv] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0) {
        const int nw = blockDim.x >> 6;
        for (int i = 0; i < nw; ++i) s += lds[i];
    }
    __syncthreads();
    return s;
}

// rows.used: row r sums its first rows.n[r] partials (packed models: each model's own count), else n;
// the second set of partials (z.q) starts at part + n in every row
__global__ __launch_bounds__(1024) void k_finish(const double *__restrict__ part, int n, int mode, Scal *sc,
                                                 int max_iter, double *means, const int *counts, int comp, int ps,
                                                 Scal *mirror, FinRows rows, int quads, int stamp)
{
    __shared__ double red[16];
    part += (long long)blockIdx.x * ps;
    if (sc) sc += blockIdx.x;
    // a stopped right side keeps its scalars; the flag is loaded with the partials and tested after them
    // (a test first would put one more memory round trip before the loads)
    const bool may_stop =
        mode == FIN_ALPHA || mode == FIN_RR || mode == FIN_BETA0 || mode == FIN_BETA || mode == FIN_BETA_STD;
    const int stopped = may_stop ? sc->done : 0;
    const int nr = rows.used ? rows.n[blockIdx.x] : n;
    // eight independent loads in flight per thread and round, summed in a fixed order (deterministic)
    constexpr int U = 8;
    const int nt = blockDim.x;
    double a = 0.0, b = 0.0;
    for (int i0 = threadIdx.x; i0 < nr; i0 += U * nt) {
        double v[U], w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + u * nt;
            if (quads) {
                double p[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) p[k] = 4 * i + k < quads ? part[4 * i + k] : 0.0;
                v[u] = ((p[0] + p[1]) + p[2]) + p[3];
                w[u] = 0.0;
                continue;
            }
            v[u] = i < nr ? part[i] : 0.0;
            w[u] = mode == FIN_BETA && i < nr ? part[n + i] : 0.0;
        }
        a += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        b += ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7]));
    }
    if (stopped) {
        if (threadIdx.x == 0) store_mirror(mirror, sc, stamp, blockIdx.x);
        return;
    }
    a = block_sum_any(a, red);
    if (mode == FIN_BETA) b = block_sum_any(b, red);
    if (threadIdx.x != 0) return;
    switch (mode) {
    case FIN_BB:
        *sc = Scal{};   // a new right side
        sc->bb = a;
        break;
    case FIN_ALPHA: {
        sc->pq = a;
        double alpha = sc->rz / a;
        if (!(a > 0.0) || !isfinite(alpha)) {
            alpha = 0.0;
            sc->status = 6;
            sc->done = 1;
        }
        sc->alpha = alpha;
        break;
    }
    case FIN_RR:
        sc->rr = a;
        sc->iters += 1;
        sc->hcount += 1;   // the step's search direction and step size are kept
        if (a <= sc->tol2) {
            sc->done = 1;
        } else if (!isfinite(a)) {
            sc->status = 6;
            sc->done = 1;
        } else if (sc->iters >= max_iter) {
            sc->status = 5;
            sc->done = 1;
        }
        break;
    case FIN_BETA0:
    case FIN_BETA:
    case FIN_BETA_STD: {
        double beta = 0.0;
        if (mode == FIN_BETA) beta = -sc->alpha * b / sc->rz;
        if (mode == FIN_BETA_STD) beta = a / sc->rz;
        if (!(a > 0.0) || !isfinite(beta)) {
            sc->status = 6;
            sc->done = 1;
            beta = 0.0;
        }
        sc->zq = b;
        sc->rz = a;
        sc->beta = beta;
        break;
    }
    case FIN_RESID0:
        sc->rr = a;
        if (a <= sc->tol2) sc->done = 1;
        break;
    case FIN_RESID1:
        sc->zq = a;
        break;
    case FIN_MEAN:
        means[comp] = counts[comp] > 0 ? a / (double)counts[comp] : 0.0;
        break;
    }
    if (sc) store_mirror(mirror, sc, stamp, blockIdx.x);
}

hipError_t launch_finish(const double *part, int n, int mode, Scal *sc, int max_iter, hipStream_t s, double *means,
                         const int *counts, int comp, int nbatch, int ps, Scal *mirror, const FinRows *rows, int quads,
                         int stamp)
{
    if (mirror && !sc) return hipErrorInvalidValue;
    if (quads && (mode == FIN_BETA || quads > 4 * n || (rows && rows->used))) return hipErrorInvalidValue;
    if (rows && rows->used && nbatch > MAX_MODELS) return hipErrorInvalidValue;
    const FinRows fr = rows ? *rows : FinRows{};
    SPFD_LAUNCH(k_finish, dim3(nbatch), dim3(1024), 0, s, part, n, mode, sc, max_iter, means, counts, comp, ps,
                mirror, fr, quads, stamp);
    return hipGetLastError();
}

// x += sum_j alpha_j p_j over the search directions kept in the window and not yet added (slots happlied ..
// hcount-1, filled in step order), in step order: x receives the same sequence of updates as with one
// update per step, whatever the window length and whenever the updates happen.  k_hist_reset then starts
// the next window (full) or marks the directions added (an update before the window is full).
template <typename TP>
__global__ __launch_bounds__(NT) void k_x_flush(Topo topo, double *__restrict__ x, const TP *__restrict__ ph,
                                                long long hs, const double *__restrict__ ahist, int nh, long long vs,
                                                const Scal *sc)
{
    int loc, row;
    const int bk = topo_brick(topo, loc, row);
    if (bk < 0) return;
    const double *ah = ahist + (long long)row * nh;
    const int m = min(sc[row].hcount, nh);
    const int lo = max(sc[row].happlied, 0);
    if (m <= lo) return;
    // a node column without unknowns holds zeros in x and every p: nothing to read or write
    if (topo.cmask && !((topo.cmask[bk] >> (threadIdx.x & 63)) & 1ull)) return;
    const long long n = row * vs + (long long)bk * BS + threadIdx.x;
    // every direction's load in flight (fully unrolled, wave-uniform conditions: no indexed private
    // array), then the updates in step order
    double a[MAX_PHIST];
    TP pv[MAX_PHIST];
#pragma unroll
    for (int j = 0; j < MAX_PHIST; ++j) {
        a[j] = 0.0;
        pv[j] = TP(0);
        if (j >= lo && j < m) {
            a[j] = ah[j];
            pv[j] = ph[(long long)j * hs + n];
        }
    }
    double xv = x[n];
#pragma unroll
    for (int j = 0; j < MAX_PHIST; ++j)
        if (j >= lo && j < m) xv = __builtin_fma(a[j], (double)pv[j], xv);
    x[n] = xv;
}

// full: the next window starts empty; else the window goes on, its directions so far marked as added
__global__ void k_hist_reset(Scal *sc, int n, int full)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (full) {
        sc[i].hcount = 0;
        sc[i].happlied = 0;
    } else {
        sc[i].happlied = sc[i].hcount;
    }
}

template <typename TP>
hipError_t launch_x_flush(Topo topo, double *x, const TP *ph, long long hs, const double *ahist, int nh, Scal *sc,
                          const Batch &bt, hipStream_t s, int full)
{
    if (topo.nb <= 0 || bt.n <= 0) return hipSuccess;
    if (nh < 2 || nh > MAX_PHIST || !ph || !ahist || !sc) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_x_flush<TP>, topo_grid(topo, 1, bt.n), dim3(NT), 0, s, topo, x, ph, hs, ahist, nh,
                bt.vs, sc);
    SPFD_LAUNCH(k_hist_reset, dim3((bt.n + 63) / 64), dim3(64), 0, s, sc, bt.n, full);
    return hipGetLastError();
}
template hipError_t launch_x_flush<float>(Topo, double *, const float *, long long, const double *, int, Scal *,
                                          const Batch &, hipStream_t, int);
template hipError_t launch_x_flush<double>(Topo, double *, const double *, long long, const double *, int, Scal *,
                                           const Batch &, hipStream_t, int);

// r -= alpha q, ||r||^2 partials and the FP32 copy of r (x is updated once per window of steps, k_x_flush)
__global__ __launch_bounds__(NT) void k_rupdate(Topo topo, double *__restrict__ r, const double *__restrict__ q,
                                                double *part, const Scal *sc, long long vs, int ps,
                                                float *__restrict__ r32, double *ahist, int nh)
{
    __shared__ double red[8];
    int loc, row;
    const int bk = topo_brick(topo, loc, row);
    if (bk < 0) return;
    sc += row;
    // the step size of this search direction (window slot hcount), for the update of x at the window's end
    if (loc == 0 && threadIdx.x == 0 && sc->done == 0 && sc->hcount < nh) ahist[row * nh + sc->hcount] = sc->alpha;
    const long long n = row * vs + (long long)bk * BS + threadIdx.x;
    // The loads do not wait for the stop flag (a test before them would cost one more memory round
    // trip): a stopped right side loads, but stores nothing.
    const double rv = r[n], qv = q[n];
    const bool run = sc->done == 0;
    const double rn = rv - sc->alpha * qv;
    if (run) {
        r[n] = rn;
        if (r32) r32[n] = (float)rn;
    }
    const double tot = block_sum(run ? rn * rn : 0.0, red);
    if (threadIdx.x == 0 && run) part[(long long)row * ps + loc] = tot;
}

hipError_t launch_rupdate(Topo topo, double *r, const double *q, double *part, Scal *sc, const Batch &bt, float *r32,
                          hipStream_t s, double *ahist, int nh)
{
    if (topo.nb <= 0) return hipSuccess;
    if (!ahist || nh < 2 || nh > MAX_PHIST) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_rupdate, topo_grid(topo, 1, bt.n), dim3(NT), 0, s, topo, r, q, part, sc, bt.vs,
                bt.ps, r32, ahist, nh);
    return hipGetLastError();
}

// partials of r.z and z.q (flexible beta follows in k_finish), one per brick: a wave per brick, a lane per node column,
// the layers' wave sums in order.  (A workgroup per brick, a wave per layer: 16 packed models, 2.9 M unknowns, 23.6
// us; this form 8.)
constexpr int DOTS_WAVES = 4;

template <typename TZ>
__global__ __launch_bounds__(64 * DOTS_WAVES) void k_dots(Topo topo, const TZ *__restrict__ z,
                                                          const double *__restrict__ r,
                                                          const double *__restrict__ q, double *part, const Scal *sc,
                                                          int first, long long vs, int ps)
{
    int row;
    int2 range;
    const int g = topo_group(topo, DOTS_WAVES, row, range);
    if (g < 0) return;
    const int loc = g * DOTS_WAVES + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (loc >= range.y || sc[row].done) return;
    const long long n = row * vs + (long long)(range.x + loc) * BS + lane;
    part += (long long)row * ps;
    double zv[BD], a[BD];
#pragma unroll
    for (int k = 0; k < BD; ++k) zv[k] = (double)z[n + 64 * k];
#pragma unroll
    for (int k = 0; k < BD; ++k) a[k] = r[n + 64 * k];
    auto layers = [&]() {   // a: the lane's products, then the sum over the brick
        double v = wave_rows<BD>(a), sum = 0.0;
#pragma unroll
        for (int k = 0; k < BD; ++k) sum += __shfl(v, 64 / BD * k, 64);
        return sum;
    };
#pragma unroll
    for (int k = 0; k < BD; ++k) a[k] *= zv[k];
    const double rz = layers();
    double zq = 0.0;
    if (!first) {
#pragma unroll
        for (int k = 0; k < BD; ++k) a[k] = zv[k] * q[n + 64 * k];
        zq = layers();
    }
    if (lane == 0) {
        // z.q partials follow the topo_count(topo) partials of r.z
        part[loc] = rz;
        part[topo_count(topo) + loc] = zq;
    }
}

template <typename TZ>
hipError_t launch_dots(Topo topo, const TZ *z, const double *r, const double *q, double *part, Scal *sc, int first,
                       const Batch &bt, hipStream_t s)
{
    if (topo.nb <= 0) return hipSuccess;
    SPFD_LAUNCH(k_dots<TZ>, topo_grid(topo, DOTS_WAVES, bt.n), dim3(64 * DOTS_WAVES), 0, s, topo, z, r, q, part, sc,
                first, bt.vs, bt.ps);
    return hipGetLastError();
}
template hipError_t launch_dots<double>(Topo, const double *, const double *, const double *, double *, Scal *, int,
                                        const Batch &, hipStream_t);
template hipError_t launch_dots<float>(Topo, const float *, const double *, const double *, double *, Scal *, int,
                                       const Batch &, hipStream_t);

// ---------------------------------------------------------------- multigrid level kernels
__device__ __forceinline__ bool stopped(const Scal *sc)
{
    return sc && sc[blockIdx.y].done;   // set by an earlier kernel than the one that asks: a plain (scalar) load
}

// x += s * P x_c
template <typename T>
__global__ __launch_bounds__(NT) void k_prolong(Topo topo, T *__restrict__ x, const T *__restrict__ xc,
                                                const int *__restrict__ parent_slot, const int4 *__restrict__ fcoord,
                                                T scale, const Scal *sc, long long vs, long long vsc)
{
    if (stopped(sc)) return;
    const int bk = xcd_brick(blockIdx.x, topo.nb);
    if (bk < 0) return;
    x += blockIdx.y * vs;
    xc += blockIdx.y * vsc;
    const int t = threadIdx.x;
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    const int4 c = fcoord[bk];
    const int cxl = (c.x & 1) * 4 + (tx >> 1), cyl = (c.y & 1) * 4 + (ty >> 1), czl = (c.z & 1) * 4 + (tz >> 1);
    const long long n = (long long)bk * BS + t;
    x[n] += scale * xc[(long long)parent_slot[bk] * BS + cxl + 8 * cyl + 64 * czl];
}

// coarsest solve z_c = A_c^+ r_c (dense FP64 GEMV); 4 rows per workgroup of 256
template <typename T, typename TB>
__global__ __launch_bounds__(256) void k_coarse_apply(const TB *__restrict__ bc, T *__restrict__ xc,
                                                      const double *__restrict__ Ainv,
                                                      const int *__restrict__ node_of_dof, int n, const Scal *sc,
                                                      long long vs)
{
    __shared__ double rv[1024];
    bc += blockIdx.y * vs;
    xc += blockIdx.y * vs;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + wv;
    // the wave's row of the inverse is loaded first (n <= 1024: 16 values per
    // lane), in flight together with the gather of b_c and the stop flag
    const double *a = Ainv + (long long)(row < n ? row : n - 1) * n;
    double av[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int j = lane + 64 * k;
        av[k] = a[j < n ? j : n - 1];
    }
    for (int i = threadIdx.x; i < n; i += blockDim.x) rv[i] = (double)bc[node_of_dof[i]];
    const bool stop = stopped(sc);
    __syncthreads();
    if (stop || row >= n) return;
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int j = lane + 64 * k;
        if (j < n) s += av[k] * rv[j];
    }
    s = wave_sum(s);
    if (lane == 0) xc[node_of_dof[row]] = (T)s;
}

template <typename T>
hipError_t launch_prolong(Topo topo, T *x, const T *xc, const int *parent_slot, const int4 *fcoord, T scale,
                          const Scal *sc, const Batch &bt, hipStream_t s)
{
    if (topo.nb <= 0) return hipSuccess;
    SPFD_LAUNCH(k_prolong<T>, dim3(xcd_grid(topo.nb), bt.n), dim3(NT), 0, s, topo, x, xc, parent_slot, fcoord,
                       scale, sc, bt.vs, bt.vsc);
    return hipGetLastError();
}

template <typename T, typename TB>
hipError_t launch_coarse_apply(const TB *bc, T *xc, const double *Ainv, const int *node_of_dof, int n, const Scal *sc,
                               const Batch &bt, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n > 1024) return hipErrorInvalidValue;
    SPFD_LAUNCH((k_coarse_apply<T, TB>), dim3((n + 3) / 4, bt.n), dim3(256), 0, s, bc, xc, Ainv, node_of_dof, n,
                       sc, bt.vs);
    return hipGetLastError();
}

template hipError_t launch_prolong<double>(Topo, double *, const double *, const int *, const int4 *, double,
                                           const Scal *, const Batch &, hipStream_t);
template hipError_t launch_prolong<float>(Topo, float *, const float *, const int *, const int4 *, float, const Scal *,
                                          const Batch &, hipStream_t);
template hipError_t launch_coarse_apply<double, double>(const double *, double *, const double *, const int *, int,
                                                        const Scal *, const Batch &, hipStream_t);
template hipError_t launch_coarse_apply<float, float>(const float *, float *, const double *, const int *, int,
                                                      const Scal *, const Batch &, hipStream_t);
template hipError_t launch_coarse_apply<float, double>(const double *, float *, const double *, const int *, int,
                                                       const Scal *, const Batch &, hipStream_t);

// ============================================================================
// gauge, output, post-processing
// ============================================================================

// Component means in a fixed summation order (bitwise reproducible for any
// number of components): up to COMP_PASS components per pass; every brick
// workgroup forms the sum of each component over its 512 nodes (wave sums,
// then the eight waves in order) and stores one partial per (component,
// brick); one workgroup per component then adds its partials in brick order.
constexpr int COMP_PASS = 16;

__global__ __launch_bounds__(NT) void k_comp_sum(Topo topo, const double *__restrict__ x, const int *__restrict__ comp,
                                                 int c0, int nk, double *part)
{
    __shared__ double red[COMP_PASS][NT / 64];
    const int bk = xcd_brick(blockIdx.x, topo.nb);
    if (bk < 0) return;
    const long long n = (long long)bk * BS + threadIdx.x;
    const int c = comp[n] - c0;
    const double v = x[n];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    for (int k = 0; k < nk; ++k) {
        // (few components meet in a wave: the sum of the others' zeros is not formed.  16 packed models, 24.6 k
        // bricks: 116 us with all 16 sums in every wave, now 19)
        const double t = __any(c == k) ? wave_sum(c == k ? v : 0.0) : 0.0;
        if (lane == 0) red[k][wv] = t;
    }
    __syncthreads();
    if ((int)threadIdx.x < nk) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) t += red[threadIdx.x][w];
        part[(long long)threadIdx.x * topo.nb + bk] = t;
    }
}

// mean of component c0 + blockIdx.x: its nb partials summed in a fixed order
__global__ __launch_bounds__(1024) void k_comp_finish(const double *__restrict__ part, int nb, int c0,
                                                      const int *__restrict__ counts, double *means)
{
    __shared__ double red[16];
    const int k = blockIdx.x;
    const double *p = part + (long long)k * nb;
    double t = 0.0;
    for (int i = threadIdx.x; i < nb; i += blockDim.x) t += p[i];
    t = wave_sum(t);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
        const int cnt = counts[c0 + k];
        means[c0 + k] = cnt > 0 ? s / (double)cnt : 0.0;
    }
}

size_t comp_mean_parts(int nb) { return (size_t)COMP_PASS * (nb > 0 ? nb : 1); }

hipError_t launch_comp_mean(Topo topo, const double *x, const int *comp, int ncomp, const int *counts, double *means,
                            double *part, hipStream_t s)
{
    if (topo.nb <= 0 || ncomp <= 0) return hipSuccess;
    for (int c0 = 0; c0 < ncomp; c0 += COMP_PASS) {
        const int nk = ncomp - c0 < COMP_PASS ? ncomp - c0 : COMP_PASS;
        SPFD_LAUNCH(k_comp_sum, dim3(xcd_grid(topo.nb)), dim3(NT), 0, s, topo, x, comp, c0, nk, part);
        SPFD_LAUNCH(k_comp_finish, dim3(nk), dim3(1024), 0, s, part, topo.nb, c0, counts, means);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- several voxel models in one handle
// model m's labels (nx, ny, nz voxels) into the packed label grid (NX, NY voxels per layer) from voxel
// layer zoff on; the rest of the packed grid stays as it is (air)
__global__ void k_pack_labels(const uint8_t *__restrict__ src, int nx, int ny, int nz, uint8_t *__restrict__ dst,
                              int NX, int NY, int zoff)
{
    const long long n = (long long)nx * ny * nz;
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(v % nx), j = (int)((v / nx) % ny), k = (int)(v / ((long long)nx * ny));
        dst[i + (long long)NX * (j + (long long)NY * (k + zoff))] = src[v];
    }
}

hipError_t launch_pack_labels(const uint8_t *src, int nx, int ny, int nz, uint8_t *dst, int NX, int NY, int zoff,
                              hipStream_t s)
{
    const long long n = (long long)nx * ny * nz;
    const unsigned gb = (unsigned)((n + 255) / 256 > 65536 ? 65536 : (n + 255) / 256);
    SPFD_LAUNCH(k_pack_labels, dim3(gb), dim3(256), 0, s, src, nx, ny, nz, dst, NX, NY, zoff);
    return hipGetLastError();
}

// conductivity of every voxel of the packed grid: its model's table at its label (tables [np][256]),
// 0 outside every model's box
__global__ void k_pack_sigma(const uint8_t *__restrict__ labels, Grid g, ModelBoxes mb,
                             const double *__restrict__ tables, double *__restrict__ sig)
{
    const long long n = (long long)g.nx * g.ny * g.nz;
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(v % g.nx), j = (int)((v / g.nx) % g.ny), k = (int)(v / ((long long)g.nx * g.ny));
        double sv = 0.0;
        for (int m = 0; m < mb.np; ++m)
            if (k >= mb.zoff[m] && k < mb.zoff[m] + mb.nz[m] && i < mb.nx[m] && j < mb.ny[m])
                sv = tables[m * MAX_LABELS + labels[v]];
        sig[v] = sv;
    }
}

__global__ __launch_bounds__(256) void k_brick_models(const int4 *__restrict__ coord, int nb, ModelBoxes mb,
                                                      int *__restrict__ nbr)
{
    const int b = blockIdx.x * 256 + threadIdx.x;
    if (b >= nb) return;
    const int z0 = coord[b].z * BD;
    int m = 0;
    while (m + 1 < mb.np && z0 >= mb.zoff[m + 1]) ++m;
    nbr[b * NBR + NTAB] = m * MAX_LABELS;
}

hipError_t launch_brick_models(const int4 *coord, int nb, const ModelBoxes &mb, int *nbr, hipStream_t s)
{
    if (nb <= 0 || mb.np < 1) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_brick_models, dim3((nb + 255) / 256), dim3(256), 0, s, coord, nb, mb, nbr);
    return hipGetLastError();
}

hipError_t launch_pack_sigma(const uint8_t *labels, const Grid &g, const ModelBoxes &mb, const double *tables,
                             double *sig, hipStream_t s)
{
    const long long n = (long long)g.nx * g.ny * g.nz;
    const unsigned gb = (unsigned)((n + 255) / 256 > 65536 ? 65536 : (n + 255) / 256);
    SPFD_LAUNCH(k_pack_sigma, dim3(gb), dim3(256), 0, s, labels, g, mb, tables, sig);
    return hipGetLastError();
}

// dense node array from the brick layout: psi = x - mean(component), 0 outside the conductor.  g: the grid of the
// output and of the brick layout; with packed models (MODELS, one launch row each) g is the packed grid and the
// models' own grids come from `models`.
constexpr int PSI_ROWS = 8;   // node rows per workgroup: the eight y rows of one brick row

template <bool MODELS>
__global__ __launch_bounds__(256) void k_psi_out(const double *__restrict__ x, const int *__restrict__ comp,
                                                 const double *__restrict__ means, const int *__restrict__ slot_of,
                                                 Grid g, const ModelOut *__restrict__ models, double *psi)
{
    // workgroup: node rows j0..j0+7 of layer k (contiguous stores, no 64-bit index division).  The eight
    // rows lie in the same bricks, so one slot lookup per lane serves all of them, and each lane keeps the
    // eight rows' loads in flight together.  Rows past the grid's end (the last brick row) are loaded, as
    // they lie inside their bricks, but not stored.
    ModelOut o{g.Nx, g.Ny, g.Nz, 0, 0};
    if (MODELS) o = models[blockIdx.y];
    const int gy = (o.Ny + PSI_ROWS - 1) / PSI_ROWS;
    const int jb = blockIdx.x % gy, k = blockIdx.x / gy;
    if (MODELS && k >= o.Nz) return;
    const int kb = k + o.zoff, j0 = jb * PSI_ROWS;
    const int nr = o.Ny - j0 < PSI_ROWS ? o.Ny - j0 : PSI_ROWS;
    const int *srow = slot_of + g.Gx * (jb + g.Gy * (kb >> 3));
    double *prow = psi + o.at + ((long long)k * o.Ny + j0) * o.Nx;
    for (int i = threadIdx.x; i < o.Nx; i += blockDim.x) {
        const int sl = srow[i >> 3];
        // slot 0 stands in outside the bricks; the values are masked below
        const long long base = sl >= 0 ? (long long)sl * BS + (i & 7) + 64 * (kb & 7) : 0;
        int c[PSI_ROWS];
        double xv[PSI_ROWS];
#pragma unroll
        for (int r = 0; r < PSI_ROWS; ++r) {
            const long long idx = sl >= 0 ? base + 8 * r : 0;
            c[r] = comp[idx];
            xv[r] = x[idx];
        }
#pragma unroll
        for (int r = 0; r < PSI_ROWS; ++r) {
            const double m = means[c[r] >= 0 ? c[r] : 0];
            if (r < nr) prow[(long long)r * o.Nx + i] = (sl >= 0 && c[r] >= 0) ? xv[r] - m : 0.0;
        }
    }
}

hipError_t launch_psi_out(const double *x, const int *comp, const double *means, const int *slot_of, const Grid &g,
                          double *psi, hipStream_t s, const ModelOut *models, int nmodels, int groups_most)
{
    if (models) {
        if (nmodels < 1 || groups_most < 1) return hipErrorInvalidValue;
        SPFD_LAUNCH(k_psi_out<true>, dim3(groups_most, nmodels), dim3(256), 0, s, x, comp, means, slot_of, g, models,
                    psi);
        return hipGetLastError();
    }
    const long long groups = (long long)psi_groups(g.Ny, g.Nz);
    if (groups <= 0 || g.Nx <= 0) return hipSuccess;
    SPFD_LAUNCH(k_psi_out<false>, dim3((unsigned)groups), dim3(256), 0, s, x, comp, means, slot_of, g, nullptr, psi);
    return hipGetLastError();
}

int psi_groups(int Ny, int Nz) { return (Ny + PSI_ROWS - 1) / PSI_ROWS * Nz; }

// start of a solve from x = 0: x = 0, r = b (right side i at b + i*bvs, vectors at i*n) and, for an
// FP32 cycle, the FP32 copy of r that the first cycle reads
__global__ void k_start(long long n, const double *__restrict__ b, long long bvs, double *__restrict__ x,
                        double *__restrict__ r, float *__restrict__ r32, const float *__restrict__ dinv)
{
    const long long off = (long long)blockIdx.y * n;
    b += (long long)blockIdx.y * bvs;
    for (long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (long long)gridDim.x * blockDim.x) {
        const double v = b[k];
        x[off + k] = 0.0;
        r[off + k] = v;
        if (r32) r32[off + k] = dinv ? (float)(v * (double)dinv[k]) : (float)v;
    }
}

hipError_t launch_start(long long n, const double *b, long long bvs, double *x, double *r, float *r32, int nvec,
                        hipStream_t s, const float *dinv)
{
    if (n <= 0 || nvec <= 0) return hipSuccess;
    if (dinv && !r32) return hipErrorInvalidValue;
    const long long blocks = (n + 255) / 256;
    SPFD_LAUNCH(k_start, dim3((unsigned)(blocks > 65536 ? 65536 : blocks), nvec), dim3(256), 0, s, n, b, bvs, x, r, r32,
                dinv);
    return hipGetLastError();
}

// brick layout from a dense node array (start iterate), 0 outside the conductor
__global__ void k_psi_in(const double *__restrict__ psi, const int *__restrict__ comp, const int4 *__restrict__ coord,
                         Grid g, double *x)
{
    const int b = blockIdx.x, t = threadIdx.x;
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    const int4 c = coord[b];
    const int i = c.x * 8 + tx, j = c.y * 8 + ty, k = c.z * 8 + tz;
    const long long idx = (long long)b * BS + t;
    double v = 0.0;
    if (comp[idx] >= 0) v = psi[i + (long long)g.Nx * (j + (long long)g.Ny * k)];
    x[idx] = v;
}

hipError_t launch_psi_in(const double *psi, const int *comp, const int4 *coord, int nb, const Grid &g, double *x,
                         hipStream_t s)
{
    if (nb <= 0) return hipSuccess;
    SPFD_LAUNCH(k_psi_in, dim3(nb), dim3(NT), 0, s, psi, comp, coord, g, x);
    return hipGetLastError();
}

// Columns of FCOL layers: the lanes of a workgroup hold consecutive (i, j) of a layer (contiguous loads and
// stores, one division per thread, no idle lanes at the row ends), each for FCOL layers of z.  What
// neighbouring layers share (voxel flags, potentials, edge voltages) is read once, and all loads of a thread
// are in flight together.  A layer has fewer than 2^32 columns (a grid of two node layers has at most 2^33 - 4 nodes),
// so a column is counted in 32 bits without a sign; the blocks of layers go along the launch's y dimension, in several
// launches where they are more than it takes.
constexpr int FCOL = 4;
constexpr int FCOL_T = 256;
constexpr int FCOL_Y = 65535;   // most workgroups along y

// LAUNCH(grid, first block of layers) over the columns of an nx x ny layer and the blocks of nz layers
template <typename F>
static hipError_t launch_columns(int nx, int ny, int nz, const F &launch)
{
    if (nx <= 0 || ny <= 0 || nz <= 0) return hipSuccess;
    const unsigned long long cols = (unsigned long long)nx * ny;
    if (cols > 0xffffffffull) return hipErrorInvalidValue;
    const int blocks = nz / FCOL + (nz % FCOL != 0);
    for (int b0 = 0; b0 < blocks; b0 += FCOL_Y) {
        launch(dim3((unsigned)((cols + FCOL_T - 1) / FCOL_T), (unsigned)(blocks - b0 < FCOL_Y ? blocks - b0 : FCOL_Y)),
               b0);
        HIP_RETURN_IF(hipGetLastError());
    }
    return hipSuccess;
}

// cond[l]: label l conducts (all threads of the workgroup call this)
__device__ __forceinline__ void stage_cond(const double *__restrict__ table, bool per_voxel, unsigned char *cond)
{
    if (!per_voxel)
        for (int l = threadIdx.x; l < MAX_LABELS; l += blockDim.x) cond[l] = table[l] > 0.0;
    __syncthreads();
}

// the FCOL voxels (i, j, k0 ..) of a column as bits (bit m: layer k0 + m conducts; 0 outside the grid)
__device__ __forceinline__ unsigned col_cond(const uint8_t *__restrict__ labels, const double *__restrict__ sig_vox,
                                             const unsigned char *cond, const Grid &g, int i, int j, int k0, int n)
{
    const bool in = i >= 0 && i < g.nx && j >= 0 && j < g.ny;
    const long long plane = (long long)g.nx * g.ny;
    const long long base = (in ? i + (long long)g.nx * j : 0) + plane * (k0 > 0 ? k0 : 0);
    unsigned bits = 0u;
    if (sig_vox) {
        double v[FCOL + 1];
#pragma unroll
        for (int m = 0; m <= FCOL; ++m) {
            const int k = k0 + m;
            v[m] = (in && m < n && k >= 0 && k < g.nz) ? sig_vox[base + plane * (k0 >= 0 ? m : m - 1)] : 0.0;
        }
#pragma unroll
        for (int m = 0; m <= FCOL; ++m) bits |= (v[m] > 0.0 ? 1u : 0u) << m;
    } else {
        int l[FCOL + 1];
#pragma unroll
        for (int m = 0; m <= FCOL; ++m) {
            const int k = k0 + m;
            l[m] = (in && m < n && k >= 0 && k < g.nz) ? labels[base + plane * (k0 >= 0 ? m : m - 1)] : -1;
        }
#pragma unroll
        for (int m = 0; m <= FCOL; ++m) bits |= (l[m] >= 0 && cond[l[m] >= 0 ? l[m] : 0] ? 1u : 0u) << m;
    }
    return bits;
}

// Eq. (1) and the voxel average: for a conducting voxel, u = a + G psi on its
// twelve edges (all conducting), ubar_d = mean of the four d-edges and
// |E| = omega * sqrt(sum (ubar_d / h_d)^2); air voxels get 0.  Bound by memory
// (labels and |E| of every voxel, a and psi of the conductor).  A layer adds
// twelve loads per voxel to those of the layer below, against twenty for a
// voxel on its own, and the voxels' loads no longer wait one after the other
// behind label and conductivity (250 x 150 x 900 body: 243 -> 197 us).
__global__ __launch_bounds__(FCOL_T) void k_efield(const uint8_t *__restrict__ labels, const double *__restrict__ table,
                                                   const double *__restrict__ sig_vox, Grid g, double hx, double hy,
                                                   double hz, double omega, const double *__restrict__ a,
                                                   const double *__restrict__ psi, double *__restrict__ emag, int b0)
{
    __shared__ unsigned char cond[MAX_LABELS];
    stage_cond(table, sig_vox != nullptr, cond);
    const unsigned e = blockIdx.x * FCOL_T + threadIdx.x;
    if (e >= (unsigned)g.nx * (unsigned)g.ny) return;
    const int i = (int)(e % (unsigned)g.nx), j = (int)(e / (unsigned)g.nx), k0 = (b0 + (int)blockIdx.y) * FCOL;
    const int nk = g.nz - k0 < FCOL ? g.nz - k0 : FCOL;
    const long long nn = (long long)g.Nx * g.Ny * g.Nz;
    const long long sy = g.Nx, sz = (long long)g.Nx * g.Ny;
    const long long vplane = (long long)g.nx * g.ny;
    const unsigned bits = col_cond(labels, sig_vox, cond, g, i, j, k0, nk);
    double out[FCOL];
#pragma unroll
    for (int m = 0; m < FCOL; ++m) out[m] = 0.0;
    if (bits) {
        const long long n0 = i + sy * j + sz * k0;
        // layers of the column that are read: nodes k0 .. k0 + nk
        double p[FCOL + 1][4], ax[FCOL + 1][2], ay[FCOL + 1][2], az[FCOL][4];
#pragma unroll
        for (int m = 0; m <= FCOL; ++m) {
            const long long n = n0 + sz * (m < nk ? m : nk);
            p[m][0] = psi[n];
            p[m][1] = psi[n + 1];
            p[m][2] = psi[n + sy];
            p[m][3] = psi[n + sy + 1];
            ax[m][0] = a[n];
            ax[m][1] = a[n + sy];
            ay[m][0] = a[nn + n];
            ay[m][1] = a[nn + n + 1];
        }
#pragma unroll
        for (int m = 0; m < FCOL; ++m) {
            const long long n = 2 * nn + n0 + sz * (m < nk ? m : nk - 1);
            az[m][0] = a[n];
            az[m][1] = a[n + 1];
            az[m][2] = a[n + sy];
            az[m][3] = a[n + sy + 1];
        }
        auto ux = [&](int m, int y) { return (ax[m][y] + p[m][2 * y + 1]) - p[m][2 * y]; };
        auto uy = [&](int m, int x) { return (ay[m][x] + p[m][2 + x]) - p[m][x]; };
#pragma unroll
        for (int m = 0; m < FCOL; ++m) {
            const double sx = ((ux(m, 0) + ux(m, 1)) + ux(m + 1, 0)) + ux(m + 1, 1);
            const double sv = ((uy(m, 0) + uy(m, 1)) + uy(m + 1, 0)) + uy(m + 1, 1);
            double sw = 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) sw += (az[m][q] + p[m + 1][q]) - p[m][q];
            const double fx = 0.25 * sx / hx, fy = 0.25 * sv / hy, fz = 0.25 * sw / hz;
            if ((bits >> m) & 1u) out[m] = omega * sqrt(fx * fx + fy * fy + fz * fz);
        }
    }
#pragma unroll
    for (int m = 0; m < FCOL; ++m)
        if (m < nk) emag[e + vplane * (k0 + m)] = out[m];
}

hipError_t launch_efield(const uint8_t *labels, const double *table, const double *sig_vox, const Grid &g,
                         const double h[3], double omega, const double *a, const double *psi, double *emag,
                         hipStream_t s)
{
    return launch_columns(g.nx, g.ny, g.nz, [&](dim3 grid, int b0) {
        SPFD_LAUNCH(k_efield, grid, dim3(FCOL_T), 0, s, labels, table, sig_vox, g, h[0], h[1], h[2], omega, a, psi,
                    emag, b0);
    });
}

// u = a + G psi on conducting edges (any of the four voxels around the edge conducts), 0 elsewhere.  Bound by
// the 24 bytes stored per node of the whole grid (250 x 150 x 900 body: 719 us with twelve label lookups
// per node, 278 us now, 4.1 TB/s).
__global__ __launch_bounds__(FCOL_T) void k_uedges(const uint8_t *__restrict__ labels, const double *__restrict__ table,
                                                   const double *__restrict__ sig_vox, Grid g,
                                                   const double *__restrict__ a, const double *__restrict__ psi,
                                                   double *__restrict__ u, int b0)
{
    __shared__ unsigned char cond[MAX_LABELS];
    stage_cond(table, sig_vox != nullptr, cond);
    const unsigned e = blockIdx.x * FCOL_T + threadIdx.x;
    if (e >= (unsigned)g.Nx * (unsigned)g.Ny) return;
    const int i = (int)(e % (unsigned)g.Nx), j = (int)(e / (unsigned)g.Nx), k0 = (b0 + (int)blockIdx.y) * FCOL;
    const int nk = g.Nz - k0 < FCOL ? g.Nz - k0 : FCOL;
    const long long nn = (long long)g.Nx * g.Ny * g.Nz;
    const long long sy = g.Nx, sz = (long long)g.Nx * g.Ny;
    // voxel columns around the node column, bit m: layer k0 - 1 + m
    const unsigned c00 = col_cond(labels, sig_vox, cond, g, i - 1, j - 1, k0 - 1, nk + 1);
    const unsigned c10 = col_cond(labels, sig_vox, cond, g, i, j - 1, k0 - 1, nk + 1);
    const unsigned c01 = col_cond(labels, sig_vox, cond, g, i - 1, j, k0 - 1, nk + 1);
    const unsigned c11 = col_cond(labels, sig_vox, cond, g, i, j, k0 - 1, nk + 1);
    // x-edges of layer k0 + m: voxels (i, j-1..j, k-1..k); y: (i-1..i, j, k-1..k); z: (i-1..i, j-1..j, k)
    const unsigned ex = (c10 | c11) | ((c10 | c11) >> 1), ey = (c01 | c11) | ((c01 | c11) >> 1);
    const unsigned ez = (c00 | c10 | c01 | c11) >> 1;
    double ux[FCOL], uy[FCOL], uz[FCOL];
#pragma unroll
    for (int m = 0; m < FCOL; ++m) ux[m] = uy[m] = uz[m] = 0.0;
    if (ex | ey | ez) {
        const long long n0 = e + sz * k0;
        double p[FCOL + 1], px[FCOL], py[FCOL], av[3][FCOL];
        // an edge that leaves the grid has no conducting voxel: a stand-in index is read there
#pragma unroll
        for (int m = 0; m < FCOL; ++m) {
            const long long n = n0 + sz * (m < nk ? m : 0);
            p[m] = psi[n];
            px[m] = psi[n + (i < g.nx ? 1 : 0)];
            py[m] = psi[n + (j < g.ny ? sy : 0)];
            av[0][m] = a[n];
            av[1][m] = a[nn + n];
            av[2][m] = a[2 * nn + n];
        }
        p[FCOL] = psi[n0 + sz * (k0 + FCOL < g.Nz ? FCOL : 0)];
#pragma unroll
        for (int m = 0; m < FCOL; ++m) {
            if ((ex >> m) & 1u) ux[m] = (av[0][m] + px[m]) - p[m];
            if ((ey >> m) & 1u) uy[m] = (av[1][m] + py[m]) - p[m];
            if ((ez >> m) & 1u) uz[m] = (av[2][m] + p[m + 1]) - p[m];
        }
    }
#pragma unroll
    for (int m = 0; m < FCOL; ++m)
        if (m < nk) {
            const long long n = e + sz * (k0 + m);
            u[n] = ux[m];
            u[nn + n] = uy[m];
            u[2 * nn + n] = uz[m];
        }
}

hipError_t launch_uedges(const uint8_t *labels, const double *table, const double *sig_vox, const Grid &g,
                         const double *a, const double *psi, double *u, hipStream_t s)
{
    return launch_columns(g.Nx, g.Ny, g.Nz, [&](dim3 grid, int b0) {
        SPFD_LAUNCH(k_uedges, grid, dim3(FCOL_T), 0, s, labels, table, sig_vox, g, a, psi, u, b0);
    });
}

}  // namespace spfd

namespace spfd {

// ============================================================================
// adjoint gradient of an objective J(|E|) with respect to the conductivities
// ============================================================================
// With A Psi = -G^T M a, u = a + G Psi and dA = G^T dM G, a change of M gives
// A dPsi = -G^T dM u; for dJ = g^T du = (G^T g)^T dPsi the adjoint solve
// A lambda = G^T g yields dJ = -(G lambda)^T dM u, and dM_e/dsigma_v = (dual
// area / length)/4 for the four voxels v around edge e.

// per conducting voxel: c_d = dJ/d|E| * omega^2 * ubar_d / (4 h_d^2 |E|), the
// derivative of J with respect to each of the voxel's four d-edge voltages
__global__ void k_adj_voxel(const uint8_t *__restrict__ labels, const double *__restrict__ table,
                            const double *__restrict__ sig_vox, Grid g, double hx, double hy, double hz, double omega,
                            const double *__restrict__ a, const double *__restrict__ psi,
                            const double *__restrict__ grad_emag, double *c)
{
    const long long nvox = (long long)g.nx * g.ny * g.nz;
    const long long nn = (long long)g.Nx * g.Ny * g.Nz;
    const long long sy = g.Nx, sz = (long long)g.Nx * g.Ny;
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (long long)gridDim.x * blockDim.x) {
        const double s = sig_vox ? sig_vox[v] : table[labels[v]];
        double cx = 0.0, cy = 0.0, cz = 0.0;
        if (s > 0.0) {
            const long long i = v % g.nx, j = (v / g.nx) % g.ny, k = v / ((long long)g.nx * g.ny);
            const long long n0 = i + g.Nx * (j + (long long)g.Ny * k);
            const long long ex[4] = {n0, n0 + sy, n0 + sz, n0 + sy + sz};
            const long long ey[4] = {n0, n0 + 1, n0 + sz, n0 + 1 + sz};
            const long long ez[4] = {n0, n0 + 1, n0 + sy, n0 + 1 + sy};
            double ux = 0.0, uy = 0.0, uz = 0.0;
            for (int q = 0; q < 4; ++q) {
                ux += (a[ex[q]] + psi[ex[q] + 1]) - psi[ex[q]];
                uy += (a[nn + ey[q]] + psi[ey[q] + sy]) - psi[ey[q]];
                uz += (a[2 * nn + ez[q]] + psi[ez[q] + sz]) - psi[ez[q]];
            }
            const double fx = 0.25 * ux / hx, fy = 0.25 * uy / hy, fz = 0.25 * uz / hz;
            const double E = omega * sqrt(fx * fx + fy * fy + fz * fz);
            if (E > 0.0) {
                const double ge = grad_emag[v];
                cx = ge * omega * omega * (0.25 * ux) / (4.0 * hx * hx * E);
                cy = ge * omega * omega * (0.25 * uy) / (4.0 * hy * hy * E);
                cz = ge * omega * omega * (0.25 * uz) / (4.0 * hz * hz * E);
            }
        }
        c[v] = cx;
        c[nvox + v] = cy;
        c[2 * nvox + v] = cz;
    }
}

// adjoint right side at the nodes: (G^T g)_n, where each of the 8 voxels
// around n passes its d-edge through n; n is the head of that edge when the
// voxel lies on the minus side along d (+c) and its tail otherwise (-c)
__global__ __launch_bounds__(NT) void k_adj_rhs(Topo topo, const int4 *__restrict__ coord, Grid g,
                                                const double *__restrict__ c, double *b, double *part)
{
    __shared__ double red[8];
    const int bk = xcd_brick(blockIdx.x, topo.nb);
    if (bk < 0) return;
    const int t = threadIdx.x;
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    const int4 q = coord[bk];
    const int i = q.x * 8 + tx, j = q.y * 8 + ty, k = q.z * 8 + tz;
    const long long nvox = (long long)g.nx * g.ny * g.nz;
    double s = 0.0;
    for (int oz = -1; oz <= 0; ++oz)
        for (int oy = -1; oy <= 0; ++oy)
            for (int ox = -1; ox <= 0; ++ox) {
                const int vi = i + ox, vj = j + oy, vk = k + oz;
                if (vi < 0 || vj < 0 || vk < 0 || vi >= g.nx || vj >= g.ny || vk >= g.nz) continue;
                const long long v = vi + (long long)g.nx * (vj + (long long)g.ny * vk);
                s += (ox < 0 ? c[v] : -c[v]);
                s += (oy < 0 ? c[nvox + v] : -c[nvox + v]);
                s += (oz < 0 ? c[2 * nvox + v] : -c[2 * nvox + v]);
            }
    b[(long long)bk * BS + t] = s;
    const double tot = block_sum(s * s, red);
    if (t == 0) part[bk] = tot;
}

// dJ/dsigma_v = -sum over the 12 edges of v of (area/length/4) (G lambda)_e u_e,
// and per-block partial sums per label (LDS atomics, then a fixed-order sum)
__global__ __launch_bounds__(256) void k_adj_grad(const uint8_t *__restrict__ labels, const double *__restrict__ table,
                                                  const double *__restrict__ sig_vox, Grid g, double gx, double gy,
                                                  double gz, const double *__restrict__ a,
                                                  const double *__restrict__ psi, const double *__restrict__ lam,
                                                  double *grad, double *lab_part, int nlab)
{
    __shared__ double hist[MAX_LABELS];
    for (int l = threadIdx.x; l < nlab; l += blockDim.x) hist[l] = 0.0;
    __syncthreads();
    const long long nvox = (long long)g.nx * g.ny * g.nz;
    const long long nn = (long long)g.Nx * g.Ny * g.Nz;
    const long long sy = g.Nx, sz = (long long)g.Nx * g.Ny;
    const double geo[3] = {gx, gy, gz};
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (long long)gridDim.x * blockDim.x) {
        const double s = sig_vox ? sig_vox[v] : table[labels[v]];
        double out = 0.0;
        if (s > 0.0) {
            const long long i = v % g.nx, j = (v / g.nx) % g.ny, k = v / ((long long)g.nx * g.ny);
            const long long n0 = i + g.Nx * (j + (long long)g.Ny * k);
            const long long e[3][4] = {{n0, n0 + sy, n0 + sz, n0 + sy + sz},
                                       {n0, n0 + 1, n0 + sz, n0 + 1 + sz},
                                       {n0, n0 + 1, n0 + sy, n0 + 1 + sy}};
            const long long st[3] = {1, sy, sz};
            double acc = 0.0;
            for (int d = 0; d < 3; ++d)
                for (int q = 0; q < 4; ++q) {
                    const long long n = e[d][q];
                    const double glam = lam[n + st[d]] - lam[n];
                    const double u = (a[d * nn + n] + psi[n + st[d]]) - psi[n];
                    acc += geo[d] * glam * u;
                }
            out = -acc;
            if (labels[v] < nlab) atomicAdd(hist + labels[v], out);
        }
        grad[v] = out;
    }
    __syncthreads();
    for (int l = threadIdx.x; l < nlab; l += blockDim.x) lab_part[(long long)blockIdx.x * nlab + l] = hist[l];
}

// per-label totals: fixed-order sum of the block partials
__global__ void k_adj_labsum(const double *__restrict__ lab_part, int nblocks, int nlab, double *out)
{
    const int l = blockIdx.x;
    __shared__ double red[8];
    double s = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) s += lab_part[(long long)b * nlab + l];
    s = block_sum(s, red);
    if (threadIdx.x == 0) out[l] = s;
}

hipError_t launch_adj_voxel(const uint8_t *labels, const double *table, const double *sig_vox, const Grid &g,
                            const double h[3], double omega, const double *a, const double *psi,
                            const double *grad_emag, double *c, hipStream_t s)
{
    const long long nvox = (long long)g.nx * g.ny * g.nz;
    const unsigned gb = (unsigned)((nvox + 255) / 256 > 131072 ? 131072 : (nvox + 255) / 256);
    SPFD_LAUNCH(k_adj_voxel, dim3(gb), dim3(256), 0, s, labels, table, sig_vox, g, h[0], h[1], h[2], omega, a,
                       psi, grad_emag, c);
    return hipGetLastError();
}

hipError_t launch_adj_rhs(Topo topo, const int4 *coord, const Grid &g, const double *c, double *b, double *part,
                          hipStream_t s)
{
    if (topo.nb <= 0) return hipSuccess;
    SPFD_LAUNCH(k_adj_rhs, dim3(xcd_grid(topo.nb)), dim3(NT), 0, s, topo, coord, g, c, b, part);
    return hipGetLastError();
}

int adj_grad_blocks(const Grid &g)
{
    const long long nvox = (long long)g.nx * g.ny * g.nz;
    const long long b = (nvox + 255) / 256;
    return (int)(b > 8192 ? 8192 : b);
}

hipError_t launch_adj_grad(const uint8_t *labels, const double *table, const double *sig_vox, const Grid &g,
                           const double geo4[3], const double *a, const double *psi, const double *lam, double *grad,
                           double *lab_part, int nlab, double *lab_out, hipStream_t s)
{
    const int gb = adj_grad_blocks(g);
    SPFD_LAUNCH(k_adj_grad, dim3(gb), dim3(256), 0, s, labels, table, sig_vox, g, geo4[0], geo4[1], geo4[2], a,
                       psi, lam, grad, lab_part, nlab);
    SPFD_LAUNCH(k_adj_labsum, dim3(nlab), dim3(NT), 0, s, lab_part, gb, nlab, lab_out);
    return hipGetLastError();
}

}  // namespace spfd
