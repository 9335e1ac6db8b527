// Shared device-side definitions of the SPFD library (gfx950, wave64).
//
// Node arrays of every multigrid level live in 8x8x8 bricks: only bricks that
// hold unknowns are stored, brick b occupies elements [b*512, b*512+512) and
// node (tx,ty,tz) of a brick sits at tx + 8*ty + 64*tz.  A workgroup of 512
// threads owns one brick, so each wave covers one 8x8 z-slice (512 contiguous
// bytes in FP64).  Neighbour bricks come from a table of [nb][NBR] ints, the first
// six of a brick's (-1 = absent).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spfd {

constexpr int BD = 8;              // brick edge in nodes
constexpr int BS = 512;            // nodes per brick
constexpr int TILE = 9;            // label tile edge: the brick's voxels plus one layer on the minus side
constexpr int TILE_VOX = 729;
constexpr int TILE_BYTES = 768;    // 729 padded
constexpr int MAX_LABELS = 256;
constexpr int NT = 512;            // threads per brick workgroup

// neighbour slots
enum { NMX = 0, NPX = 1, NMY = 2, NPY = 3, NMZ = 4, NPZ = 5 };

// per right-hand side scalars of the outer CG, resident in device memory
struct Scal {
    double rz;       // r.z of the current iterate
    double pq;       // p.q
    double alpha;
    double beta;
    double rr;       // ||r||^2
    double bb;       // ||b||^2
    double zq;       // z.q (flexible beta)
    double tol2;     // (rel_tol)^2 * ||b||^2
    int done;        // 1 = converged or stopped: later kernels of this solve return at once
    int iters;
    int status;      // 0 ok, 5 not converged, 6 breakdown
    int hcount;      // CG steps of the current window of kept search directions (the next one's slot)
    int happlied;    // of these, the directions already added to x (an update of x before the window is full)
    int stamp;       // host copies only: number of the launch that wrote the copy, stored after the rest of it
    double rzn;      // r.z of the step under way, where the CG kernels finish the sums themselves: the CG step reads
                     // rz and leaves the new value here, the residual update reads it here and moves it to rz
};

constexpr int MAX_MODELS = 16;     // voxel models packed into one handle

// ints per brick's record; in it, where the brick's table of conductivities starts (packed models: each its own)
constexpr int NBR = 8, NTAB = 6;

struct Topo {
    int nb;                                    // active bricks
    const int *nbr;                            // [nb*NBR]: the six neighbours' slots (-1: absent), then NTAB
    const unsigned long long *cmask = nullptr; // [nb]: bit tx + 8 ty set when the node column (tx,ty,*)
                                               // holds an unknown (nullptr: all columns)
    // np > 0: the bricks of np voxel models packed into one level, model m's being [prange[m].x, prange[m].x +
    // prange[m].y), with its own scalars and partial sums (row m).  The workgroups of all models follow each other in
    // one launch dimension, and each finds its model in the ranges (topo_group): a launch row per model, as long as
    // the largest one's, left most workgroups of uneven models empty.  The ranges live in device memory (uniform
    // loads; entries up to MAX_MODELS can be read), not in the kernel arguments: an argument array indexed by a row
    // would be copied to scratch memory in every kernel.
    int np = 0;
    int pmax = 0;                    // largest range
    int psum = 0;                    // bricks of all ranges
    const int2 *prange = nullptr;    // [np] (first brick, bricks)
};

// bricks per launch row: all bricks, or the largest model's
__host__ __device__ __forceinline__ int topo_count(const Topo &t) { return t.np ? t.pmax : t.nb; }

// XCD-aware workgroup -> brick map: the hardware hands consecutive workgroup
// ids to the 8 XCDs in turn; giving each XCD a contiguous run of bricks keeps
// neighbour bricks (halo reads) in the same L2.  Returns -1 for padding ids.
__device__ __forceinline__ int xcd_brick(int wg, int nb)
{
    int per = (nb + 7) >> 3;
    int b = (wg & 7) * per + (wg >> 3);
    return b < nb ? b : -1;
}

__host__ __device__ __forceinline__ int xcd_grid(int nb) { return ((nb + 7) >> 3) << 3; }

// Row, range of bricks and group of `per` bricks within it (-1 for padding) of a workgroup: launch row blockIdx.y
// works on all bricks, or, with packed models, the workgroups go through the models' groups one after the other
// (MODELS false: a kernel that is launched without).
template <bool MODELS = true>
__device__ __forceinline__ int topo_group(const Topo &t, int per, int &row, int2 &range)
{
    row = blockIdx.y;
    range = make_int2(0, t.nb);
    if (!MODELS || t.np == 0) return xcd_brick(blockIdx.x, (t.nb + per - 1) / per);
    int groups[MAX_MODELS], total = 0;
#pragma unroll
    for (int m = 0; m < MAX_MODELS; ++m) {
        groups[m] = m < t.np ? (t.prange[m].y + per - 1) / per : 0;
        total += groups[m];
    }
    // (the launch may be a little longer than the groups: topo_grid counts a partial one for every model)
    int g = (int)blockIdx.x < xcd_grid(total) ? xcd_brick(blockIdx.x, total) : -1;
    row = 0;
    if (g >= 0) {
#pragma unroll
        for (int m = 0; m + 1 < MAX_MODELS; ++m)
            if (row == m && g >= groups[m]) {
                g -= groups[m];
                row = m + 1;
            }
    }
    range = t.prange[row];
    return g;
}

// launch grid of such workgroups (n launch rows unless models are packed)
__host__ __forceinline__ dim3 topo_grid(const Topo &t, int per, int n)
{
    return t.np ? dim3(xcd_grid((t.psum + per - 1) / per + t.np), 1) : dim3(xcd_grid((t.nb + per - 1) / per), n);
}

// the brick of a one-brick workgroup (-1 for padding), its row and its index there (local, that of its partial sum)
__device__ __forceinline__ int topo_brick(const Topo &t, int &local, int &row)
{
    int2 range;
    local = topo_group(t, 1, row, range);
    return local < 0 ? -1 : range.x + local;
}

__device__ __forceinline__ void brick_xyz(int t, int &tx, int &ty, int &tz)
{
    tx = t & 7;
    ty = (t >> 3) & 7;
    tz = t >> 6;
}

// Index of each face neighbour of node t of brick b.  A neighbour in an absent
// brick is never a conductor node, and the edge to it has conductance 0, so
// it is replaced by the node itself: every lane issues exactly one load per
// direction and the stencil term w (x_n - x_n) vanishes.
__device__ __forceinline__ void nbr_index(long long base, int t, int tx, int ty, int tz, const int *nb,
                                          long long I[6])
{
    const long long self = base + t;
    I[NMX] = tx > 0 ? self - 1 : (nb[NMX] >= 0 ? (long long)nb[NMX] * BS + t + 7 : self);
    I[NPX] = tx < 7 ? self + 1 : (nb[NPX] >= 0 ? (long long)nb[NPX] * BS + t - 7 : self);
    I[NMY] = ty > 0 ? self - 8 : (nb[NMY] >= 0 ? (long long)nb[NMY] * BS + t + 56 : self);
    I[NPY] = ty < 7 ? self + 8 : (nb[NPY] >= 0 ? (long long)nb[NPY] * BS + t - 56 : self);
    I[NMZ] = tz > 0 ? self - 64 : (nb[NMZ] >= 0 ? (long long)nb[NMZ] * BS + t + 448 : self);
    I[NPZ] = tz < 7 ? self + 64 : (nb[NPZ] >= 0 ? (long long)nb[NPZ] * BS + t - 448 : self);
}

template <typename T>
__device__ __forceinline__ void nbr_vals(const T *__restrict__ x, const long long I[6], T X[6])
{
#pragma unroll
    for (int k = 0; k < 6; ++k) X[k] = x[I[k]];
}

// edge weights of node t from stored arrays w[d*stride + node] (edge to +d);
// the minus-side weights are the plus-side weights of the minus neighbours
// (0 when that neighbour's brick is absent)
template <typename T>
__device__ __forceinline__ void stored_weights(const T *__restrict__ w, long long stride, long long base, int t,
                                               const long long I[6], T W[6])
{
    const long long n = base + t;
    W[NPX] = w[n];
    W[NPY] = w[stride + n];
    W[NPZ] = w[2 * stride + n];
    const T mx = w[I[NMX]], my = w[stride + I[NMY]], mz = w[2 * stride + I[NMZ]];
    W[NMX] = I[NMX] != n ? mx : T(0);
    W[NMY] = I[NMY] != n ? my : T(0);
    W[NMZ] = I[NMZ] != n ? mz : T(0);
}

// the six neighbour slots of a brick (uniform across the workgroup: scalar loads)
__device__ __forceinline__ void brick_nbrs(const int *nbr, int b, int nb[6])
{
    const int *p = nbr + b * NBR;
#pragma unroll
    for (int k = 0; k < 6; ++k) nb[k] = p[k];
}

// Conductances of the six edges of a node from the conductivities of its eight
// surrounding voxels, held in an LDS tile s[a + 9*(b + 9*c)] where (a,b,c) =
// (tx,ty,tz) + {0,1}^3.  Edge to +x: the four voxels at a = tx+1, and so on.
// geo4[d] = (area of the dual facet) / (length) / 4 of a d-edge.  The sums keep
// the order (j-1,k-1), (j,k-1), (j-1,k), (j,k) of the other two axes.
template <typename T>
__device__ __forceinline__ void tile_weights(const T *s, int tx, int ty, int tz, const T geo4[3], T W[6])
{
    const T *p = s + tx + 9 * (ty + 9 * tz);
    const T s000 = p[0], s100 = p[1], s010 = p[9], s110 = p[10];
    const T s001 = p[81], s101 = p[82], s011 = p[90], s111 = p[91];
    W[NPX] = (((s100 + s110) + s101) + s111) * geo4[0];
    W[NMX] = (((s000 + s010) + s001) + s011) * geo4[0];
    W[NPY] = (((s010 + s110) + s011) + s111) * geo4[1];
    W[NMY] = (((s000 + s100) + s001) + s101) * geo4[1];
    W[NPZ] = (((s001 + s101) + s011) + s111) * geo4[2];
    W[NMZ] = (((s000 + s100) + s010) + s110) * geo4[2];
}

// (A x)_n = sum over edges of w (x_n - x_m); exact zero for a constant field
template <typename T>
__device__ __forceinline__ T stencil_apply(T x0, const T X[6], const T W[6])
{
    T y = W[0] * (x0 - X[0]);
    y += W[1] * (x0 - X[1]);
    y += W[2] * (x0 - X[2]);
    y += W[3] * (x0 - X[3]);
    y += W[4] * (x0 - X[4]);
    y += W[5] * (x0 - X[5]);
    return y;
}

template <typename T>
__device__ __forceinline__ T diag_of(const T W[6])
{
    return ((((W[0] + W[1]) + W[2]) + W[3]) + W[4]) + W[5];
}

// ---------------------------------------------------------------- reductions
__device__ __forceinline__ double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Wave sums of NV values a lane at once (NV a power of two up to 32): lane l returns that of row l / (64 / NV).  Each
// step over half the distance also halves the rows a lane keeps (lanes l and l ^ off keep one half each), so 16 rows
// take 17 cross-lane adds instead of 96, in the order of wave_sum.
template <int NV>
__device__ __forceinline__ double wave_rows(double (&acc)[NV])
{
    const int lane = threadIdx.x & 63;
    int off = 32;
#pragma unroll
    for (int m = NV / 2; m > 0; m /= 2, off /= 2) {
        const long long up = lane & off ? -1LL : 0LL;   // (a mask: a choice of elements becomes a search by index)
#pragma unroll
        for (int i = 0; i < m; ++i) {
            const long long lo = __double_as_longlong(acc[i]), hi = __double_as_longlong(acc[i + m]);
            const double give = __longlong_as_double((lo & up) | (hi & ~up));
            const double keep = __longlong_as_double((hi & up) | (lo & ~up));
            acc[i] = keep + __shfl_xor(give, off, 64);
        }
    }
    for (; off > 0; off >>= 1) acc[0] += __shfl_xor(acc[0], off, 64);
    return acc[0];
}

// sum over a 512-thread block, valid in thread 0; lds needs 8 doubles
__device__ __forceinline__ double block_sum(double v, double *lds)
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

// number of set flags in the threads before this one, and in *total those of all 1024 threads (count: 16 ints in LDS)
__device__ __forceinline__ int flags_before(bool flag, int *count, int *total)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const unsigned long long m = __ballot(flag);
    __syncthreads();
    if (lane == 0) count[wv] = __popcll(m);
    __syncthreads();
    int before = __popcll(m & ((1ull << lane) - 1ull)), all = 0;
    for (int k = 0; k < 16; ++k) {
        if (k < wv) before += count[k];
        all += count[k];
    }
    *total = all;
    return before;
}

// the scalars into host memory; with a stamp (> 0) the host may poll for them: it sees the stamp after the rest
__device__ __forceinline__ void store_mirror(Scal *mirror, const Scal *sc, int stamp, int row = 0)
{
    if (!mirror) return;
    Scal *m = mirror + row;
    *m = *sc;   // (the device's stamp is 0)
    if (stamp > 0) {
        __threadfence_system();
        __hip_atomic_store(&m->stamp, stamp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

}  // namespace spfd
