// Unstructured (ELL) coarse levels of the aggregation multigrid.
//
// On the coarse end of the hierarchy, 2x2x2 aggregates are split into the
// pieces that are connected inside the aggregate, so that one coarse unknown
// never glues together conductor regions that touch only through air (an arm
// and the torso across a thin gap, two legs).  A coarse unknown is then no
// longer a grid node: these levels store, per unknown, its grid position and
// up to K neighbours with conductances (ELL, column-major: entry k of row i at
// k*n + i, column -1 = empty).  The Galerkin product for piecewise-constant
// aggregation is still exact: the coarse conductance between two pieces is
// the sum of the fine conductances that join them.
#include <math.h>

#include "kernels.h"

namespace spfd {

// ---------------------------------------------------------------- union-find helpers (agent-scope, lock-free)
__device__ __forceinline__ int uf_load(const int *p, int i)
{
    return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int uf_find(int *p, int x)
{
    int px = uf_load(p, x);
    while (px != x) {
        const int ppx = uf_load(p, px);
        if (ppx != px) __hip_atomic_store(p + x, ppx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = px;
        px = ppx;
    }
    return x;
}

__device__ __forceinline__ void uf_unite(int *p, int a, int b)
{
    while (true) {
        a = uf_find(p, a);
        b = uf_find(p, b);
        if (a == b) return;
        if (a > b) { const int t = a; a = b; b = t; }
        int expected = b;
        if (__hip_atomic_compare_exchange_strong(p + b, &expected, a, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return;
    }
}

// ---------------------------------------------------------------- pieces of a structured (brick) level
// The connected pieces of every 2x2x2 aggregate of a brick (bricks start at multiples of 8, so an aggregate lies in
// one brick): reach[n] = the nodes of node n's aggregate that conducting edges inside it connect to n, as bits
// (dx + 2 dy + 4 dz), 0 for a node without a positive diagonal.  The smallest node of a piece stands for it.
// part[b] and part[nb + b]: pieces and unknowns of brick b.  (Twelve edges and eight nodes fit in a thread's
// registers; a union-find over the level took four launches.)
__global__ __launch_bounds__(NT) void k_pieces_brick(const double *__restrict__ w, long long stride, Topo topo,
                                                     uint8_t *__restrict__ reach, int *__restrict__ part)
{
    __shared__ unsigned long long e[3][8];
    __shared__ int count[2][8];
    const int b = blockIdx.x, t = threadIdx.x;
    int nb[6];
    brick_nbrs(topo.nbr, b, nb);
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    const long long base = (long long)b * BS;
    long long I[6];
    nbr_index(base, t, tx, ty, tz, nb, I);
    double W[6];
    stored_weights(w, stride, base, t, I, W);
    const unsigned long long ex = __ballot(W[NPX] > 0.0), ey = __ballot(W[NPY] > 0.0), ez = __ballot(W[NPZ] > 0.0);
    if ((t & 63) == 0) {
        e[0][tz] = ex;
        e[1][tz] = ey;
        e[2][tz] = ez;
    }
    __syncthreads();
    const int z0 = tz & ~1, s0 = (tx & ~1) + 8 * (ty & ~1);
    auto quad = [&](unsigned long long m) {   // the four nodes of a layer
        m >>= s0;
        return (unsigned)((m & 3ull) | ((m >> 6) & 12ull));
    };
    // edges by their lower node
    const unsigned X = (quad(e[0][z0]) | quad(e[0][z0 + 1]) << 4) & 0x55u;
    const unsigned Y = (quad(e[1][z0]) | quad(e[1][z0 + 1]) << 4) & 0x33u;
    const unsigned Z = quad(e[2][z0]);
    const int q = (tx & 1) + 2 * (ty & 1) + 4 * (tz & 1);
    unsigned r = 1u << q;
    for (int k = 0; k < 7; ++k)
        r |= (r & X) << 1 | (r >> 1 & X) | (r & Y) << 2 | (r >> 2 & Y) | (r & Z) << 4 | (r >> 4 & Z);
    const bool unknown = diag_of(W) > 0.0;
    reach[base + t] = unknown ? (uint8_t)r : 0;
    const int pieces = __popcll(__ballot(unknown && __ffs(r) - 1 == q)), nodes = __popcll(__ballot(unknown));
    if ((t & 63) == 0) {
        count[0][tz] = pieces;
        count[1][tz] = nodes;
    }
    __syncthreads();
    if (t < 2) {
        int sum = 0;
        for (int k = 0; k < 8; ++k) sum += count[t][k];
        part[t * topo.nb + b] = sum;
    }
}

// The pieces in the order of their smallest nodes: agg of every node, grid position at the coarse level, members (CSR
// and, as at most eight, the direct table memb[p*8 + j], -1: none).  part: exclusive sums over the bricks.
__global__ __launch_bounds__(NT) void k_pieces_write(const uint8_t *__restrict__ reach, int nb,
                                                     const int4 *__restrict__ coord, const int *__restrict__ part,
                                                     int nc, int *__restrict__ agg, int4 *__restrict__ pos,
                                                     int *__restrict__ mptr, int *__restrict__ mem,
                                                     int *__restrict__ memb)
{
    __shared__ int id[BS];
    __shared__ int count[2][8];
    const int b = blockIdx.x, t = threadIdx.x, lane = t & 63;
    int tx, ty, tz;
    brick_xyz(t, tx, ty, tz);
    const int base = b * BS;
    const unsigned r = reach[base + t];
    const int q = (tx & 1) + 2 * (ty & 1) + 4 * (tz & 1);
    const int corner = t - (tx & 1) - 8 * (ty & 1) - 64 * (tz & 1);   // node 0 of the aggregate
    auto node = [&](int k) { return corner + (k & 1) + 8 * (k >> 1 & 1) + 64 * (k >> 2); };
    const bool root = r != 0u && __ffs(r) - 1 == q;
    const unsigned long long roots = __ballot(root);
    const int size = root ? __popc(r) : 0;
    int incl = size;   // members up to and with this lane's piece
    for (int off = 1; off < 64; off <<= 1) {
        const int v = __shfl_up(incl, off, 64);
        if (lane >= off) incl += v;
    }
    if (lane == 63) {
        count[0][tz] = __popcll(roots);
        count[1][tz] = incl;
    }
    __syncthreads();
    int first = part[b], at = part[nb + b];
    for (int k = 0; k < tz; ++k) {
        first += count[0][k];
        at += count[1][k];
    }
    first += __popcll(roots & ((1ull << lane) - 1ull));
    at += incl - size;
    id[t] = first;
    __syncthreads();
    agg[base + t] = r != 0u ? id[node(__ffs(r) - 1)] : -1;
    if (!root) return;
    const int4 c = coord[b];
    pos[first] = make_int4((c.x * 8 + tx) >> 1, (c.y * 8 + ty) >> 1, (c.z * 8 + tz) >> 1, 0);
    mptr[first] = at;
    if (first == nc - 1) mptr[nc] = at + size;
    int n = 0;
    for (unsigned m = r; m != 0u; m &= m - 1u) {
        const int i = base + node(__ffs(m) - 1);
        mem[at + n] = i;
        memb[(long long)first * 8 + n] = i;
        ++n;
    }
    for (; n < 8; ++n) memb[(long long)first * 8 + n] = -1;
}

// ---------------------------------------------------------------- pieces of an ELL level
// (parent[i] = i for a row with a positive diagonal, else -1: written by the kernel that made the level)
// KR: entries of a row whose loads go out together (its columns and values, then their positions); the rest of a
// wider row goes one by one.
template <int KR>
__global__ __launch_bounds__(256) void k_piece_union_ell(int n, int K, const int *__restrict__ col,
                                                         const double *__restrict__ val, const int4 *__restrict__ pos,
                                                         int *parent)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int4 pi = pos[i];
    auto together = [&](const int4 &pj) {
        return (pi.x >> 1) == (pj.x >> 1) && (pi.y >> 1) == (pj.y >> 1) && (pi.z >> 1) == (pj.z >> 1);
    };
    int j[KR];
    double w[KR];
    int4 pj[KR];
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        j[k] = col[(long long)k * n + i];
        w[k] = val[(long long)k * n + i];
    }
#pragma unroll
    for (int k = 0; k < KR; ++k) pj[k] = pos[j[k] >= 0 ? j[k] : i];
#pragma unroll
    for (int k = 0; k < KR; ++k)
        if (j[k] > i && w[k] > 0.0 && together(pj[k])) uf_unite(parent, i, j[k]);
    for (int k = KR; k < K; ++k) {
        const int m = col[(long long)k * n + i];
        if (m > i && val[(long long)k * n + i] > 0.0 && together(pos[m])) uf_unite(parent, i, m);
    }
}

// root of every row (-1: none), number of the roots before it in its workgroup's rows, and their total
constexpr int ROOTS_WG = 256;
__global__ __launch_bounds__(ROOTS_WG) void k_piece_roots(int *parent, int n, int *__restrict__ root,
                                                          int *__restrict__ idx, int *__restrict__ part)
{
    __shared__ int count[ROOTS_WG / 64];
    const int i = blockIdx.x * ROOTS_WG + threadIdx.x, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int r = -1;
    if (i < n && uf_load(parent, i) >= 0) r = uf_find(parent, i);
    const unsigned long long m = __ballot(r >= 0 && r == i);
    if (lane == 0) count[wv] = __popcll(m);
    __syncthreads();
    int before = __popcll(m & ((1ull << lane) - 1ull)), total = 0;
    for (int k = 0; k < ROOTS_WG / 64; ++k) {
        if (k < wv) before += count[k];
        total += count[k];
    }
    if (i < n) {
        root[i] = r;
        idx[i] = before;
    }
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

// aggregate of every row, position of its pieces, number of members (count cleared before)
__global__ void k_piece_assign(int n, const int *__restrict__ root, const int *__restrict__ idx,
                               const int *__restrict__ part, const int4 *__restrict__ fpos, int *__restrict__ agg,
                               int4 *__restrict__ pos, int *count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int r = root[i];
    const int a = r >= 0 ? idx[r] + part[r / ROOTS_WG] : -1;
    agg[i] = a;
    if (a < 0) return;
    atomicAdd(count + a, 1);
    if (r == i) {
        const int4 p = fpos[i];
        pos[a] = make_int4(p.x >> 1, p.y >> 1, p.z >> 1, 0);
    }
}

// members of each coarse unknown; put in increasing fine index (deterministic order) by the sort, which also writes
// the direct table and sets stat->over when an aggregate has more than eight (the restriction then keeps the CSR form)
__global__ void k_members_fill(const int *__restrict__ agg, int n, const int *__restrict__ mptr, int *cursor, int *mem)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int a = agg[i];
    if (a >= 0) mem[mptr[a] + atomicAdd(cursor + a, 1)] = i;
}

__global__ void k_members_sort(int nc, const int *__restrict__ mptr, int *mem, int *__restrict__ memb, EllStat *stat)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= nc) return;
    const int b = mptr[p], e = mptr[p + 1];
    if (e - b <= 8) {   // in registers: odd-even transposition, absent members last
        unsigned v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = b + j < e ? (unsigned)mem[b + j] : 0xffffffffu;
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int j = r & 1; j + 1 < 8; j += 2) {
                const unsigned lo = v[j] < v[j + 1] ? v[j] : v[j + 1], hi = v[j] < v[j + 1] ? v[j + 1] : v[j];
                v[j] = lo;
                v[j + 1] = hi;
            }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (b + j < e) mem[b + j] = (int)v[j];
            memb[(long long)p * 8 + j] = (int)v[j];   // (absent: -1)
        }
        return;
    }
    for (int i = b + 1; i < e; ++i) {
        const int v = mem[i];
        int j = i - 1;
        while (j >= b && mem[j] > v) {
            mem[j + 1] = mem[j];
            --j;
        }
        mem[j + 1] = v;
    }
    stat->over = 1;
}

// ---------------------------------------------------------------- Galerkin rows
constexpr int GAL_MAX = 48;   // distinct coarse neighbours a row may collect

// visit the edges of fine unknown i: f(j, w) for every neighbour j with w > 0
struct FineLevel {
    // structured
    const double *w;
    long long stride;
    const int *nbr;
    // ELL
    int n, K;
    const int *col;
    const double *val;
};

template <typename F>
__device__ __forceinline__ void fine_edges(const FineLevel &f, int i, F &&fn)
{
    if (f.w) {
        const int b = i / BS, t = i % BS;
        int tx, ty, tz;
        brick_xyz(t, tx, ty, tz);
        int nb[6];
        brick_nbrs(f.nbr, b, nb);
        long long I[6];
        nbr_index((long long)b * BS, t, tx, ty, tz, nb, I);
        double W[6];
        stored_weights(f.w, f.stride, (long long)b * BS, t, I, W);
        for (int k = 0; k < 6; ++k)
            if (W[k] > 0.0 && I[k] != i) fn((int)I[k], W[k]);
    } else {
        for (int k = 0; k < f.K; ++k) {
            const int j = f.col[(long long)k * f.n + i];
            if (j >= 0 && f.val[(long long)k * f.n + i] > 0.0) fn(j, f.val[(long long)k * f.n + i]);
        }
    }
}

// pass 0: row lengths (len[p]); pass 1: fill ELL with width K (entries in
// order of first appearance over members and their edges; sums in that order)
__global__ void k_galerkin_rows(FineLevel f, const int *__restrict__ agg, int nc, const int *__restrict__ mptr,
                                const int *__restrict__ mem, int pass, int *len, int K, int *col, double *val64,
                                float *val32, int *overflow)
{
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < nc; p += gridDim.x * blockDim.x) {
        int cols[GAL_MAX];
        double ws[GAL_MAX];
        int m = 0;
        bool over = false;
        for (int q = mptr[p]; q < mptr[p + 1]; ++q) {
            const int i = mem[q];
            fine_edges(f, i, [&](int j, double wj) {
                const int a = agg[j];
                if (a < 0 || a == p) return;
                int s = 0;
                while (s < m && cols[s] != a) ++s;
                if (s == m) {
                    if (m == GAL_MAX) { over = true; return; }
                    cols[m] = a;
                    ws[m] = 0.0;
                    ++m;
                }
                ws[s] += wj;
            });
        }
        if (over) *overflow = 1;
        if (pass == 0) {
            len[p] = m;
        } else {
            for (int k = 0; k < K; ++k) {
                const long long e = (long long)k * nc + p;
                if (k < m) {
                    col[e] = cols[k];
                    val64[e] = ws[k];
                    val32[e] = (float)ws[k];
                } else {
                    col[e] = -1;
                    val64[e] = 0.0;
                    val32[e] = 0.0f;
                }
            }
        }
    }
}

__global__ void k_max_int(const int *__restrict__ v, int n, int *out)
{
    __shared__ int s[256];
    int m = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) m = max(m, v[i]);
    s[threadIdx.x] = m;
    __syncthreads();
    for (int d = 128; d > 0; d >>= 1) {
        if (threadIdx.x < d) s[threadIdx.x] = max(s[threadIdx.x], s[threadIdx.x + d]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = s[0];
}

// Rows of at most ELL_K8 entries, which nearly all levels have, in one pass: eight lanes per row.  Lane q collects the
// edges of member q (of each round of eight members), then the eight lanes go through all of them in the order of
// the general kernel, lane s holding entry s of the row.  The row's diagonal, its inverse and its start value of the
// next level's union-find follow.  A row with more entries sets stat->longest, and the level is built by the
// general kernel.  (One thread per row with its entries in scratch memory, once to count and once to fill: 2 x 45 us
// for 21 k rows, 2 x 70 us for 3 k, and five waits of the host per level; this form 13 and 16 us.)
template <bool BRICK>
__global__ __launch_bounds__(256) void k_galerkin_rows8(FineLevel f, const int *__restrict__ agg, int nc,
                                                        const int *__restrict__ mptr, const int *__restrict__ mem,
                                                        int *__restrict__ col, double *__restrict__ val64,
                                                        float *__restrict__ val32, double *__restrict__ d64,
                                                        float *__restrict__ d32, int *__restrict__ parent, EllStat *stat)
{
    constexpr int E = BRICK ? 6 : ELL_K8;
    const int lane = threadIdx.x & 63, s = lane & 7, first = lane & ~7;
    const int p = blockIdx.x * 32 + (threadIdx.x >> 3);
    const bool row = p < nc;
    const int mb = row ? mptr[p] : 0, me = row ? mptr[p + 1] : 0;
    int c = -1, m = 0;
    double ws = 0.0;
    for (int r = mb; __any(r < me); r += 8) {
        int a[E];
        double w[E];
        const bool have = r + s < me;
        const int i = have ? mem[r + s] : 0;
        if (BRICK) {
            const int b = i / BS, t = i % BS;
            int tx, ty, tz;
            brick_xyz(t, tx, ty, tz);
            int nb[6];
            brick_nbrs(f.nbr, b, nb);
            long long I[6];
            nbr_index((long long)b * BS, t, tx, ty, tz, nb, I);
            double W[6];
            stored_weights(f.w, f.stride, (long long)b * BS, t, I, W);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                a[k] = agg[I[k]];
                w[k] = W[k];
                if (!(have && W[k] > 0.0 && I[k] != i && a[k] != p)) a[k] = -1;
            }
        } else {
#pragma unroll
            for (int k = 0; k < E; ++k) {
                a[k] = f.col[(long long)k * f.n + i];
                w[k] = f.val[(long long)k * f.n + i];
            }
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const int j = a[k];
                a[k] = agg[j >= 0 ? j : i];
                if (!(have && j >= 0 && w[k] > 0.0 && a[k] != p)) a[k] = -1;
            }
        }
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const int A = __shfl(a[k], first + q, 64);
                const double v = __shfl(w[k], first + q, 64);
                const bool match = A >= 0 && c == A;
                const bool found = ((__ballot(match) >> first) & 255ull) != 0ull;
                if (match) ws += v;
                if (A >= 0 && !found) {
                    if (s == m) {
                        c = A;
                        ws = v;
                    }
                    ++m;
                }
            }
    }
    if (m > ELL_K8 && s == 0) atomicMax(&stat[blockIdx.x % LEVEL_STATS].longest, (unsigned)m);
    if (row) {
        const long long e = (long long)s * nc + p;
        col[e] = c;
        val64[e] = ws;
        val32[e] = (float)ws;
    }
    double d = 0.0;
    for (int q = 0; q < 8; ++q) d += __shfl(ws, first + q, 64);
    const bool unknown = row && s == 0 && d > 0.0;
    const int count = __popcll(__ballot(unknown));
    if (lane == 0 && count) atomicAdd(&stat[blockIdx.x % LEVEL_STATS].count, (unsigned)count);
    if (row && s == 0) {
        const double v = d > 0.0 ? 1.0 / d : 0.0;
        if (d64) d64[p] = v;
        if (d32) d32[p] = (float)v;
        parent[p] = d > 0.0 ? p : -1;
    }
}

static unsigned gblocks(long long n, int bs = 256, long long cap = 65536)
{
    long long b = (n + bs - 1) / bs;
    if (b < 1) b = 1;
    return (unsigned)(b > cap ? cap : b);
}

hipError_t launch_pieces_brick(const double *w64, long long stride, Topo topo, uint8_t *reach, int *part, int *nc,
                               hipStream_t s)
{
    if (topo.nb <= 0) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_pieces_brick, dim3(topo.nb), dim3(NT), 0, s, w64, stride, topo, reach, part);
    HIP_RETURN_IF(hipGetLastError());
    HIP_RETURN_IF(scan_small(part, topo.nb, nc, s));
    return scan_small(part + topo.nb, topo.nb, nullptr, s);
}

hipError_t launch_pieces_write(const uint8_t *reach, int nb, const int4 *coord, const int *part, int nc, int *agg,
                               int4 *pos, int *mptr, int *mem, int *memb, hipStream_t s)
{
    if (nb <= 0 || nc <= 0) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_pieces_write, dim3(nb), dim3(NT), 0, s, reach, nb, coord, part, nc, agg, pos, mptr, mem, memb);
    return hipGetLastError();
}

int piece_parts(int n) { return (n + ROOTS_WG - 1) / ROOTS_WG; }

hipError_t launch_pieces_ell(int n, int K, const int *col, const double *val, const int4 *pos, int *parent, int *root,
                             int *idx, int *part, int *nc, hipStream_t s)
{
    if (n <= 0) return hipErrorInvalidValue;
    if (K < ELL_K8) return hipErrorInvalidValue;   // (every level is stored with that many or more)
    SPFD_LAUNCH(k_piece_union_ell<ELL_K8>, dim3((n + 255) / 256), dim3(256), 0, s, n, K, col, val, pos, parent);
    SPFD_LAUNCH(k_piece_roots, dim3(piece_parts(n)), dim3(ROOTS_WG), 0, s, parent, n, root, idx, part);
    HIP_RETURN_IF(hipGetLastError());
    return scan_small(part, piece_parts(n), nc, s);
}

hipError_t launch_members_ell(int n, const int *root, const int *idx, int *part, const int4 *fpos, int nc,
                              int *agg, int4 *pos, int *mptr, int *cursor, int *mem, int *memb, EllStat *stat,
                              hipStream_t s)
{
    if (n <= 0 || nc <= 0) return hipErrorInvalidValue;
    const dim3 rows((n + 255) / 256);
    // mptr holds the numbers of members, cleared by the caller with the cursors, and becomes their exclusive sums
    // (scratch: part, n / ROOTS_WG >= (nc + 1) / SCAN_CHUNK ints, read by then)
    SPFD_LAUNCH(k_piece_assign, rows, dim3(256), 0, s, n, root, idx, part, fpos, agg, pos, mptr);
    HIP_RETURN_IF(hipGetLastError());
    HIP_RETURN_IF(scan_ints(mptr, nc + 1, part, s));
    SPFD_LAUNCH(k_members_fill, rows, dim3(256), 0, s, agg, n, mptr, cursor, mem);
    SPFD_LAUNCH(k_members_sort, dim3((nc + 255) / 256), dim3(256), 0, s, nc, mptr, mem, memb, stat);
    return hipGetLastError();
}

static FineLevel fine_level(const FineLevelArgs &fa)
{
    FineLevel f;
    f.w = fa.w;
    f.stride = fa.stride;
    f.nbr = fa.nbr;
    f.n = fa.n;
    f.K = fa.K;
    f.col = fa.col;
    f.val = fa.val;
    return f;
}

hipError_t launch_galerkin_rows8(const FineLevelArgs &fa, const int *agg, int nc, const int *mptr, const int *mem,
                                 int *col, double *val64, float *val32, double *d64, float *d32, int *parent,
                                 EllStat *stat, hipStream_t s)
{
    if (nc <= 0 || (!fa.w && fa.K != ELL_K8)) return hipErrorInvalidValue;
    const dim3 grid((nc + 31) / 32);
    if (fa.w)
        SPFD_LAUNCH(k_galerkin_rows8<true>, grid, dim3(256), 0, s, fine_level(fa), agg, nc, mptr, mem, col, val64, val32,
                    d64, d32, parent, stat);
    else
        SPFD_LAUNCH(k_galerkin_rows8<false>, grid, dim3(256), 0, s, fine_level(fa), agg, nc, mptr, mem, col, val64,
                    val32, d64, d32, parent, stat);
    return hipGetLastError();
}

hipError_t launch_galerkin_ell(const FineLevelArgs &fa, const int *agg, int nc, const int *mptr, const int *mem,
                               int pass, int *len, int K, int *col, double *val64, float *val32, int *overflow,
                               int *maxlen, hipStream_t s)
{
    const FineLevel f = fine_level(fa);
    if (nc <= 0) return hipSuccess;
    SPFD_LAUNCH(k_galerkin_rows, dim3(gblocks(nc, 128)), dim3(128), 0, s, f, agg, nc, mptr, mem, pass, len, K,
                       col, val64, val32, overflow);
    if (pass == 0) SPFD_LAUNCH(k_max_int, dim3(1), dim3(256), 0, s, len, nc, maxlen);
    return hipGetLastError();
}

// ============================================================================
// cycle kernels on ELL levels (T = arithmetic of the cycle)
// ============================================================================
__device__ __forceinline__ bool ell_stopped(const Scal *sc)
{
    return sc && sc[blockIdx.y].done;   // set by an earlier kernel than the one that asks: a plain (scalar) load
}

// (A x)_i and the diagonal D of an ELL row.  Padding entries (col < 0) read
// the row's own value and count with weight 0: every load is unconditional,
// so a thread has all of its row's loads in flight at once (a load under a
// condition becomes a branch that waits for it).
template <typename T>
__device__ __forceinline__ T ell_row(int n, int K, const int *__restrict__ col, const T *__restrict__ val,
                                     const T *__restrict__ x, int i, T xi, T &D)
{
    T y = T(0), d = T(0);
#pragma unroll 8
    for (int k = 0; k < K; ++k) {
        const int j = col[(long long)k * n + i];
        const T v = val[(long long)k * n + i];
        const T xj = x[j >= 0 ? j : i];
        const T w = j >= 0 ? v : T(0);
        d += w;
        y += w * (xi - xj);
    }
    D = d;
    return y;
}

template <typename T>
__global__ void k_ell_cheb_first(int n, int K, const int *__restrict__ col, const T *__restrict__ val,
                                 const T *__restrict__ b, T *__restrict__ x, T c0, const Scal *sc, long long vs)
{
    if (ell_stopped(sc)) return;
    b += blockIdx.y * vs;
    x += blockIdx.y * vs;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const T bi = b[i];
        T d = T(0);
#pragma unroll 8
        for (int k = 0; k < K; ++k) {
            const int j = col[(long long)k * n + i];
            const T v = val[(long long)k * n + i];
            d += j >= 0 ? v : T(0);
        }
        x[i] = d > T(0) ? c0 * bi / d : T(0);
    }
}

// x with the coarse-grid correction of the prolongation applied: x_i + s x_c[agg_i] (agg_i < 0: none)
template <typename T>
__device__ __forceinline__ T corrected(const T *__restrict__ x, const int *__restrict__ agg, const T *__restrict__ xc,
                                       T scale, int i)
{
    const T v = x[i];
    const int a = agg[i];
    const T c = xc[a >= 0 ? a : 0];
    return a >= 0 ? v + scale * c : v;
}

// general Chebyshev step on an ELL level; with agg the prolongation from the
// coarser ELL level (x += s x_c[agg]) is applied to every value read (the
// first post-smoothing step)
template <typename T>
__global__ void k_ell_cheb_step(int n, int K, const int *__restrict__ col, const T *__restrict__ val,
                                const T *__restrict__ b, const T *__restrict__ xin, T *__restrict__ xout,
                                const T *__restrict__ din, T *__restrict__ dout, T c1, T c2, const Scal *sc,
                                long long vs, const int *__restrict__ agg, const T *__restrict__ xc, T scale,
                                long long vsc)
{
    if (ell_stopped(sc)) return;
    b += blockIdx.y * vs;
    xin += blockIdx.y * vs;
    xout += blockIdx.y * vs;
    if (din) din += blockIdx.y * vs;
    if (dout) dout += blockIdx.y * vs;
    if (agg) xc += blockIdx.y * vsc;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const T xi = agg ? corrected(xin, agg, xc, scale, i) : xin[i];
        const T bi = b[i];
        const T di = din ? din[i] : T(0);
        T D;
        T ax;
        if (agg) {
            // as ell_row, with every value read corrected (unconditional loads)
            T y = T(0), d = T(0);
#pragma unroll 8
            for (int k = 0; k < K; ++k) {
                const int j = col[(long long)k * n + i];
                const T v = val[(long long)k * n + i];
                const T xj = corrected(xin, agg, xc, scale, j >= 0 ? j : i);
                const T w = j >= 0 ? v : T(0);
                d += w;
                y += w * (xi - xj);
            }
            D = d;
            ax = y;
        } else {
            ax = ell_row(n, K, col, val, xin, i, xi, D);
        }
        T xo = T(0), dn = T(0);
        if (D > T(0)) {
            const T dold = din ? di : xi;
            dn = c1 * dold + c2 * (bi - ax) / D;
            xo = xi + dn;
        }
        xout[i] = xo;
        if (dout) dout[i] = dn;
    }
}

// (b - A x)_i of row i of the finer level (structured stencil or ELL rows)
template <typename T>
__device__ __forceinline__ T fine_resid(const FineLevelT<T> &f, const T *__restrict__ b, const T *__restrict__ x,
                                        long long i)
{
    const T xi = x[i];
    T ax;
    if (f.w) {
        const int bk = (int)(i / BS), t = (int)(i % BS);
        int tx, ty, tz;
        brick_xyz(t, tx, ty, tz);
        int nb[6];
        brick_nbrs(f.nbr, bk, nb);
        long long I[6];
        nbr_index((long long)bk * BS, t, tx, ty, tz, nb, I);
        T W[6], X[6];
        stored_weights(f.w, f.stride, (long long)bk * BS, t, I, W);
        nbr_vals(x, I, X);
        ax = stencil_apply(xi, X, W);
    } else {
        T D;
        ax = ell_row(f.n, f.K, f.col, f.val, x, (int)i, xi, D);
    }
    return b[i] - ax;
}

// Coarse right side b_c[p] = sum over the members i of p of (b - A x)_i.
// Eight lanes per aggregate (an aggregate of the split 2x2x2 aggregation has
// at most eight members): lane j forms the residuals of members j, j+8, ...
// and the eight partial sums meet in a fixed butterfly, so the result does not
// depend on scheduling.  With xc: also the coarse level's first Chebyshev
// step, xc = c0 D^-1 b_c.
constexpr int RLANES = 8;

template <typename T>
__global__ __launch_bounds__(256) void k_restrict_rows(FineLevelT<T> f, int nc, const int *__restrict__ mptr,
                                                       const int *__restrict__ mem, const T *__restrict__ b,
                                                       const T *__restrict__ x, T *__restrict__ bc, const Scal *sc,
                                                       long long vs, long long vsc, T *__restrict__ xc,
                                                       const T *__restrict__ dinv, T c0)
{
    const bool done = ell_stopped(sc);
    b += blockIdx.y * vs;
    x += blockIdx.y * vs;
    bc += blockIdx.y * vsc;
    if (xc) xc += blockIdx.y * vsc;
    const int j = threadIdx.x % RLANES;
    // the eight lanes of a group share p, so they run the same rounds (the butterfly needs all of them)
    for (int p = (blockIdx.x * blockDim.x + threadIdx.x) / RLANES; p < nc; p += gridDim.x * blockDim.x / RLANES) {
        const int q0 = mptr[p], q1 = mptr[p + 1];
        T s = T(0);
        for (int q = q0 + j; q < q1; q += RLANES) s += fine_resid(f, b, x, mem[q]);
#pragma unroll
        for (int m = 1; m < RLANES; m <<= 1) s += __shfl_xor(s, m, RLANES);
        if (j == 0 && !done) {
            bc[p] = s;
            if (xc) xc[p] = c0 * s * dinv[p];
        }
    }
}

// The same restriction from the direct member table (aggregates of at most eight members; lane j of a
// group takes member j): the member index, then the member's row or stencil, then the neighbours, with no
// wait inside a round.  FELL: the finer level is an ELL level stored with 8 entries per row; otherwise a
// structured level with stored weights.  The stop flag only guards the stores.
template <typename T, bool FELL>
__global__ __launch_bounds__(256) void k_restrict8(FineLevelT<T> f, int nc, const int *__restrict__ memb,
                                                   const T *__restrict__ b, const T *__restrict__ x,
                                                   T *__restrict__ bc, const Scal *sc, long long vs, long long vsc,
                                                   T *__restrict__ xc, const T *__restrict__ dinv, T c0)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int p = (int)(t / RLANES), j = (int)(t % RLANES);
    const bool inr = p < nc;   // (every lane of a group reaches the butterfly)
    const int stop = sc[blockIdx.y].done;
    b += blockIdx.y * vs;
    x += blockIdx.y * vs;
    bc += blockIdx.y * vsc;
    // unconditional loads at clamped indices (a load under a condition becomes a branch that waits for it)
    const int mi = memb[inr ? (long long)p * RLANES + j : 0];
    const T dq = (xc ? dinv : b)[inr ? p : 0];
    const int i = inr ? mi : -1;
    const T dp = xc ? dq : T(0);
    const long long ii = i >= 0 ? i : 0;   // a valid row for the loads of a lane without a member
    T r;
    if constexpr (FELL) {
        int jj[ELL_K8];
        T vv[ELL_K8];
#pragma unroll
        for (int k = 0; k < ELL_K8; ++k) {
            jj[k] = f.col[(long long)k * f.n + ii];
            vv[k] = f.val[(long long)k * f.n + ii];
        }
        const T xi = x[ii], bi = b[ii];
        T xj[ELL_K8];
#pragma unroll
        for (int k = 0; k < ELL_K8; ++k) xj[k] = x[jj[k] >= 0 ? jj[k] : ii];
        T y = T(0);
#pragma unroll
        for (int k = 0; k < ELL_K8; ++k) y += (jj[k] >= 0 ? vv[k] : T(0)) * (xi - xj[k]);
        r = bi - y;
    } else {
        r = fine_resid(f, b, x, ii);
    }
    T sum = i >= 0 ? r : T(0);
#pragma unroll
    for (int m = 1; m < RLANES; m <<= 1) sum += __shfl_xor(sum, m, RLANES);
    if (j == 0 && inr && !stop) {
        bc[p] = sum;
        if (xc) xc[blockIdx.y * vsc + p] = c0 * sum * dp;
    }
}

// inverse diagonals (0 where the diagonal vanishes) of an ELL level
__global__ __launch_bounds__(256) void k_ell_setup(int n, int K, const int *__restrict__ col,
                                                   const double *__restrict__ val, double *__restrict__ d64,
                                                   float *__restrict__ d32, int *__restrict__ parent, EllStat *stat)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    double d = 0.0;
    if (i < n) {
        for (int k = 0; k < K; ++k)
            if (col[(long long)k * n + i] >= 0) d += val[(long long)k * n + i];
        const double v = d > 0.0 ? 1.0 / d : 0.0;
        if (d64) d64[i] = v;
        if (d32) d32[i] = (float)v;
        parent[i] = d > 0.0 ? i : -1;
    }
    const int count = __popcll(__ballot(d > 0.0));
    if ((threadIdx.x & 63) == 0 && count) atomicAdd(&stat[blockIdx.x % LEVEL_STATS].count, (unsigned)count);
}

// inverse diagonals, start of the next level's union-find and number of unknowns of a level made by the general kernel
hipError_t launch_ell_setup(int n, int K, const int *col, const double *val, double *d64, float *d32, int *parent,
                            EllStat *stat, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    SPFD_LAUNCH(k_ell_setup, dim3((n + 255) / 256), dim3(256), 0, s, n, K, col, val, d64, d32, parent, stat);
    return hipGetLastError();
}

// The same step for levels stored with ELL_K8 entries per row (every level with rows of at most that many;
// the build pads them to it), one row per thread, written so that a
// thread's loads go out in two rounds without a wait in between the loads of a round: first its row (the
// eight column indices and values, b, d and its own x, and with the prolongation its aggregate), then the
// gathers of the neighbours' x (and their aggregates and coarse values).  The stop flag is loaded with the
// first round and tested after it was issued (the opaque copy keeps the compiler from testing it first,
// which would put one more memory round trip in front of the loads).
// (No __restrict__ here: with it the compiler may move the row loads past the opaque flag and its test.)
template <typename T, bool PRO>
__global__ __launch_bounds__(256) void k_ell_cheb_step8(int n, int K, const int *col, const T *val, const T *b,
                                                        const T *xin, T *xout, const T *din, T *dout, T c1, T c2,
                                                        const Scal *sc, long long vs, const int *agg, const T *xc,
                                                        T scale, long long vsc)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int stop = sc[blockIdx.y].done;
    b += blockIdx.y * vs;
    xin += blockIdx.y * vs;
    xout += blockIdx.y * vs;
    const bool has_d = din != nullptr;
    const T *dsrc = has_d ? din + blockIdx.y * vs : xin;   // (a valid address either way)
    if (dout) dout += blockIdx.y * vs;
    if (PRO) xc += blockIdx.y * vsc;
    int j[ELL_K8];
    T v[ELL_K8];
#pragma unroll
    for (int k = 0; k < ELL_K8; ++k) {
        j[k] = col[(long long)k * n + i];
        v[k] = val[(long long)k * n + i];
    }
    const T bi = b[i];
    const T dd = dsrc[i];
    const T x0 = xin[i];
    const int a0 = PRO ? agg[i] : -1;
    asm volatile("" : "+s"(stop) : : "memory");
    if (stop) return;
    // second round: the neighbours (padding entries read the row's own slot with weight 0)
    T xj[ELL_K8];
    int aj[ELL_K8];
#pragma unroll
    for (int k = 0; k < ELL_K8; ++k) {
        const int jj = j[k] >= 0 ? j[k] : i;
        xj[k] = xin[jj];
        if (PRO) aj[k] = agg[jj];
    }
    T xi = x0;
    if (PRO) {
        const T c0v = xc[a0 >= 0 ? a0 : 0];
        T cj[ELL_K8];
#pragma unroll
        for (int k = 0; k < ELL_K8; ++k) cj[k] = xc[aj[k] >= 0 ? aj[k] : 0];
        xi = a0 >= 0 ? x0 + scale * c0v : x0;
#pragma unroll
        for (int k = 0; k < ELL_K8; ++k) xj[k] = aj[k] >= 0 ? xj[k] + scale * cj[k] : xj[k];
    }
    T y = T(0), d = T(0);
#pragma unroll
    for (int k = 0; k < ELL_K8; ++k) {
        const T w = j[k] >= 0 ? v[k] : T(0);
        d += w;
        y += w * (xi - xj[k]);
    }
    T xo = T(0), dn = T(0);
    if (d > T(0)) {
        const T dold = has_d ? dd : xi;
        dn = c1 * dold + c2 * (bi - y) / d;
        xo = xi + dn;
    }
    xout[i] = xo;
    if (dout) dout[i] = dn;
}

// x_f += scale * x_c[agg]
template <typename T>
__global__ void k_prolong_agg(long long n, const int *__restrict__ agg, T *__restrict__ x, const T *__restrict__ xc,
                              T scale, const Scal *sc, long long vs, long long vsc)
{
    // the stop flag guards the stores only (tested before the loads it would cost one more round trip)
    const bool stop = ell_stopped(sc);
    x += blockIdx.y * vs;
    xc += blockIdx.y * vsc;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
        const int a = agg[i];
        const T xv = x[i];
        const T cv = xc[a >= 0 ? a : 0];
        // (stored unconditionally, unchanged where nothing applies, so that the load of x is not moved
        // behind the aggregate's)
        x[i] = a >= 0 && !stop ? xv + scale * cv : xv;
    }
}

template <typename T>
hipError_t launch_ell_cheb_first(int n, int K, const int *col, const T *val, const T *b, T *x, T c0, const Scal *sc,
                                 const Batch &bt, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    SPFD_LAUNCH(k_ell_cheb_first<T>, dim3(gblocks(n), bt.n), dim3(256), 0, s, n, K, col, val, b, x, c0, sc,
                       bt.vs);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_ell_cheb_step(int n, int K, const int *col, const T *val, const T *b, const T *xin, T *xout,
                                const T *din, T *dout, T c1, T c2, const Scal *sc, const Batch &bt, hipStream_t s,
                                const int *agg, const T *xc, T scale)
{
    if (n <= 0) return hipSuccess;
    if (agg && !xc) return hipErrorInvalidValue;
    const long long nb = (n + 255) / 256;
    if (K == ELL_K8 && sc && nb <= 65536) {
        if (agg)
            SPFD_LAUNCH((k_ell_cheb_step8<T, true>), dim3((unsigned)nb, bt.n), dim3(256), 0, s, n, K, col, val, b, xin,
                        xout, din, dout, c1, c2, sc, bt.vs, agg, xc, scale, bt.vsc);
        else
            SPFD_LAUNCH((k_ell_cheb_step8<T, false>), dim3((unsigned)nb, bt.n), dim3(256), 0, s, n, K, col, val, b, xin,
                        xout, din, dout, c1, c2, sc, bt.vs, agg, xc, scale, bt.vsc);
        return hipGetLastError();
    }
    SPFD_LAUNCH(k_ell_cheb_step<T>, dim3(gblocks(n), bt.n), dim3(256), 0, s, n, K, col, val, b, xin, xout, din, dout,
                c1, c2, sc, bt.vs, agg, xc, scale, bt.vsc);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_restrict_members(const FineLevelT<T> &f, long long nrows, const T *b, const T *x, int nc,
                                   const int *mptr, const int *mem, T *bc, const Scal *sc, const Batch &bt,
                                   hipStream_t s, T *xc, const T *dinv_c, T c0, const int *memb)
{
    if (nc <= 0 || nrows <= 0) return hipSuccess;
    if (xc && !dinv_c) return hipErrorInvalidValue;
    const long long nt = (long long)nc * RLANES, nbk = (nt + 255) / 256;
    if (memb && sc && nbk <= 65536 && (f.w || f.K == ELL_K8)) {
        if (f.w)
            SPFD_LAUNCH((k_restrict8<T, false>), dim3((unsigned)nbk, bt.n), dim3(256), 0, s, f, nc, memb, b, x, bc, sc,
                        bt.vs, bt.vsc, xc, dinv_c, c0);
        else
            SPFD_LAUNCH((k_restrict8<T, true>), dim3((unsigned)nbk, bt.n), dim3(256), 0, s, f, nc, memb, b, x, bc, sc,
                        bt.vs, bt.vsc, xc, dinv_c, c0);
        return hipGetLastError();
    }
    SPFD_LAUNCH(k_restrict_rows<T>, dim3(gblocks((long long)nc * RLANES, 256), bt.n), dim3(256), 0, s, f, nc, mptr,
                mem, b, x, bc, sc, bt.vs, bt.vsc, xc, dinv_c, c0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_prolong_agg(long long n, const int *agg, T *x, const T *xc, T scale, const Scal *sc,
                              const Batch &bt, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    SPFD_LAUNCH(k_prolong_agg<T>, dim3(gblocks(n), bt.n), dim3(256), 0, s, n, agg, x, xc, scale, sc, bt.vs,
                       bt.vsc);
    return hipGetLastError();
}

#define SPFD_INST_ELL(T)                                                                                            \
    template hipError_t launch_ell_cheb_first<T>(int, int, const int *, const T *, const T *, T *, T, const Scal *, \
                                                 const Batch &, hipStream_t);                                       \
    template hipError_t launch_ell_cheb_step<T>(int, int, const int *, const T *, const T *, const T *, T *,         \
                                                const T *, T *, T, T, const Scal *, const Batch &, hipStream_t,     \
                                                const int *, const T *, T);                                         \
    template hipError_t launch_restrict_members<T>(const FineLevelT<T> &, long long, const T *, const T *, int,      \
                                                   const int *, const int *, T *, const Scal *, const Batch &,      \
                                                   hipStream_t, T *, const T *, T, const int *);                    \
    template hipError_t launch_prolong_agg<T>(long long, const int *, T *, const T *, T, const Scal *,             \
                                              const Batch &, hipStream_t);
SPFD_INST_ELL(double)
SPFD_INST_ELL(float)

// ---------------------------------------------------------------- coarsest level given as ELL
// unknowns = rows with D > 0, in row order; adjacency among them
__global__ __launch_bounds__(1024) void k_coarse_enum_ell(int n, int K, const int *__restrict__ col, const double *__restrict__ val,
                                  int *dof_of_row, int *row_of_dof, int *ndof, int maxdof)
{
    __shared__ int count[16];
    const int t = threadIdx.x;
    int carry = 0;
    for (int base = 0; base < n; base += 1024) {
        const int i = base + t;
        double d = 0.0;
        if (i < n)
            for (int k = 0; k < K; ++k)
                if (col[(long long)k * n + i] >= 0) d += val[(long long)k * n + i];
        const bool isdof = d > 0.0;
        int total;
        const int id = carry + flags_before(isdof, count, &total);
        if (i < n) {
            dof_of_row[i] = isdof ? id : -1;
            if (isdof && id < maxdof) row_of_dof[id] = i;
        }
        carry += total;
    }
    if (t == 0) *ndof = carry;
}

hipError_t launch_coarse_enum_ell(int n, int K, const int *col, const double *val, int *dof_of_row, int *row_of_dof,
                                  int *ndof, int maxdof, hipStream_t s)
{
    SPFD_LAUNCH(k_coarse_enum_ell, dim3(1), dim3(1024), 0, s, n, K, col, val, dof_of_row, row_of_dof, ndof,
                       maxdof);
    return hipGetLastError();
}

// dense matrix of the coarsest ELL level over its unknowns (row-major n x n)
__global__ void k_coarse_dense_ell(int nrow, int K, const int *__restrict__ col, const double *__restrict__ val,
                                   const int *__restrict__ dof_of_row, const int *__restrict__ row_of_dof, int n,
                                   double *A)
{
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < (long long)n * n;
         e += (long long)gridDim.x * blockDim.x)
        A[e] = 0.0;
}

__global__ void k_coarse_fill_ell(int nrow, int K, const int *__restrict__ col, const double *__restrict__ val,
                                  const int *__restrict__ dof_of_row, const int *__restrict__ row_of_dof, int n,
                                  double *A)
{
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < n; q += gridDim.x * blockDim.x) {
        const int i = row_of_dof[q];
        double d = 0.0;
        for (int k = 0; k < K; ++k) {
            const int j = col[(long long)k * nrow + i];
            if (j < 0) continue;
            const double w = val[(long long)k * nrow + i];
            d += w;
            const int m = dof_of_row[j];
            if (m >= 0) A[(long long)q * n + m] -= w;
        }
        A[(long long)q * n + q] += d;
    }
}

hipError_t launch_coarse_dense_ell(int nrow, int K, const int *col, const double *val, const int *dof_of_row,
                                   const int *row_of_dof, int n, double *A, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    SPFD_LAUNCH(k_coarse_dense_ell, dim3(gblocks((long long)n * n)), dim3(256), 0, s, nrow, K, col, val,
                       dof_of_row, row_of_dof, n, A);
    SPFD_LAUNCH(k_coarse_fill_ell, dim3(gblocks(n)), dim3(256), 0, s, nrow, K, col, val, dof_of_row,
                       row_of_dof, n, A);
    return hipGetLastError();
}

}  // namespace spfd
