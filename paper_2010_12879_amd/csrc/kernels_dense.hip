// Dense inverse of the coarsest-level matrix by blocked Gauss-Jordan
// elimination on 64x64 tiles, one launch per tile step.
//
// The matrix (after the rank-one regularisation of every connected component,
// which makes it symmetric positive definite) is copied into an ld x ld work
// array, ld = n rounded up to 64, with the identity on the padding.  For each
// diagonal tile k, with P = A_kk^-1:
//   A_kk <- P,   A_kj <- P A_kj,   A_ik <- -A_ik P,
//   A_ij <- A_ij - (A_ik P) A_kj            (i, j != k; old A_ik, A_kj)
// Every tile of step k reads only the previous matrix and writes the next one
// (two work matrices used in turn), so one launch covers the whole step.  The
// workgroup of the next diagonal tile comes first and goes on to invert it
// (P of the next step), while the others update their tiles: a step lasts as
// long as that one workgroup, whose 64 pivots are a serial chain.  The products
// are FP64 matrix instructions, whose sum over k is the chain of multiply-adds
// in ascending k to the last bit.  No pivoting is needed for a symmetric
// positive definite matrix.  640 unknowns, 10 steps: 34 us of inverse and 26 us
// of update in turn, 0.65 ms in all; then 20 + 19 us a step in one launch,
// 0.43 ms; with matrix instructions and the inverse on four waves 18 + 11 us, 0.31 ms.
#include "kernels.h"

namespace spfd {

constexpr int GT = 64;        // tile edge
// LDS row strides of a left and a right factor: the 32 lanes of a read take 16 rows by 2 columns of the left one, 2
// rows by 16 columns of the right one, which these spread over all 64 banks
constexpr int GA = GT + 2, GB = GT + 16;
constexpr int GI = 4;         // rows and columns per thread in the tile inverse (256 threads)

__global__ __launch_bounds__(256) void k_gj_pad(int n, int ld, const double *__restrict__ A, double *__restrict__ W)
{
    const long long tot = (long long)ld * ld;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < tot;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(e / ld), j = (int)(e % ld);
        W[e] = (i < n && j < n) ? A[(long long)i * n + j] : (i == j ? 1.0 : 0.0);
    }
}

__global__ __launch_bounds__(256) void k_gj_unpad(int n, int ld, const double *__restrict__ W, double *__restrict__ A)
{
    const long long tot = (long long)n * n;
    for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < tot;
         e += (long long)gridDim.x * blockDim.x) {
        const int i = (int)(e / n), j = (int)(e % n);
        A[e] = W[(long long)i * ld + j];
    }
}

template <int S>
__device__ __forceinline__ void tile_load(const double *__restrict__ src, int ld, int r0, int c0, double *t)
{
    for (int e = threadIdx.x; e < GT * GT; e += blockDim.x) {
        const int r = e / GT, c = e % GT;
        t[r * S + c] = src[(long long)(r0 + r) * ld + c0 + c];
    }
}

typedef double double4v __attribute__((ext_vector_type(4)));

// a * b for LDS tiles (row strides GA, GB), 16 waves: wave w the 16x16 block (w / 4, w % 4); entry r of lane l is row
// l / 16 + 4 r, column l % 16 of it
__device__ __forceinline__ double4v tile_mul(const double *a, const double *b)
{
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double *ap = a + (16 * (w >> 2) + (l & 15)) * GA + (l >> 4);
    const double *bp = b + (l >> 4) * GB + 16 * (w & 3) + (l & 15);
    double4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < GT; k += 4) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ap[k], bp[k * GB], acc, 0, 0, 0);
    return acc;
}

// In-place Gauss-Jordan inverse of a 64x64 tile held by 256 threads: thread t
// holds rows 4 (t/16) .. +3 by columns 4 (t%16) .. +3.  For pivot p with d = A_pp:
//   A_pj <- A_pj / d (j != p),  A_pp <- 1/d,
//   A_ij <- A_ij - (A_ip / d) A_pj (i, j != p),  A_ip <- -A_ip / d,
// that is, one multiply-add per entry once row p carries 1 in place of d and
// the entries of column p outside row p start from 0.  Row p (with 1/d
// beside it) and column p pass through LDS; the threads that own row and
// column p + 1 publish them right after their update for pivot p, into the
// other of two buffers, so each pivot needs one barrier.  (Sixteen entries a
// thread need 64 B of row and column per pivot; with four entries each, 1024
// threads read 2.7 times as much from LDS and met at a barrier of 16 waves:
// 20 us for the 64 pivots, now 18.)
struct InvLds {
    double row[2][GT + 2];   // [GT]: reciprocal pivot; rows 16-byte aligned for wide loads
    double col[2][GT];
};

__device__ __forceinline__ void tile_inverse(double a[GI][GI], InvLds &L)
{
    const int ib = threadIdx.x >> 4, jb = threadIdx.x & 15;
    // (pivot p = GI pb + q, q known at compile time)
    auto publish = [&](int pb, int q, int buf) {
        if (ib == pb) {
            if (jb == pb) L.row[buf][GT] = 1.0 / a[q][q];
#pragma unroll
            for (int k = 0; k < GI; ++k) L.row[buf][GI * jb + k] = (k == q && jb == pb) ? 1.0 : a[q][k];
        }
        if (jb == pb) {
#pragma unroll
            for (int i = 0; i < GI; ++i) L.col[buf][GI * ib + i] = a[i][q];
        }
    };
    publish(0, 0, 0);
    __syncthreads();
    for (int pb = 0; pb < GT / GI; ++pb) {
#pragma unroll
        for (int q = 0; q < GI; ++q) {
            const int cur = q & 1;   // (GI even)
            const double piv = L.row[cur][GT];
            double r[GI], c[GI];
#pragma unroll
            for (int k = 0; k < GI; ++k) {
                r[k] = L.row[cur][GI * jb + k];
                c[k] = L.col[cur][GI * ib + k];
            }
            if (jb == pb) {
#pragma unroll
                for (int i = 0; i < GI; ++i) a[i][q] = 0.0;
            }
#pragma unroll
            for (int i = 0; i < GI; ++i) {
                const double cp = c[i] * piv;
#pragma unroll
                for (int k = 0; k < GI; ++k) a[i][k] = __builtin_fma(-cp, r[k], a[i][k]);
            }
            if (ib == pb) {
#pragma unroll
                for (int k = 0; k < GI; ++k) a[q][k] = r[k] * piv;
            }
            if (q + 1 < GI)
                publish(pb, q + 1, cur ^ 1);
            else if (pb + 1 < GT / GI)
                publish(pb + 1, 0, cur ^ 1);
            __syncthreads();
        }
    }
}

// P = A_00^-1 (the first diagonal tile)
__global__ __launch_bounds__(256) void k_gj_diag(int ld, const double *__restrict__ W, double *__restrict__ P)
{
    __shared__ __align__(16) InvLds L;
    const int i0 = (threadIdx.x >> 4) * GI, j0 = (threadIdx.x & 15) * GI;
    double a[GI][GI];
#pragma unroll
    for (int i = 0; i < GI; ++i)
#pragma unroll
        for (int j = 0; j < GI; ++j) a[i][j] = W[(long long)(i0 + i) * ld + j0 + j];
    tile_inverse(a, L);
#pragma unroll
    for (int i = 0; i < GI; ++i)
#pragma unroll
        for (int j = 0; j < GI; ++j) P[(i0 + i) * GT + j0 + j] = a[i][j];
}

// Step k: the tiles of Wn from Wo and P = (Wo)_kk^-1, and (not in the last step) Pn = (Wn)_{k+1,k+1}^-1
__global__ __launch_bounds__(1024) void k_gj_step(int ld, int nt, int k, const double *__restrict__ Wo,
                                                  double *__restrict__ Wn, const double *__restrict__ P,
                                                  double *__restrict__ Pn)
{
    __shared__ __align__(16) double ta[GT * GA];
    __shared__ __align__(16) double tb[GT * GB];
    __shared__ __align__(16) double tc[GT * GB];
    __shared__ __align__(16) InvLds L;
    // the next diagonal tile first (tile 0 takes its place)
    const int next = k + 1 < nt ? (k + 1) * (nt + 1) : 0;
    const int id = blockIdx.x == 0 ? next : (int)blockIdx.x == next ? 0 : blockIdx.x;
    const int bi = id / nt, bj = id % nt;
    const int k0 = k * GT, i0 = bi * GT, j0 = bj * GT;
    // the thread's entries of a product (tile_mul)
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r0 = 16 * (w >> 2) + (l >> 4), c0 = 16 * (w & 3) + (l & 15);
    if (bi == k && bj == k) {   // A_kk <- P
        for (int e = threadIdx.x; e < GT * GT; e += blockDim.x) Wn[(long long)(k0 + e / GT) * ld + k0 + e % GT] = P[e];
        return;
    }
    if (bi == k || bj == k) {   // A_kj <- P A_kj,  A_ik <- -A_ik P
        if (bi == k) {
            tile_load<GA>(P, GT, 0, 0, ta);
            tile_load<GB>(Wo, ld, k0, j0, tb);
        } else {
            tile_load<GA>(Wo, ld, i0, k0, ta);
            tile_load<GB>(P, GT, 0, 0, tb);
        }
        __syncthreads();
        const double4v acc = tile_mul(ta, tb);
        const double sg = bi == k ? 1.0 : -1.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) Wn[(long long)(i0 + r0 + 4 * r) * ld + j0 + c0] = sg * acc[r];
        return;
    }
    // other tiles: A_ij - (A_ik P) A_kj; all three tiles and the old A_ij loaded up front
    double old[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) old[r] = Wo[(long long)(i0 + r0 + 4 * r) * ld + j0 + c0];
    tile_load<GA>(Wo, ld, i0, k0, ta);
    tile_load<GB>(P, GT, 0, 0, tb);
    tile_load<GB>(Wo, ld, k0, j0, tc);
    __syncthreads();
    double4v acc = tile_mul(ta, tb);      // T = A_ik P
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) ta[(r0 + 4 * r) * GA + c0] = acc[r];
    __syncthreads();
    acc = tile_mul(ta, tc);               // T A_kj
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        acc[r] = old[r] - acc[r];
        Wn[(long long)(i0 + r0 + 4 * r) * ld + j0 + c0] = acc[r];
    }
    if (blockIdx.x != 0 || k + 1 == nt) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) tb[(r0 + 4 * r) * GB + c0] = acc[r];
    __syncthreads();
    if (threadIdx.x >= 256) return;       // (waves that have ended do not count at a barrier)
    const int ia = (threadIdx.x >> 4) * GI, ja = (threadIdx.x & 15) * GI;
    double a[GI][GI];
#pragma unroll
    for (int i = 0; i < GI; ++i)
#pragma unroll
        for (int j = 0; j < GI; ++j) a[i][j] = tb[(ia + i) * GB + ja + j];
    tile_inverse(a, L);
#pragma unroll
    for (int i = 0; i < GI; ++i)
#pragma unroll
        for (int j = 0; j < GI; ++j) Pn[(ia + i) * GT + ja + j] = a[i][j];
}

size_t dense_inverse_work_doubles(int n)
{
    const long long ld = ((long long)n + GT - 1) / GT * GT;
    return (size_t)(2 * ld * ld + 2 * GT * GT);
}

hipError_t launch_dense_inverse(int n, double *A, double *work, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const int ld = (n + GT - 1) / GT * GT;
    const int nt = ld / GT;
    double *W[2] = {work, work + (long long)ld * ld};
    double *P[2] = {work + 2LL * ld * ld, work + 2LL * ld * ld + GT * GT};
    auto blocks = [](long long m) { return (unsigned)((m + 255) / 256 > 65536 ? 65536 : (m + 255) / 256); };
    SPFD_LAUNCH(k_gj_pad, dim3(blocks((long long)ld * ld)), dim3(256), 0, s, n, ld, A, W[0]);
    SPFD_LAUNCH(k_gj_diag, dim3(1), dim3(256), 0, s, ld, W[0], P[0]);
    for (int k = 0; k < nt; ++k)
        SPFD_LAUNCH(k_gj_step, dim3(nt * nt), dim3(1024), 0, s, ld, nt, k, W[k & 1], W[(k + 1) & 1], P[k & 1],
                    P[(k + 1) & 1]);
    SPFD_LAUNCH(k_gj_unpad, dim3(blocks((long long)n * n)), dim3(256), 0, s, n, ld, W[nt & 1], A);
    return hipGetLastError();
}

}  // namespace spfd
