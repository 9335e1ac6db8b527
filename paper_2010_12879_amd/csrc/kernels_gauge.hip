// Edge potentials from facet fluxes, Eq. (2) b = C a, in a tree-cotree gauge
// (technical summary of Sec. II.A, step 3).
//
// On the structured voxel grid a spanning tree of the nodes is fixed: every
// z-edge, the y-edges of the node plane k = 0 and the x-edges of the node line
// j = k = 0 carry a = 0.  Every cotree edge then closes one facet whose other
// three edges are known, so the over-determined system becomes prefix sums:
//   plane k = 0 (z-facets):  a_x(i, j+1, 0) = a_x(i, j, 0) - b_z(i, j, 0)   (one thread per i)
//   columns (y- and x-facets): a_x(i, j, k+1) = a_x(i, j, k) + b_y(i, j, k),
//                              a_y(i, j, k+1) = a_y(i, j, k) - b_x(i, j, k)  (one thread per (i, j))
// and the remaining z-facets hold when the fluxes are divergence-free.  Arrays
// are [3][Nz][Ny][Nx] node-anchored (flux of normal d and edge along d start
// at node (i, j, k)), as the sources of spfd_set_source.  The sums run in the
// order of the recurrences.
#include "kernels.h"

namespace spfd {

// Plane and columns are serial chains (their sums keep the order of the recurrence), few against the chip's
// lanes.  Columns: the component is the launch's y index (a_x, a_y, the zeros of a_z), so that the chains of
// a_x and a_y run on different waves, in one-wave workgroups that spread over all CUs, and every lane loads
// the next TC_U fluxes while it adds and stores the present ones.  Plane and columns of the 250 x 150 x 900
// body: 63 + 667 us with one load after the other, 11 + 393 us now (1.36 GB, 3.5 TB/s).
constexpr int TC_U = 16;
constexpr int TC_T = 64;

__global__ __launch_bounds__(TC_T) void k_tc_plane(const double *__restrict__ flux, double *__restrict__ a, Grid g)
{
    const int i = blockIdx.x * TC_T + threadIdx.x;
    if (i >= g.nx) return;
    const long long nn = (long long)g.Nx * g.Ny * g.Nz;
    const double *bz = flux + 2 * nn + i;
    double acc = 0.0, cur[TC_U], nxt[TC_U];
    a[i] = 0.0;
#pragma unroll
    for (int u = 0; u < TC_U; ++u) cur[u] = bz[(long long)(u < g.ny ? u : g.ny - 1) * g.Nx];
    for (int j = 0; j < g.ny; j += TC_U) {
#pragma unroll
        for (int u = 0; u < TC_U; ++u) {
            const int l = j + TC_U + u;
            nxt[u] = bz[(long long)(l < g.ny ? l : g.ny - 1) * g.Nx];
        }
#pragma unroll
        for (int u = 0; u < TC_U; ++u)
            if (j + u < g.ny) {
                acc -= cur[u];
                a[(long long)(j + u + 1) * g.Nx + i] = acc;
            }
#pragma unroll
        for (int u = 0; u < TC_U; ++u) cur[u] = nxt[u];
    }
}

__global__ __launch_bounds__(TC_T) void k_tc_columns(const double *__restrict__ flux, double *__restrict__ a, Grid g)
{
    // (a layer has fewer than 2^32 columns)
    const unsigned e = blockIdx.x * TC_T + threadIdx.x;
    if (e >= (unsigned)g.Nx * (unsigned)g.Ny) return;
    const int i = (int)(e % (unsigned)g.Nx), j = (int)(e / (unsigned)g.Nx);
    const long long nn = (long long)g.Nx * g.Ny * g.Nz;
    const long long plane = (long long)g.Nx * g.Ny;
    const int d = blockIdx.y;
    double *o = a + d * nn + e;
    if (d == 2) {
        for (int k = 0; k <= g.nz; ++k) o[k * plane] = 0.0;
        return;
    }
    const bool in = d == 0 ? i < g.nx : j < g.ny;
    // a_x: the plane k = 0, written by k_tc_plane (zero beyond the grid); a_y starts at 0
    double s = d == 0 && in ? o[0] : 0.0;
    if (d == 1 || !in) o[0] = 0.0;
    if (!in) {
        for (int k = 1; k <= g.nz; ++k) o[k * plane] = 0.0;
        return;
    }
    const double *f = flux + (d == 0 ? nn : 0) + e;   // b_y adds to a_x, b_x subtracts from a_y
    double cur[TC_U], nxt[TC_U];
#pragma unroll
    for (int u = 0; u < TC_U; ++u) cur[u] = f[(u < g.nz ? u : g.nz - 1) * plane];
    for (int k = 0; k < g.nz; k += TC_U) {
#pragma unroll
        for (int u = 0; u < TC_U; ++u) {
            const int l = k + TC_U + u;
            nxt[u] = f[(l < g.nz ? l : g.nz - 1) * plane];
        }
#pragma unroll
        for (int u = 0; u < TC_U; ++u)
            if (k + u < g.nz) {
                s = d == 0 ? s + cur[u] : s - cur[u];
                o[(k + u + 1) * plane] = s;
            }
#pragma unroll
        for (int u = 0; u < TC_U; ++u) cur[u] = nxt[u];
    }
}

hipError_t launch_tree_cotree(const double *flux, double *a, const Grid &g, hipStream_t s)
{
    SPFD_LAUNCH(k_tc_plane, dim3((g.nx + TC_T - 1) / TC_T), dim3(TC_T), 0, s, flux, a, g);
    const unsigned long long cols = (unsigned long long)g.Nx * g.Ny;
    if (cols > 0xffffffffull) return hipErrorInvalidValue;
    SPFD_LAUNCH(k_tc_columns, dim3((unsigned)((cols + TC_T - 1) / TC_T), 3), dim3(TC_T), 0, s, flux, a, g);
    return hipGetLastError();
}

}  // namespace spfd
