// One leg of the multigrid cycle on a small structured level in one kernel.
//
// A workgroup owns one brick (on the smallest levels an eighth of one).  It
// loads it and H nodes around it (H = the level's smoothing degree), runs
// every Chebyshev step of the leg on that region, exchanging x through LDS,
// and stores what its own nodes give:
//   down: the steps from the level's first iterate, the residual and its
//         restriction (with the coarser level's first iterate);
//   up:   the coarse-grid correction and the steps; on the finest level also
//         the partial sums of z.r of the outer CG.
// The nodes around the brick are smoothed again by every workgroup that needs
// them: a node at distance d of the brick takes part in the first H - d steps
// only, so no value crosses workgroups inside a leg.
//
// Why: a level of some hundred bricks has all its waves resident at once and
// each of its kernels lasts one wave's latency, about 5.5 us with the gap to
// the next; the degree-4 level alone is eight of them per cycle.  The region
// is 2.7 (H = 2) to 5.2 (H = 4) times the brick, so the leg pays while the
// workgroups together leave the chip idle, and loses on levels that fill it
// (leg_max).
//
// Every node is computed as the separate kernels compute it, to the last bit,
// so the choice of the form may depend on the number of right sides and moves
// no result.  (With the FP32 cycle a solve to 1e-8 answers roundings by more
// than their size on bodies of coarse voxels: a rounding up or down of every
// source value moves |E| of a body at 4 mm, driven by potentials in the
// tree-cotree gauge, by up to 4.8e-8 in the 2-norm and 1.5e-7 of its largest
// value, at 2 mm by 2.8e-12; with the FP64 cycle by 1.7e-13.)  The separate kernels
// leave their multiply-adds to the compiler; here they are written out as it
// forms them there, and nothing else is contracted:
//   * A x starts with the +x edge's product, the others are added to it;
//   * 1/D and D b of the label form take D from fused products of the
//     conductivity sums, except that of the edge below a node that shares it
//     with the node below in the same column segment;
//   * a corrected iterate is one multiply-add, but a product and a sum where
//     a segment sees it across an x or y face of its brick;
//   * the difference to a first iterate c0 D^-1 b beyond a segment's z ends is
//     one multiply-add.
#include <type_traits>
#include <hip/hip_fp16.h>

#include "kernels.h"

namespace spfd {

// (as the column kernels: the hardware reciprocal in FP32, a division in FP64)
template <typename T>
__device__ __forceinline__ T brecip(T d) { return T(1) / d; }
template <>
__device__ __forceinline__ float brecip<float>(float d) { return __builtin_amdgcn_rcpf(d); }

__device__ __forceinline__ float fmadd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmadd(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Block of one workgroup: the brick, or a part of it (BX x BY x BZ nodes)
template <int H, int BX, int BY, int BZ>
struct BrickGeom {
    static constexpr int EX = BX + 2 * H, EY = BY + 2 * H, EZ = BZ + 2 * H;   // region
    static constexpr int ZS = EZ / 4;                                         // nodes per thread, consecutive in z
    static constexpr int NTH = 4 * EX * EY;                                   // threads
    static constexpr int EC = EX * EY * EZ;
    static constexpr int NX = 8 / BX, NY = 8 / BY, PARTS = NX * NY * (8 / BZ);
    static_assert(EZ % 4 == 0 && NTH <= 1024 && EC >= BS && NTH >= BX * BY * BZ, "one region, one workgroup");
};

// distance of region coordinate e from the block (B nodes) along its axis
template <int H, int B>
__device__ __forceinline__ int halo_depth(int e)
{
    return e < H ? H - e : (e >= B + H ? e - (B - 1) - H : 0);
}

enum { BR_LABEL = 0, BR_STORED = 1, BR_HALF = 2 };

// ||r||^2 and the stop test of the step before (k_finish, FIN_RR) for up to RR_MOST partials, one a thread; red: LDS
__device__ __forceinline__ void finish_rr(const RrIn &in, int row, double *red)
{
    const int t = threadIdx.x;
    const double *part = in.part + (long long)row * in.ps;
    Scal *sc = in.sc + row;
    const int stopped = sc->done;
    double a = t < in.n ? part[t] : 0.0;
    a = wave_sum(a);
    if ((t & 63) == 0) red[t >> 6] = a;
    __syncthreads();
    if (t != 0) return;
    if (!stopped) {
        a = 0.0;
        for (int w = 0; w < RR_MOST / 64; ++w) a += red[w];
        sc->rr = a;
        sc->iters += 1;
        sc->hcount += 1;   // the step's search direction and step size are kept
        if (a <= sc->tol2) {
            sc->done = 1;
        } else if (!isfinite(a)) {
            sc->status = 6;
            sc->done = 1;
        } else if (sc->iters >= in.max_iter) {
            sc->status = 5;
            sc->done = 1;
        }
    }
    store_mirror(in.mirror, sc, in.stamp, row);
}

// OPK: the operator (label form, stored weights, FP16 weights).  FINE: the finest level (down: the first
// iterate is c0 D^-1 b, formed here; up: the dot products).  UP: the upward leg.  CELL: the coarser level is
// an ELL level (member table, aggregate map).
template <typename T, int H, int BX, int BY, int BZ, int OPK, bool FINE, bool UP, bool CELL>
__global__ __launch_bounds__((BrickGeom<H, BX, BY, BZ>::NTH)) void k_brick_leg(BrickLeg<T> A)
{
#pragma clang fp contract(off)
    using G = BrickGeom<H, BX, BY, BZ>;
    constexpr int SEG = sizeof(T) == 4 ? 8 : 4;   // nodes per lane of the column kernels on the finest level
    constexpr int EX = G::EX, EY = G::EY, EZ = G::EZ, EL = EX * EY, ZS = G::ZS, NTH = G::NTH;
    constexpr bool LABEL = OPK == BR_LABEL;
    constexpr int VX = EX + 1, VY = EY + 1, VL = VX * VY, NV = LABEL ? VL * (EZ + 1) : 1;
    auto depth_x = [](int e) { return halo_depth<H, BX>(e); };
    auto depth_y = [](int e) { return halo_depth<H, BY>(e); };
    auto depth_z = [](int e) { return halo_depth<H, BZ>(e); };
    __shared__ T xs[2][G::EC], xe[FINE && !UP ? G::EC : 1];
    __shared__ T sig[NV], tab[LABEL ? MAX_LABELS : 1];
    __shared__ int nslot[27], npar[27], stop;
    if constexpr (FINE && !UP) {
        // The right side may turn out to be done here: the leg's own workgroups do not wait for it (they write
        // nothing but the cycle's vectors, all of them again in the next cycle), and the kernels behind see the flag.
        // As it may change while they start, one thread of each reads it for its whole workgroup.
        if (A.rr.n > 0 && blockIdx.x == gridDim.x - 1) {
            finish_rr(A.rr, blockIdx.y, (double *)xs);
            return;
        }
    }
    const int part = xcd_brick(blockIdx.x, A.nb * G::PARTS);
    if (part < 0) return;
    const int b = part / G::PARTS;
    // the block's place in the brick, and the brick's node at region coordinate 0
    const int ox = part % G::NX * BX, oy = part / G::NX % G::NY * BY, oz = part % G::PARTS / (G::NX * G::NY) * BZ;
    const int rx = ox - H, ry = oy - H, rz = oz - H;
    const int t = threadIdx.x;
    if (t == 0) stop = A.sc[blockIdx.y].done;
    const int4 fc = A.coord[b];
    const unsigned long long cm = A.cmask[b];
    if (t < 27) {
        const int s = A.nbr27[b * 27 + t];
        nslot[t] = s;
        if constexpr (!CELL) npar[t] = A.parent_slot[s >= 0 ? s : 0];
    }
    if constexpr (LABEL) {
        const T *table = A.models ? A.table + A.models[b * NBR + NTAB] : A.table;
        for (int l = t; l < MAX_LABELS; l += NTH) tab[l] = l < A.nlab ? table[l] : T(0);
    }
    const long long vo = blockIdx.y * A.vs;
    // the thread's nodes: region column (ex, ey), layers ez0 .. ez0 + ZS - 1
    const int ex = t % EX, ey = (t / EX) % EY, ez0 = (t / EL) * ZS;
    const int hxy = depth_x(ex) + depth_y(ey);
    const int lx = (ex + rx) & 7, ly = (ey + ry) & 7;
    const bool own_xy = hxy == 0;
    const bool act = own_xy && ((cm >> (lx + 8 * ly)) & 1ull);
    // voxel labels of the region (voxel layer v lies below node layer v): one round of loads, no use yet
    constexpr int NL = LABEL ? (NV + NTH - 1) / NTH : 1;
    int lab[NL];
    if constexpr (LABEL) {
#pragma unroll
        for (int k = 0; k < NL; ++k) {
            const int e = t + k * NTH;
            const int i = 8 * fc.x + e % VX + rx - 1, j = 8 * fc.y + (e / VX) % VY + ry - 1,
                      l = 8 * fc.z + e / VL + rz - 1;
            const bool in = e < NV && i >= 0 && j >= 0 && l >= 0 && i < A.g.nx && j < A.g.ny && l < A.g.nz;
            lab[k] = in ? A.labels[i + (long long)A.g.nx * (j + (long long)A.g.ny * l)] : 0;
        }
    }
    __syncthreads();
    if (stop) return;   // (uniform: read once, above)
    auto brick_of = [&](int x, int y, int z) {   // index into nslot / npar of a region coordinate
        return ((x + rx) >> 3) + 1 + 3 * (((y + ry) >> 3) + 1) + 9 * (((z + rz) >> 3) + 1);
    };
    auto slot_of = [&](int x, int y, int z) -> long long {   // slot of a region node, -1 in an absent brick
        const int s = nslot[brick_of(x, y, z)];
        return s < 0 ? -1 : (long long)s * BS + ((x + rx) & 7) + 8 * ((y + ry) & 7) + 64 * ((z + rz) & 7);
    };
    // every load of the node data in one round: b, the iterate (down on the finest level: D^-1), the weights
    T bv[ZS], xv[ZS], xf[ZS], W[ZS][6], D[ZS];
    int ag[CELL ? ZS : 1];
    long long n[ZS];
    const T *xsrc = FINE && !UP ? A.dinv : A.xin + vo;
    const bool scaled = FINE && A.bscale;
#pragma unroll
    for (int z = 0; z < ZS; ++z) {
        const int h = hxy + depth_z(ez0 + z);
        n[z] = h <= H ? slot_of(ex, ey, ez0 + z) : -1;
        bv[z] = xv[z] = T(0);
        if (CELL) ag[z] = -1;
        if (n[z] >= 0) {
            bv[z] = A.b[vo + n[z]];
            if (!(FINE && !UP && scaled)) xv[z] = xsrc[n[z]];
            if (CELL) ag[z] = A.agg[n[z]];
        }
    }
    if constexpr (!LABEL) {
        // W[z][k]: first the loaded values (FP16: their bits), minus sides from the minus neighbours
        uint16_t hw[OPK == BR_HALF ? ZS : 1][6];
#pragma unroll
        for (int z = 0; z < ZS; ++z) {
            const bool in = n[z] >= 0 && hxy + depth_z(ez0 + z) < H;
            const long long mx = in ? slot_of(ex - 1, ey, ez0 + z) : -1, my = in ? slot_of(ex, ey - 1, ez0 + z) : -1;
            const long long mz = in && z == 0 ? slot_of(ex, ey, ez0 - 1) : -1;
            const long long st = A.stride;
            if constexpr (OPK == BR_HALF) {
                hw[z][NPX] = in ? A.wh[n[z]] : 0;
                hw[z][NPY] = in ? A.wh[st + n[z]] : 0;
                hw[z][NPZ] = n[z] >= 0 ? A.wh[2 * st + n[z]] : 0;
                hw[z][NMX] = mx >= 0 ? A.wh[mx] : 0;
                hw[z][NMY] = my >= 0 ? A.wh[st + my] : 0;
                hw[z][NMZ] = mz >= 0 ? A.wh[2 * st + mz] : 0;
            } else {
                W[z][NPX] = in ? A.w[n[z]] : T(0);
                W[z][NPY] = in ? A.w[st + n[z]] : T(0);
                W[z][NPZ] = n[z] >= 0 ? A.w[2 * st + n[z]] : T(0);
                W[z][NMX] = mx >= 0 ? A.w[mx] : T(0);
                W[z][NMY] = my >= 0 ? A.w[st + my] : T(0);
                W[z][NMZ] = mz >= 0 ? A.w[2 * st + mz] : T(0);
            }
        }
        if constexpr (OPK == BR_HALF) {
#pragma unroll
            for (int z = 0; z < ZS; ++z)
#pragma unroll
                for (int k = 0; k < 6; ++k) W[z][k] = (T)__half2float(__ushort_as_half(hw[z][k])) * (T)A.whs;
        }
        // inside the thread's run the lower edge of a node is the upper edge of the node below (which is why
        // that edge is loaded one node further out)
#pragma unroll
        for (int z = 1; z < ZS; ++z) W[z][NMZ] = W[z - 1][NPZ];
    }
    // up: the coarse-grid correction of every value read
    if constexpr (UP) {
        const T *xc = A.xc + blockIdx.y * A.vsc;
        T cv[ZS];
#pragma unroll
        for (int z = 0; z < ZS; ++z) {
            cv[z] = T(0);
            if constexpr (CELL) {
                if (n[z] >= 0) cv[z] = xc[ag[z] >= 0 ? ag[z] : 0];
            } else if (n[z] >= 0) {
                const int ez = ez0 + z, p = npar[brick_of(ex, ey, ez)];
                // fine node (8 f + l) -> node (4 (f & 1) + l / 2) of the parent brick
                const int px = (((ex + rx + 8 * fc.x) >> 3) & 1) * 4 + (lx >> 1);
                const int py = (((ey + ry + 8 * fc.y) >> 3) & 1) * 4 + (ly >> 1);
                const int pz = (((ez + rz + 8 * fc.z) >> 3) & 1) * 4 + (((ez + rz) & 7) >> 1);
                cv[z] = xc[(long long)p * BS + px + 8 * py + 64 * pz];
            }
        }
#pragma unroll
        for (int z = 0; z < ZS; ++z) {
            xf[z] = xv[z] + A.scale * cv[z];   // as seen across an x or y face of its brick
            if (!CELL || ag[z] >= 0) xv[z] = fmadd(A.scale, cv[z], xv[z]);
        }
    }
    // down: what the restriction reads besides the residual, loaded ahead; the thread's aggregate in the brick
    const int cx = ox / 2 + t % (BX / 2), cy = oy / 2 + t / (BX / 2) % (BY / 2), cz = oz / 2 + t / (BX * BY / 4);
    int rp = -1, rm[8] = {-1, -1, -1, -1, -1, -1, -1, -1};
    long long rn = 0;
    T rdc = T(0);
    if constexpr (!UP) {
        if constexpr (CELL) {
            if (t < BX * BY * BZ) {   // the first member of a piece stores it
                const int own = b * BS + ox + t % BX + 8 * (oy + t / BX % BY) + 64 * (oz + t / (BX * BY));
                const int p = A.agg[own];
                if (p >= 0) {
                    const int4 m0 = ((const int4 *)A.memb)[2 * (long long)p], m1 = ((const int4 *)A.memb)[2 * (long long)p + 1];
                    rm[0] = m0.x, rm[1] = m0.y, rm[2] = m0.z, rm[3] = m0.w;
                    rm[4] = m1.x, rm[5] = m1.y, rm[6] = m1.z, rm[7] = m1.w;
                    if (rm[0] == own) {
                        rp = p;
                        if (A.xcout) rdc = A.dinv_c[p];
                    }
                }
            }
        } else if (t < BX * BY * BZ / 8) {
            rn = (long long)npar[13] * BS + ((fc.x & 1) * 4 + cx) + 8 * ((fc.y & 1) * 4 + cy) + 64 * ((fc.z & 1) * 4 + cz);
            rp = 0;
            if (A.xcout) rdc = A.dinv_c[rn];
        }
    }
    if constexpr (LABEL) {
#pragma unroll
        for (int k = 0; k < NL; ++k)
            if (t + k * NTH < NV) sig[t + k * NTH] = tab[lab[k]];
        __syncthreads();
        T lo[4], hi[4];
        auto plane = [&](int v, T q[4]) {
            const T *p = sig + VL * v + VX * ey + ex;
            q[0] = p[0];
            q[1] = p[1];
            q[2] = p[VX];
            q[3] = p[VX + 1];
        };
        plane(ez0, lo);
#pragma unroll
        for (int z = 0; z < ZS; ++z) {
            plane(ez0 + z + 1, hi);
            // conductivity sums in the order of the setup kernel: (j-1,k-1), (j,k-1), (j-1,k), (j,k)
            const T spx = ((lo[1] + lo[3]) + hi[1]) + hi[3], smx = ((lo[0] + lo[2]) + hi[0]) + hi[2];
            const T spy = ((lo[2] + lo[3]) + hi[2]) + hi[3], smy = ((lo[0] + lo[1]) + hi[0]) + hi[1];
            const T spz = ((hi[0] + hi[1]) + hi[2]) + hi[3], smz = ((lo[0] + lo[1]) + lo[2]) + lo[3];
            W[z][NPX] = spx * A.geo4[0];
            W[z][NMX] = smx * A.geo4[0];
            W[z][NPY] = spy * A.geo4[1];
            W[z][NMY] = smy * A.geo4[1];
            W[z][NPZ] = spz * A.geo4[2];
            W[z][NMZ] = smz * A.geo4[2];
            T d = fmadd(A.geo4[0], smx, W[z][NPX]);
            d = fmadd(A.geo4[1], smy, d);
            d = fmadd(A.geo4[1], spy, d);
            d = ((ez0 + z + rz) & (SEG - 1)) == 0 ? fmadd(A.geo4[2], smz, d) : d + W[z][NMZ];
            D[z] = fmadd(A.geo4[2], spz, d);
#pragma unroll
            for (int k = 0; k < 4; ++k) lo[k] = hi[k];
        }
    }
    // first iterate, b as the cycle takes it, 1/D
    T bz[ZS], rd[ZS], di1[ZS], xp[ZS];
#pragma unroll
    for (int z = 0; z < ZS; ++z) {
        if constexpr (!LABEL) {
            const T *w = W[z];
            D[z] = ((((w[0] + w[1]) + w[2]) + w[3]) + w[4]) + w[5];
        }
        rd[z] = D[z] > T(0) ? brecip(D[z]) : T(0);
        bz[z] = scaled ? D[z] * bv[z] : bv[z];
        di1[z] = rd[z];
        if constexpr (FINE && !UP) {
            xf[z] = scaled ? bv[z] : A.c0 * bv[z];   // the first iterate's factors
            di1[z] = scaled ? rd[z] : xv[z];         // (the stored inverse diagonal, also in the step after it)
            xv[z] = scaled ? A.c0 * bv[z] : xf[z] * di1[z];
        }
        xp[z] = T(0);
    }
    int cur = 0;
    const int at = ex + EX * ey + EL * ez0;
    const int oxm = ex > 0 ? -1 : 0, oxp = ex < EX - 1 ? 1 : 0, oym = ey > 0 ? -EX : 0, oyp = ey < EY - 1 ? EX : 0;
    const int ozm = ez0 > 0 ? -EL : 0, ozp = ez0 + ZS < EZ ? EL : 0;
    auto publish = [&]() {
#pragma unroll
        for (int z = 0; z < ZS; ++z) xs[cur][at + EL * z] = xv[z];
        __syncthreads();
    };
    // neighbours of the thread's node z (at the region's faces stand-ins whose results are not used)
    auto nbrs = [&](int z, T N[6]) {
        const T *p = xs[cur] + at + EL * z;
        N[NMX] = p[oxm];
        N[NPX] = p[oxp];
        N[NMY] = p[oym];
        N[NPY] = p[oyp];
        N[NMZ] = z > 0 ? xv[z - 1] : p[ozm];
        N[NPZ] = z < ZS - 1 ? xv[z + 1] : p[ozp];
    };
    // A x from the differences x - N along the six edges
    auto apply = [&](const T d[6], const T w[6]) {
        T y = w[1] * d[1];
        y = fmadd(w[0], d[0], y);
        y = fmadd(w[2], d[2], y);
        y = fmadd(w[3], d[3], y);
        y = fmadd(w[4], d[4], y);
        return fmadd(w[5], d[5], y);
    };
    // the first step reads a second form of the iterate from xs[1]: the corrected one as seen across an x or y
    // face (up, structured coarser level); the factors of c0 D^-1 b (down, finest level)
    constexpr bool FACES = UP && !CELL, FACTORS = FINE && !UP;
    if constexpr (FACES || FACTORS) {
#pragma unroll
        for (int z = 0; z < ZS; ++z) {
            xs[1][at + EL * z] = xf[z];
            if constexpr (FACTORS) xe[at + EL * z] = di1[z];
        }
    }
    publish();
    constexpr int NST = UP ? H : H - 1;
#pragma unroll
    for (int s = 0; s < NST; ++s) {
        // up: step 0 has no previous update; down: the first step's previous update is the first iterate
        const int k = UP ? s : s + 1;
        const T c1 = UP && s == 0 ? T(0) : A.c1[k], c2 = UP && s == 0 ? A.c0 : A.c2[k];
        T nx[ZS];
#pragma unroll
        for (int z = 0; z < ZS; ++z) {
            T N[6], d[6];
            nbrs(z, N);
            const T *f = xs[1] + at + EL * z;
            if constexpr (FACES) {
                if (s == 0) {
                    if (lx == 0) N[NMX] = f[oxm];
                    if (lx == 7) N[NPX] = f[oxp];
                    if (ly == 0) N[NMY] = f[oym];
                    if (ly == 7) N[NPY] = f[oyp];
                }
            }
#pragma unroll
            for (int e = 0; e < 6; ++e) d[e] = xv[z] - N[e];
            if constexpr (FACTORS) {
                if (s == 0) {
                    const int lz = (ez0 + z + rz) & (SEG - 1);
                    const int om = z > 0 ? -EL : ozm, op = z < ZS - 1 ? EL : ozp;
                    const T *g = xe + at + EL * z;
                    if (lz == 0) d[NMZ] = scaled ? fmadd(-A.c0, f[om], xv[z]) : fmadd(-f[om], g[om], xv[z]);
                    if (lz == SEG - 1) d[NPZ] = scaled ? fmadd(-A.c0, f[op], xv[z]) : fmadd(-f[op], g[op], xv[z]);
                }
            }
            const T dv = (s == 0) ? xv[z] : xv[z] - xp[z];
            const T di = !UP && s == 0 ? di1[z] : rd[z];
            T xo = T(0);
            if (di > T(0)) {
                const T y = apply(d, W[z]);
                const T r = FACTORS && s == 0 && scaled ? fmadd(D[z], bv[z], -y) : bz[z] - y;
                xo = xv[z] + fmadd(c1, dv, (c2 * r) * di);
            }
            nx[z] = xo;
        }
#pragma unroll
        for (int z = 0; z < ZS; ++z) {
            xp[z] = xv[z];
            xv[z] = nx[z];
        }
        if ((FACES || FACTORS) && s == 0) __syncthreads();   // (xs[1] has been read)
        cur ^= 1;
        if (s < NST - 1 || !UP) publish();
    }
    // own nodes
    T *xo = A.xout + vo;
#pragma unroll
    for (int z = 0; z < ZS; ++z)
        if (act && depth_z(ez0 + z) == 0) xo[n[z]] = xv[z];
    if constexpr (UP) {
        if constexpr (FINE && G::PARTS == 1) {
            if (!A.part) return;
            // z.b of the own nodes, summed as the column kernels' waves do: lane = node column, the nodes of a
            // segment in order, then the wave's sum; one partial per segment (4 of them to a group)
            T *xd = xs[cur], *bd = xs[cur] + BS;   // (nobody reads this buffer any more)
#pragma unroll
            for (int z = 0; z < ZS; ++z)
                if (own_xy && depth_z(ez0 + z) == 0) {
                    const int l = lx + 8 * ly + 64 * (ez0 + z + rz);
                    xd[l] = act ? xv[z] : T(0);
                    bd[l] = act ? bz[z] : T(0);
                }
            __syncthreads();
            constexpr int NSEG = 8 / SEG;
            if (t < 64 * NSEG) {
                double d = 0.0;
#pragma unroll
                for (int z = 0; z < SEG; ++z) {
                    const int l = t % 64 + 64 * (z + SEG * (t / 64));
                    d = fmadd((double)xd[l], (double)bd[l], d);
                }
                d = wave_sum(d);
                if (t % 64 == 0) A.part[(long long)blockIdx.y * A.ps + (long long)b * NSEG + t / 64] = d;
            }
        }
        return;
    }
    // residual of the own nodes (0 in columns without unknowns) into LDS
    T *rs = xs[cur ^ 1];
#pragma unroll
    for (int z = 0; z < ZS; ++z) {
        T N[6];
        nbrs(z, N);
        if (own_xy && depth_z(ez0 + z) == 0) {
            T d[6];
            const T x0 = scaled ? xv[z] - bv[z] : xv[z];
#pragma unroll
            for (int e = 0; e < 6; ++e) d[e] = x0 - N[e];
            const T y = apply(d, W[z]);
            const T r = scaled ? -y : bv[z] - y;
            rs[lx + 8 * ly + 64 * (ez0 + z + rz)] = act ? r : T(0);
        }
    }
    __syncthreads();
    if (rp < 0) return;
    T *bc = A.bc + blockIdx.y * A.vsc;
    T sum;
    if constexpr (CELL) {
        T v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = rm[j] >= 0 ? rs[rm[j] & (BS - 1)] : T(0);
        sum = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        rn = rp;
    } else {
        const T *q = rs + 2 * cx + 16 * cy + 128 * cz;
        const T a00 = q[0] + q[64], a10 = q[1] + q[65], a01 = q[8] + q[72], a11 = q[9] + q[73];
        sum = (a00 + a10) + (a01 + a11);
    }
    bc[rn] = sum;
    // (0 at a coarse node without conductance whatever the sum is, as the separate kernel)
    if (A.xcout) A.xcout[blockIdx.y * A.vsc + rn] = rdc > T(0) ? A.c0 * sum * rdc : T(0);
}

// the 27 bricks around each brick (index (dx+1) + 3 (dy+1) + 9 (dz+1); -1: absent)
__global__ __launch_bounds__(256) void k_nbr27(const int *__restrict__ slot_of, const int4 *__restrict__ coord, int nb,
                                               int gx, int gy, int gz, int *__restrict__ out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nb * 27) return;
    const int b = i / 27, k = i % 27;
    const int4 c = coord[b];
    const int x = c.x + k % 3 - 1, y = c.y + (k / 3) % 3 - 1, z = c.z + k / 9 - 1;
    out[i] = x >= 0 && y >= 0 && z >= 0 && x < gx && y < gy && z < gz ? slot_of[x + gx * (y + gy * z)] : -1;
}

hipError_t launch_nbr27(const int *slot_of, const int4 *coord, int nb, const int G[3], int *out, hipStream_t s)
{
    if (nb <= 0) return hipSuccess;
    SPFD_LAUNCH(k_nbr27, dim3((unsigned)((nb * 27 + 255) / 256)), dim3(256), 0, s, slot_of, coord, nb, G[0], G[1],
                G[2], out);
    return hipGetLastError();
}

// Up to this many bricks (times right sides) a brick is dealt to eight workgroups, an eighth (4x4x4 nodes) each: the
// regions are 1.7 to 6.8 times smaller than the brick's own (H = 4: 1,728 nodes for 4,096; H = 2: 512 for 1,728), and
// 384 workgroups still run at once.  Solves, whole bricks -> eighths on the levels named: 31^3 (48 and 8 bricks) 591
// -> 545 us, 64x48x56 (25) 728 -> 685, 96x80x120 (30) 837 -> 759; with 66 bricks (131x97x203) 1,210 -> 1,344 us, with
// 80 (128x96x256) 1,041 -> 1,198.  Quarters (8x4x4) there: 1,210 -> 1,242 in FP64, 1,053 -> 1,010 in FP32.  In FP64
// the H = 4 region keeps a compute unit busy by itself, so there one workgroup per unit: with 36 bricks (56^3) FP64
// takes 589 -> 627 us, FP32 559 -> 533.  Finest levels of 50 to 78 bricks (balls of 32 to 41 voxels) gain 0 to 2 %, so
// the line stays below the 66 bricks of degree 4 that lose 11 %.
template <typename T, int H>
constexpr long long leg_eighths_most() { return sizeof(T) == 8 && H == 4 ? 32 : 48; }

template <typename T, int H, int BX, int BY, int BZ, int OPK, bool FINE, bool CELL>
static hipError_t leg_parts(const BrickLeg<T> &A, int up, int n, hipStream_t s)
{
    using G = BrickGeom<H, BX, BY, BZ>;
    const dim3 grid(xcd_grid(A.nb * G::PARTS) + (!up && A.rr.n > 0 ? 1 : 0), n), block(G::NTH);
    static_assert(G::NTH >= RR_MOST, "one partial a thread");
    if (up)
        SPFD_LAUNCH((k_brick_leg<T, H, BX, BY, BZ, OPK, FINE, true, CELL>), grid, block, 0, s, A);
    else
        SPFD_LAUNCH((k_brick_leg<T, H, BX, BY, BZ, OPK, FINE, false, CELL>), grid, block, 0, s, A);
    return hipGetLastError();
}

template <typename T, int H, int OPK, bool FINE, bool CELL>
static hipError_t leg(const BrickLeg<T> &A, int up, int n, hipStream_t s)
{
    // (the partial sums run over the columns of a whole brick)
    const bool whole = FINE && up && A.part;
    if (!whole && (long long)A.nb * n <= leg_eighths_most<T, H>())
        return leg_parts<T, H, 4, 4, 4, OPK, FINE, CELL>(A, up, n, s);
    return leg_parts<T, H, 8, 8, 8, OPK, FINE, CELL>(A, up, n, s);
}

template <typename T>
hipError_t launch_brick_leg(const BrickLeg<T> &A, int degree, int fine, int up, int nrhs, hipStream_t s)
{
    const bool cell = A.agg != nullptr, label = A.labels != nullptr, half = A.wh != nullptr;
    if (A.nb <= 0 || nrhs <= 0) return hipSuccess;
    if (!A.nbr27 || !A.cmask || !A.coord || !A.sc || !A.b || !A.xout || (!label && !half && !A.w) ||
        (!cell && !A.parent_slot) || (up ? !A.xin || !A.xc : !A.bc || (cell && !A.memb) || (A.xcout && !A.dinv_c)) ||
        (fine && !up && !A.bscale && !A.dinv) || (!fine && !A.xin) || (label && !fine) ||
        (A.rr.n > 0 && (A.rr.n > RR_MOST || !fine || up || !A.rr.sc || !A.rr.part)))
        return hipErrorInvalidValue;
    if (fine) {
        if (degree != 2 || cell || half) return hipErrorInvalidValue;
        return label ? leg<T, 2, BR_LABEL, true, false>(A, up, nrhs, s) : leg<T, 2, BR_STORED, true, false>(A, up, nrhs, s);
    }
    if (half) {
        if constexpr (std::is_same<T, float>::value) {
            if (cell) return hipErrorInvalidValue;
            if (degree == 4) return leg<T, 4, BR_HALF, false, false>(A, up, nrhs, s);
            if (degree == 2) return leg<T, 2, BR_HALF, false, false>(A, up, nrhs, s);
        }
        return hipErrorInvalidValue;
    }
    if (degree == 4)
        return cell ? leg<T, 4, BR_STORED, false, true>(A, up, nrhs, s) : leg<T, 4, BR_STORED, false, false>(A, up, nrhs, s);
    if (degree == 2)
        return cell ? leg<T, 2, BR_STORED, false, true>(A, up, nrhs, s) : leg<T, 2, BR_STORED, false, false>(A, up, nrhs, s);
    return hipErrorInvalidValue;
}
template hipError_t launch_brick_leg<float>(const BrickLeg<float> &, int, int, int, int, hipStream_t);
template hipError_t launch_brick_leg<double>(const BrickLeg<double> &, int, int, int, int, hipStream_t);

}  // namespace spfd
