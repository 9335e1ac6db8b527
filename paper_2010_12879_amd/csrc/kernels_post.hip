// Post-processing on the voxel field: nearest-rank quantiles of |E|.
//
// Step 6 of the paper's technical summary (Sec. II.A) takes the 99th
// percentile of the voxel-averaged field (Sec. III.F) to exclude unphysical
// field enhancements.  The quantile of rank k = ceil(q n) among the n
// conducting voxels (whole body, and per tissue label) is found exactly from
// the 64-bit patterns of |E|: for non-negative doubles the unsigned bit
// pattern orders like the value.  Two forms:
//
//  * launch_quantiles_bins: two scans of the voxels.  The first builds one
//    histogram per group over bins that are monotone in the key; the second
//    copies the keys of each group's bin that holds rank k to that group's
//    stretch of a candidate buffer, and one workgroup per group selects among
//    its candidates.  It needs a buffer; when the candidates do not fit
//    (nearly equal fields) it says so and the caller takes the other form.
//  * launch_quantiles: radix select over the whole key, eight scans with
//    8-bit digits, most significant first, in a small fixed work area (the
//    allocation-free entry point).
//
// Both count with integer atomics only: exact and independent of order.
#include <math.h>

#include "kernels.h"

namespace spfd {

constexpr int SEL_BINS = 256;

// per group: prefix of the selected key, the rank still to find (1-based) and the count
struct SelState {
    unsigned long long prefix;
    long long k;
    long long n;
};

__global__ __launch_bounds__(256) void k_sel_hist(const uint8_t *__restrict__ labels, const double *__restrict__ table,
                                                  const double *__restrict__ sig_vox, long long nvox,
                                                  const double *__restrict__ emag, int ngroups, int shift,
                                                  const SelState *__restrict__ st, unsigned int *hist, int use_lds)
{
    extern __shared__ unsigned int lh[];
    const int nb = ngroups * SEL_BINS;
    if (use_lds) {
        for (int i = threadIdx.x; i < nb; i += blockDim.x) lh[i] = 0;
        __syncthreads();
    }
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (long long)gridDim.x * blockDim.x) {
        const double s = sig_vox ? sig_vox[v] : table[labels[v]];
        if (!(s > 0.0)) continue;
        const unsigned long long key = (unsigned long long)__double_as_longlong(emag[v]);
        const int digit = (int)((key >> shift) & 0xff);
        const int lab = labels[v];
        // group 0: whole body; group 1 + label: that tissue
        const int g2 = 1 + lab < ngroups ? 1 + lab : -1;
        const bool m0 = shift == 56 || (key >> (shift + 8)) == (st[0].prefix >> (shift + 8));
        const bool m2 = g2 >= 0 && (shift == 56 || (key >> (shift + 8)) == (st[g2].prefix >> (shift + 8)));
        if (use_lds) {
            if (m0) atomicAdd(lh + digit, 1u);
            if (m2) atomicAdd(lh + g2 * SEL_BINS + digit, 1u);
        } else {
            if (m0) atomicAdd(hist + digit, 1u);
            if (m2) atomicAdd(hist + g2 * SEL_BINS + digit, 1u);
        }
    }
    if (use_lds) {
        __syncthreads();
        for (int i = threadIdx.x; i < nb; i += blockDim.x)
            if (lh[i]) atomicAdd(hist + i, lh[i]);
    }
}

// pick the digit that holds rank k of each group: one wave per group, four bins per lane and a wave scan (one
// thread per group summing 256 bins in turn, twice: 27 us a pass; this form 3)
__global__ __launch_bounds__(64) void k_sel_pick(int shift, double q, SelState *st, unsigned int *hist)
{
    const int g = blockIdx.x, t = threadIdx.x;
    unsigned int *h = hist + g * SEL_BINS + 4 * t;
    const unsigned c[4] = {h[0], h[1], h[2], h[3]};
    const long long mine = (long long)c[0] + c[1] + c[2] + c[3];
    long long incl = mine;
    for (int d = 1; d < 64; d <<= 1) {
        const long long o = __shfl_up(incl, d, 64);
        if (t >= d) incl += o;
    }
    const long long total = __shfl(incl, 63, 64);
    long long n, k;
    if (shift == 56) {
        n = total;
        k = (long long)ceil(q * (double)n);
        if (k < 1) k = 1;
        if (t == 0) {
            st[g].n = n;
            st[g].k = k;
            st[g].prefix = 0ull;
        }
    } else {
        n = st[g].n;
        k = st[g].k;
    }
    const unsigned long long prefix = shift == 56 ? 0ull : st[g].prefix;
    long long below = incl - mine;
    if (n > 0 && below < k && k <= incl) {   // exactly one lane
        int d = 0;
        while (d < 3 && below + c[d] < k) below += c[d++];
        st[g].k = k - below;
        st[g].prefix = prefix | (unsigned long long)(4 * t + d) << shift;
    }
    h[0] = h[1] = h[2] = h[3] = 0u;
}

__global__ void k_sel_out(int ngroups, const SelState *st, double *out)
{
    for (int g = threadIdx.x; g < ngroups; g += blockDim.x)
        out[g] = st[g].n > 0 ? __longlong_as_double((long long)st[g].prefix) : nan("");
}

size_t sel_work_bytes(int ngroups)
{
    return (size_t)ngroups * (sizeof(SelState) + SEL_BINS * sizeof(unsigned int) + sizeof(double)) + 256;
}

// work: sel_work_bytes(ngroups) bytes of device memory; out: ngroups doubles (device)
hipError_t launch_quantiles(const uint8_t *labels, const double *table, const double *sig_vox, long long nvox,
                            const double *emag, int ngroups, double q, void *work, double *out, hipStream_t s)
{
    SelState *st = (SelState *)work;
    unsigned int *hist = (unsigned int *)(st + ngroups);
    // cleared by a kernel, not a memset node: callers may capture this into a graph
    hipError_t e = launch_fill<int>((int *)hist, (long long)ngroups * SEL_BINS, 0, s);
    if (e != hipSuccess) return e;
    long long blocks = (nvox + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    const size_t lds = (size_t)ngroups * SEL_BINS * sizeof(unsigned int);
    const int use_lds = lds <= 64 * 1024;
    for (int shift = 56; shift >= 0; shift -= 8) {
        SPFD_LAUNCH(k_sel_hist, dim3((unsigned)blocks), dim3(256), use_lds ? lds : 0, s, labels, table, sig_vox,
                           nvox, emag, ngroups, shift, st, hist, use_lds);
        SPFD_LAUNCH(k_sel_pick, dim3(ngroups), dim3(64), 0, s, shift, q, st, hist);
    }
    SPFD_LAUNCH(k_sel_out, dim3(1), dim3(256), 0, s, ngroups, st, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- two scans with a candidate buffer
//
// A scan is bound by reading the labels of all voxels and |E| of the
// conducting ones.  The eight digit passes of the radix form read them eight
// times, each wave waiting for label, conductivity and field one after the
// other: 8 x (150 + 28) us on the 250 x 150 x 900 body.  Here every lane has
// SCAN_U labels and then SCAN_U fields in flight, conductivity flags and bins
// are in LDS, and the voxels are read twice (scans of 53 and 38 us, selection
// 18 us, the rest 22 us): the kernels of a quantile 1,540 -> 131 us.
//
// Bins: 32 octaves of |E| ending one octave above that of a sampled maximum, body
// 128 bins per octave, each label up to 16; keys beyond either end fall into
// the end bins (the map stays monotone, so the choice of the window and the
// sample decide the speed and never the result).
constexpr int SCAN_T = 1024;          // threads of a scan workgroup (its histograms take most of a CU's LDS)
constexpr int SCAN_U = 8;             // voxels per thread and iteration
constexpr int OCT = 32;               // octaves of the bin window
constexpr int BODY_SH = 45;           // key bits below a body bin: 128 bins per octave
constexpr int BODY_BINS = OCT << (52 - BODY_SH);
constexpr int LAB_BINS = 512;         // most bins of a label: 16 per octave
constexpr int LAB_FULL = 64;          // labels that get LAB_BINS bins each (LDS); up to twice as many get half, ...
constexpr int HIST_WORDS = BODY_BINS + (LAB_FULL + 1) * LAB_BINS;
constexpr int SEL_GROUPS = 1 + MAX_LABELS;
constexpr int LIST_CAP = 8192;        // candidates a workgroup collects in LDS before its one append
constexpr int PICK_T = 256;
constexpr int FIN_T = 1024;           // threads of a final selection
constexpr int FIN_BINS = 2048;        // its 11-bit digits
constexpr int FIN_LIST = 4096;        // keys it keeps in LDS

constexpr int SAMPLE_WG = 1 + (HIST_WORDS + SCAN_T - 1) / SCAN_T;   // workgroups of k_bin_start

struct BinState {
    unsigned long long top[SAMPLE_WG];// largest sampled keys (finite), one per workgroup of k_bin_start
    unsigned present[MAX_LABELS / 32];// labels that occur (only read when the labels exceed LAB_FULL)
    int bin[SEL_GROUPS];              // the bin that holds rank k of a group (-1: no voxels)
    long long k[SEL_GROUPS];          // the rank to find inside that bin
    long long n[SEL_GROUPS];          // voxels of the group
    unsigned count[SEL_GROUPS];       // keys in that bin
    unsigned cursor[SEL_GROUPS];      // keys appended so far
};

// where the histograms of the labels lie: compact index per label, bins per label
struct LabelMap {
    int n, sh, bins;
};

__device__ __forceinline__ int key_bin(unsigned long long key, unsigned long long base, int sh, int bins)
{
    const unsigned long long d = key >> sh, b = base >> sh;
    if (d <= b) return 0;
    const unsigned long long r = d - b;
    return r < (unsigned long long)bins ? (int)r : bins - 1;
}

// map[l] = compact histogram index of label l (labels that occur, in order); all threads call this
__device__ __forceinline__ LabelMap label_map(const BinState *st, int nlab, unsigned char *map, int *nsh)
{
    if (nlab <= LAB_FULL + 1) {
        for (int l = threadIdx.x; l < MAX_LABELS; l += blockDim.x) map[l] = l < nlab ? (unsigned char)l : 0;
        __syncthreads();
        return LabelMap{nlab, 52 - 4, LAB_BINS};
    }
    for (int l = threadIdx.x; l < MAX_LABELS; l += blockDim.x) {
        int c = 0;
        for (int w = 0; w < l >> 5; ++w) c += __popc(st->present[w]);
        const unsigned low = st->present[l >> 5] & ((1u << (l & 31)) - 1u);
        c += __popc(low);
        map[l] = (unsigned char)c;
        if (l == MAX_LABELS - 1) *nsh = c + (int)(st->present[l >> 5] >> 31);
    }
    __syncthreads();
    LabelMap m{*nsh, 52 - 4, LAB_BINS};
    while (m.n * m.bins > (LAB_FULL + 1) * LAB_BINS) {
        m.bins >>= 1;
        ++m.sh;
    }
    return m;
}

// Clears the histograms, the presence mask and the cursors, and samples the largest finite |E|: every thread
// reads SAMPLES voxels, each somewhere in a stretch of its own (a plain stride can stay in one column of the
// grid).  One workgroup with 32,768 samples took 70 us, each being a line of its own from memory.
constexpr int SAMPLES = 4;

__global__ __launch_bounds__(SCAN_T) void k_bin_start(const double *__restrict__ emag, long long nvox, BinState *st,
                                                      unsigned *__restrict__ hist)
{
    const int t = threadIdx.x;
    if (blockIdx.x > 0) {
        const int i = ((int)blockIdx.x - 1) * SCAN_T + t;
        if (i < HIST_WORDS) hist[i] = 0u;
    } else {
        if (t < MAX_LABELS / 32) st->present[t] = 0u;
        for (int g = t; g < SEL_GROUPS; g += SCAN_T) st->cursor[g] = 0u;
    }
    __shared__ unsigned long long sm[SCAN_T / 64];
    const unsigned long long INF = 0x7ff0000000000000ull;
    const unsigned long long n = (unsigned long long)nvox, ns = (unsigned long long)SAMPLE_WG * SCAN_T * SAMPLES;
    const unsigned long long step = (n + ns - 1) / ns;
    unsigned long long v[SAMPLES], m = 0ull;
#pragma unroll
    for (int j = 0; j < SAMPLES; ++j) {
        const unsigned long long k = ((unsigned long long)j * SAMPLE_WG + blockIdx.x) * SCAN_T + t;
        const unsigned long long i = k * step + (k * 2654435761ull >> 8) % step;
        v[j] = (unsigned long long)__double_as_longlong(emag[i < n ? i : i % n]);
    }
#pragma unroll
    for (int j = 0; j < SAMPLES; ++j) m = v[j] < INF && v[j] > m ? v[j] : m;
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_down(m, off, 64);
        m = o > m ? o : m;
    }
    if ((t & 63) == 0) sm[t >> 6] = m;
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < SCAN_T / 64; ++w) m = sm[w] > m ? sm[w] : m;
        st->top[blockIdx.x] = m;
    }
}

// lowest key of the window (all lanes of a wave call this)
__device__ __forceinline__ unsigned long long bin_base(const BinState *st)
{
    static_assert(SAMPLE_WG <= 64, "one wave reads them");
    const int lane = threadIdx.x & 63;
    unsigned long long m = lane < SAMPLE_WG ? st->top[lane] : 0ull;
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(m, off, 64);
        m = o > m ? o : m;
    }
    const unsigned long long top = (m >> 52) + 2ull;
    return (top > OCT ? top - OCT : 0ull) << 52;
}

// which labels occur (only for tables longer than LAB_FULL + 1)
__global__ __launch_bounds__(256) void k_bin_labels(const uint8_t *__restrict__ labels, long long nvox, BinState *st)
{
    __shared__ unsigned p[MAX_LABELS / 32];
    if (threadIdx.x < MAX_LABELS / 32) p[threadIdx.x] = 0u;
    __syncthreads();
    int last = -1;
    for (long long v = (long long)blockIdx.x * blockDim.x + threadIdx.x; v < nvox; v += (long long)gridDim.x * blockDim.x) {
        const int l = labels[v];
        if (l != last) atomicOr(p + (l >> 5), 1u << (l & 31));
        last = l;
    }
    __syncthreads();
    if (threadIdx.x < MAX_LABELS / 32 && p[threadIdx.x]) atomicOr(&st->present[threadIdx.x], p[threadIdx.x]);
}

// one iteration's voxels of a thread: labels, conducting flags and keys (all loads of a kind in flight together)
struct ScanVox {
    int lab[SCAN_U];
    bool on[SCAN_U];
    unsigned long long key[SCAN_U];

    __device__ __forceinline__ void load(const uint8_t *__restrict__ labels, const double *__restrict__ sig_vox,
                                         const unsigned char *cond, const double *__restrict__ emag, long long nvox,
                                         long long v0)
    {
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) {
            const long long v = v0 + (long long)u * SCAN_T;
            on[u] = v < nvox;
            lab[u] = labels[on[u] ? v : nvox - 1];
        }
        if (sig_vox) {
            double sv[SCAN_U];
#pragma unroll
            for (int u = 0; u < SCAN_U; ++u) {
                const long long v = v0 + (long long)u * SCAN_T;
                sv[u] = sig_vox[v < nvox ? v : nvox - 1];
            }
#pragma unroll
            for (int u = 0; u < SCAN_U; ++u) on[u] = on[u] && sv[u] > 0.0;
        } else {
#pragma unroll
            for (int u = 0; u < SCAN_U; ++u) on[u] = on[u] && cond[lab[u]];
        }
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u) {
            key[u] = 0ull;
            if (on[u]) key[u] = (unsigned long long)__double_as_longlong(emag[v0 + (long long)u * SCAN_T]);
        }
    }
};

__global__ __launch_bounds__(SCAN_T) void k_bin_hist(const uint8_t *__restrict__ labels,
                                                     const double *__restrict__ table,
                                                     const double *__restrict__ sig_vox, long long nvox,
                                                     const double *__restrict__ emag, int nlab,
                                                     const BinState *__restrict__ st, unsigned *hist)
{
    __shared__ unsigned lh[HIST_WORDS];
    __shared__ unsigned char map[MAX_LABELS], cond[MAX_LABELS];
    __shared__ int nsh;
    const int t = threadIdx.x;
    const LabelMap m = label_map(st, nlab, map, &nsh);
    const int words = BODY_BINS + m.n * m.bins;
    for (int i = t; i < words; i += SCAN_T) lh[i] = 0u;
    for (int l = t; l < MAX_LABELS; l += SCAN_T) cond[l] = !sig_vox && l < nlab && table[l] > 0.0;
    const unsigned long long base = bin_base(st);
    __syncthreads();
    const long long stride = (long long)SCAN_T * SCAN_U;
    for (long long c = (long long)blockIdx.x * stride; c < nvox; c += (long long)gridDim.x * stride) {
        ScanVox x;
        x.load(labels, sig_vox, cond, emag, nvox, c + t);
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u)
            if (x.on[u]) {
                atomicAdd(lh + key_bin(x.key[u], base, BODY_SH, BODY_BINS), 1u);
                atomicAdd(lh + BODY_BINS + (int)map[x.lab[u]] * m.bins + key_bin(x.key[u], base, m.sh, m.bins), 1u);
            }
    }
    __syncthreads();
    for (int i = t; i < words; i += SCAN_T)
        if (lh[i]) atomicAdd(hist + i, lh[i]);
}

// one workgroup per group: the bin that holds rank ceil(q n), the rank inside it
__global__ __launch_bounds__(PICK_T) void k_bin_pick(int nlab, double q, BinState *st, const unsigned *__restrict__ hist)
{
    __shared__ unsigned char map[MAX_LABELS];
    __shared__ int nsh;
    __shared__ unsigned part[PICK_T];
    const int g = blockIdx.x, t = threadIdx.x;
    const LabelMap m = label_map(st, nlab, map, &nsh);
    const bool occurs = g == 0 || nlab <= LAB_FULL + 1 || ((st->present[(g - 1) >> 5] >> ((g - 1) & 31)) & 1u);
    const int bins = g == 0 ? BODY_BINS : m.bins;
    const unsigned *h = hist + (g == 0 ? 0 : BODY_BINS + (int)map[g - 1] * m.bins);
    const int per = (bins + PICK_T - 1) / PICK_T;
    unsigned mine = 0u;
    if (occurs)
        for (int j = 0; j < per; ++j) {
            const int b = t * per + j;
            if (b < bins) mine += h[b];
        }
    part[t] = mine;
    __syncthreads();
    for (int off = 1; off < PICK_T; off <<= 1) {   // inclusive sums
        const unsigned v = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    const long long n = part[PICK_T - 1];
    long long k = (long long)ceil(q * (double)n);
    if (k < 1) k = 1;
    if (t == 0) {
        st->n[g] = n;
        if (n == 0) {
            st->bin[g] = -1;
            st->count[g] = 0u;
            st->k[g] = 0;
        }
    }
    long long below = (long long)part[t] - mine;
    if (n > 0 && below < k && k <= below + mine)   // exactly one thread
        for (int j = 0; j < per; ++j) {
            const int b = t * per + j;
            const unsigned c = b < bins ? h[b] : 0u;
            if (k <= below + c) {
                st->bin[g] = b;
                st->k[g] = k - below;
                st->count[g] = c;
                break;
            }
            below += c;
        }
}

// first candidate of each group (the groups in order); all threads of the workgroup call this; returns the total
__device__ __forceinline__ unsigned long long group_offsets(const BinState *st, int ngroups, unsigned *off,
                                                            unsigned long long *total)
{
    if (threadIdx.x < 64) {   // one wave: running sums over blocks of 64 groups
        unsigned long long run = 0ull;
        for (int g0 = 0; g0 < ngroups; g0 += 64) {
            const int g = g0 + threadIdx.x;
            const unsigned long long c = g < ngroups ? st->count[g] : 0u;
            unsigned long long inc = c;
            for (int d = 1; d < 64; d <<= 1) {
                const unsigned long long o = __shfl_up(inc, d, 64);
                if ((int)threadIdx.x >= d) inc += o;
            }
            if (g < ngroups) off[g] = (unsigned)(run + inc - c);
            run += __shfl(inc, 63, 64);
        }
        if (threadIdx.x == 0) *total = run;
    }
    __syncthreads();
    return *total;
}

__global__ __launch_bounds__(SCAN_T) void k_bin_gather(const uint8_t *__restrict__ labels,
                                                       const double *__restrict__ table,
                                                       const double *__restrict__ sig_vox, long long nvox,
                                                       const double *__restrict__ emag, int nlab, BinState *st,
                                                       unsigned long long *__restrict__ cand, unsigned long long cap)
{
    __shared__ unsigned long long lkey[LIST_CAP];
    __shared__ unsigned short lgrp[LIST_CAP], lpos[LIST_CAP];
    __shared__ unsigned off[SEL_GROUPS], cnt[SEL_GROUPS], at[SEL_GROUPS];
    __shared__ int sbin[SEL_GROUPS];
    __shared__ unsigned char map[MAX_LABELS], cond[MAX_LABELS];
    __shared__ int nsh;
    __shared__ unsigned fill;
    __shared__ unsigned long long total;
    const int t = threadIdx.x, ngroups = 1 + nlab;
    const LabelMap m = label_map(st, nlab, map, &nsh);
    if (group_offsets(st, ngroups, off, &total) > cap) return;   // does not fit: the caller takes the radix form
    for (int g = t; g < ngroups; g += SCAN_T) {
        cnt[g] = 0u;
        sbin[g] = st->bin[g];
    }
    for (int l = t; l < MAX_LABELS; l += SCAN_T) cond[l] = !sig_vox && l < nlab && table[l] > 0.0;
    if (t == 0) fill = 0u;
    const unsigned long long base = bin_base(st);
    __syncthreads();
    // a key of group g: into the LDS list, or straight to its stretch when the list is full
    auto put = [&](int g, unsigned long long key) {
        const unsigned p = atomicAdd(&fill, 1u);
        if (p < LIST_CAP) {
            lkey[p] = key;
            lgrp[p] = (unsigned short)g;
            lpos[p] = (unsigned short)atomicAdd(cnt + g, 1u);
        } else {
            cand[off[g] + atomicAdd(&st->cursor[g], 1u)] = key;
        }
    };
    const long long stride = (long long)SCAN_T * SCAN_U;
    for (long long c = (long long)blockIdx.x * stride; c < nvox; c += (long long)gridDim.x * stride) {
        ScanVox x;
        x.load(labels, sig_vox, cond, emag, nvox, c + t);
#pragma unroll
        for (int u = 0; u < SCAN_U; ++u)
            if (x.on[u]) {
                if (key_bin(x.key[u], base, BODY_SH, BODY_BINS) == sbin[0]) put(0, x.key[u]);
                const int g = 1 + x.lab[u];
                if (g < ngroups && key_bin(x.key[u], base, m.sh, m.bins) == sbin[g]) put(g, x.key[u]);
            }
    }
    __syncthreads();
    for (int g = t; g < ngroups; g += SCAN_T) at[g] = cnt[g] ? off[g] + atomicAdd(&st->cursor[g], cnt[g]) : 0u;
    __syncthreads();
    const unsigned have = fill < LIST_CAP ? fill : LIST_CAP;
    for (unsigned i = t; i < have; i += SCAN_T) cand[at[lgrp[i]] + lpos[i]] = lkey[i];
}

// One workgroup per group selects rank k among its candidates: repeatedly an
// 11-bit histogram below the highest bit in which the remaining keys differ.
// Few keys (the usual case) are held in LDS from the start; more are read
// from the buffer until those that are left fit.
__global__ __launch_bounds__(FIN_T) void k_bin_select(int nlab, const BinState *__restrict__ st,
                                                      const unsigned long long *__restrict__ cand,
                                                      unsigned long long cap, double *__restrict__ out)
{
    __shared__ unsigned h[FIN_BINS];
    __shared__ unsigned part[FIN_T];
    __shared__ unsigned long long list[2][FIN_LIST];
    __shared__ unsigned long long wand[FIN_T / 64], wor[FIN_T / 64];
    __shared__ unsigned off[SEL_GROUPS];
    __shared__ unsigned long long total;
    __shared__ unsigned fill, bin_sh;
    __shared__ long long k_sh;
    const int g = blockIdx.x, t = threadIdx.x;
    const bool fits = group_offsets(st, 1 + nlab, off, &total) <= cap;
    if (g == 0 && t == 0) out[1 + nlab] = fits ? 0.0 : 1.0;
    if (!fits) return;
    if (st->n[g] == 0) {
        if (t == 0) out[g] = nan("");
        return;
    }
    const unsigned long long *src = cand + off[g];   // the keys still in question: those of src with the prefix
    unsigned n = st->count[g];
    long long k = st->k[g];
    unsigned long long prefix = 0ull, mask = 0ull;
    int cur = 0;
    if (n <= FIN_LIST) {
        for (unsigned i = t; i < n; i += FIN_T) list[0][i] = src[i];
        src = list[0];
        __syncthreads();
    }
    while (true) {
        unsigned long long a = ~0ull, o = 0ull;
#pragma unroll 8
        for (unsigned i = t; i < n; i += FIN_T) {
            const unsigned long long v = src[i];
            if ((v & mask) == prefix) {
                a &= v;
                o |= v;
            }
        }
        for (int d = 32; d > 0; d >>= 1) {
            a &= __shfl_xor(a, d, 64);
            o |= __shfl_xor(o, d, 64);
        }
        if ((t & 63) == 0) {
            wand[t >> 6] = a;
            wor[t >> 6] = o;
        }
        for (int i = t; i < FIN_BINS; i += FIN_T) h[i] = 0u;
        if (t == 0) fill = 0u;
        __syncthreads();
        for (int w = 0; w < FIN_T / 64; ++w) {
            a &= wand[w];
            o |= wor[w];
        }
        const unsigned long long diff = a ^ o;
        if (diff == 0ull) {   // all that are left are equal
            if (t == 0) out[g] = __longlong_as_double((long long)a);
            return;
        }
        const int top = 63 - __clzll((long long)diff);
        const int sh = top >= 10 ? top - 10 : 0;
#pragma unroll 8
        for (unsigned i = t; i < n; i += FIN_T) {
            const unsigned long long v = src[i];
            if ((v & mask) == prefix) atomicAdd(h + (int)((v >> sh) & (FIN_BINS - 1)), 1u);
        }
        __syncthreads();
        constexpr int PER = FIN_BINS / FIN_T;
        unsigned mine = 0u;
        for (int j = 0; j < PER; ++j) mine += h[t * PER + j];
        part[t] = mine;
        __syncthreads();
        for (int d = 1; d < FIN_T; d <<= 1) {
            const unsigned v = t >= d ? part[t - d] : 0u;
            __syncthreads();
            part[t] += v;
            __syncthreads();
        }
        long long below = (long long)part[t] - mine;
        if (below < k && k <= below + mine)
            for (int j = 0; j < PER; ++j) {
                const unsigned c = h[t * PER + j];
                if (k <= below + c) {
                    bin_sh = (unsigned)(t * PER + j);
                    k_sh = k - below;
                    break;
                }
                below += c;
            }
        __syncthreads();
        const unsigned b = bin_sh;
        const unsigned left = h[b];
        k = k_sh;
        // bits above the digit agree in all keys that were in question (their common prefix is a's)
        const unsigned long long above = top >= 63 ? 0ull : ~0ull << (top + 1);
        const unsigned long long digit = (unsigned long long)(FIN_BINS - 1) << sh;
        const unsigned long long old_mask = mask, old_prefix = prefix;
        prefix = (a & above) | ((unsigned long long)b << sh);
        mask = above | digit;
        if (top < 10) prefix = (a & above & ~digit) | (unsigned long long)b;
        if (left <= FIN_LIST) {
            for (unsigned i = t; i < n; i += FIN_T) {
                const unsigned long long v = src[i];
                if ((v & old_mask) == old_prefix && ((v >> sh) & (FIN_BINS - 1)) == b)
                    list[cur ^ 1][atomicAdd(&fill, 1u)] = v;
            }
            __syncthreads();
            cur ^= 1;
            src = list[cur];
            n = left;
        }
        __syncthreads();
    }
}

size_t bin_state_bytes() { return (sizeof(BinState) + 255) / 256 * 256 + HIST_WORDS * sizeof(unsigned); }

// Candidates kept: a sixteenth of the voxels covers about 5 % of a conductor that fills the box; the
// smallest buffer covers grids of up to 64 K voxels whole (every voxel a candidate of the body and its label).
long long bin_candidates(long long nvox)
{
    const long long n = nvox / 16;
    return n < (1 << 17) ? 1 << 17 : (n > (1 << 24) ? 1 << 24 : n);
}

// work: bin_state_bytes(), cand: bin_candidates(nvox) keys; out: nlab + 2 doubles, the last one nonzero when
// the candidates did not fit (then nothing else is valid)
hipError_t launch_quantiles_bins(const uint8_t *labels, const double *table, const double *sig_vox, long long nvox,
                                 const double *emag, int nlab, double q, void *work, unsigned long long *cand,
                                 double *out, hipStream_t s)
{
    BinState *st = (BinState *)work;
    unsigned *hist = (unsigned *)((uint8_t *)work + (sizeof(BinState) + 255) / 256 * 256);
    const unsigned long long cap = (unsigned long long)bin_candidates(nvox);
    const long long chunk = (long long)SCAN_T * SCAN_U;
    long long blocks = (nvox + chunk - 1) / chunk;
    if (blocks > 256) blocks = 256;   // one workgroup per CU: its histograms fill the LDS
    SPFD_LAUNCH(k_bin_start, dim3(SAMPLE_WG), dim3(SCAN_T), 0, s, emag, nvox, st, hist);
    if (nlab > LAB_FULL + 1) {
        long long lb = (nvox + 4095) / 4096;
        if (lb > 2048) lb = 2048;
        SPFD_LAUNCH(k_bin_labels, dim3((unsigned)lb), dim3(256), 0, s, labels, nvox, st);
    }
    SPFD_LAUNCH(k_bin_hist, dim3((unsigned)blocks), dim3(SCAN_T), 0, s, labels, table, sig_vox, nvox, emag, nlab, st,
                hist);
    SPFD_LAUNCH(k_bin_pick, dim3(1 + nlab), dim3(PICK_T), 0, s, nlab, q, st, hist);
    SPFD_LAUNCH(k_bin_gather, dim3((unsigned)blocks), dim3(SCAN_T), 0, s, labels, table, sig_vox, nvox, emag, nlab, st,
                cand, cap);
    SPFD_LAUNCH(k_bin_select, dim3(1 + nlab), dim3(FIN_T), 0, s, nlab, st, cand, cap, out);
    return hipGetLastError();
}

}  // namespace spfd
