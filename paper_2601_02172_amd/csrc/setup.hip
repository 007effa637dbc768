// Setup of a problem on the device (Sec. 2, Sec. 3):
//  1. snap: L/h in voxel units, |L| < snap_eps -> 0 (Sec. 3); input validation;
//  2. classify every voxel: an element is cut when it has vertices with L > 0
//     and with L < 0; a voxel is irregular when it holds a cut element or
//     elements of different materials; vertices of cut elements are marked as
//     enriched nodes (eq. X-FEM space);
//  3. ordered compaction (block counts, one-block scan, in-order emit) of the
//     irregular voxels and of the enriched nodes (numbered by node index);
//  4. per irregular voxel: enriched index and level set of its corners and the
//     labels of its elements (decided once, in FP64);
//  5. D0_jj = sum over the cut elements at j of int ||M (grad N_X^j (x) I3)||^2
//     (eq. scaling factors) = 2 sum int |grad N_X^j|^2, gathered per enriched
//     node from its eight voxels through the per-side moments (element.h);
//  6. FFT twiddles exp(-2 pi i t / n) and half-angle tables sin, cos(pi k / n).
#include "kernels.h"
#include "element.h"
#include "fft_lines.h"

#include <cmath>
#include <cstring>
#include <vector>

namespace xfft {

namespace {

constexpr int SCAN_T = 256, SCAN_PER = 16, SCAN_CH = SCAN_T * SCAN_PER;

__device__ __forceinline__ int wrapn(int a, int n) { return a < 0 ? a + n : (a >= n ? a - n : a); }

__device__ __forceinline__ int64_t corner_node(int i, int j, int k, int c, int n0, int n1, int n2) {
    return wrapn(i + (c & 1), n0) + (int64_t)n0 * (wrapn(j + ((c >> 1) & 1), n1) + (int64_t)n1 * wrapn(k + (c >> 2), n2));
}

__global__ void k_snap(int64_t N, const double *L, double inv_h, double eps, const int32_t *phase, int nphase,
                       double *Ls, int *err) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const double v = L[i] * inv_h;
    if (!isfinite(v)) atomicOr(err, 1);
    const int ph = phase[i];
    if (ph < 0 || ph >= nphase) atomicOr(err, 2);
    Ls[i] = fabs(v) < eps ? 0.0 : v;
}

template <int t>
__device__ __forceinline__ void classify_tet(const double (&Lc)[8], const int (&pc)[8], bool &cut, int &lab_uncut,
                                             int &lp, int &ln, bool &ml) {
    double L[4];
    int lab[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) { L[a] = Lc[tet_corner(t, a)]; lab[a] = pc[tet_corner(t, a)]; }
    const bool anyp = L[0] > 0 || L[1] > 0 || L[2] > 0 || L[3] > 0;
    const bool anyn = L[0] < 0 || L[1] < 0 || L[2] < 0 || L[3] < 0;
    cut = anyp && anyn;
    element_labels<double>(L, lab, lab_uncut, lp, ln, ml);
}

__global__ void k_classify(int n0, int n1, int n2, const double *Ls, const int32_t *phase, int p1, uint8_t *vflag,
                           int32_t *vlab, uint8_t *jflag, unsigned long long *counts) {
    const int64_t N = (int64_t)n0 * n1 * n2;
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    const int i = (int)(v % n0), j = (int)((v / n0) % n1), k = (int)(v / ((int64_t)n0 * n1));
    double Lc[8];
    int pc[8];
    int64_t nodes[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        nodes[c] = corner_node(i, j, k, c, n0, n1, n2);
        Lc[c] = Ls[nodes[c]];
        pc[c] = phase[nodes[c]];
    }
    if (p1) {
        // voxel-segmented P1: the level set at the voxel centre (mean of the
        // corners) picks the side; the corner with the largest |L| on that side
        // gives the material (first in corner order on ties)
        double sum = 0.0;
#pragma unroll
        for (int c = 0; c < 8; ++c) sum += Lc[c];
        const bool pos = sum >= 0.0;
        double best = -1.0;
        int lab = pc[0];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const bool on = pos ? Lc[c] >= 0.0 : Lc[c] < 0.0;
            if (on && fabs(Lc[c]) > best) { best = fabs(Lc[c]); lab = pc[c]; }
        }
        vflag[v] = 0;
        vlab[v] = lab;
        return;
    }
    bool cut[6], ml[6];
    int lu[6], lp[6], ln[6];
    classify_tet<0>(Lc, pc, cut[0], lu[0], lp[0], ln[0], ml[0]);
    classify_tet<1>(Lc, pc, cut[1], lu[1], lp[1], ln[1], ml[1]);
    classify_tet<2>(Lc, pc, cut[2], lu[2], lp[2], ln[2], ml[2]);
    classify_tet<3>(Lc, pc, cut[3], lu[3], lp[3], ln[3], ml[3]);
    classify_tet<4>(Lc, pc, cut[4], lu[4], lp[4], ln[4], ml[4]);
    classify_tet<5>(Lc, pc, cut[5], lu[5], lp[5], ln[5], ml[5]);
    bool irregular = false;
    int ncut = 0, nml = 0;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        if (cut[t]) { irregular = true; ++ncut; nml += ml[t] ? 1 : 0; }
        if (lu[t] != lu[0]) irregular = true;
    }
    vflag[v] = irregular ? 1 : 0;
    vlab[v] = lu[0];
    if (ncut) {
        // vertices of cut elements are enriched (plain stores of the same value)
#pragma unroll
        for (int t = 0; t < 6; ++t) {
            if (cut[t]) {
#pragma unroll
                for (int a = 0; a < 4; ++a) jflag[nodes[tet_corner(t, a)]] = 1;
            }
        }
        atomicAdd(&counts[0], (unsigned long long)ncut);
        if (nml) atomicAdd(&counts[1], (unsigned long long)nml);
    }
}

__global__ __launch_bounds__(SCAN_T) void k_scan_count(int64_t n, const uint8_t *flag, int32_t *cnt) {
    __shared__ double red[4];
    const int64_t base = (int64_t)blockIdx.x * SCAN_CH;
    double c[1] = {0.0};
    for (int q = 0; q < SCAN_PER; ++q) {
        const int64_t i = base + (int64_t)threadIdx.x * SCAN_PER + q;
        if (i < n && flag[i]) c[0] += 1.0;
    }
    block_sum<1>(c, red);
    if (threadIdx.x == 0) cnt[blockIdx.x] = (int32_t)c[0];
}

__global__ __launch_bounds__(1024) void k_scan_offsets(int nb, const int32_t *cnt, int32_t *off, int64_t *total) {
    __shared__ int64_t buf[1024];
    __shared__ int64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nb; base += 1024) {
        const int i = base + threadIdx.x;
        const int64_t v = (i < nb) ? cnt[i] : 0;
        buf[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            const int64_t add = (threadIdx.x >= o) ? buf[threadIdx.x - o] : 0;
            __syncthreads();
            buf[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < nb) off[i] = (int32_t)(carry + buf[threadIdx.x] - v);
        __syncthreads();
        if (threadIdx.x == 1023) carry += buf[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

// Emit in order: for voxels, irr[pos] = v and vmat[v] = -(pos + 1) (or the label);
// for nodes, jlist[pos] = node and jmap[node] = pos (or -1).  comp, if given,
// takes the others in order.
__global__ __launch_bounds__(SCAN_T) void k_scan_emit(int64_t n, const uint8_t *flag, const int32_t *off,
                                                       int32_t *list, int32_t *map, const int32_t *lab,
                                                       int32_t *comp) {
    __shared__ int32_t pre[SCAN_T];
    const int64_t base = (int64_t)blockIdx.x * SCAN_CH + (int64_t)threadIdx.x * SCAN_PER;
    int c = 0;
    for (int q = 0; q < SCAN_PER; ++q) {
        const int64_t i = base + q;
        if (i < n && flag[i]) ++c;
    }
    pre[threadIdx.x] = c;
    __syncthreads();
    for (int o = 1; o < SCAN_T; o <<= 1) {
        const int add = (threadIdx.x >= o) ? pre[threadIdx.x - o] : 0;
        __syncthreads();
        pre[threadIdx.x] += add;
        __syncthreads();
    }
    int pos = off[blockIdx.x] + pre[threadIdx.x] - c;
    for (int q = 0; q < SCAN_PER; ++q) {
        const int64_t i = base + q;
        if (i >= n) break;
        if (flag[i]) {
            list[pos] = (int32_t)i;
            map[i] = lab ? -(pos + 1) : pos;
            ++pos;
        } else {
            map[i] = lab ? lab[i] : -1;
            if (comp) comp[i - pos] = (int32_t)i;
        }
    }
}

// labels of element t of an irregular voxel; returns whether it is cut
template <int t>
__device__ __forceinline__ bool irr_labels_tet(const double (&Lc)[8], const int (&pc)[8], int32_t *out,
                                               int64_t stride) {
    bool cut, ml;
    int lu, lp, ln;
    classify_tet<t>(Lc, pc, cut, lu, lp, ln, ml);
    out[(2 * t) * stride] = cut ? lp : lu;
    out[(2 * t + 1) * stride] = cut ? ln : lu;
    return cut;
}

// corner tables and element labels of the irregular voxels and, per element
// 6 q + t, whether it is cut
__global__ void k_irr_tables(int64_t nirr, int n0, int n1, int n2, const int32_t *irr, const double *Ls,
                             const int32_t *phase, const int32_t *jmap, int32_t *irr_j, int32_t *irr_node,
                             int32_t *irr_lab, double *irr_L64, float *irr_L32, uint8_t *cut) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nirr) return;
    const int64_t v = irr[q];
    const int i = (int)(v % n0), j = (int)((v / n0) % n1), k = (int)(v / ((int64_t)n0 * n1));
    double Lc[8];
    int pc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int64_t nd = corner_node(i, j, k, c, n0, n1, n2);
        Lc[c] = Ls[nd];
        pc[c] = phase[nd];
        irr_j[c * nirr + q] = jmap[nd];
        irr_node[c * nirr + q] = (int32_t)nd;
        irr_L64[c * nirr + q] = Lc[c];
        irr_L32[c * nirr + q] = (float)Lc[c];
    }
    int32_t *lab = irr_lab + q;
    uint8_t *ct = cut + 6 * q;
    ct[0] = irr_labels_tet<0>(Lc, pc, lab, nirr);
    ct[1] = irr_labels_tet<1>(Lc, pc, lab, nirr);
    ct[2] = irr_labels_tet<2>(Lc, pc, lab, nirr);
    ct[3] = irr_labels_tet<3>(Lc, pc, lab, nirr);
    ct[4] = irr_labels_tet<4>(Lc, pc, lab, nirr);
    ct[5] = irr_labels_tet<5>(Lc, pc, lab, nirr);
}

// first cut element of every run of IRR_VB irregular voxels (lower bound of 6 q0 in the ascending list)
__global__ void k_blk_cut(int nblk, int64_t ncut, const int32_t *tet_cut, int32_t *blk_cut) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b > nblk) return;
    const int64_t key = (int64_t)6 * IRR_VB * b;
    int64_t lo = 0, hi = ncut;
    while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (tet_cut[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    blk_cut[b] = (int32_t)lo;
}

__global__ void k_uncut_lab(int64_t n, int64_t nirr, const int32_t *tet_uncut, const int32_t *irr_lab, int32_t *lab) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int q = tet_uncut[i] / 6, t = tet_uncut[i] - 6 * q;
    lab[i] = irr_lab[(int64_t)(2 * t) * nirr + q];
}

// Side moments of every cut element (exact integration over its two sides):
// geometry only, so they are computed once per setup in FP64 instead of in every
// operator application.  Stored as 10 values [e][i] (element fastest, so that
// the lanes of a wave read consecutive words): the upper triangle (row by row)
// of the moments of the side with the smaller volume, whose entry 0 carries the
// sign bit when that side is the - side (all moments are >= 0), and the labels
// of the smaller and the larger side.  The operator forms the other side as the
// complement M^tet - Ms, which is accurate in FP32 because it is the larger side.
__global__ void k_cut_moments(int64_t ncut, int64_t nirr, const int32_t *tet_cut, const double *irr_L64,
                              const int32_t *irr_lab, double *M64, float *M32, int32_t *cut_lab) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ncut) return;
    const int q = tet_cut[i] / 6, t = tet_cut[i] - 6 * q;
    double L[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) L[a] = irr_L64[tet_corner(t, a) * nirr + q];
    double Ms[4][4];
    bool pos = small_side_moments<double>(L, 1.0 / 6.0, Ms);
    // keep the side of smaller volume (sum of the moments): its complement is
    // then the larger side and is formed accurately in FP32
    const double Vt = (1.0 / 6.0) * 0.05;
    double vs = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int d = 0; d < 4; ++d) vs += Ms[c][d];
    if (vs > 0.5 * (20.0 * Vt)) {      // the whole tet: sum of V (1 + delta_cd) / 20 = V
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int d = 0; d < 4; ++d) Ms[c][d] = Vt * (c == d ? 2.0 : 1.0) - Ms[c][d];
        pos = !pos;
    }
    double v[10];
    int k = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int d = c; d < 4; ++d, ++k) v[k] = Ms[c][d];
    if (!pos) v[0] = -v[0];                       // sign bit marks the - side (also for +0)
#pragma unroll
    for (int e = 0; e < 10; ++e) {
        M64[e * ncut + i] = v[e];
        M32[e * ncut + i] = (float)v[e];
    }
    const int lp = irr_lab[(int64_t)(2 * t) * nirr + q], ln = irr_lab[(int64_t)(2 * t + 1) * nirr + q];
    cut_lab[i] = pos ? lp : ln;
    cut_lab[ncut + i] = pos ? ln : lp;
}

// int over both sides of |grad N_X^a|^2 for vertex a of cut Kuhn tet t
template <int t>
__device__ __forceinline__ double d0_tet(const double (&Lc)[8], int corner) {
    double L[4];
    int a = -1;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        L[v] = Lc[tet_corner(t, v)];
        if (tet_corner(t, v) == corner) a = v;
    }
    if (a < 0) return 0.0;
    const bool anyp = L[0] > 0 || L[1] > 0 || L[2] > 0 || L[3] > 0;
    const bool anyn = L[0] < 0 || L[1] < 0 || L[2] < 0 || L[3] < 0;
    if (!(anyp && anyn)) return 0.0;
    double Mp[4][4], Mm[4][4];
    side_moments<double>(L, 1.0 / 6.0, Mp, Mm);
    double ga[3];
    kuhn_g<t, double>(a, ga);
    const double g2 = ga[0] * ga[0] + ga[1] * ga[1] + ga[2] * ga[2];
    double tot = 0.0;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const double sg = side == 0 ? 1.0 : -1.0;
        double w[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) w[b] = fabs(L[b]) - sg * L[b];
        double G[3] = {0, 0, 0};
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            double gb[3];
            kuhn_g<t, double>(b, gb);
            G[0] += w[b] * gb[0]; G[1] += w[b] * gb[1]; G[2] += w[b] * gb[2];
        }
        // int |w_c g_a + delta_ac G|^2 weights: g2 w^T M w + 2 (g_a . G) (M w)_a + M_aa |G|^2
        double wMw = 0.0, Mwa = 0.0, Maa = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double rowc = 0.0;
#pragma unroll
            for (int d = 0; d < 4; ++d) rowc += (side == 0 ? Mp[c][d] : Mm[c][d]) * w[d];
            wMw += w[c] * rowc;
            if (c == a) { Mwa = rowc; Maa = side == 0 ? Mp[c][c] : Mm[c][c]; }
        }
        const double gG = ga[0] * G[0] + ga[1] * G[1] + ga[2] * G[2];
        const double G2 = G[0] * G[0] + G[1] * G[1] + G[2] * G[2];
        tot += g2 * wMw + 2.0 * gG * Mwa + Maa * G2;
    }
    return tot;
}

__global__ void k_d0(int64_t nX, int n0, int n1, int n2, const int32_t *jlist, const int32_t *vmat,
                     const double *irr_L64, int64_t nirr, double scale, double *d0, double *d0is64,
                     float *d0is32) {
    const int64_t jn = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (jn >= nX) return;
    const int64_t node = jlist[jn];
    const int i = (int)(node % n0), j = (int)((node / n0) % n1), k = (int)(node / ((int64_t)n0 * n1));
    double acc = 0.0;
    for (int c = 0; c < 8; ++c) {
        const int64_t vox = wrapn(i - (c & 1), n0) + (int64_t)n0 * (wrapn(j - ((c >> 1) & 1), n1) + (int64_t)n1 * wrapn(k - (c >> 2), n2));
        const int m = vmat[vox];
        if (m >= 0) continue;
        const int64_t q = -(int64_t)m - 1;
        double Lc[8];
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) Lc[cc] = irr_L64[cc * nirr + q];
        acc += d0_tet<0>(Lc, c) + d0_tet<1>(Lc, c) + d0_tet<2>(Lc, c) + d0_tet<3>(Lc, c) + d0_tet<4>(Lc, c) +
               d0_tet<5>(Lc, c);
    }
    // eq. scaling factors with the norm of the scalar function's gradient:
    // D0_jj = int |grad N_X^j|^2 (the reading that gives the paper's iteration
    // counts for the Hashin inclusion, Sec. 4.2)
    const double D = acc * scale;
    d0[jn] = D;
    d0is64[jn] = 1.0 / sqrt(D);
    d0is32[jn] = (float)(1.0 / sqrt(D));
}

__global__ void k_enr_src(int64_t nX, int n0, int n1, int n2, const int32_t *jlist, const int32_t *vmat,
                          int32_t *src) {
    const int64_t jn = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (jn >= nX) return;
    const int64_t node = jlist[jn];
    const int i = (int)(node % n0), j = (int)((node / n0) % n1), k = (int)(node / ((int64_t)n0 * n1));
    for (int c = 0; c < 8; ++c) {
        const int64_t vox = wrapn(i - (c & 1), n0) + (int64_t)n0 * (wrapn(j - ((c >> 1) & 1), n1) + (int64_t)n1 * wrapn(k - (c >> 2), n2));
        const int m = vmat[vox];
        src[jn * 8 + c] = (m < 0) ? (int32_t)(8 * (-(int64_t)m - 1) + c) : -1;
    }
}

__device__ __forceinline__ double2 twiddle(int t, int n) {
    double s, c;
    sincospi(-2.0 * (double)t / (double)n, &s, &c);
    return make_double2(c, s);
}

// Twiddles exp(-2 pi i t / n), half-angle tables, and the twiddles in the stage
// order of the compile-time plans: st* for the plan of the line passes, pl* (null:
// none) for the plan of the xy-plane kernels, which is the narrow one in FP64.
__global__ void k_fft_tables(int n, double2 *tw64, float2 *tw32, double *half64, float *half32, double2 *st64,
                             float2 *st32, double2 *pl64, float2 *pl32) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n) return;
    const auto narrow = [](double2 w) { return make_float2((float)w.x, (float)w.y); };
    const double2 w = twiddle(t, n);
    tw64[t] = w;
    tw32[t] = narrow(w);
    double hs, hc;
    sincospi((double)t / (double)n, &hs, &hc);
    half64[2 * t] = hs;
    half64[2 * t + 1] = hc;
    half32[2 * t] = (float)hs;
    half32[2 * t + 1] = (float)hc;
    // entry t of the stage order; 1 where a length has no compile-time plan
    const int i = t < n - 1 ? fft_stage_index(n, t) : -1;
    const double2 ws = i >= 0 ? twiddle(i, n) : make_double2(1.0, 0.0);
    st64[t] = ws;
    st32[t] = narrow(ws);
    if (pl64) {
        const int ip = t < n - 1 ? fft_stage_index(n, t, true) : -1;
        pl64[t] = ip >= 0 ? twiddle(ip, n) : make_double2(1.0, 0.0);
        pl32[t] = narrow(ws);
    }
}

__global__ void k_lame(int n, const double *lame, float *lame32) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < 2 * n) lame32[t] = (float)lame[t];
}

constexpr int XFFT_EDEVICE_INTERNAL = -3;
constexpr int XFFT_ENOMEM_INTERNAL = -2;
constexpr int XFFT_EINVAL_INTERNAL = -1;

int scan_blocks(int64_t n) { return (int)((n + SCAN_CH - 1) / SCAN_CH); }

// Ordered compaction of n flags in two halves, so that the host waits once for all
// list lengths it needs: scan leaves the block offsets in off and the length in
// total, emit writes the lists.
void scan_flags(hipStream_t s, int64_t n, const uint8_t *flag, int32_t *cnt, int32_t *off, int64_t *total) {
    const int nb = scan_blocks(n);
    k_scan_count<<<nb, SCAN_T, 0, s>>>(n, flag, cnt);
    k_scan_offsets<<<1, 1024, 0, s>>>(nb, cnt, off, total);
}
void emit_lists(hipStream_t s, int64_t n, const uint8_t *flag, const int32_t *off, int32_t *list, int32_t *map,
                const int32_t *lab, int32_t *comp) {
    k_scan_emit<<<scan_blocks(n), SCAN_T, 0, s>>>(n, flag, off, list, map, lab, comp);
}

// Device memory of several arrays.  The runtime hands out less than 2 MB from chunks
// that it keeps (1 us, also right after a free), more by a call into the driver each
// (12 us, up to 250 us for memory that is not at hand, as much for the free): arrays
// of 2 MB and more share one allocation, the others are packed into allocations of up
// to 1 MB.  A 24^3 problem (3 MB of tables) built while others live takes 0.52 ms so
// and 0.75 ms with all of it in one allocation; 128^3 is freed in 0.57 instead of 2.6 ms.
class DeviceArrays {
public:
    template <typename P> void add(P *&ptr, int64_t count) {
        rq_.push_back({&ptr, (sizeof(P) * (size_t)count + 255) & ~(size_t)255});
    }
    // false when an allocation fails; what was allocated is in own either way
    bool allocate(std::vector<void *> &own) {
        constexpr size_t LARGE = (size_t)2 << 20, PACK = (size_t)1 << 20;
        std::vector<const Request *> part;
        size_t size = 0;
        const auto flush = [&]() {
            if (part.empty()) return true;
            void *block = nullptr;
            if (hipMalloc(&block, size ? size : 1) != hipSuccess) return false;
            own.push_back(block);
            size_t at = 0;
            for (const Request *q : part) {
                void *v = static_cast<unsigned char *>(block) + at;
                std::memcpy(q->ptr, &v, sizeof(v));
                at += q->bytes;
            }
            part.clear();
            size = 0;
            return true;
        };
        for (const Request &q : rq_) {
            if (q.bytes >= LARGE) continue;
            if (size + q.bytes > PACK && !flush()) return false;
            part.push_back(&q);
            size += q.bytes;
        }
        if (!flush()) return false;
        for (const Request &q : rq_) {
            if (q.bytes < LARGE) continue;
            part.push_back(&q);
            size += q.bytes;
        }
        return flush();
    }

private:
    struct Request {
        void *ptr;          // where the pointer goes
        size_t bytes;
    };
    std::vector<Request> rq_;
};

// what the host reads back from a setup, in the order of the kernels that fill it
struct SetupCounts {
    unsigned long long elements[2];   // cut elements, of these with several labels on a side
    int64_t irregular, enriched, cut; // list lengths
    int err, pad;
};

}  // namespace

// L_dev_raw: device copy of the caller's level set (units of len).
//
// A small grid pays for the calls of its setup and not for the kernels, so the host
// waits for the list lengths once and for the end once, and arrays share
// allocations.  With 62 allocations, 17 frees, 10 waits and 26 launches 16^3 took
// 440 us to build, 64^3 750 us and 128^3 2.5 ms, and 24^3 and 64^3 0.68 and 1.85 ms
// while other problems live; with 9 (16^3), 3, 3 and 21 they take 320 us, 660 us,
// 2.15 ms, 0.52 and 1.54 ms.
int run_setup(xfft_problem *p, const double *L_dev_raw) {
    hipStream_t s = p->stream;
    Geometry &g = p->g;
    const int64_t N = g.N;
    const int tb = 256;
    const auto blocks = [&](int64_t n) { return (unsigned)((n + tb - 1) / tb); };
    SetupCounts *cnt = nullptr;
    uint8_t *jflag = nullptr, *vflag = nullptr, *cut = nullptr;
    int32_t *vlab = nullptr, *jmap = nullptr, *sc[3] = {}, *so[3] = {};
    std::vector<void *> scratch;
    {
        DeviceArrays d;
        const int64_t scan_n[3] = {N, N, 6 * N};
        d.add(cnt, 1);
        for (int q = 0; q < 3; ++q) {
            d.add(sc[q], scan_blocks(scan_n[q]));
            d.add(so[q], scan_blocks(scan_n[q]));
        }
        d.add(jflag, N);
        d.add(vflag, N);
        d.add(vlab, N);
        d.add(jmap, N);
        if (!d.allocate(scratch)) {
            for (void *q : scratch) (void)hipFree(q);
            return XFFT_ENOMEM_INTERNAL;
        }
    }
    int rc = 0;
    SetupCounts h;
    const auto fetch = [&]() {
        if (hipMemcpyAsync(&h, cnt, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            rc = XFFT_EDEVICE_INTERNAL;
    };
    if (hipMemsetAsync(cnt, 0, sizeof(SetupCounts), s) != hipSuccess || hipMemsetAsync(jflag, 0, N, s) != hipSuccess)
        rc = XFFT_EDEVICE_INTERNAL;
    if (!rc) {
        k_snap<<<blocks(N), tb, 0, s>>>(N, L_dev_raw, 1.0 / p->h, p->snap_eps, p->phase, g.nphase, p->Ls, &cnt->err);
        k_classify<<<blocks(N), tb, 0, s>>>(g.n0, g.n1, g.n2, p->Ls, p->phase, p->p1, vflag, vlab, jflag,
                                            cnt->elements);
        scan_flags(s, N, vflag, sc[0], so[0], &cnt->irregular);
        scan_flags(s, N, jflag, sc[1], so[1], &cnt->enriched);
        fetch();
    }
    if (!rc && h.err) rc = XFFT_EINVAL_INTERNAL;
    if (!rc) {
        g.nirr = h.irregular;
        g.nX = h.enriched;
        p->n_cut_elements = (int64_t)h.elements[0];
        p->n_multilabel = (int64_t)h.elements[1];
    }
    const int64_t nirr = g.nirr, nX = g.nX, nc = p->n_cut_elements, nu = 6 * nirr - nc;
    const int nblk = (int)((nirr + IRR_VB - 1) / IRR_VB);
    if (!rc) {
        DeviceArrays d;
        d.add(p->irr, nirr);
        d.add(p->jlist, nX);
        d.add(p->irr_j, 8 * nirr);
        d.add(p->irr_node, 8 * nirr);
        d.add(p->irr_lab, 12 * nirr);
        d.add(p->t64.irr_L, 8 * nirr);
        d.add(p->t32.irr_L, 8 * nirr);
        d.add(p->tet_cut, nc);
        d.add(p->tet_uncut, nu);
        d.add(p->cut_pos, 6 * nirr);
        d.add(p->blk_cut, nblk + 1);
        d.add(p->cut_lab, 2 * nc);
        d.add(p->uncut_lab, nu);
        d.add(p->t64.cut_M, 10 * nc);
        d.add(p->t32.cut_M, 10 * nc);
        d.add(p->d0, nX);
        d.add(p->t64.d0is, nX);
        d.add(p->t32.d0is, nX);
        d.add(p->enr_src, 8 * nX);
        DeviceArrays tmp;
        tmp.add(cut, 6 * nirr);
        if (!d.allocate(p->tables) || !tmp.allocate(scratch)) rc = XFFT_ENOMEM_INTERNAL;
    }
    if (!rc) {
        emit_lists(s, N, vflag, so[0], p->irr, p->vmat, vlab, nullptr);
        emit_lists(s, N, jflag, so[1], p->jlist, jmap, nullptr, nullptr);
    }
    if (!rc && nirr > 0) {
        k_irr_tables<<<blocks(nirr), tb, 0, s>>>(nirr, g.n0, g.n1, g.n2, p->irr, p->Ls, p->phase, jmap, p->irr_j,
                                                 p->irr_node, p->irr_lab, p->t64.irr_L, p->t32.irr_L, cut);
        // lists of the cut and the uncut elements; their lengths are known from the
        // classification, which decides by the same comparisons
        scan_flags(s, 6 * nirr, cut, sc[2], so[2], &cnt->cut);
        emit_lists(s, 6 * nirr, cut, so[2], p->tet_cut, p->cut_pos, nullptr, p->tet_uncut);
        k_blk_cut<<<(unsigned)((nblk + 256) / 256), 256, 0, s>>>(nblk, nc, p->tet_cut, p->blk_cut);
        if (nc)
            k_cut_moments<<<blocks(nc), tb, 0, s>>>(nc, nirr, p->tet_cut, p->t64.irr_L, p->irr_lab, p->t64.cut_M,
                                                    p->t32.cut_M, p->cut_lab);
        if (nu) k_uncut_lab<<<blocks(nu), tb, 0, s>>>(nu, nirr, p->tet_uncut, p->irr_lab, p->uncut_lab);
    }
    if (!rc && nX > 0) {
        k_d0<<<blocks(nX), tb, 0, s>>>(nX, g.n0, g.n1, g.n2, p->jlist, p->vmat, p->t64.irr_L, nirr, p->d0_scale, p->d0,
                                       p->t64.d0is, p->t32.d0is);
        k_enr_src<<<blocks(nX), tb, 0, s>>>(nX, g.n0, g.n1, g.n2, p->jlist, p->vmat, p->enr_src);
    }
    if (!rc) fetch();
    if (!rc && (hipGetLastError() != hipSuccess || (nirr > 0 && h.cut != nc))) rc = XFFT_EDEVICE_INTERNAL;
    for (void *q : scratch) (void)hipFree(q);
    return rc;
}

int compute_tables(xfft_problem *p) {
    hipStream_t s = p->stream;
    const int n[3] = {p->g.n0, p->g.n1, p->g.n2};
    const int np = p->g.nphase;
    const bool plane = fft_variants<double>(p->g) & 1 || fft_variants<float>(p->g) & 1;
    DeviceArrays d;
    for (int a = 0; a < 3; ++a) {
        d.add(p->t64.tw[a], n[a]);
        d.add(p->t32.tw[a], n[a]);
        d.add(p->t64.half[a], 2 * n[a]);
        d.add(p->t32.half[a], 2 * n[a]);
        d.add(p->t64.tws[a], n[a]);
        d.add(p->t32.tws[a], n[a]);
    }
    if (plane) {
        d.add(p->t64.twp, n[0]);
        d.add(p->t32.twp, n[0]);
    }
    d.add(p->t64.lame, 2 * np);
    d.add(p->t32.lame, 2 * np);
    if (!d.allocate(p->tables)) return XFFT_ENOMEM_INTERNAL;
    for (int a = 0; a < 3; ++a) {
        p->plan[a] = make_plan(n[a]);
        const auto c64 = [](cpx<double> *q) { return reinterpret_cast<double2 *>(q); };
        const auto c32 = [](cpx<float> *q) { return reinterpret_cast<float2 *>(q); };
        k_fft_tables<<<(n[a] + 255) / 256, 256, 0, s>>>(n[a], c64(p->t64.tw[a]), c32(p->t32.tw[a]), p->t64.half[a],
                                                        p->t32.half[a], c64(p->t64.tws[a]), c32(p->t32.tws[a]),
                                                        a == 0 ? c64(p->t64.twp) : nullptr,
                                                        a == 0 ? c32(p->t32.twp) : nullptr);
    }
    if (hipMemcpyAsync(p->t64.lame, p->lame_host.data(), sizeof(double) * 2 * np, hipMemcpyHostToDevice, s) !=
        hipSuccess)
        return XFFT_EDEVICE_INTERNAL;
    k_lame<<<(2 * np + 255) / 256, 256, 0, s>>>(np, p->t64.lame, p->t32.lame);
    if (hipStreamSynchronize(s) != hipSuccess) return XFFT_EDEVICE_INTERNAL;
    return 0;
}

}  // namespace xfft
