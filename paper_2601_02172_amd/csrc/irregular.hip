// Irregular voxels of the matrix-free operator (eqs. linearSystem_element,
// resVector): voxels with a cut element or elements of different materials.
//
// k_irregular evaluates the elements one per lane.  All Kuhn tetrahedra are the
// same element up to the order of the axes, and the materials are isotropic, so
// a lane reads its element's vectors with the components permuted to the local
// axes (p0, p1, p2) and every lane runs the same instructions.  A workgroup
// takes the elements of VB consecutive voxels: it stages the corner values in
// LDS, works through its list of cut elements and its list of uncut ones, leaves
// the vertex forces of every element in LDS and sums them per corner in element
// order (no atomics).
//
// Bound by: vector issue (about 890 instructions per wave with an active load, 85
// per voxel and load: at full rate 59 of 102 us at 128^3 FP32 with six loads) and
// latency, the gathers of the corner values (22 cache-line accesses per wave load)
// above all: its waves wait for 61 % of their time.  One thread per voxel looping over its six elements, the form before,
// held the 96 corner values and sums in registers (211 VGPRs in FP32, 256 + 158
// AGPRs in FP64: two and one waves per SIMD), ran the cut path for uncut elements
// too and chained six elements' loads.  Per launch, before -> now: 128^3 FP32
// with six loads (5.2 active) 123 -> 106 us, one FP64 load 73 -> 56; 64^3 one
// FP64 load 29.8 -> 16.7, six 60.5 -> 54.8; 16^3 six FP32 loads 21.2 -> 9.5 us;
// 256^3 FP32 790 -> 620.
#include "kernels.h"
#include "op_common.h"

#include <algorithm>

namespace xfft {

namespace {

constexpr int VB = IRR_VB;          // voxels per workgroup: 192 cut and 60 uncut elements on average, four waves
constexpr int BT = 256;
static_assert(6 * VB <= BT, "every element of a workgroup's voxels has a lane");

// local axis s of Kuhn tet t (lexicographic permutations), at run time
__device__ __forceinline__ void tet_axes(int t, int &p0, int &p1, int &p2) {
    p0 = t >> 1;
    const int lo = p0 == 0 ? 1 : 0, hi = p0 == 2 ? 1 : 2;
    p1 = (t & 1) ? hi : lo;
    p2 = (t & 1) ? lo : hi;
}

// Strain of a local displacement gradient H (columns u1 - u0, u2 - u1, u3 - u2):
// normal components and engineering shears 2 e_12, 2 e_02, 2 e_01.
template <typename T> struct Eng { T n[3], g[3]; };

template <typename T>
__device__ __forceinline__ Eng<T> eng_strain(const T (&v)[4][3]) {
    Eng<T> e;
    T h[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int i = 0; i < 3; ++i) h[c][i] = v[c + 1][i] - v[c][i];
    e.n[0] = h[0][0]; e.n[1] = h[1][1]; e.n[2] = h[2][2];
    e.g[0] = h[2][1] + h[1][2]; e.g[1] = h[2][0] + h[0][2]; e.g[2] = h[1][0] + h[0][1];
    return e;
}

// stress lam tr(e) I + 2 mu e, returned in the same slots (shears are stresses)
template <typename T>
__device__ __forceinline__ Eng<T> eng_hooke(const Eng<T> &e, T lam, T mu) {
    const T tr = lam * (e.n[0] + e.n[1] + e.n[2]), mu2 = mu + mu;
    return {{tr + mu2 * e.n[0], tr + mu2 * e.n[1], tr + mu2 * e.n[2]}, {mu * e.g[0], mu * e.g[1], mu * e.g[2]}};
}

template <typename T>
__device__ __forceinline__ void eng_vec(const Eng<T> &s, const T (&G)[3], T (&r)[3]) {
    r[0] = s.n[0] * G[0] + s.g[2] * G[1] + s.g[1] * G[2];
    r[1] = s.g[2] * G[0] + s.n[1] * G[1] + s.g[0] * G[2];
    r[2] = s.g[1] * G[0] + s.g[0] * G[1] + s.n[2] * G[2];
}

// a x + b y + sym(p (x) G)
template <typename T>
__device__ __forceinline__ Eng<T> eng_comb(T a, const Eng<T> &x, T b, const Eng<T> &y, const T (&p)[3], const T (&G)[3]) {
    Eng<T> r;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int j = (i + 1) % 3, k = (i + 2) % 3;
        r.n[i] = a * x.n[i] + b * y.n[i] + p[i] * G[i];
        r.g[i] = a * x.g[i] + b * y.g[i] + p[j] * G[k] + p[k] * G[j];
    }
    return r;
}

template <typename T>
__device__ __forceinline__ void eng_add(Eng<T> &y, const Eng<T> &x) {
#pragma unroll
    for (int i = 0; i < 3; ++i) { y.n[i] += x.n[i]; y.g[i] += x.g[i]; }
}

// vertex forces S g_a, g = -e0, e0 - e1, e1 - e2, e2, added to f
template <typename T>
__device__ __forceinline__ void eng_scatter(const Eng<T> &S, T (&f)[4][3]) {
    const T c[3][3] = {{S.n[0], S.g[2], S.g[1]}, {S.g[2], S.n[1], S.g[0]}, {S.g[1], S.g[0], S.n[2]}};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        f[0][i] -= c[0][i];
        f[1][i] += c[0][i] - c[1][i];
        f[2][i] += c[1][i] - c[2][i];
        f[3][i] += c[2][i];
    }
}

// One cut element in local axes: level set L, FE and enriched (scaled by
// D0^-1/2) vertex values, moments ms of the side of smaller volume (upper
// triangle; pos: it is the + side) and the moduli of both sides.  The side's
// integrals need its nodal stresses sigma_c = C (e_F + w_c e_q + sym(q_c (x) G))
// only through
//   sum_c M_ac sigma_c = C (m_a e_F + (M w)_a e_q + sym(y_a (x) G)),
//   m_a = sum_c M_ac,  y_a = sum_c M_ac q_c,
// of which the FE forces take the sum over a, the forces of the enriched
// gradient the sum weighted by w, and the rest is its product with G,
//   m_a C e_F G + (M w)_a C e_q G + (lambda + mu) (y_a . G) G + mu |G|^2 y_a.
// The larger side is the complement M^tet - M, M^tet_cd = V (1 + delta_cd) / 20,
// accurate because it is the larger one; its y follow from the sum of q.
// eF: FE strain including the macro strain.  S: stress integral; fe: enriched
// vertex forces (not yet scaled).
template <typename T>
__device__ __forceinline__ void cut_element(const T (&L)[4], const Eng<T> &eF, const T (&q)[4][3], const T (&ms)[10],
                                            bool pos, T lam_s, T mu_s, T lam_l, T mu_l, Eng<T> &S, T (&fe)[4][3]) {
    const T V = (T)(1.0 / 6.0), V20 = V * (T)0.05;
    const Eng<T> eq = eng_strain<T>(q);
    T M[4][4];
    {
        int k = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int d = c; d < 4; ++d, ++k) M[c][d] = M[d][c] = ms[k];
    }
    T m[4], y[4][3];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        m[a] = M[a][0] + M[a][1] + M[a][2] + M[a][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
            y[a][i] = M[a][0] * q[0][i] + M[a][1] * q[1][i] + M[a][2] * q[2][i] + M[a][3] * q[3][i];
    }
    Eng<T> Sw;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const T lam = side == 0 ? lam_s : lam_l, mu = side == 0 ? mu_s : mu_l;
        const T sg = (side == 0) == pos ? (T)1 : (T)-1;
        if (side == 1) {
            // complement
            T qs[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) qs[i] = V20 * (q[0][i] + q[1][i] + q[2][i] + q[3][i]);
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                m[a] = (T)5 * V20 - m[a];
#pragma unroll
                for (int i = 0; i < 3; ++i) y[a][i] = (qs[i] + V20 * q[a][i]) - y[a][i];
#pragma unroll
                for (int c = a; c < 4; ++c) M[a][c] = M[c][a] = (a == c ? (T)2 * V20 : V20) - M[a][c];
            }
        }
        T w[4], Mw[4], G[3];
#pragma unroll
        for (int a = 0; a < 4; ++a) w[a] = fabs(L[a]) - sg * L[a];
#pragma unroll
        for (int i = 0; i < 3; ++i) G[i] = w[i + 1] - w[i];
        T vs = 0, sw = 0, ww = 0, p[3] = {0, 0, 0}, pw[3] = {0, 0, 0};
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            Mw[a] = M[a][0] * w[0] + M[a][1] * w[1] + M[a][2] * w[2] + M[a][3] * w[3];
            vs += m[a];
            sw += Mw[a];
            ww += w[a] * Mw[a];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                p[i] += y[a][i];
                pw[i] += w[a] * y[a][i];
            }
        }
        const Eng<T> st = eng_hooke(eng_comb(vs, eF, sw, eq, p, G), lam, mu);
        const Eng<T> sv = eng_hooke(eng_comb(sw, eF, ww, eq, pw, G), lam, mu);
        if (side == 0) { S = st; Sw = sv; }
        else { eng_add(S, st); eng_add(Sw, sv); }
        T tF[3], tq[3];
        eng_vec(eng_hooke(eF, lam, mu), G, tF);
        eng_vec(eng_hooke(eq, lam, mu), G, tq);
        const T g2 = mu * (G[0] * G[0] + G[1] * G[1] + G[2] * G[2]), lm = lam + mu;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const T yg = lm * (y[a][0] * G[0] + y[a][1] * G[1] + y[a][2] * G[2]);
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const T v = m[a] * tF[i] + Mw[a] * tq[i] + yg * G[i] + g2 * y[a][i];
                fe[a][i] = side == 0 ? v : fe[a][i] + v;
            }
        }
    }
    eng_scatter(Sw, fe);
}

template <typename T> struct IrrArgs {
    const T *x, *xe;          // inputs of load 0 (null: zero); loads 3 N / 3 nX apart
    T *cutbuf;                // corner-force buffer of load 0
    const double *ebar;       // [rhs][6] Mandel
    const Flags *flags;
    int parity;
    const int32_t *irr, *irr_node, *irr_j;
    const T *irr_L;
    const int32_t *tet_cut, *tet_uncut, *blk_cut;
    const int32_t *cut_lab, *uncut_lab;
    const T *cut_M;
    const T *d0is, *lame;
    double *partial;
    int nslots, slot0;
    double *vstress;          // [rhs][6][N] voxel-average Mandel stress, or null
    int64_t N, nX, nirr, ncut;
    int blocks;               // workgroups per right-hand side
};

// Odd strides per voxel and element: the same place of neighbouring voxels falls on
// different banks.  Lanes at different corners and elements still meet: 2.4 conflict
// cycles per LDS instruction, about 14 of 102 us at 128^3 FP32 with six loads.
constexpr int IN_S = 51, OUT_T = 25, OUT_S = 6 * OUT_T + 1, L_S = 9;
constexpr int CS_S = 25;          // corner sums, FE and enriched halves: 2 x 25 values in place of a voxel's corner values
static_assert(2 * CS_S <= IN_S, "the corner sums fit in the place of the corner values");
template <typename T> struct IrrShared {
    T in[VB * IN_S];          // [voxel][corner][6]: u, then D0^-1/2 u~
    T out[VB * OUT_S];        // [voxel][element][vertex][6]: FE, then enriched vertex forces
    T L[VB * L_S], sc[VB * L_S];
    double red[4 * 7];
};

template <typename T, bool HX, bool EB, bool ST>
__global__ __launch_bounds__(BT) void k_irregular(IrrArgs<T> A) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    IrrShared<T> &sh = *reinterpret_cast<IrrShared<T> *>(smem_raw);
    const int64_t lb = xcd_remap(blockIdx.x, gridDim.x);
    const int r = (int)(lb / A.blocks), blk = (int)(lb % A.blocks);
    if (A.flags && A.flags[r].active[A.parity] == 0) return;
    const int tid = threadIdx.x;
    const uint32_t q0 = (uint32_t)blk * VB, nirr = (uint32_t)A.nirr;
    const int nv = min(VB, (int)(nirr - q0));
    const T *x = HX ? A.x + (int64_t)r * 3 * A.N : nullptr;
    const T *xe = HX ? A.xe + (int64_t)r * 3 * A.nX : nullptr;
    // the first element of the lane: its geometry is loaded together with the corner values
    const int c0 = A.blk_cut[blk], c1 = A.blk_cut[blk + 1];
    const int u0 = 6 * (int)q0 - c0, u1 = 6 * ((int)q0 + nv) - c1;
    int desc = 0;
    T ms[10] = {}, mod[4] = {};
    if (c0 + tid < c1) {
        const int i = c0 + tid;
        desc = elem(A.tet_cut, (uint32_t)i);
        const int ls = elem(A.cut_lab, (uint32_t)i), ll = elem(A.cut_lab + A.ncut, (uint32_t)i);
#pragma unroll
        for (int e = 0; e < 10; ++e) ms[e] = elem(A.cut_M + e * A.ncut, (uint32_t)i);
        mod[0] = A.lame[2 * ls]; mod[1] = A.lame[2 * ls + 1];
        mod[2] = A.lame[2 * ll]; mod[3] = A.lame[2 * ll + 1];
    }
    // corner values, corner by corner (rows of the tables)
    for (int it = tid; it < 8 * VB; it += BT) {
        const int c = it / VB, v = it - c * VB;
        if (v < nv) {
            const uint32_t row = (uint32_t)c * nirr + q0 + (uint32_t)v;
            const int jc = elem(A.irr_j, row);
            sh.L[v * L_S + c] = elem(A.irr_L, row);
            T sc = 0, u[3] = {0, 0, 0}, e[3] = {0, 0, 0};
            if constexpr (HX) {
                const uint32_t node = (uint32_t)elem(A.irr_node, row);
#pragma unroll
                for (int i = 0; i < 3; ++i) u[i] = elem(x + (int64_t)i * A.N, node);
            }
            if (jc >= 0) {
                sc = elem(A.d0is, (uint32_t)jc);
                if constexpr (HX) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) e[i] = sc * elem(xe + (int64_t)i * A.nX, (uint32_t)jc);
                }
            }
            sh.sc[v * L_S + c] = sc;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                sh.in[v * IN_S + 6 * c + i] = u[i];
                sh.in[v * IN_S + 6 * c + 3 + i] = e[i];
            }
        }
    }
    T eb[6] = {0, 0, 0, 0, 0, 0};
    if constexpr (EB) {
        const Sym<T> s = load_ebar<T>(A.ebar + 6 * r);
        eb[0] = s.xx; eb[1] = s.yy; eb[2] = s.zz; eb[3] = s.yz; eb[4] = s.xz; eb[5] = s.xy;
    }
    // macro strain of a diagonal / off-diagonal pair in local axes
    auto add_macro = [&](Eng<T> &e, int p0, int p1, int p2) {
        if constexpr (EB) {
            auto pick = [&](int o, int p) { return p == 0 ? eb[o] : (p == 1 ? eb[o + 1] : eb[o + 2]); };
            e.n[0] += pick(0, p0); e.n[1] += pick(0, p1); e.n[2] += pick(0, p2);
            e.g[0] += (T)2 * pick(3, p0); e.g[1] += (T)2 * pick(3, p1); e.g[2] += (T)2 * pick(3, p2);
        }
    };
    __syncthreads();
    double acc7[7] = {0, 0, 0, 0, 0, 0, 0};
    if (c0 + tid < c1) {
        const int qv = desc / 6, t = desc - 6 * qv, v = qv - (int)q0;
        const bool pos = !signbit(ms[0]);
        ms[0] = fabs(ms[0]);
        int p0, p1, p2;
        tet_axes(t, p0, p1, p2);
        const int cn[4] = {0, 1 << p0, (1 << p0) | (1 << p1), 7};
        T L[4], u[4][3], q[4][3];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const T *in = sh.in + v * IN_S + 6 * cn[a];
            L[a] = sh.L[v * L_S + cn[a]];
            u[a][0] = in[p0]; u[a][1] = in[p1]; u[a][2] = in[p2];
            q[a][0] = in[3 + p0]; q[a][1] = in[3 + p1]; q[a][2] = in[3 + p2];
        }
        Eng<T> eF = eng_strain<T>(u);
        add_macro(eF, p0, p1, p2);
        Eng<T> S;
        T f[4][3], fe[4][3];
        cut_element<T>(L, eF, q, ms, pos, mod[0], mod[1], mod[2], mod[3], S, fe);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int d = 0; d < 3; ++d) f[a][d] = acc_zero<T>();
        eng_scatter(S, f);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            T *o = sh.out + v * OUT_S + OUT_T * t + 6 * a;
            o[p0] = f[a][0]; o[p1] = f[a][1]; o[p2] = f[a][2];
            o[3 + p0] = fe[a][0]; o[3 + p1] = fe[a][1]; o[3 + p2] = fe[a][2];
        }
    }
    // uncut elements, from the last thread down (the waves with the fewest cut ones)
    if (const int i = u0 + (BT - 1 - tid); i < u1) {
        const int desc = elem(A.tet_uncut, (uint32_t)i);
        const int qv = desc / 6, t = desc - 6 * qv, v = qv - (int)q0;
        const int lm = elem(A.uncut_lab, (uint32_t)i);
        const T V = (T)(1.0 / 6.0);
        const T lam = V * A.lame[2 * lm], mu = V * A.lame[2 * lm + 1];
        int p0, p1, p2;
        tet_axes(t, p0, p1, p2);
        const int cn[4] = {0, 1 << p0, (1 << p0) | (1 << p1), 7};
        T u[4][3];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const T *in = sh.in + v * IN_S + 6 * cn[a];
            u[a][0] = in[p0]; u[a][1] = in[p1]; u[a][2] = in[p2];
        }
        Eng<T> eF = eng_strain<T>(u);
        add_macro(eF, p0, p1, p2);
        T f[4][3];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int d = 0; d < 3; ++d) f[a][d] = acc_zero<T>();
        eng_scatter(eng_hooke(eF, lam, mu), f);
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            T *o = sh.out + v * OUT_S + OUT_T * t + 6 * a;
            o[p0] = f[a][0]; o[p1] = f[a][1]; o[p2] = f[a][2];
            o[3] = o[4] = o[5] = 0;
        }
    }
    __syncthreads();
    // corner sums: corner 0 is vertex 0 of all six elements, corner 7 vertex 3,
    // corner e_a vertex 1 of the two elements that start along a, corner 7 - e_l
    // vertex 2 of the two that end along l
    T *cb = A.cutbuf + (int64_t)r * cut_rows(A.nirr) * 48;
    T *cbe = cb + cut_rows(A.nirr) * 24;
    for (int it = tid; it < 8 * VB; it += BT) {
        const int c = it / VB, v = it - c * VB;
        if (v < nv) {
            T s[6];
            const T *o = sh.out + v * OUT_S;
            if (c == 0 || c == 7) {
                const int a = c == 0 ? 0 : 3;
#pragma unroll
                for (int d = 0; d < 6; ++d) s[d] = o[6 * a + d];
#pragma unroll
                for (int t = 1; t < 6; ++t)
#pragma unroll
                    for (int d = 0; d < 6; ++d) s[d] += o[OUT_T * t + 6 * a + d];
            } else {
                // first: elements 2a, 2a + 1; last axis l = 0, 1, 2: elements 3, 5; 1, 4; 0, 2
                const bool one = c == 1 || c == 2 || c == 4;
                const int l = c == 6 ? 0 : (c == 5 ? 1 : 2);
                const int ta = one ? 2 * (c >> 1) : (l == 0 ? 3 : (l == 1 ? 1 : 0));
                const int tb = one ? ta + 1 : (l == 0 ? 5 : (l == 1 ? 4 : 2));
                const int a = one ? 1 : 2;
#pragma unroll
                for (int d = 0; d < 6; ++d) s[d] = o[OUT_T * ta + 6 * a + d] + o[OUT_T * tb + 6 * a + d];
            }
            if constexpr (ST) {
                // stress integral of the voxel: sum over the corners of force (x) position
                const T dx = (T)(c & 1), dy = (T)((c >> 1) & 1), dz = (T)(c >> 2);
                const Sym<T> w = {dx * s[0], dy * s[1], dz * s[2], dz * s[1], dz * s[0], dy * s[0]};
                add_sym(acc7, w);
            }
            // the corner values are no longer needed: their place takes the sums
            const T sc = sh.sc[v * L_S + c];
            T *w = sh.in + v * CS_S + 3 * c;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                w[i] = s[i];
                w[VB * CS_S + i] = sc * s[3 + i];
            }
        }
    }
    __syncthreads();
    // one contiguous stream per half of the buffer (written corner by corner the
    // stores took 36 cache-line writes per wave instruction instead of 4)
    for (int it = tid; it < 24 * nv; it += BT) {
        const int v = it / 24, k = it - 24 * v;
        elem(cb, cut_index(q0, it)) = sh.in[v * CS_S + k];
        elem(cbe, cut_index(q0, it)) = sh.in[VB * CS_S + v * CS_S + k];
    }
    if constexpr (ST) {
        if (A.vstress && tid < nv) {
            // voxel stress: corner forces again, by elements of the voxel of this thread
            double w[6] = {0, 0, 0, 0, 0, 0};
            for (int t = 0; t < 6; ++t) {
                int p0, p1, p2;
                tet_axes(t, p0, p1, p2);
                const int cn[4] = {0, 1 << p0, (1 << p0) | (1 << p1), 7};
                for (int a = 1; a < 4; ++a) {
                    const T *o = sh.out + tid * OUT_S + OUT_T * t + 6 * a;
                    const double dx = cn[a] & 1, dy = (cn[a] >> 1) & 1, dz = cn[a] >> 2;
                    w[0] += dx * (double)o[0]; w[1] += dy * (double)o[1]; w[2] += dz * (double)o[2];
                    w[3] += dz * (double)o[1]; w[4] += dz * (double)o[0]; w[5] += dy * (double)o[0];
                }
            }
            const Sym<double> sv = {w[0], w[1], w[2], w[3], w[4], w[5]};
            store_vstress(A.vstress + (int64_t)r * 6 * A.N, A.N, A.irr[q0 + tid], sv);
        }
        block_sum<7>(acc7, sh.red);
    }
    if (tid == 0) {
        double *P = A.partial + ((int64_t)r * A.nslots + A.slot0 + blk) * NPART;
#pragma unroll
        for (int q = 0; q < 7; ++q) P[q] = acc7[q];
    }
}

// ---------------------------------------------------------------- cached voxel matrices
// Column k of the matrix of irregular voxel q: the voxel's forces for the unit
// input dof k (k < 24: FE component k % 3 of corner k / 3; k >= 24: enriched
// dof (k - 24) of the corner, entering scaled by D0^-1/2), by the moment form
// above in FP64; the outputs are the FE corner forces and the scaled enriched
// corner forces, as the irregular-voxel kernel writes them.  Column k supplies
// the rows i <= k of the packed upper triangle and the stress integral.
__global__ __launch_bounds__(128) void k_vm_build(IrrArgs<double> A, const int32_t *irr_lab, const int32_t *cut_pos,
                                                  double *K64, float *K32) {
    __shared__ double col[48][128];
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t q = t0 / 48;
    const int k = (int)(t0 - q * 48), tid = threadIdx.x;
    if (q >= A.nirr) return;
    for (int i = 0; i < 48; ++i) col[i][tid] = 0.0;
    double st[6] = {0, 0, 0, 0, 0, 0};
    const int kc = (k < 24 ? k : k - 24) / 3, kd = (k < 24 ? k : k - 24) % 3;
    const int jk = A.irr_j[(int64_t)kc * A.nirr + q];
    const double sk = jk >= 0 ? A.d0is[jk] : 0.0;
    for (int t = 0; t < 6; ++t) {
        int p0, p1, p2;
        tet_axes(t, p0, p1, p2);
        const int cn[4] = {0, 1 << p0, (1 << p0) | (1 << p1), 7};
        const int ax[3] = {p0, p1, p2};
        double L[4], u[4][3], qe[4][3];
        for (int a = 0; a < 4; ++a) {
            L[a] = A.irr_L[cn[a] * A.nirr + q];
            for (int s = 0; s < 3; ++s) {
                const bool hit = cn[a] == kc && ax[s] == kd;
                u[a][s] = hit && k < 24 ? 1.0 : 0.0;
                qe[a][s] = hit && k >= 24 ? sk : 0.0;
            }
        }
        const Eng<double> eF = eng_strain<double>(u);
        Eng<double> S;
        double f[4][3] = {}, fe[4][3] = {};
        const int32_t i = cut_pos[6 * q + t];
        if (i >= 0) {
            double ms[10];
            for (int e = 0; e < 10; ++e) ms[e] = A.cut_M[e * A.ncut + i];
            const bool pos = !signbit(ms[0]);
            ms[0] = fabs(ms[0]);
            const int ls = A.cut_lab[i], ll = A.cut_lab[A.ncut + i];
            cut_element<double>(L, eF, qe, ms, pos, A.lame[2 * ls], A.lame[2 * ls + 1], A.lame[2 * ll],
                                A.lame[2 * ll + 1], S, fe);
        } else {
            const int lm = irr_lab[(int64_t)(2 * t) * A.nirr + q];
            S = eng_hooke(eF, A.lame[2 * lm] / 6.0, A.lame[2 * lm + 1] / 6.0);
        }
        eng_scatter(S, f);
        for (int a = 0; a < 4; ++a)
            for (int s = 0; s < 3; ++s) {
                col[3 * cn[a] + ax[s]][tid] += f[a][s];
                col[24 + 3 * cn[a] + ax[s]][tid] += fe[a][s];
            }
        for (int s = 0; s < 3; ++s) {
            st[ax[s]] += S.n[s];
            st[3 + ax[s]] += S.g[s];
        }
    }
    double *k64 = K64 + q * VM_STRIDE;
    float *k32 = K32 ? K32 + q * VM_STRIDE : nullptr;
    for (int i = 0; i <= k; ++i) {
        double v = col[i][tid];
        if (i >= 24) {
            const int jc = A.irr_j[(int64_t)((i - 24) / 3) * A.nirr + q];
            v *= jc >= 0 ? A.d0is[jc] : 0.0;
        }
        k64[vm_row(i) + k] = v;
        if (k32) k32[vm_row(i) + k] = (float)v;
    }
    for (int m = 0; m < 6; ++m) {
        k64[VM_KP + 48 * m + k] = st[m];
        if (k32) k32[VM_KP + 48 * m + k] = (float)st[m];
    }
    if (k < VM_KP - VM_K) {
        k64[VM_K + k] = 0.0;
        if (k32) k32[VM_K + k] = 0.0f;
    }
}

template <typename T>
IrrArgs<T> irr_args(const xfft_problem *p, const Tables<T> &tb) {
    const Geometry &g = p->g;
    IrrArgs<T> A{};
    A.irr = p->irr; A.irr_node = p->irr_node; A.irr_j = p->irr_j; A.irr_L = tb.irr_L;
    A.tet_cut = p->tet_cut; A.tet_uncut = p->tet_uncut; A.blk_cut = p->blk_cut;
    A.cut_lab = p->cut_lab; A.uncut_lab = p->uncut_lab; A.cut_M = tb.cut_M;
    A.d0is = tb.d0is; A.lame = tb.lame;
    A.N = g.N; A.nX = g.nX; A.nirr = g.nirr; A.ncut = p->n_cut_elements;
    A.blocks = p->slots.cut_n;
    return A;
}

template <typename T, bool HX, bool EB, bool ST>
void launch_irr(int device, const IrrArgs<T> &A, int nrhs, hipStream_t s) {
    const size_t lds = sizeof(IrrShared<T>);
    static std::atomic<uint64_t> lds_ok{0};
    allow_lds(lds_ok, device, k_irregular<T, HX, EB, ST>, lds);
    k_irregular<T, HX, EB, ST><<<(unsigned)(A.blocks * nrhs), BT, lds, s>>>(A);
}

}  // namespace

template <typename T>
void launch_irregular(xfft_problem *p, const Tables<T> &tb, const T *x, const T *xe, const double *ebar, bool use_ebar,
                      int nrhs, const Flags *flags, int parity, double *vstress, hipStream_t s, bool stress, T *cutbuf,
                      double *partial) {
    IrrArgs<T> A = irr_args<T>(p, tb);
    A.x = x; A.xe = xe; A.cutbuf = cutbuf; A.ebar = ebar; A.flags = flags; A.parity = parity;
    A.partial = partial; A.nslots = p->nslots; A.slot0 = p->slots.cut0; A.vstress = vstress;
    const bool hx = x != nullptr;
    xfft_prof_mark(p, -1, s);
    if (hx && use_ebar) launch_irr<T, true, true, true>(p->device, A, nrhs, s);
    else if (hx && stress) launch_irr<T, true, false, true>(p->device, A, nrhs, s);
    else if (hx) launch_irr<T, true, false, false>(p->device, A, nrhs, s);
    else if (use_ebar) launch_irr<T, false, true, true>(p->device, A, nrhs, s);
    else launch_irr<T, false, false, false>(p->device, A, nrhs, s);
    xfft_prof_mark(p, K_IRREGULAR + (sizeof(T) == 8 ? K_COUNT : 0), s);
}

template void launch_irregular<double>(xfft_problem *, const Tables<double> &, const double *, const double *,
                                       const double *, bool, int, const Flags *, int, double *, hipStream_t, bool,
                                       double *, double *);
template void launch_irregular<float>(xfft_problem *, const Tables<float> &, const float *, const float *,
                                      const double *, bool, int, const Flags *, int, double *, hipStream_t, bool,
                                      float *, double *);

void launch_vm_build(xfft_problem *p, double *K64, float *K32) {
    const IrrArgs<double> A = irr_args<double>(p, p->t64);
    const int64_t nt = p->g.nirr * 48;
    k_vm_build<<<(unsigned)((nt + 127) / 128), 128, 0, p->stream>>>(A, p->irr_lab, p->cut_pos, K64, K32);
}

}  // namespace xfft
