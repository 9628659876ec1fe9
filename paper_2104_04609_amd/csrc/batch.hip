// Matrix-free product of the permuted PMCHWT operator (Sec. 2.7) with several
// vectors: every separated triangle pair is integrated once per batch and the
// vectors are multiplied on the matrix cores.
//
// The sums are those of the single-vector pair kernel (6 x 6 rule, point pairs
// of triangles sharing no vertex).  For one triangle pair (tau, sigma) they are
// the four complex 3 x 3 local blocks
//   V_ab = sum w_i w_j phi_a(x_i) phi_b(y_j) (G_0 + rho G_1)
//   K_ab = sum w_i w_j phi_a phi_b F (y_j - x_i).n_sigma      (row 1, phi; negated)
//   P_ab = sum w_i w_j phi_a phi_b F (x_i - y_j).n_tau        (row 2, psi)
//   D_ab = curl_a . curl_b sum w_i w_j (G_0 + G_1 / rho)
//          - k_0^2 (n_tau . n_sigma) sum w_i w_j phi_a phi_b (G_0 + n_10 G_1)
// times the trial triangle's vertex values; the curl part of D acts on
// differences of phi, so that a constant phi cancels before rounding.
// A lane forms the blocks of one pair: lane l of a wavefront holds tau = l % 16,
// sigma = l / 16, which is the A operand of v_mfma_f32_16x16x4 and
// v_mfma_f64_16x16x4 (row l % 16, k = l / 16), so a block entry goes to the
// matrix core as it stands.  The B operand is |sigma| times the vertex values
// (or the curl) of the four sigma in 16 real columns (8 vectors, re and im
// interleaved) and, for the imaginary parts of the blocks, the same columns
// times i.
//
// FP32 (batch_kernel): the blocks are summed over all 36 points before the
// product, 72 matrix instructions per 64 triangle pairs and 16 columns.  The
// evaluation (about 60 VALU instructions and 5 transcendentals per point pair)
// does not depend on the number of vectors; with C > 1 the four wavefronts of a
// workgroup form 4 / C tiles of 16 test triangles, C wavefronts evaluate
// different sigma of one tile, exchange their blocks through LDS and multiply
// 16 columns each, so that one evaluation serves 8 C vectors.
// 16 vectors at 6 252 vertices: 15.7 ms, from 81.3 ms with four vectors per launch
// on the vector units; matrix and vector instructions of two wavefronts hardly
// overlap (VALU issue 72 %, matrix cores 33 % of the cycles), so their sum counts.
// FP64 (batch64_kernel): the blocks of a pair would take 144 registers, which
// spill to accumulation registers at four moves per update; the sums over the
// test points alone (48 registers) are multiplied for every trial point, 162
// matrix instructions, at two wavefronts per SIMD.
#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <type_traits>

#include "batch_split.h"
#include "bem_internal.h"
#include "entries.h"

namespace bem {

namespace {

using entries::DCoefT;
using entries::DIntT;
using entries::DM;
using entries::qb;
using entries::qw;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr double INV4PI = 0.079577471545947667884441881686257;
constexpr int BT_THREADS = 256;   // four wavefronts
constexpr int BT_TAU = 16;        // test triangles per wavefront tile
constexpr int BT_COLS = 16;       // real columns per matrix tile: 8 vectors
constexpr int BT_BLK = 72;        // 4 complex 3 x 3 blocks
// Weights of the sums over the test points.  w phi_a is o at the two other points
// of an orbit and o + d at the own one (o_1, d_1; o_2, d_2), so that
//   sum_i w_i phi_a(x_i) v_i = d_1 (c_a + BW_C (c_0 + c_1 + c_2) + BW_U U),
//   c_a = v_a + BW_D v_{a+3},  U = v_3 + v_4 + v_5:
// 12 operations for three a instead of 18.  d_1 goes into the final scale.  FP32
// trial weights are taken times BT_SCALE, for which all of them are FP32 numbers
// to 6e-10: their rounding, the same for every pair, would not average out.
constexpr double BW_O1 = qw(0) * qb(0, 1), BW_D1 = qw(0) * (qb(0, 0) - qb(0, 1));
constexpr double BW_O2 = qw(3) * qb(3, 1), BW_D2 = qw(3) * (qb(3, 0) - qb(3, 1));
constexpr double BW_D = BW_D2 / BW_D1, BW_C = BW_O1 / BW_D1;
constexpr double BW_U = (BW_O2 - BW_D * BW_O1) / BW_D1;
constexpr double BT_SCALE = 1.8680741340591038;
// the blocks carry this factor
template <class R> constexpr double bt_scale() {
    return (std::is_same<R, float>::value ? BT_SCALE : 1.0) / BW_D1;
}

// staged trial triangle: points, normal, plane offset (odd stride: the four
// sigma of a step in distinct banks); vertex ids and object
constexpr int BG_N = 18, BG_C = 21, BG_C1 = GEO_STRIDE, BG_VALS = 23;

template <class R> struct Mx;
template <> struct Mx<float> {
    using Acc = f32x4;
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // accumulator element v of lane l: row 4 (l / 16) + v, column l % 16
    static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
    static __device__ __forceinline__ float swap(float v) {   // neighbouring lane (l ^ 1)
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1,
                                                                  0xF, 0xF, true));
    }
};
template <> struct Mx<double> {
    using Acc = f64x4;
    static __device__ __forceinline__ Acc mma(double a, double b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // accumulator element v of lane l: row l / 16 + 4 v, column l % 16
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
    static __device__ __forceinline__ double swap(double v) {
        const long long b = __builtin_bit_cast(long long, v);
        const int lo = __builtin_amdgcn_mov_dpp((int)b, 0xB1, 0xF, 0xF, true);
        const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0xB1, 0xF, 0xF, true);
        return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
    }
};

__device__ __forceinline__ float fmaC(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaC(double a, double b, double c) { return __builtin_fma(a, b, c); }

// sin and cos of the phase t (phase units).  FP32 phases stay below 256
// revolutions here, inside which the hardware functions reduce exactly; FP64 ones
// below PHASE64_NARROW (the lossy variants are 5 % slower with the wide form,
// which spills six more registers)
__device__ __forceinline__ void sc_rev(float t, float &s, float &c, const double2 *) {
    s = __builtin_amdgcn_sinf(t);
    c = __builtin_amdgcn_cosf(t);
}
__device__ __forceinline__ void sc_rev(double t, double &s, double &c, const double2 *tab) {
    sincos_256<false>(t, s, c, tab);
}

// w_j phi_b(y_j), read with a point index that is uniform over the wavefront
#define BEM_WB(j) qw(j) * qb(j, 0), qw(j) * qb(j, 1), qw(j) * qb(j, 2)
__constant__ double kWB64[18] = {BEM_WB(0), BEM_WB(1), BEM_WB(2), BEM_WB(3), BEM_WB(4), BEM_WB(5)};
#undef BEM_WB
#define BEM_WB1(j, b) (float)(BT_SCALE * qw(j) * qb(j, b))
#define BEM_WB(j) BEM_WB1(j, 0), BEM_WB1(j, 1), BEM_WB1(j, 2)
__constant__ float kWB32[18] = {BEM_WB(0), BEM_WB(1), BEM_WB(2), BEM_WB(3), BEM_WB(4), BEM_WB(5)};
#undef BEM_WB
#undef BEM_WB1
template <class R> __device__ __forceinline__ R wb_at(int k) {
    if constexpr (std::is_same<R, float>::value) return kWB32[k];
    else return kWB64[k];
}

// 2^x for x <= 0 (decay of lossy media)
__device__ __forceinline__ float decay(float x, const double *) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ double decay(double x, const double *tab) { return decay64(x, tab); }

// x [nr][2N] -> xt [N][2][cols], vector r in columns 2r (re) and 2r + 1 (im),
// zeros beyond nr
__global__ __launch_bounds__(256) void batch_gather_kernel(const double2 *__restrict__ x, int nr,
                                                           int64_t N, int cols,
                                                           double *__restrict__ xt) {
    const int half = cols / 2;
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (id >= 2 * N * half) return;
    const int64_t vh = id / half;
    const int r = (int)(id - vh * half);
    const int64_t v = vh >> 1, h = vh & 1;
    const double2 z = r < nr ? x[(int64_t)r * 2 * N + h * N + v] : make_double2(0.0, 0.0);
    reinterpret_cast<double2 *>(xt)[id] = z;
}

// One row of a staged trial triangle (both kernels).
template <class R>
__device__ __forceinline__ void stage_tile(const R *__restrict__ geo, const int32_t *__restrict__ tobj,
                                           const int32_t *__restrict__ tri,
                                           const double *__restrict__ tst, int T, int base,
                                           bool multi, R *g, int32_t *gi, double *gt) {
    for (int idx = threadIdx.x; idx < BT_TILE * BG_C1; idx += BT_THREADS) {
        const int sl = idx / BG_C1, f = idx - sl * BG_C1;
        const int s = min(base + sl, T - 1);   // (finite values beyond the end)
        g[sl * BG_VALS + f] = geo[(int64_t)GEO_STRIDE * s + f];
    }
    if (threadIdx.x < BT_TILE * 4) {
        const int sl = threadIdx.x >> 2, f = threadIdx.x & 3;
        const int s = min(base + sl, T - 1);
        gi[threadIdx.x] = f < 3 ? tri[3 * s + f] : (multi ? tobj[s] : 0);
    }
    for (int idx = threadIdx.x; idx < BT_TILE * TST_STRIDE; idx += BT_THREADS)
        gt[idx] = tst[min((int64_t)base * TST_STRIDE + idx, (int64_t)T * TST_STRIDE - 1)];
}

// Sums over the six test points x_i, weights w_i phi_a(x_i), of the kernel
// values at one trial point y, over d_1: c[q][a], q = G_0 re im, G_1 re im,
// F (y - x).n_y re im, F re im.
template <class R, bool CK0, bool CK1>
__device__ __forceinline__ void point_sums(R yx, R yy, R yz, const R (&px)[6], const R (&py)[6],
                                           const R (&pz)[6], const R (&dny)[6], bool dead,
                                           const DCoefT<R> &cf, const DIntT<R> &c1,
                                           const double2 *etab, const double *xtab, R (&c)[8][3]) {
    R S[8], U[8];   // sums of c, sums over the second orbit
#pragma unroll
    for (int i = 0; i < 6; i++) {
        const R dx = yx - px[i], dy = yy - py[i], dz = yz - pz[i];
        const R r2 = dx * dx + dy * dy + dz * dz;
        R ri = DM<R>::rsq(r2);
        ri = dead ? (R)0 : ri;   // all values of a dead pair vanish
        const R r = r2 * ri;
        R E0r, E0i, E1r, E1i;
        sc_rev(r * cf.krev0, E0i, E0r, etab);
        sc_rev(r * c1.krev1, E1i, E1r, etab);
        if (CK0) {
            const R d0 = decay(r * cf.kdec0, xtab);
            E0r *= d0;
            E0i *= d0;
        }
        if (CK1) {
            const R d1 = decay(r * c1.kdec1, xtab);
            E1r *= d1;
            E1i *= d1;
        }
        const R G0r = E0r * ri, G0i = E0i * ri, G1r = E1r * ri, G1i = E1i * ri;
        R Fr = fmaC(c1.ns1, G1r, -G0r), Fi = fmaC(c1.ns1, G1i, -G0i);
        Fr = fmaC(-cf.k0r, E0i, Fr);
        Fi = fmaC(cf.k0r, E0r, Fi);
        Fr = fmaC(-c1.k1r, E1i, Fr);
        Fi = fmaC(c1.k1r, E1r, Fi);
        if (CK0) {
            Fr = fmaC(-cf.k0i, E0r, Fr);
            Fi = fmaC(-cf.k0i, E0i, Fi);
        }
        if (CK1) {
            Fr = fmaC(-c1.k1i, E1r, Fr);
            Fi = fmaC(-c1.k1i, E1i, Fi);
        }
        const R ri2 = ri * ri;
        Fr *= ri2;
        Fi *= ri2;
        const R val[8] = {G0r, G0i, G1r, G1i, Fr * dny[i], Fi * dny[i], Fr, Fi};
#pragma unroll
        for (int q = 0; q < 8; q++) {
            if (i < 3) c[q][i] = val[q];
            else c[q][i - 3] = fmaC((R)BW_D, val[q], c[q][i - 3]);
            U[q] = i == 3 ? val[q] : i > 3 ? U[q] + val[q] : (R)0;
        }
    }
#pragma unroll
    for (int q = 0; q < 8; q++) {
        S[q] = fmaC((R)BW_C, c[q][0] + c[q][1] + c[q][2], (R)BW_U * U[q]);
#pragma unroll
        for (int a = 0; a < 3; a++) c[q][a] += S[q];
    }
}

// Geometry and ids of a lane's test triangle.
template <class R> struct Test {
    R px[6], py[6], pz[6], nx, ny, nz, c;
    int v0, v1, v2, obj;
    __device__ __forceinline__ void load(const R *geo, const int32_t *tri, const int32_t *tobj,
                                         int t, bool multi) {
        for (int i = 0; i < 6; i++) {
            px[i] = geo[GEO_STRIDE * t + 3 * i];
            py[i] = geo[GEO_STRIDE * t + 3 * i + 1];
            pz[i] = geo[GEO_STRIDE * t + 3 * i + 2];
        }
        nx = geo[GEO_STRIDE * t + 18];
        ny = geo[GEO_STRIDE * t + 19];
        nz = geo[GEO_STRIDE * t + 20];
        c = geo[GEO_STRIDE * t + 21];
        v0 = tri[3 * t];
        v1 = tri[3 * t + 1];
        v2 = tri[3 * t + 2];
        obj = multi ? tobj[t] : 0;
    }
    __device__ __forceinline__ bool touches(const int32_t *s) const {
        return s[0] == v0 || s[0] == v1 || s[0] == v2 || s[1] == v0 || s[1] == v1 || s[1] == v2 ||
               s[2] == v0 || s[2] == v1 || s[2] == v2;
    }
};

// interior coefficients of a trial triangle's object; zero where the triangles
// belong to different objects (the interior operators act within each)
template <class R, bool MULTI>
__device__ __forceinline__ DIntT<R> interior_of(const DCoefT<R> &cf, const DIntT<R> *__restrict__ itab,
                                                int obj, int own) {
    if constexpr (!MULTI) return cf.in;
    DIntT<R> c1 = itab[obj];
    if (obj != own) c1.k1r = c1.k1i = c1.rho = c1.irho = c1.n10r = c1.n10i = c1.ns1 = (R)0;
    return c1;
}

template <int C> constexpr size_t batch_ex() {
    return C > 1 ? (size_t)(BT_THREADS / 64) * BT_BLK * 64 : 1;
}

// FP32.  Two wavefronts per SIMD (two workgroups per CU: one evaluates while the
// other multiplies).
template <bool CK0, bool CK1, bool MULTI, int C>
__global__ __launch_bounds__(BT_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void batch_kernel(
    const float *__restrict__ geo, const double *__restrict__ tst, const int32_t *__restrict__ tobj,
    const int32_t *__restrict__ tri, int T, int split_len, DCoefT<float> cf,
    const DIntT<float> *__restrict__ itab, const double *__restrict__ xt,
    double *__restrict__ part) {
    using R = float;
    using M = Mx<float>;
    constexpr int W = BT_THREADS / 64 / C;   // test tiles per workgroup
    constexpr int COLS = BT_COLS * C;
    __shared__ R g[BT_TILE * BG_VALS];
    __shared__ int32_t gi[BT_TILE * 4];
    __shared__ double gt[BT_TILE * TST_STRIDE];   // areas and curls
    __shared__ R ex[batch_ex<C>()];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wt = wave / C, wc = wave % C;
    const int col = lane & 15, kq = lane >> 4;
    const int tau0 = ((int)blockIdx.x * W + wt) * BT_TAU;
    const int tau = tau0 + col;
    const int tt = tau < T ? tau : T - 1;
    const int s_begin = (int)blockIdx.y * split_len, s_end = min(T, s_begin + split_len);
    Test<R> te;
    te.load(geo, tri, tobj, tt, MULTI);
    R cu[9];
    for (int c = 0; c < 9; c++) cu[c] = (R)tst[(int64_t)TST_STRIDE * tt + 1 + c];
    const R rot = (lane & 1) ? (R)1 : (R)-1;   // columns times i: re <- -im, im <- re

    double sum[2][3][4];   // FP64 sums over the groups of four sigma
    for (int q = 0; q < 2; q++)
        for (int a = 0; a < 3; a++)
            for (int v = 0; v < 4; v++) sum[q][a][v] = 0.0;

    for (int base = s_begin; base < s_end; base += BT_TILE) {
        const int cnt = min(BT_TILE, s_end - base);
        __syncthreads();
        stage_tile<R>(geo, tobj, tri, tst, T, base, MULTI, g, gi, gt);
        __syncthreads();
        for (int s0 = 0; s0 < cnt; s0 += 4 * C) {
            const int sl = s0 + 4 * wc + kq;   // (< BT_TILE: the tile is whole steps)
            const R *src = g + sl * BG_VALS;
            const int *si = gi + 4 * sl;
            const bool dead = tau >= T || sl >= cnt || te.touches(si);
            const R nsx = src[BG_N], nsy = src[BG_N + 1], nsz = src[BG_N + 2], cs = src[BG_C];
            const DIntT<R> c1 = interior_of<R, MULTI>(cf, itab, si[3], te.obj);
            R dny[6];
            for (int i = 0; i < 6; i++)
                dny[i] = cs - (te.px[i] * nsx + te.py[i] * nsy + te.pz[i] * nsz);
            // blocks of G_0, G_1, F (y - x).n_y and F (x - y).n_x: [comp][3 a + b]
            R blk[8][9];
            for (int q = 0; q < 8; q++)
                for (int e = 0; e < 9; e++) blk[q][e] = (R)0;
#pragma unroll 1
            for (int j = 0; j < 6; j++) {
                const int ju = __builtin_amdgcn_readfirstlane(j);
                const R yx = src[3 * j], yy = src[3 * j + 1], yz = src[3 * j + 2];
                const R dnx = te.c - (yx * te.nx + yy * te.ny + yz * te.nz);
                R c[8][3];
                point_sums<R, CK0, CK1>(yx, yy, yz, te.px, te.py, te.pz, dny, dead, cf, c1, nullptr,
                                        nullptr, c);
#pragma unroll
                for (int q = 0; q < 8; q++)
#pragma unroll
                    for (int a = 0; a < 3; a++) {
                        const R v = q >= 6 ? c[q][a] * dnx : c[q][a];
#pragma unroll
                        for (int b = 0; b < 3; b++)
                            blk[q][3 * a + b] = fmaC(wb_at<R>(3 * ju + b), v, blk[q][3 * a + b]);
                    }
            }
            // vertex values of this lane's sigma in group q, this column: loaded
            // ahead of the product that uses them
            struct Vals {
                double p[3], f[3];
            };
            auto fetch = [&](int q) {
                const int *vi = gi + 4 * (s0 + 4 * q + kq);
                Vals v;
#pragma unroll
                for (int b = 0; b < 3; b++) {
                    const double *xv = xt + (int64_t)vi[b] * 2 * COLS + BT_COLS * wc + col;
                    v.p[b] = xv[0];
                    v.f[b] = xv[COLS];
                }
                return v;
            };
            Vals xq = fetch(0);
            // V and D from the G_0 and G_1 blocks; -K; the curl weight G_0 + G_1 / rho
            const R nn = te.nx * nsx + te.ny * nsy + te.nz * nsz;
            R w0r = (R)0, w0i = (R)0, w1r = (R)0, w1i = (R)0;
#pragma unroll
            for (int e = 0; e < 9; e++) {
                w0r += blk[0][e];
                w0i += blk[1][e];
                w1r += blk[2][e];
                w1i += blk[3][e];
            }
            const R gwr = fmaC(c1.irho, w1r, w0r), gwi = fmaC(c1.irho, w1i, w0i);
            const R gnr = -cf.n0r * nn, gni = -cf.n0i * nn;
            R lb[8][9];   // V re im, -K re im, P re im, D re im
#pragma unroll
            for (int e = 0; e < 9; e++) {
                R nr = fmaC(c1.n10r, blk[2][e], blk[0][e]), ni = fmaC(c1.n10r, blk[3][e], blk[1][e]);
                if (CK0 || CK1) {
                    nr = fmaC(-c1.n10i, blk[3][e], nr);
                    ni = fmaC(c1.n10i, blk[2][e], ni);
                }
                lb[0][e] = fmaC(c1.rho, blk[2][e], blk[0][e]);
                lb[1][e] = fmaC(c1.rho, blk[3][e], blk[1][e]);
                lb[2][e] = -blk[4][e];
                lb[3][e] = -blk[5][e];
                lb[4][e] = blk[6][e];
                lb[5][e] = blk[7][e];
                lb[6][e] = gnr * nr;
                lb[7][e] = gnr * ni;
                if (CK0) {
                    lb[6][e] = fmaC(-gni, ni, lb[6][e]);
                    lb[7][e] = fmaC(gni, nr, lb[7][e]);
                }
            }
            // phi enters as phi_0, phi_1 - phi_0, phi_2 - phi_0: the curl part of D
            // acts on the differences alone (the three curls add to zero)
#pragma unroll
            for (int a = 0; a < 3; a++) {
#pragma unroll
                for (int q = 2; q < 8; q += (q == 3 ? 3 : 1))
                    lb[q][3 * a] += lb[q][3 * a + 1] + lb[q][3 * a + 2];
#pragma unroll
                for (int b = 1; b < 3; b++) {
                    const double *cb = gt + TST_STRIDE * sl + 1 + 3 * b;
                    const R cc = cu[3 * a] * (R)cb[0] + cu[3 * a + 1] * (R)cb[1] + cu[3 * a + 2] * (R)cb[2];
                    lb[6][3 * a + b] = fmaC(cc, gwr, lb[6][3 * a + b]);
                    lb[7][3 * a + b] = fmaC(cc, gwi, lb[7][3 * a + b]);
                }
            }
            // group q of four sigma times 16 columns; its blocks in lb or, with
            // C > 1, in LDS at blkp
            auto multiply = [&](int q, const Vals &xq, const R *blkp) {
                M::Acc acc[2][3];
                for (int h = 0; h < 2; h++)
                    for (int a = 0; a < 3; a++)
                        for (int v = 0; v < 4; v++) acc[h][a][v] = (R)0;
                const double area = gt[TST_STRIDE * (s0 + 4 * q + kq)];
#pragma unroll
                for (int b = 0; b < 3; b++) {
                    const R p1 = (R)(area * xq.p[b]);
                    const R f1 = (R)(area * (b ? xq.f[b] - xq.f[0] : xq.f[0]));
                    const R p2 = rot * M::swap(p1), f2 = rot * M::swap(f1);
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        // k = 0: V (psi), 1: -K (phi); 2: P (psi), 3: D (phi)
                        const R x1 = (k & 1) ? f1 : p1, x2 = (k & 1) ? f2 : p2;
                        // (the three sums in turn: a product never waits for the last)
#pragma unroll
                        for (int h = 0; h < 2; h++)
#pragma unroll
                            for (int a = 0; a < 3; a++) {
                                const int q8 = 2 * k + h, e = 3 * a + b;
                                R v;
                                if constexpr (C > 1) v = blkp[(9 * q8 + e) * 64];
                                else v = lb[q8][e];
                                acc[k >> 1][a] = M::mma(v, h ? x2 : x1, acc[k >> 1][a]);
                            }
                    }
                }
                // 48 products per FP32 sum (the single-vector kernel's 448 are
                // sums at one of six points each, added in FP64)
                for (int h = 0; h < 2; h++)
                    for (int a = 0; a < 3; a++)
                        for (int v = 0; v < 4; v++) sum[h][a][v] += (double)acc[h][a][v];
            };
            if constexpr (C == 1) {
                multiply(0, xq, nullptr);
            } else {
                R *mine = ex + (size_t)wave * BT_BLK * 64 + lane;
#pragma unroll
                for (int q = 0; q < 8; q++)
#pragma unroll
                    for (int e = 0; e < 9; e++) mine[(9 * q + e) * 64] = lb[q][e];
                __syncthreads();
#pragma unroll 2
                for (int q = 0; q < C; q++) {
                    const Vals now = xq;
                    if (q + 1 < C) xq = fetch(q + 1);
                    multiply(q, now, ex + (size_t)(wt * C + q) * BT_BLK * 64 + lane);
                }
                __syncthreads();
            }
        }
    }
    // part[split][tau][3 q + a][COLS]
    for (int v = 0; v < 4; v++) {
        const int t = tau0 + M::row(lane, v);
        if (t >= T) continue;
        double *o = part + ((int64_t)blockIdx.y * T + t) * 6 * COLS + BT_COLS * wc + col;
        for (int q = 0; q < 2; q++)
            for (int a = 0; a < 3; a++) o[(3 * q + a) * COLS] = sum[q][a][v];
    }
}

// FP64, 8 vectors.  For every trial point the 24 sums over the test points are
// multiplied by the trial functions' values there.
template <bool CK0, bool CK1, bool MULTI>
__global__ __launch_bounds__(BT_THREADS) __attribute__((amdgpu_waves_per_eu(2))) void batch64_kernel(
    const double *__restrict__ geo, const double *__restrict__ tst,
    const int32_t *__restrict__ tobj, const int32_t *__restrict__ tri, int T, int split_len,
    DCoefT<double> cf, const DIntT<double> *__restrict__ itab, const double *__restrict__ xt,
    double *__restrict__ part) {
    using R = double;
    using M = Mx<double>;
    constexpr int W = BT_THREADS / 64, COLS = BT_COLS;
    __shared__ R g[BT_TILE * BG_VALS];
    __shared__ int32_t gi[BT_TILE * 4];
    __shared__ double gt[BT_TILE * TST_STRIDE];   // areas and curls
    __shared__ double2 etab[256];
    __shared__ double xtab[DECAY_TAB];
    __shared__ double cu[W * BT_TAU * 9];   // curls of the test triangles
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = lane & 15, kq = lane >> 4;
    DM<R>::fill_table(etab);
    if (CK0 || CK1) decay_table(xtab);
    for (int n = threadIdx.x; n < W * BT_TAU * 9; n += BT_THREADS) {
        const int t = min((int)blockIdx.x * W * BT_TAU + n / 9, T - 1);
        cu[n] = tst[(int64_t)TST_STRIDE * t + 1 + n % 9];
    }   // (the first tile's barrier orders these writes)
    const int tau0 = ((int)blockIdx.x * W + wave) * BT_TAU;
    const int tau = tau0 + col;
    const int tt = tau < T ? tau : T - 1;
    const int s_begin = (int)blockIdx.y * split_len, s_end = min(T, s_begin + split_len);
    Test<R> te;
    te.load(geo, tri, tobj, tt, MULTI);
    const R rot = (lane & 1) ? (R)1 : (R)-1;
    M::Acc acc[2][3];
    for (int q = 0; q < 2; q++)
        for (int a = 0; a < 3; a++)
            for (int v = 0; v < 4; v++) acc[q][a][v] = (R)0;

    for (int base = s_begin; base < s_end; base += BT_TILE) {
        const int cnt = min(BT_TILE, s_end - base);
        __syncthreads();
        stage_tile<R>(geo, tobj, tri, tst, T, base, MULTI, g, gi, gt);
        __syncthreads();
        for (int s0 = 0; s0 < cnt; s0 += 4) {
            const int sl = s0 + kq;
            const R *src = g + sl * BG_VALS;
            const int *si = gi + 4 * sl;
            const bool dead = tau >= T || sl >= cnt || te.touches(si);
            const R nsx = src[BG_N], nsy = src[BG_N + 1], nsz = src[BG_N + 2], cs = src[BG_C];
            const DIntT<R> c1 = interior_of<R, MULTI>(cf, itab, si[3], te.obj);
            R dny[6];
            for (int i = 0; i < 6; i++)
                dny[i] = cs - (te.px[i] * nsx + te.py[i] * nsy + te.pz[i] * nsz);
            const R nn = te.nx * nsx + te.ny * nsy + te.nz * nsz;
            const R gnr = -cf.n0r * nn, gni = -cf.n0i * nn;
            const double *ts = gt + TST_STRIDE * sl;
            R xp[3], xf[3];   // |sigma| psi, |sigma| phi at sigma's vertices, this column
#pragma unroll
            for (int b = 0; b < 3; b++) {
                const double *xv = xt + (int64_t)si[b] * 2 * COLS + col;
                xp[b] = ts[0] * xv[0];
                xf[b] = ts[0] * xv[COLS];
            }
            R gwr = 0, gwi = 0;
#pragma unroll 1
            for (int j = 0; j < 6; j++) {
                const int ju = __builtin_amdgcn_readfirstlane(j);
                const R yx = src[3 * j], yy = src[3 * j + 1], yz = src[3 * j + 2];
                const R w0 = wb_at<R>(3 * ju), w1 = wb_at<R>(3 * ju + 1), w2 = wb_at<R>(3 * ju + 2);
                const R dnx = te.c - (yx * te.nx + yy * te.ny + yz * te.nz);
                R c[8][3];
                point_sums<R, CK0, CK1>(yx, yy, yz, te.px, te.py, te.pz, dny, dead, cf, c1, etab, xtab,
                                        c);
                // weighted trial values at y_j
                const R p1 = w0 * xp[0] + w1 * xp[1] + w2 * xp[2];
                const R f1 = w0 * xf[0] + w1 * xf[1] + w2 * xf[2];
                const R p2 = rot * M::swap(p1), f2 = rot * M::swap(f1);
                const R wj = w0 + w1 + w2;
                gwr = fmaC(wj, fmaC(c1.irho, c[2][0] + c[2][1] + c[2][2], c[0][0] + c[0][1] + c[0][2]), gwr);
                gwi = fmaC(wj, fmaC(c1.irho, c[3][0] + c[3][1] + c[3][2], c[1][0] + c[1][1] + c[1][2]), gwi);
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    acc[0][a] = M::mma(fmaC(c1.rho, c[2][a], c[0][a]), p1, acc[0][a]);
                    acc[0][a] = M::mma(fmaC(c1.rho, c[3][a], c[1][a]), p2, acc[0][a]);
                    acc[0][a] = M::mma(-c[4][a], f1, acc[0][a]);
                    acc[0][a] = M::mma(-c[5][a], f2, acc[0][a]);
                    acc[1][a] = M::mma(c[6][a] * dnx, p1, acc[1][a]);
                    acc[1][a] = M::mma(c[7][a] * dnx, p2, acc[1][a]);
                    R nr = fmaC(c1.n10r, c[2][a], c[0][a]), ni = fmaC(c1.n10r, c[3][a], c[1][a]);
                    if (CK0 || CK1) {
                        nr = fmaC(-c1.n10i, c[3][a], nr);
                        ni = fmaC(c1.n10i, c[2][a], ni);
                    }
                    R dr = gnr * nr, di = gnr * ni;
                    if (CK0) {
                        dr = fmaC(-gni, ni, dr);
                        di = fmaC(gni, nr, di);
                    }
                    acc[1][a] = M::mma(dr, f1, acc[1][a]);
                    acc[1][a] = M::mma(di, f2, acc[1][a]);
                }
            }
            // curl part: curl_a . (|sigma| curl phi) times the curl weight
            asm volatile("" ::: "memory");   // (the curls stay in LDS)
            const double *cl = cu + (wave * BT_TAU + col) * 9;
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const R x1 = ts[1 + k] * xf[0] + ts[4 + k] * xf[1] + ts[7 + k] * xf[2];
                const R x2 = rot * M::swap(x1);
#pragma unroll
                for (int a = 0; a < 3; a++) {
                    acc[1][a] = M::mma(cl[3 * a + k] * gwr, x1, acc[1][a]);
                    acc[1][a] = M::mma(cl[3 * a + k] * gwi, x2, acc[1][a]);
                }
            }
        }
    }
    for (int v = 0; v < 4; v++) {
        const int t = tau0 + M::row(lane, v);
        if (t >= T) continue;
        double *o = part + ((int64_t)blockIdx.y * T + t) * 6 * COLS + col;
        for (int q = 0; q < 2; q++)
            for (int a = 0; a < 3; a++) o[(3 * q + a) * COLS] = acc[q][a][v];
    }
}

// y_r[i] = sum over the star of vertex i of scale |tau| times its rows
// (splits in order) + near-field CSR row times x.  BF_LANES lanes per (vertex,
// vector), the vectors of a vertex on adjacent groups.
constexpr int BF_LANES = 4;
__global__ __launch_bounds__(256) void batch_finish_kernel(
    const double *__restrict__ part, int nsplit, int T, const double *__restrict__ tst,
    const int32_t *__restrict__ star_ptr, const int32_t *__restrict__ star_idx,
    const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col,
    const double2 *__restrict__ nf, int64_t nnz, const double *__restrict__ xt, int64_t N, int nr,
    int cols, double scale, double2 *__restrict__ y) {
    const int half = cols / 2;
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    // lanes of one (vertex, vector) are `half` apart, so that a vertex's
    // vectors read neighbouring columns
    const int64_t i = id / (half * BF_LANES);
    const int rem = (int)(id - i * half * BF_LANES);
    const int sub = rem / half, r = rem - sub * half;
    double y1r = 0, y1i = 0, y2r = 0, y2i = 0;
    if (i < N && r < nr) {
        const int s0 = star_ptr[i], s1 = star_ptr[i + 1];
        for (int e = s0 + sub; e < s1; e += BF_LANES) {
            const int ta = star_idx[e], t = ta / 3, a = ta - 3 * t;
            double ar = 0, ai = 0, br = 0, bi = 0;
            for (int sp = 0; sp < nsplit; sp++) {
                const double2 *p = reinterpret_cast<const double2 *>(
                    part + (((int64_t)sp * T + t) * 6 + a) * cols) + r;
                const double2 u = p[0], w = p[3 * half];
                ar += u.x;
                ai += u.y;
                br += w.x;
                bi += w.y;
            }
            const double sc = scale * tst[(int64_t)TST_STRIDE * t];
            y1r += sc * ar;
            y1i += sc * ai;
            y2r += sc * br;
            y2i += sc * bi;
        }
        const double2 *C11 = nf, *C12 = nf + nnz, *C21 = nf + 2 * nnz, *C22 = nf + 3 * nnz;
        const int e1 = rowptr[i + 1];
        for (int e = rowptr[i] + sub; e < e1; e += BF_LANES) {
            const double2 *xv = reinterpret_cast<const double2 *>(xt) + (int64_t)col[e] * cols + r;
            const double2 p = xv[0], f = xv[half];
            const double2 a = C11[e], b = C12[e], c = C21[e], d = C22[e];
            y1r += a.x * p.x - a.y * p.y + b.x * f.x - b.y * f.y;
            y1i += a.x * p.y + a.y * p.x + b.x * f.y + b.y * f.x;
            y2r += c.x * p.x - c.y * p.y + d.x * f.x - d.y * f.y;
            y2i += c.x * p.y + c.y * p.x + d.x * f.y + d.y * f.x;
        }
    }
    // the lanes of one (vertex, vector), in lane order through LDS
    __shared__ double s[4][256];
    s[0][threadIdx.x] = y1r;
    s[1][threadIdx.x] = y1i;
    s[2][threadIdx.x] = y2r;
    s[3][threadIdx.x] = y2i;
    __syncthreads();   // (256 is a multiple of half * BF_LANES)
    if (sub != 0 || i >= N || r >= nr) return;
    for (int k = 1; k < BF_LANES; k++) {
        const int o = threadIdx.x + k * half;
        y1r += s[0][o];
        y1i += s[1][o];
        y2r += s[2][o];
        y2i += s[3][o];
    }
    y[(int64_t)r * 2 * N + i] = make_double2(y1r, y1i);
    y[(int64_t)r * 2 * N + N + i] = make_double2(y2r, y2i);
}

// Launch variant: complex k_0 alone takes the variant of two complex
// wavenumbers (code of entries::variant_code: 4 ck0 + 2 ck1 + several objects).
template <class R> using BatchFn = void (*)(const R *, const double *, const int32_t *,
                                            const int32_t *, int, int, DCoefT<R>,
                                            const DIntT<R> *, const double *, double *);
template <class R, int C, bool A, bool B, bool MU> BatchFn<R> variant_fn() {
    if constexpr (std::is_same<R, float>::value) return batch_kernel<A, B, MU, C>;
    else return batch64_kernel<A, B, MU>;
}
template <class R, int C> BatchFn<R> batch_fn(int code) {
    const bool multi = code & 1;
    if (code & 4) return multi ? variant_fn<R, C, true, true, true>() : variant_fn<R, C, true, true, false>();
    if (code & 2) return multi ? variant_fn<R, C, false, true, true>() : variant_fn<R, C, false, true, false>();
    return multi ? variant_fn<R, C, false, false, true>() : variant_fn<R, C, false, false, false>();
}

// Workgroups of a variant resident on the device (cached per device and kernel).
int batch_slots(const void *kern) {
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, int> cache;
    int dev = 0;
    BEM_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> gd(mu);
    auto it = cache.find({dev, kern});
    if (it != cache.end()) return it->second;
    int cus = 0, per = 0;
    BEM_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    BEM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, BT_THREADS, 0));
    return cache[{dev, kern}] = std::max(1, cus * per);
}

template <class R, int C>
void batch_plan(const bem_mesh *m, int code, int *nsplit, int *len) {
    const int W = BT_THREADS / 64 / C, T = (int)m->T;
    batch_split(T, (T + W * BT_TAU - 1) / (W * BT_TAU), batch_slots((const void *)batch_fn<R, C>(code)),
                (int64_t)T * 6 * BT_COLS * C * (int64_t)sizeof(double), nsplit, len);
}

template <class R, int C>
void batch_apply(bem_mesh *m, const NearOperator &nf, double2 k0, const double2 *x, double2 *y,
                 int nr, hipStream_t s) {
    constexpr bool F32 = std::is_same<R, float>::value;
    constexpr int W = BT_THREADS / 64 / C, cols = BT_COLS * C;
    const int T = (int)m->T, code = entries::variant_code(m, k0, nf);
    const int64_t N = m->N;
    int nsplit = 1, len = T;
    batch_plan<R, C>(m, code, &nsplit, &len);
    const size_t np = (size_t)nsplit * T * 6 * cols, nx = (size_t)N * 2 * cols;
    if (m->batch_part.n < np + nx) m->batch_part.alloc(np + nx);
    double *part = m->batch_part.p, *xt = part + np;
    auto &itab = [&]() -> auto & {
        if constexpr (F32) return nf.dtab32;
        else return nf.dtab64;
    }();
    if (m->nobj > 1 && !itab.p) {   // per-object interior parts
        constexpr size_t K = sizeof(DIntT<R>) / sizeof(R);
        std::vector<R> h((size_t)m->nobj * K);
        for (int o = 0; o < m->nobj; o++) {
            const DIntT<R> c = entries::make_dint<R>(k0, nf.k1o[o], nf.rhoo[o], nf.s1);
            std::copy((const R *)&c, (const R *)&c + K, h.data() + (size_t)o * K);
        }
        itab.upload(h);
    }
    hipLaunchKernelGGL(batch_gather_kernel, dim3((unsigned)((N * cols + 255) / 256)), dim3(256), 0, s,
                       x, nr, N, cols, xt);
    BEM_LAUNCH_CHECK();
    const R *geo;
    if constexpr (F32) geo = m->geo32.p;
    else geo = m->geo64.p;
    {
        Timer tm(F32 ? "farfield_fp32_multi" : "farfield_fp64_multi", s);
        hipLaunchKernelGGL((batch_fn<R, C>(code)), dim3((T + W * BT_TAU - 1) / (W * BT_TAU), nsplit),
                           dim3(BT_THREADS), 0, s, geo, m->tst.p, m->tobj_d.p, m->tri_d.p, T, len,
                           entries::make_dcoef<R>(k0, nf), (const DIntT<R> *)itab.p, xt, part);
        BEM_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(batch_finish_kernel, dim3((unsigned)((N * (cols / 2) * BF_LANES + 255) / 256)),
                       dim3(256), 0, s, part, nsplit, T, m->tst.p, m->star_ptr.p, m->star_idx.p,
                       m->nf_rowptr.p, m->nf_col.p, (const double2 *)nf.vals.p, m->nf_nnz, xt, N, nr,
                       cols, INV4PI / bt_scale<R>(), y);
    BEM_LAUNCH_CHECK();
}

template <class R, int C> int64_t batch_bytes(const bem_mesh *m, int code) {
    int nsplit = 1, len = 0;
    batch_plan<R, C>(m, code, &nsplit, &len);
    return ((int64_t)nsplit * m->T * 6 + m->N * 2) * BT_COLS * C * (int64_t)sizeof(double);
}

}   // namespace

int farfield_mx_max(int precision) { return precision == BEM_FP32 ? 32 : 8; }

void farfield_mx_apply(bem_mesh *m, const NearOperator &nf, double2 k0, const double2 *x, double2 *y,
                       int nr, int precision, hipStream_t s) {
    if (precision != BEM_FP32) batch_apply<double, 1>(m, nf, k0, x, y, nr, s);
    else if (nr <= 8) batch_apply<float, 1>(m, nf, k0, x, y, nr, s);
    else if (nr <= 16) batch_apply<float, 2>(m, nf, k0, x, y, nr, s);
    else batch_apply<float, 4>(m, nf, k0, x, y, nr, s);
}

int64_t farfield_mx_bytes(const bem_mesh *m, int precision, double2 k0, double2 k1, int R) {
    const int code = (k0.y != 0 ? 4 : 0) | (k1.y != 0 ? 2 : 0) | (m->nobj > 1 ? 1 : 0);
    if (precision != BEM_FP32) return batch_bytes<double, 1>(m, code);
    int64_t b = batch_bytes<float, 1>(m, code);
    if (R > 8) b = std::max(b, batch_bytes<float, 2>(m, code));
    if (R > 16) b = std::max(b, batch_bytes<float, 4>(m, code));
    return b;
}

}   // namespace bem
