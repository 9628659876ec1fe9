// Near-field operator of the permuted PMCHWT matvec (FP64, built once per
// (k_ext, k_int, rho, s1) and kept on the device).
//
// For every ordered triangle pair (tau, sigma) sharing at least one vertex the
// four combined 3x3 blocks
//   B11 = V_0 + rho V_1,  B12 = -(K_0 + K_1),  B21 = K'_0 + K'_1,
//   B22 = D_0 + D_1 / rho          (Sec. 2.7; operators of Sec. 2.2)
// are integrated with the singular rule of the pair's class (coincident,
// common edge, common vertex); the matrix-free pair kernel skips exactly these
// pairs.  The blocks are summed into a vertex-by-vertex CSR matrix in a fixed
// order.  The interior terms of a pair use its object's material.  With s1 =
// -1 the interior terms enter with the opposite sign and the
// coincident pairs add the local P1 mass matrix |tau| (1 + delta_ab) / 12 to
// B12 and B21: the Mueller operator I + A_0 - A^_1 of Sec. 2.2 on the
// permuted unknowns, whose identity pairs each trace row with its own trace.
#include <algorithm>
#include <cmath>

#include "bem_internal.h"
#include "fp64_math.h"

namespace bem {

namespace {

struct NearCoef {
    double2 k0;
    double s1;   // +1 PMCHWT, -1 Mueller
};

// Wavenumber in the units of the tables: phase in 256ths of a revolution per
// length, decay in powers of two per length (0: none).
struct NearK {
    double u, d;
};
__device__ inline NearK near_k(double2 k) {
    return NearK{k.x * (PHASE64 / 6.283185307179586476925286766559),
                 k.y * -1.4426950408889634073599246810019};
}

// e^{i k r} / (4 pi r) and (i k r - 1) e^{i k r} / (4 pi r^3), ir = 1 / r
__device__ __forceinline__ void green(double2 k, NearK nk, double r, double ir,
                                      const double2 *etab, const double *dtab, double2 &G,
                                      double2 &F) {
    double s, c;
    sincos_256(nk.u * r, s, c, etab);
    double mag = 0.079577471545947667884441881686257 * ir;
    if (nk.d < 0.0) mag *= decay64(nk.d * r, dtab);
    else if (nk.d > 0.0) mag *= ::exp2(nk.d * r);
    G = make_double2(c * mag, s * mag);
    const double ir2 = ir * ir;
    const double tx = (-1.0 - k.y * r) * ir2, ty = k.x * ir;   // (i k r - 1) / r^2
    F = make_double2(G.x * tx - G.y * ty, G.x * ty + G.y * tx);
}

constexpr int NACC = 74;   // 4 x 9 complex blocks (B22 normal part) + 1 complex

// One step of the wave's sums: of the N values that a lane holds, lanes with bit
// O of their index clear keep the first ceil(N / 2), the others the rest (and a
// zero when N is odd), each added to its partner's.  Six steps leave the sums
// of all lanes, one or two to a lane.
template <int N, int O>
__device__ __forceinline__ void near_fold(double *acc, int lane) {
    constexpr int H = (N + 1) / 2;
    const bool up = lane & O;
#pragma unroll
    for (int i = 0; i < H; i++) {
        const double lo = acc[i], hi = i + H < N ? acc[i + H] : 0.0;
        const double keep = up ? hi : lo, give = up ? lo : hi;
        acc[i] = keep + __shfl_xor(give, O, 64);
    }
    if constexpr (O > 1) near_fold<H, O / 2>(acc, lane);
}
// What the folds leave: NEAR_LEFT values to a lane, value v being the sum with
// index near_base(lane) + v where v < near_valid(lane), a fill beyond.
constexpr int near_left(int n, int o) { return o ? near_left((n + 1) / 2, o / 2) : n; }
constexpr int NEAR_LEFT = near_left(NACC, 32);
constexpr int near_base(int lane, int n = NACC, int o = 32) {
    return o ? (lane & o ? (n + 1) / 2 : 0) + near_base(lane, (n + 1) / 2, o / 2) : 0;
}
constexpr int near_valid(int lane, int n = NACC, int o = 32, int valid = NACC) {
    if (!o) return valid;
    const int h = (n + 1) / 2, left = lane & o ? valid - h : (valid < h ? valid : h);
    return near_valid(lane, h, o / 2, left > 0 ? left : 0);
}
constexpr int near_lane(int index) {   // the lane that is left with a sum
    for (int l = 0; l < 64; l++)
        if (index >= near_base(l) && index < near_base(l) + near_valid(l)) return l;
    return -1;
}

// One wave per ordered pair, NEAR_WAVES waves a workgroup, `per` pairs a wave.
// Bound by the FP64 units: 1536, 1024 or 512 points a pair (coincident, edge,
// vertex), two kernels and 74 sums each.  Points keep the order of their rule's
// vertices (the pair's permutation is applied to the two triangles' vertices
// and to the stored block); the phases come from the table of the pair kernels
// and the sums of a wave are folded, 76 exchanges instead of 444.
// 20 480 triangles: 6.2 -> 2.1 ms, 320 triangles: 135 -> 62 us.
constexpr int NEAR_WAVES = 4;
__global__ __launch_bounds__(64 * NEAR_WAVES, 2) void near_pairs_kernel(
    const int32_t *__restrict__ pairs, int64_t n_pairs, int per, const double *__restrict__ P,
    const int32_t *__restrict__ tri, const double *__restrict__ tst,
    const double *__restrict__ geo, const double *__restrict__ tab, int off0, int off1,
    int off2, int off3, NearCoef cf, const int32_t *__restrict__ tobj,
    const double *__restrict__ omat, double2 *__restrict__ blocks) {
    __shared__ double2 etab[256];
    __shared__ double dtab[DECAY_TAB];
    phase_table(etab);
    decay_table(dtab);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const double k0sq_r = cf.k0.x * cf.k0.x - cf.k0.y * cf.k0.y, k0sq_i = 2 * cf.k0.x * cf.k0.y;
    const NearK nk0 = near_k(cf.k0);
    for (int it = 0; it < per; it++) {
        const int64_t p = ((int64_t)blockIdx.x * per + it) * NEAR_WAVES + wave;
        if (p >= n_pairs) return;
        const int t = pairs[4 * p], s = pairs[4 * p + 1], cls = pairs[4 * p + 2],
                  perm = pairs[4 * p + 3];
        double vt[3][3], vs[3][3];   // in the order of the rule
        for (int r = 0; r < 3; r++) {
            const int a = tri[3 * t + ((perm >> (2 * r)) & 3)];
            const int b = tri[3 * s + ((perm >> (6 + 2 * r)) & 3)];
            for (int c = 0; c < 3; c++) {
                vt[r][c] = P[3 * a + c];
                vs[r][c] = P[3 * b + c];
            }
        }
        const double at = tst[TST_STRIDE * t], as = tst[TST_STRIDE * s];
        const double *nt = geo + GEO_STRIDE * t + 18, *ns = geo + GEO_STRIDE * s + 18;
        const double nn = nt[0] * ns[0] + nt[1] * ns[1] + nt[2] * ns[2];

        const int rb = cls == 0 ? off0 : (cls == 1 ? off1 : off2);
        const int re = cls == 0 ? off1 : (cls == 1 ? off2 : off3);
        const int nss = re - rb;

        double acc[NACC];
#pragma unroll
        for (int i = 0; i < NACC; i++) acc[i] = 0.0;
        // interior material of the pair's object (a pair sharing a vertex lies
        // within one object): omat[object] = (Re k_1, Im k_1, rho)
        const int ob = tobj[t];
        const double2 k1 = make_double2(omat[3 * ob], omat[3 * ob + 1]);
        const NearK nk1 = near_k(k1);
        const double rho = omat[3 * ob + 2];
        const double k1sq_r = cf.s1 * (k1.x * k1.x - k1.y * k1.y) / rho,
                     k1sq_i = cf.s1 * 2 * k1.x * k1.y / rho;
        const double rho1 = cf.s1 * rho, irho1 = cf.s1 / rho;

        for (int q = lane; q < nss; q += 64) {
            const double *row = tab + 5 * (int64_t)(rb + q);
            const double lx[3] = {1.0 - row[0], row[0] - row[1], row[1]};
            const double ly[3] = {1.0 - row[2], row[2] - row[3], row[3]};
            const double w = 4.0 * at * as * row[4];
            double d[3];
#pragma unroll
            for (int c = 0; c < 3; c++) {
                double xc = lx[0] * vt[0][c] + lx[1] * vt[1][c] + lx[2] * vt[2][c];
                double yc = ly[0] * vs[0][c] + ly[1] * vs[1][c] + ly[2] * vs[2][c];
                d[c] = xc - yc;   // x - y
            }
            const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
            const double ir = rsqrt64(r2), r = r2 * ir;
            double2 G0, F0, G1, F1;
            green(cf.k0, nk0, r, ir, etab, dtab, G0, F0);
            green(k1, nk1, r, ir, etab, dtab, G1, F1);
            double2 GV = make_double2(G0.x + rho1 * G1.x, G0.y + rho1 * G1.y);
            double2 GW = make_double2(G0.x + irho1 * G1.x, G0.y + irho1 * G1.y);
            double2 GN =
                make_double2(k0sq_r * G0.x - k0sq_i * G0.y + k1sq_r * G1.x - k1sq_i * G1.y,
                             k0sq_r * G0.y + k0sq_i * G0.x + k1sq_r * G1.y + k1sq_i * G1.x);
            double2 FK = make_double2(F0.x + cf.s1 * F1.x, F0.y + cf.s1 * F1.y);
            const double dny = d[0] * ns[0] + d[1] * ns[1] + d[2] * ns[2];   // (x-y).n_y
            const double dnx = d[0] * nt[0] + d[1] * nt[1] + d[2] * nt[2];   // (x-y).n_x
            const double2 FY = make_double2(FK.x * dny, FK.y * dny);
            const double2 FX = make_double2(FK.x * dnx, FK.y * dnx);
#pragma unroll
            for (int a = 0; a < 3; a++) {
                const double wa = w * lx[a];
#pragma unroll
                for (int b = 0; b < 3; b++) {
                    const double pp = wa * ly[b];
                    const int e = 2 * (3 * a + b);
                    acc[e] += GV.x * pp;
                    acc[e + 1] += GV.y * pp;
                    acc[18 + e] += FY.x * pp;
                    acc[18 + e + 1] += FY.y * pp;
                    acc[36 + e] += FX.x * pp;
                    acc[36 + e + 1] += FX.y * pp;
                    acc[54 + e] += GN.x * pp;
                    acc[54 + e + 1] += GN.y * pp;
                }
            }
            acc[72] += GW.x * w;
            acc[73] += GW.y * w;
        }
        near_fold<NACC, 32>(acc, lane);   // fixed order
        constexpr int l72 = near_lane(72), l73 = near_lane(73);
        static_assert(l72 >= 0 && l73 >= 0, "every sum is left with a lane");
        const double gwr = __shfl(acc[72 - near_base(l72)], l72, 64);
        const double gwi = __shfl(acc[73 - near_base(l73)], l73, 64);
        const int base = near_base(lane), nv = near_valid(lane);
#pragma unroll
        for (int v = 0; v < NEAR_LEFT; v++) {
            const int i = base + v;
            if (v >= nv || i >= 72) continue;
            const int blk = i / 18, ab = (i % 18) >> 1, im = i & 1;
            const int a = (perm >> (2 * (ab / 3))) & 3, b = (perm >> (6 + 2 * (ab % 3))) & 3;
            double x = acc[v];
            if (blk == 3) {
                const double *ca = tst + TST_STRIDE * t + 1 + 3 * a;
                const double *cb = tst + TST_STRIDE * s + 1 + 3 * b;
                const double cc = ca[0] * cb[0] + ca[1] * cb[1] + ca[2] * cb[2];
                x = cc * (im ? gwi : gwr) - nn * x;
            }
            if (im == 0 && cf.s1 < 0 && t == s && (blk == 1 || blk == 2))
                x += at * (a == b ? 2.0 : 1.0) / 12.0;   // Mueller identity: P1 mass
            ((double *)blocks)[2 * (36 * p + 9 * blk + 3 * a + b) + im] = x;
        }
    }
}


// CSR values: C[blk][e] = sum over the entry's contributions (fixed order).
__global__ __launch_bounds__(256) void near_csr_kernel(
    const int32_t *__restrict__ cptr, const int32_t *__restrict__ contrib, int64_t nnz,
    const double2 *__restrict__ blocks, double2 *__restrict__ vals) {
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nnz) return;
    double2 acc[4];
    for (int b = 0; b < 4; b++) acc[b] = make_double2(0.0, 0.0);
    for (int c = cptr[e]; c < cptr[e + 1]; c++) {
        int code = contrib[c];
        int64_t p = code / 9;
        int ab = code - 9 * (int)p;
        for (int b = 0; b < 4; b++) {
            double2 v = blocks[36 * p + 9 * b + ab];
            acc[b].x += v.x;
            acc[b].y += v.y;
        }
    }
    for (int b = 0; b < 4; b++) vals[b * nnz + e] = acc[b];
}

}   // namespace

NearKey near_key(const bem_mesh *m, double2 k0, double2 k1, double rho, int s1,
                 const ObjMaterials *om) {
    s1 = s1 < 0 ? -1 : 1;
    NearKey key{k0.x, k0.y, k1.x, k1.y, rho, s1, {}};
    if (om) {
        bool same = true;
        for (int o = 1; o < m->nobj; o++)
            same = same && om->k[o].x == om->k[0].x && om->k[o].y == om->k[0].y &&
                   om->rho[o] == om->rho[0];
        key.k1r = om->k[0].x;
        key.k1i = om->k[0].y;
        key.rho = om->rho[0];
        if (!same)
            for (int o = 0; o < m->nobj; o++) {
                key.om.push_back(om->k[o].x);
                key.om.push_back(om->k[o].y);
                key.om.push_back(om->rho[o]);
            }
    }
    return key;
}

std::unique_ptr<NearOperator> nearfield_build(bem_mesh *m, double2 k0, double2 k1,
                                              double rho, hipStream_t s, int s1,
                                              const ObjMaterials *om) {
    auto op = std::make_unique<NearOperator>();
    op->s1 = s1 < 0 ? -1 : 1;
    op->k1o.assign(m->nobj, k1);
    op->rhoo.assign(m->nobj, rho);
    if (om) {
        op->k1o = om->k;
        op->rhoo = om->rho;
    }
    std::vector<double> mat(3 * (size_t)m->nobj);
    bool complex_k = false;
    op->k1_plan = op->k1o[0];
    for (int o = 0; o < m->nobj; o++) {
        mat[3 * o] = op->k1o[o].x;
        mat[3 * o + 1] = op->k1o[o].y;
        mat[3 * o + 2] = op->rhoo[o];
        complex_k = complex_k || op->k1o[o].y != 0.0;
        if (std::fabs(op->k1o[o].x) > std::fabs(op->k1_plan.x)) op->k1_plan = op->k1o[o];
    }
    if (complex_k && op->k1_plan.y == 0.0) op->k1_plan.y = 1.0;   // any complex k_m: complex variant
    op->vals.alloc(4 * (size_t)m->nf_nnz * 2);
    DevBuf<double> Pd, matd;
    std::vector<double> Ph(m->P);
    Pd.upload(Ph);
    matd.upload(mat);
    DevBuf<double2> blocks(36 * (size_t)m->n_near);
    NearCoef cf{k0, (double)op->s1};
    {
        Timer tm("nearfield_build", s);
        // up to 4 pairs a wave (the tables are filled once per workgroup), fewer
        // while that leaves the 256 compute units less than 8 workgroups each
        const int per = (int)std::min<int64_t>(
            4, std::max<int64_t>(1, m->n_near / (256 * 8 * NEAR_WAVES)));
        const int64_t wgs = (m->n_near + per * NEAR_WAVES - 1) / (per * NEAR_WAVES);
        hipLaunchKernelGGL(near_pairs_kernel, dim3((unsigned)wgs), dim3(64 * NEAR_WAVES), 0, s,
                           m->near_pairs.p, m->n_near, per, Pd.p, m->tri_d.p, m->tst.p,
                           m->geo64.p, m->ss_tab.p, m->ss_off[0], m->ss_off[1],
                           m->ss_off[2], m->ss_off[3], cf, m->tobj_d.p, matd.p, blocks.p);
        BEM_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(near_csr_kernel, dim3((unsigned)((m->nf_nnz + 255) / 256)), dim3(256),
                       0, s, m->nf_cptr.p, m->nf_contrib.p, m->nf_nnz, blocks.p,
                       (double2 *)op->vals.p);
    BEM_LAUNCH_CHECK();
    BEM_HIP(hipStreamSynchronize(s));
    return op;
}

const NearOperator &nearfield_get(bem_mesh *m, double2 k0, double2 k1, double rho,
                                  hipStream_t s, int s1, const ObjMaterials *om) {
    const NearKey key = near_key(m, k0, k1, rho, s1, om);
    auto it = m->near_cache.find(key);
    if (it != m->near_cache.end()) return *it->second;
    if (m->near_cache.size() >= 8) m->near_cache.erase(m->near_cache.begin());
    auto op = nearfield_build(m, k0, make_double2(key.k1r, key.k1i), key.rho, s, key.s1,
                              key.om.empty() ? nullptr : om);
    auto &ref = *op;
    m->near_cache.emplace(key, std::move(op));
    return ref;
}

}   // namespace bem
