// Total field at points off the surface (FP64), from a boundary solution
// x = [psi; phi] of the plane wave u_inc = exp(i k_ext d.p).
//
// Representation formulas of Sec. 2.2 with the surface potentials of the
// total field (psi~+ = -psi, phi~+ = -phi outside; psi~- = rho psi,
// phi~- = phi inside, the interior Neumann trace being rho times the
// exterior one):
//   outside every object:  u = u_inc + sum over all triangles of
//       int [ -G_0 psi + (n_y . grad_y G_0) phi ] dy
//   inside object m:       u = int over object m of
//       [ rho_m G_m psi - (n_y . grad_y G_m) phi ] dy
// (k_m, rho_m the object's interior material)
// with n_y . grad_y G(p, y) = ((y - p) . n_y) G (i k r - 1) / r^2; the
// factor (y - p) . n_y = c_sigma - p . n_sigma is constant on a flat
// triangle.  6-point rule per triangle (the sources w |sigma| psi_h and
// w |sigma| phi_h at the rule's points are formed once per call).
//
// Regions: point p is inside object m when the solid angle of m's closed
// surface at p is 4 pi (0 outside); per flat triangle with vertices a, b, c
// relative to p (Van Oosterom and Strackee, 1983):
//   tan(Omega / 2) = a.(b x c) / (|a||b||c| + (a.b)|c| + (a.c)|b| + (b.c)|a|).
// With disjoint objects one pass gives both the total solid angle and, from
// the object-weighted sum, the object that encloses the point; points outside
// every object's bounding box need none.  All sums are
// accumulated in a fixed order (split partials added in split order).
#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <type_traits>

#include "bem_internal.h"
#include "fp64_math.h"

namespace bem {

namespace {

constexpr double DUN_A1 = 0.44594849091596488631832925388305;
constexpr double DUN_W1 = 0.22338158967801146569500700843312;
constexpr double DUN_A2 = 0.091576213509770743459571463402202;
constexpr double DUN_W2 = 0.10995174365532186763832632490021;
__device__ constexpr double qw(int i) { return i < 3 ? DUN_W1 : DUN_W2; }
__device__ inline double qb(int i, int a) {
    const double al = i < 3 ? DUN_A1 : DUN_A2;
    return (a == i % 3) ? (1.0 - 2.0 * al) : al;
}

constexpr double INV4PI = 0.079577471545947667884441881686257;
constexpr double TWO_PI = 6.283185307179586476925286766559;
constexpr double INV2PI = 0.15915494309189533576888376337251;

// per triangle: the 6 rule points, w |sigma| psi_h and w |sigma| phi_h there
constexpr int SRC_STRIDE = 42;   // [0,18) points, [18,30) s_psi, [30,42) s_phi
constexpr int FT = 64;           // triangles per LDS tile
constexpr int FS = 48;           // tile doubles per triangle: SRC + normal, c, object

__global__ __launch_bounds__(256) void field_sources_kernel(
    const double *__restrict__ P, const int32_t *__restrict__ tri,
    const double *__restrict__ tst, const double2 *__restrict__ x, int64_t N, int T,
    double *__restrict__ src) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    double v[3][3];
    double2 ps[3], ph[3];
    for (int b = 0; b < 3; b++) {
        const int vi = tri[3 * t + b];
        for (int c = 0; c < 3; c++) v[b][c] = P[3 * vi + c];
        ps[b] = x[vi];
        ph[b] = x[N + vi];
    }
    const double area = tst[TST_STRIDE * t];
    double *o = src + (int64_t)SRC_STRIDE * t;
    for (int q = 0; q < 6; q++) {
        const double wa = qw(q) * area;
        double pr = 0, pi = 0, fr = 0, fi = 0;
        for (int b = 0; b < 3; b++) {
            const double l = qb(q, b);
            pr += l * ps[b].x;
            pi += l * ps[b].y;
            fr += l * ph[b].x;
            fi += l * ph[b].y;
        }
        for (int c = 0; c < 3; c++)
            o[3 * q + c] = qb(q, 0) * v[0][c] + qb(q, 1) * v[1][c] + qb(q, 2) * v[2][c];
        o[18 + 2 * q] = wa * pr;
        o[18 + 2 * q + 1] = wa * pi;
        o[30 + 2 * q] = wa * fr;
        o[30 + 2 * q + 1] = wa * fi;
    }
}

// ------------------------------------------------------------------ regions
// A point outside the bounding box of every object is outside all of them; the
// others are listed (in any order: their regions do not depend on each other) and
// their solid angles summed over ranges of the triangles.
constexpr int WS = 10;          // winding tile doubles per triangle: 3 vertices, object
constexpr int64_t FIELD_POINTS = 1 << 22;   // points per pass (bounds the workspace)
constexpr int WIND_GROUPS = 2048;   // workgroups of the solid-angle sums

__global__ __launch_bounds__(64) void count_zero_kernel(int32_t *count) { *count = 0; }

__global__ __launch_bounds__(256) void region_box_kernel(const double *__restrict__ pts, int64_t n,
                                                         const double *__restrict__ box, int nobj,
                                                         int32_t *__restrict__ region,
                                                         int32_t *__restrict__ list,
                                                         int32_t *__restrict__ count) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    const double x = pts[3 * p], y = pts[3 * p + 1], z = pts[3 * p + 2];
    bool in = false;
    for (int o = 0; o < nobj; o++) {
        const double *b = box + 6 * o;
        in = in || (x >= b[0] && y >= b[1] && z >= b[2] && x <= b[3] && y <= b[4] && z <= b[5]);
    }
    region[p] = 0;
    if (in) list[atomicAdd(count, 1)] = (int32_t)p;
}

// Triangle ranges for `count` listed points (the same for every kernel): about
// WIND_GROUPS workgroups in all.
__device__ __forceinline__ int wind_splits(int count, int max_split) {
    const int pb = (count + 255) / 256;
    return pb == 0 ? 0 : min(max_split, max(1, WIND_GROUPS / pb));
}

// Solid angles of the triangles of a range at the listed points:
// [0] sum Omega_t, [1] sum Omega_t (object_t + 1).  Omega_t / 2 is the argument of
// den + i num, so a sum of arguments is the argument of a product plus 2 pi for
// every time the product passes the negative real axis: one atan2 per range and
// object (and per change of object) instead of one per triangle, and 1/sqrt for
// the three norms (1.33 ms for 10 201 points and 20 480 triangles with sqrt and
// atan2 each, all points).
__global__ __launch_bounds__(256) void winding_kernel(
    const double *__restrict__ P, const int32_t *__restrict__ tri,
    const int32_t *__restrict__ tobj, int T, const double *__restrict__ pts,
    const int32_t *__restrict__ list, const int32_t *__restrict__ countp, int max_split,
    double *__restrict__ part) {
    __shared__ double tile[FT * WS];
    const int count = *countp, nsplit = wind_splits(count, max_split);
    const int pb = (count + 255) / 256, len = nsplit > 0 ? (T + nsplit - 1) / nsplit : 0;
    // unit: 256 listed points and one range (uniform over the workgroup)
    for (int unit = blockIdx.x; unit < pb * nsplit; unit += gridDim.x) {
        const int split = unit / pb, idx0 = (unit - split * pb) * 256 + threadIdx.x;
        const int64_t pp = list[min(idx0, count - 1)];
        const double px = pts[3 * pp], py = pts[3 * pp + 1], pz = pts[3 * pp + 2];
        const int t0 = split * len, t1 = min(T, t0 + len);
        struct Sums {
            double om = 0.0, ow = 0.0;     // closed sums
            double zr = 1.0, zi = 0.0;     // running product
            int turns = 0, obj = -1;
            bool lost = false;             // a product that was closed was zero
        } s;
        auto close = [&]() {   // the product's argument into the sums
            const double o = 2.0 * (atan2(s.zi, s.zr) + TWO_PI * s.turns);
            s.om += o;
            s.ow += o * (s.obj + 1);
            s.lost = s.lost || (s.zr == 0 && s.zi == 0);
            s.zr = 1.0;
            s.zi = 0.0;
            s.turns = 0;
        };
        // the triangles of the staged tile; `skip`: leaves out factors that are zero
        auto sweep = [&](int cnt, auto skip) {
            for (int sl = 0; sl < cnt; sl++) {
                const double *v = tile + sl * WS;
                if ((int)v[9] != s.obj) {   // uniform
                    if (s.obj >= 0) close();
                    s.obj = (int)v[9];
                }
                const double a0 = v[0] - px, a1 = v[1] - py, a2 = v[2] - pz;
                const double b0 = v[3] - px, b1 = v[4] - py, b2 = v[5] - pz;
                const double c0 = v[6] - px, c1 = v[7] - py, c2 = v[8] - pz;
                const double aa = a0 * a0 + a1 * a1 + a2 * a2, bb = b0 * b0 + b1 * b1 + b2 * b2,
                             cc = c0 * c0 + c1 * c1 + c2 * c2;
                // (a point at a vertex: the norm is 0, as are num and den)
                const double ra = aa > 0 ? rsqrt64(aa) : 0.0, rb = bb > 0 ? rsqrt64(bb) : 0.0,
                             rc = cc > 0 ? rsqrt64(cc) : 0.0;
                const double la = aa * ra, lb = bb * rb, lc = cc * rc;
                const double num = a0 * (b1 * c2 - b2 * c1) + a1 * (b2 * c0 - b0 * c2) +
                                   a2 * (b0 * c1 - b1 * c0);
                const double den = la * lb * lc + (a0 * b0 + a1 * b1 + a2 * b2) * lc +
                                   (a0 * c0 + a1 * c1 + a2 * c2) * lb +
                                   (b0 * c0 + b1 * c1 + b2 * c2) * la;
                // over 4 |a||b||c|: the modulus is at most 1, near 1 for small triangles
                const double sc = 0.25 * ra * rb * rc;
                const double nr = den * sc, ni = num * sc;
                if (skip.value && nr == 0 && ni == 0) continue;
                const double wr = s.zr * nr - s.zi * ni, wi = s.zr * ni + s.zi * nr;
                // past pi, or past -pi.  The sign bit is the side that atan2 takes an
                // argument of a zero imaginary part on (pi or -pi, 0 or -0)
                const bool sz = __builtin_signbit(s.zi), sn = __builtin_signbit(ni),
                           sw = __builtin_signbit(wi);
                if (sz == sn && sn != sw) s.turns += sw ? 1 : -1;
                s.zr = wr;
                s.zi = wi;
            }
        };
        for (int base = t0; base < t1; base += FT) {
            const int cnt = min(FT, t1 - base);
            __syncthreads();
            for (int idx = threadIdx.x; idx < cnt * WS; idx += 256) {
                const int sl = idx / WS, f = idx - sl * WS;
                const int64_t t = base + sl;
                tile[idx] = f < 9 ? P[3 * tri[3 * t + f / 3] + f % 3] : (double)tobj[t];
            }
            __syncthreads();
            const Sums before = s;
            sweep(cnt, std::false_type{});
            // a product of zero: the point is at a vertex or on an edge of some triangle,
            // which has no angle of its own; the tile again without such triangles
            if (s.lost || (s.zr == 0 && s.zi == 0)) {
                s = before;
                sweep(cnt, std::true_type{});
                s.lost = false;
            }
            // keep the product's size (its argument stays)
            const double big = fmax(fabs(s.zr), fabs(s.zi));
            const double inv = big > 0 ? 1.0 / big : 1.0;
            s.zr *= inv;
            s.zi *= inv;
        }
        if (s.obj >= 0) close();
        if (idx0 < count) {
            part[2 * ((int64_t)split * count + idx0)] = s.om;
            part[2 * ((int64_t)split * count + idx0) + 1] = s.ow;
        }
    }
}

// Closed disjoint surfaces: the total solid angle is 4 pi inside one object
// and 0 outside all; inside object m the object-weighted sum is (m + 1) times
// the total, since every other surface subtends 0.
__global__ __launch_bounds__(256) void region_kernel(const double *__restrict__ part,
                                                     const int32_t *__restrict__ list,
                                                     const int32_t *__restrict__ countp, int max_split,
                                                     int nobj, int32_t *__restrict__ region) {
    const int count = *countp, nsplit = wind_splits(count, max_split);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    double om = 0.0, ow = 0.0;
#pragma unroll 4
    for (int sp = 0; sp < nsplit; sp++) {
        om += part[2 * ((int64_t)sp * count + i)];
        ow += part[2 * ((int64_t)sp * count + i) + 1];
    }
    int r = 0;
    if (fabs(om) > TWO_PI) r = min(nobj, max(1, (int)lround(ow / om)));
    region[list[i]] = r;
}

// ------------------------------------------------------------------- layers
// partial single- and double-layer sums of the split's triangles at each
// point, with the wavenumber and the triangles of the point's region.  Bound by
// FP64 VALU issue: about 50 instructions per (point, trial point) with the
// functions of fp64_math.h and F = (i k E - G) / r^2; the complex variant (LOSSY)
// is a kernel of its own, a branch per pair otherwise (96 instructions, 3.20 ms for
// 10 201 points and 20 480 triangles).
template <bool LOSSY>
__global__ __launch_bounds__(256) void field_kernel(
    const double *__restrict__ src, const double *__restrict__ geo,
    const int32_t *__restrict__ tobj, int T, int split_len, const double *__restrict__ pts,
    const int32_t *__restrict__ region, int64_t n, double2 k0, const double *__restrict__ omat,
    double *__restrict__ part) {
    __shared__ double tile[FT * FS];
    __shared__ double2 etab[256];
    __shared__ double xtab[DECAY_TAB];
    phase_table(etab);
    if (LOSSY) decay_table(xtab);
    // (the first tile's barrier orders these writes before any read)
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t pp = p < n ? p : 0;
    const double px = pts[3 * pp], py = pts[3 * pp + 1], pz = pts[3 * pp + 2];
    const int reg = region[pp];
    const bool ext = reg == 0;
    // interior material of the enclosing object: omat[object] = (Re k, Im k, rho)
    const double2 k = ext ? k0 : make_double2(omat[3 * (reg - 1)], omat[3 * (reg - 1) + 1]);
    const double krev = k.x * (INV2PI * PHASE64);
    // whole revolutions to the first trial point, taken off every phase: what is
    // left does not grow with the point's distance
    const double x0 = src[0] - px, y0 = src[1] - py, z0 = src[2] - pz;
    const double turns =
        PHASE64 * __builtin_rint(krev * sqrt(x0 * x0 + y0 * y0 + z0 * z0) * (1.0 / PHASE64));
    const double kdec = -k.y * 1.4426950408889634073599246810019;   // log2 of the decay
    const int t0 = blockIdx.y * split_len, t1 = min(T, t0 + split_len);
    double sr = 0, si = 0, dr = 0, di = 0;
    for (int base = t0; base < t1; base += FT) {
        const int cnt = min(FT, t1 - base);
        __syncthreads();
        for (int idx = threadIdx.x; idx < cnt * FS; idx += blockDim.x) {
            const int sl = idx / FS, f = idx - sl * FS;
            const int64_t t = base + sl;
            double v;
            if (f < SRC_STRIDE) v = src[SRC_STRIDE * t + f];
            else if (f < SRC_STRIDE + 3) v = geo[GEO_STRIDE * t + 18 + (f - SRC_STRIDE)];
            else if (f == SRC_STRIDE + 3) v = geo[GEO_STRIDE * t + 21];
            else v = (double)tobj[t];
            tile[idx] = v;
        }
        __syncthreads();
        for (int sl = 0; sl < cnt; sl++) {
            const double *s = tile + sl * FS;
            if (!ext && (int)s[SRC_STRIDE + 4] != reg - 1) continue;
            // (y - p) . n_sigma, constant on the flat triangle
            const double dn = s[SRC_STRIDE + 3] -
                              (px * s[SRC_STRIDE] + py * s[SRC_STRIDE + 1] + pz * s[SRC_STRIDE + 2]);
            double fr = 0, fi = 0;
#pragma unroll
            for (int q = 0; q < 6; q++) {
                const double ex = s[3 * q] - px, ey = s[3 * q + 1] - py, ez = s[3 * q + 2] - pz;
                const double r2 = ex * ex + ey * ey + ez * ez;
                const double ri = rsqrt64(r2);
                const double r = r2 * ri;
                double Er, Ei;
                sincos_256(__builtin_fma(krev, r, -turns), Ei, Er, etab);
                if (LOSSY) {
                    const double d = decay64(kdec * r, xtab);
                    Er *= d;
                    Ei *= d;
                }
                const double Gr = Er * ri, Gi = Ei * ri;     // 4 pi G
                // 4 pi G (i k r - 1) / r^2 = (i k E - G) / r^2
                double Fr = __builtin_fma(-k.x, Ei, -Gr), Fi = __builtin_fma(k.x, Er, -Gi);
                if (LOSSY) {
                    Fr = __builtin_fma(-k.y, Er, Fr);
                    Fi = __builtin_fma(-k.y, Ei, Fi);
                }
                const double ri2 = ri * ri;
                Fr *= ri2;
                Fi *= ri2;
                const double ar = s[18 + 2 * q], ai = s[18 + 2 * q + 1];
                const double br = s[30 + 2 * q], bi = s[30 + 2 * q + 1];
                sr = __builtin_fma(Gr, ar, __builtin_fma(-Gi, ai, sr));
                si = __builtin_fma(Gr, ai, __builtin_fma(Gi, ar, si));
                fr = __builtin_fma(Fr, br, __builtin_fma(-Fi, bi, fr));
                fi = __builtin_fma(Fr, bi, __builtin_fma(Fi, br, fi));
            }
            dr = __builtin_fma(dn, fr, dr);
            di = __builtin_fma(dn, fi, di);
        }
    }
    if (p < n) {
        double *o = part + 4 * ((int64_t)blockIdx.y * n + p);
        o[0] = sr;
        o[1] = si;
        o[2] = dr;
        o[3] = di;
    }
}

// splits added in order; coefficients of the region; incident wave outside
__global__ __launch_bounds__(256) void field_reduce_kernel(
    const double *__restrict__ part, int nsplit, const double *__restrict__ pts,
    const int32_t *__restrict__ region, int64_t n, double2 k0, const double *__restrict__ omat,
    double dx, double dy, double dz, double2 *__restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    double sr = 0, si = 0, dr = 0, di = 0;
#pragma unroll 4
    for (int sp = 0; sp < nsplit; sp++) {
        const double *o = part + 4 * ((int64_t)sp * n + p);
        sr += o[0];
        si += o[1];
        dr += o[2];
        di += o[3];
    }
    double ur, ui;
    const int reg = region[p];
    if (reg == 0) {
        const double dp = dx * pts[3 * p] + dy * pts[3 * p + 1] + dz * pts[3 * p + 2];
        double sn, cs;
        sincos(k0.x * dp, &sn, &cs);
        const double a = exp(-k0.y * dp);
        ur = a * cs + INV4PI * (dr - sr);
        ui = a * sn + INV4PI * (di - si);
    } else {
        const double rho = omat[3 * (reg - 1) + 2];
        ur = INV4PI * (rho * sr - dr);
        ui = INV4PI * (rho * si - di);
    }
    out[p] = make_double2(ur, ui);
}

// Triangle ranges of the layer sums: the number of equal workgroups that fills
// whole rounds of resident ones best.
int field_splits(int T, int64_t pb, const void *kern) {
    static std::mutex mu;
    static std::map<std::pair<int, const void *>, int> cache;
    int dev = 0, slots = 0;
    BEM_HIP(hipGetDevice(&dev));
    {
        std::lock_guard<std::mutex> g(mu);
        int &c = cache[{dev, kern}];
        if (c == 0) {
            int cus = 0, per = 0;
            BEM_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
            BEM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, 256, 0));
            c = std::max(1, cus * per);
        }
        slots = c;
    }
    int best = 1;
    double best_cost = 1e300;
    for (int ns = 1; ns <= 256 && (ns == 1 || ns * FT / 2 <= T); ns++) {
        const int len = (T + ns - 1) / ns;
        // + tables and the first tile, in triangles; half a round of a launch of many
        const double waves = (double)pb * ns / slots;
        const double cost = (waves <= 4 ? std::ceil(waves) : waves + 0.5) * (len + 8.0);
        if (cost < best_cost * (1 - 1e-9)) {
            best_cost = cost;
            best = ns;
        }
    }
    return best;
}

}   // namespace

void field_eval(bem_mesh *m, double2 k0, double2 k1, double rho, const double *dir,
                const double2 *x, const double *pts, int64_t n, double2 *out, int32_t *region,
                hipStream_t s, const ObjMaterials *om) {
    if (n == 0) return;
    const int T = (int)m->T, nobj = m->nobj;
    // the mesh's workspace when no other call holds it, else an own one (released
    // or free again once the stream has been waited for, below)
    bem_mesh::FieldWork own, &mw = *m->field_work;
    std::unique_lock<std::mutex> lk(mw.mu, std::try_to_lock);
    bem_mesh::FieldWork &w = lk.owns_lock() ? mw : own;
    auto grow = [](auto &b, size_t need) {
        if (b.n < need) b.alloc(need);
    };
    // per object: material (Re k, Im k, rho), then bounding box
    std::vector<double> tab(9 * (size_t)nobj);
    bool lossy = k0.y != 0.0;
    for (int o = 0; o < nobj; o++) {
        const double2 ko = om ? om->k[o] : k1;
        tab[3 * o] = ko.x;
        tab[3 * o + 1] = ko.y;
        tab[3 * o + 2] = om ? om->rho[o] : rho;
        lossy = lossy || ko.y != 0.0;
    }
    std::copy(m->obj_box.begin(), m->obj_box.end(), tab.begin() + 3 * nobj);
    w.tab.upload(tab);
    grow(w.P, (size_t)(3 * m->N));
    if (!w.have_P) {
        BEM_HIP(hipMemcpy(w.P.p, m->P.data(), m->P.size() * sizeof(double), hipMemcpyHostToDevice));
        w.have_P = true;
    }
    const double *omat = w.tab.p, *box = w.tab.p + 3 * nobj;
    const int64_t all = n;
    n = std::min(n, FIELD_POINTS);
    unsigned pb = (unsigned)((n + 255) / 256);
    const auto layers = lossy ? field_kernel<true> : field_kernel<false>;
    const int nsplit = field_splits(T, pb, (const void *)layers);
    const int split_len = (T + nsplit - 1) / nsplit;
    // solid angles: at most WIND_GROUPS workgroups' points and ranges, or one range
    const int max_split = std::max(1, T / FT);
    grow(w.src, (size_t)SRC_STRIDE * T);
    grow(w.part, std::max((size_t)nsplit * n * 4,
                          2 * std::max((size_t)n, (size_t)256 * WIND_GROUPS) + 512));
    grow(w.list, (size_t)n + 1);
    int32_t *reg = region, *count = w.list.p, *list = w.list.p + 1;
    if (!reg) {
        grow(w.region, (size_t)n);
        reg = w.region.p;
    }
    hipLaunchKernelGGL(field_sources_kernel, dim3((T + 255) / 256), dim3(256), 0, s, w.P.p, m->tri_d.p,
                       m->tst.p, x, m->N, T, w.src.p);
    BEM_LAUNCH_CHECK();
    for (int64_t p0 = 0; p0 < all; p0 += FIELD_POINTS, pts += 3 * n, out += n) {
        n = std::min(all - p0, FIELD_POINTS);
        pb = (unsigned)((n + 255) / 256);
        if (region) reg = region + p0;
        {
            Timer tm("field_winding", s);
            hipLaunchKernelGGL(count_zero_kernel, dim3(1), dim3(1), 0, s, count);
            BEM_LAUNCH_CHECK();
            hipLaunchKernelGGL(region_box_kernel, dim3(pb), dim3(256), 0, s, pts, n, box, nobj, reg, list,
                               count);
            BEM_LAUNCH_CHECK();
            hipLaunchKernelGGL(winding_kernel, dim3(WIND_GROUPS), dim3(256), 0, s, w.P.p, m->tri_d.p,
                               m->tobj_d.p, T, pts, list, count, max_split, w.part.p);
            BEM_LAUNCH_CHECK();
            hipLaunchKernelGGL(region_kernel, dim3(pb), dim3(256), 0, s, w.part.p, list, count, max_split,
                               nobj, reg);
            BEM_LAUNCH_CHECK();
        }
        {
            Timer tm("field_eval", s);
            hipLaunchKernelGGL(layers, dim3(pb, (unsigned)nsplit), dim3(256), 0, s, w.src.p, m->geo64.p,
                               m->tobj_d.p, T, split_len, pts, reg, n, k0, omat, w.part.p);
            BEM_LAUNCH_CHECK();
        }
        hipLaunchKernelGGL(field_reduce_kernel, dim3(pb), dim3(256), 0, s, w.part.p, nsplit, pts, reg, n, k0,
                           omat, dir[0], dir[1], dir[2], out);
        BEM_LAUNCH_CHECK();
    }
    BEM_HIP(hipStreamSynchronize(s));   // the workspace is free again
}

}   // namespace bem
