// Assembled form of the permuted PMCHWT Galerkin operator (Sec. 2.7;
// operators of Sec. 2.2, P1 Galerkin of Sec. 2.3) as a dense complex64
// matrix B [2N][2N] (row-major; rows [psi-row; phi-row] = [V-row; D-row],
// columns [psi; phi]), for right-hand-side batches and for GMRES iterations
// that reuse one operator many times.
//
// Entries are the same sums as the matrix-free matvec: the 6x6 rule (FP32)
// over every test/trial triangle pair sharing no vertex, plus the FP64
// near-field operator of the pairs that do.
//
// The far part is symmetric under exchange of test and trial functions (the
// same rule on both sides, a kernel symmetric in x and y): V and D are
// symmetric and K' = K^T, so B[j][i] = B[i][j], B[N+j][N+i] = B[N+i][N+j] and
// B[N+j][i] = -B[i][N+j].  Only the entries with rank(i) <= rank(j) are
// evaluated, rank being the vertex's place in a Morton order of the vertex
// coordinates (vertices of one triangle get close ranks, so that about half
// of the work remains); dense_mirror_kernel fills in the others.  Per tile J
// of trial vertices (consecutive ranks),
//   dense_pairs_kernel:  Q[tau][j][a][blk] = sum_{sigma in star(j)} local
//                        block (tau, sigma)[a][b(sigma, j)]    (thread (tau, j),
//                        only where min rank(tau) <= rank(j))
//   dense_gather_kernel: B[i][j] = sum_{(tau, a) in star(i)} Q[tau][j][a]   (thread (i, j),
//                        only where rank(i) <= rank(j))
// Each separated triangle pair is evaluated about 1.5 times (three times for
// every trial vertex without the symmetry); assembly is deterministic.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>

#include "bem_internal.h"
#include "entries.h"

namespace bem {

namespace {

using namespace entries;

typedef float fvec4 __attribute__((ext_vector_type(4)));
typedef double dvec2 __attribute__((ext_vector_type(2)));

constexpr int JT = 512;   // trial vertices per assembly tile

// At least two waves per SIMD: the FP64 instance otherwise takes 256 VGPRs
// plus AGPRs (one wave per SIMD); with the limit it keeps about 20 values in
// scratch and assembles 15 % faster.  The FP32 instances (143 VGPRs) run at 3.
template <class R, bool CK0, bool CK1, bool MULTI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void dense_pairs_kernel(
    const R *__restrict__ geo, const double *__restrict__ tst,
    const int32_t *__restrict__ tobj, const int32_t *__restrict__ tri,
    const int32_t *__restrict__ star_ptr, const int32_t *__restrict__ star_idx,
    const int32_t *__restrict__ order, int n_tau, const int32_t *__restrict__ rank,
    const int32_t *__restrict__ byrank, int T, int r0, int64_t N, DCoefT<R> cf,
    const DIntT<R> *__restrict__ itab, typename DM<R>::C *__restrict__ Q) {
    using M = DM<R>;
    __shared__ double2 etab[std::is_same<R, double>::value ? 256 : 1];   // FP64 sin/cos table
    M::fill_table(etab);
    __syncthreads();
    // test triangles in ascending order of their smallest vertex rank: the
    // first n_tau of them have a vertex ranked inside or before this tile
    const int k = blockIdx.x * 256 + threadIdx.x;
    const int tau = k < n_tau ? order[k] : T;
    const int jl = blockIdx.y;
    const int rj = r0 + jl;
    const int j = rj < N ? byrank[rj] : 0;
    const int tt = tau < T ? tau : 0;
    const int tv0 = tri[3 * tt], tv1 = tri[3 * tt + 1], tv2 = tri[3 * tt + 2];
    // Q[tau][j] is read only for rows i of tau with rank(i) <= rank(j)
    const bool active = tau < T && rj < N &&
                        min(rank[tv0], min(rank[tv1], rank[tv2])) <= rj;
    if (!active) return;
    R px[6], py[6], pz[6], ntx, nty, ntz, ct, cu[9];
    load_test(geo, tst, tt, px, py, pz, ntx, nty, ntz, ct, cu);
    R outr[12], outi[12];   // [blk * 3 + a]
    tri_vertex_entries<R, CK0, CK1, MULTI, true>(geo, tst, tobj, tri, star_ptr, star_idx, tt, j,
                                                 px, py, pz, ntx, nty, ntz, ct, cu, cf, itab,
                                                 etab, outr, outi);
    typename M::C *o = Q + ((int64_t)tau * JT + jl) * 12;
    for (int c = 0; c < 12; c++) o[c] = M::mk(outr[c], outi[c]);
}

// B[i][j], B[i][N+j], B[N+i][j], B[N+i][N+j] from the star of test vertex i,
// for the trial vertices j of the tile with rank(j) >= rank(i)
template <class C>
__global__ __launch_bounds__(256) void dense_gather_kernel(const C *__restrict__ Q,
                                                           const int32_t *__restrict__ star_ptr,
                                                           const int32_t *__restrict__ star_idx,
                                                           const int32_t *__restrict__ rank,
                                                           const int32_t *__restrict__ byrank,
                                                           int64_t N, int r0, int jt,
                                                           C *__restrict__ B) {
    const int jl = blockIdx.y * 256 + threadIdx.x;
    const int64_t i = blockIdx.x;
    if (jl >= jt || rank[i] > r0 + jl) return;
    C acc[4];
    for (int k = 0; k < 4; k++) acc[k].x = acc[k].y = 0;
    for (int e = star_ptr[i]; e < star_ptr[i + 1]; e++) {
        const int ta = star_idx[e];
        const int t = ta / 3, a = ta - 3 * t;
        const C *q = Q + ((int64_t)t * JT + jl) * 12;
        for (int k = 0; k < 4; k++) {
            acc[k].x += q[3 * k + a].x;
            acc[k].y += q[3 * k + a].y;
        }
    }
    const int64_t n2 = 2 * N, j = byrank[r0 + jl];
    B[i * n2 + j] = acc[0];
    B[i * n2 + N + j] = acc[1];
    B[(N + i) * n2 + j] = acc[2];
    B[(N + i) * n2 + N + j] = acc[3];
}

// Entries with rank(i) > rank(j) from their mirror images (blockIdx.z picks
// the block): B[i][j] = B[j][i], B[N+i][N+j] = B[N+j][N+i],
// B[N+i][j] = -B[j][N+i], B[i][N+j] = -B[N+j][i].  32 x 32 tiles transposed
// through LDS; the entries read are never written here (their row ranks lower).
template <class C>
__global__ __launch_bounds__(256) void dense_mirror_kernel(const int32_t *__restrict__ rank,
                                                           int64_t N, C *__restrict__ B) {
    __shared__ C tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int64_t I0 = (int64_t)blockIdx.x * 32, J0 = (int64_t)blockIdx.y * 32;
    const int64_t n2 = 2 * N;
    const int z = blockIdx.z;
    const int64_t ro = (z == 0 || z == 2) ? 0 : N;   // row offset of the entries read
    const int64_t co = (z == 0 || z == 3) ? 0 : N;   // column offset of the entries read
    const float sg = z < 2 ? 1.0f : -1.0f;
    // read B[ro + j][co + i] for j in the J tile, i in the I tile
    const int64_t ic = I0 + tx;
    const int ri = ic < N ? rank[ic] : 0;
    for (int rr = 0; rr < 32; rr += 8) {
        const int64_t jr = J0 + ty + rr;
        C v;
        v.x = v.y = 0;
        if (jr < N && ic < N && rank[jr] < ri) v = B[(ro + jr) * n2 + co + ic];
        tile[ty + rr][tx] = v;
    }
    __syncthreads();
    // write B[co + i][ro + j] for i in the I tile, j in the J tile
    const int64_t jc = J0 + tx;
    const int rjc = jc < N ? rank[jc] : 0;
    for (int rr = 0; rr < 32; rr += 8) {
        const int64_t ir = I0 + ty + rr;
        if (ir < N && jc < N && rank[ir] > rjc) {
            C v = tile[tx][ty + rr];
            v.x *= sg;
            v.y *= sg;
            B[(co + ir) * n2 + ro + jc] = v;
        }
    }
}

// add the FP64 near-field operator (complex64: summed in FP64, rounded once)
__global__ __launch_bounds__(256) void dense_add_near_kernel(const int32_t *__restrict__ rowptr,
                                                             const int32_t *__restrict__ col,
                                                             const double2 *__restrict__ nf,
                                                             int64_t nnz, int64_t N,
                                                             float2 *__restrict__ B) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int64_t n2 = 2 * N;
    for (int e = rowptr[i]; e < rowptr[i + 1]; e++) {
        const int64_t j = col[e];
        const int64_t pos[4] = {i * n2 + j, i * n2 + N + j, (N + i) * n2 + j,
                                (N + i) * n2 + N + j};
        for (int k = 0; k < 4; k++) {
            const double2 v = nf[k * nnz + e];
            float2 o = B[pos[k]];
            B[pos[k]] = make_float2((float)((double)o.x + v.x), (float)((double)o.y + v.y));
        }
    }
}

__global__ __launch_bounds__(256) void dense_add_near64_kernel(const int32_t *__restrict__ rowptr,
                                                               const int32_t *__restrict__ col,
                                                               const double2 *__restrict__ nf,
                                                               int64_t nnz, int64_t N,
                                                               double2 *__restrict__ B) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int64_t n2 = 2 * N;
    for (int e = rowptr[i]; e < rowptr[i + 1]; e++) {
        const int64_t j = col[e];
        const int64_t pos[4] = {i * n2 + j, i * n2 + N + j, (N + i) * n2 + j,
                                (N + i) * n2 + N + j};
        for (int k = 0; k < 4; k++) {
            const double2 v = nf[k * nnz + e];
            B[pos[k]].x += v.x;
            B[pos[k]].y += v.y;
        }
    }
}

// y = B x with the complex128 operator, one vector: two rows per wavefront,
// 16-byte loads (one complex entry), eight per row in flight per lane, B
// streamed with non-temporal loads; FP64 sums, fixed-order wave reduction.
constexpr int G64_RW = 2;
__global__ __launch_bounds__(256) void dense_gemv64_kernel(const double2 *__restrict__ B,
                                                           int64_t n2,
                                                           const double2 *__restrict__ x,
                                                           double2 *__restrict__ y) {
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * G64_RW;
    const int lane = threadIdx.x & 63;
    if (row0 >= n2) return;
    const int nrow = n2 - row0 < G64_RW ? (int)(n2 - row0) : G64_RW;
    const dvec2 *b[G64_RW];
    for (int q = 0; q < G64_RW; q++)
        b[q] = reinterpret_cast<const dvec2 *>(B + (row0 + (q < nrow ? q : 0)) * n2);
    double sr[G64_RW], si[G64_RW];
    for (int q = 0; q < G64_RW; q++) sr[q] = si[q] = 0.0;
    int64_t c0 = 0;
    for (; c0 + 512 <= n2; c0 += 512) {
        double2 v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = x[c0 + u * 64 + lane];
#pragma unroll
        for (int q = 0; q < G64_RW; q++) {
            dvec2 a[8];
#pragma unroll
            for (int u = 0; u < 8; u++) a[u] = __builtin_nontemporal_load(b[q] + c0 + u * 64 + lane);
#pragma unroll
            for (int u = 0; u < 8; u++) {
                sr[q] = __builtin_fma(a[u].x, v[u].x, __builtin_fma(-a[u].y, v[u].y, sr[q]));
                si[q] = __builtin_fma(a[u].x, v[u].y, __builtin_fma(a[u].y, v[u].x, si[q]));
            }
        }
    }
    for (int q = 0; q < G64_RW; q++)
        for (int64_t c = c0 + lane; c < n2; c += 64) {
            const dvec2 a = __builtin_nontemporal_load(b[q] + c);
            const double2 v = x[c];
            sr[q] = __builtin_fma(a.x, v.x, __builtin_fma(-a.y, v.y, sr[q]));
            si[q] = __builtin_fma(a.x, v.y, __builtin_fma(a.y, v.x, si[q]));
        }
    for (int q = 0; q < G64_RW; q++)
        for (int o = 32; o > 0; o >>= 1) {
            sr[q] += __shfl_xor(sr[q], o, 64);
            si[q] += __shfl_xor(si[q], o, 64);
        }
    if (lane == 0)
        for (int q = 0; q < nrow; q++) y[row0 + q] = make_double2(sr[q], si[q]);
}

// y_r = B x_r for NR vectors (2..8); x: [NR][n2] complex64, y_r = y + r ystride.
// Bound by HBM if the loads of B never wait.  Two rows per wavefront; each chunk of
// the NR vectors is staged in LDS by the workgroup and read by all its rows (each
// LDS value once per wavefront, for both of its rows).  Up to five vectors the next
// chunk of both is in flight while one is multiplied (two and four vectors on 5 124
// rows 43 and 51 us, without 52 and 64; on 20 484 rows 541 and 607, 570 and 610);
// beyond, the registers do not allow it, and longer chunks and more wavefronts per
// workgroup are the faster form.  16-byte loads of B (2N even: rows and vectors
// 16-byte aligned), non-temporal; FP32 partial sums per chunk added in FP64,
// fixed-order wave reduction.
constexpr int GV_RW = 2;      // rows per wavefront
template <int NR> constexpr bool gv_ahead() { return NR <= 5; }
template <int NR> constexpr int gv_chunk() { return gv_ahead<NR>() ? 128 : 256; }   // float4 per vector
template <int NR> constexpr int gv_waves() { return gv_ahead<NR>() ? 4 : 8; }       // per workgroup

template <int NR>
__global__ __launch_bounds__(64 * gv_waves<NR>()) void dense_gemv_kernel(
    const float2 *__restrict__ B, int64_t n2, const float2 *__restrict__ x, double2 *__restrict__ y,
    int64_t ystride) {
    constexpr bool AHEAD = gv_ahead<NR>();
    constexpr int CH = gv_chunk<NR>(), NT = 64 * gv_waves<NR>(), NU = CH / 64,
                  NX = (NR * CH + NT - 1) / NT;
    __shared__ fvec4 xs[AHEAD ? 2 : 1][NR * CH];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t row0 = ((int64_t)blockIdx.x * gv_waves<NR>() + wave) * GV_RW;
    const int nrow = row0 >= n2 ? 0 : (n2 - row0 < GV_RW ? (int)(n2 - row0) : GV_RW);
    const fvec4 *b4[GV_RW];
    for (int q = 0; q < GV_RW; q++)
        b4[q] = reinterpret_cast<const fvec4 *>(B + (q < nrow ? row0 + q : 0) * n2);
    const fvec4 *x4 = reinterpret_cast<const fvec4 *>(x);
    const int64_t n4 = n2 / 2;
    const fvec4 zero = fvec4{0.f, 0.f, 0.f, 0.f};
    auto load_b = [&](int64_t c0, fvec4 (&a)[GV_RW][NU]) {
#pragma unroll
        for (int q = 0; q < GV_RW; q++)
#pragma unroll
            for (int u = 0; u < NU; u++) {
                const int64_t c = c0 + u * 64 + lane;
                a[q][u] = c < n4 ? __builtin_nontemporal_load(b4[q] + c) : zero;
            }
    };
    auto load_x = [&](int64_t c0, fvec4 (&v)[NX]) {
#pragma unroll
        for (int w = 0; w < NX; w++) {
            const int idx = w * NT + threadIdx.x, r = idx / CH;
            const int64_t c = c0 + (idx - r * CH);
            v[w] = r < NR && c < n4 ? x4[r * n4 + c] : zero;
        }
    };
    auto store_x = [&](int buf, const fvec4 (&v)[NX]) {
#pragma unroll
        for (int w = 0; w < NX; w++) {
            const int idx = w * NT + threadIdx.x;
            if (idx < NR * CH) xs[buf][idx] = v[w];
        }
    };
    double sr[GV_RW][NR], si[GV_RW][NR];
    for (int q = 0; q < GV_RW; q++)
        for (int r = 0; r < NR; r++) sr[q][r] = si[q][r] = 0.0;
    auto multiply = [&](int buf, const fvec4 (&a)[GV_RW][NU]) {
#pragma unroll
        for (int r = 0; r < NR; r++) {
            float pr[GV_RW], pi[GV_RW];
#pragma unroll
            for (int q = 0; q < GV_RW; q++) pr[q] = pi[q] = 0.f;
#pragma unroll
            for (int u = 0; u < NU; u++) {
                const fvec4 v = xs[buf][r * CH + u * 64 + lane];
#pragma unroll
                for (int q = 0; q < GV_RW; q++) {
                    pr[q] += a[q][u].x * v.x - a[q][u].y * v.y;
                    pi[q] += a[q][u].x * v.y + a[q][u].y * v.x;
                    pr[q] += a[q][u].z * v.z - a[q][u].w * v.w;
                    pi[q] += a[q][u].z * v.w + a[q][u].w * v.z;
                }
            }
#pragma unroll
            for (int q = 0; q < GV_RW; q++) {
                sr[q][r] += pr[q];
                si[q][r] += pi[q];
            }
        }
    };
    fvec4 a[GV_RW][NU], xv[NX];
    if constexpr (AHEAD) {
        fvec4 an[GV_RW][NU];
        load_x(0, xv);
        load_b(0, a);
        store_x(0, xv);
        __syncthreads();
        int buf = 0;
        for (int64_t c0 = 0; c0 < n4; c0 += CH, buf ^= 1) {
            const bool more = c0 + CH < n4;   // (uniform)
            if (more) {
                load_x(c0 + CH, xv);
                load_b(c0 + CH, an);
            }
            multiply(buf, a);
            if (more) {
                store_x(buf ^ 1, xv);   // (its readers passed the previous barrier)
#pragma unroll
                for (int q = 0; q < GV_RW; q++)
#pragma unroll
                    for (int u = 0; u < NU; u++) a[q][u] = an[q][u];
            }
            __syncthreads();
        }
    } else {
        for (int64_t c0 = 0; c0 < n4; c0 += CH) {
            __syncthreads();   // the previous chunk's readers are done
            load_x(c0, xv);
            store_x(0, xv);
            __syncthreads();
            load_b(c0, a);
            multiply(0, a);
        }
    }
    if (nrow == 0) return;
    for (int q = 0; q < GV_RW; q++)
        for (int r = 0; r < NR; r++)
            for (int o = 32; o > 0; o >>= 1) {
                sr[q][r] += __shfl_xor(sr[q][r], o, 64);
                si[q][r] += __shfl_xor(si[q][r], o, 64);
            }
    if (lane == 0)
        for (int q = 0; q < nrow; q++)
            for (int r = 0; r < NR; r++) y[r * ystride + row0 + q] = make_double2(sr[q][r], si[q][r]);
}

// y = B x for one vector: GEMV1_ROWS rows per wavefront (each chunk of x, read from
// cache, serves them all), 16-byte loads (two complex entries; 2N is even, so
// every row starts 16-byte aligned), eight loads of each row in flight per
// lane, B streamed with non-temporal loads.  FP32 partial sums over chunks
// of 1024 entries are added in FP64, then a fixed-order wave reduction.
constexpr int GEMV1_ROWS = 4;   // rows per wavefront

__global__ __launch_bounds__(256) void dense_gemv1_kernel(const float2 *__restrict__ B,
                                                          int64_t n2,
                                                          const float2 *__restrict__ x,
                                                          double2 *__restrict__ y) {
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * GEMV1_ROWS;
    const int lane = threadIdx.x & 63;
    if (row0 >= n2) return;
    const int nrow = n2 - row0 < GEMV1_ROWS ? (int)(n2 - row0) : GEMV1_ROWS;
    const fvec4 *b4[GEMV1_ROWS];
    for (int q = 0; q < GEMV1_ROWS; q++)
        b4[q] = reinterpret_cast<const fvec4 *>(B + (row0 + (q < nrow ? q : 0)) * n2);
    const fvec4 *x4 = reinterpret_cast<const fvec4 *>(x);
    const int64_t n4 = n2 / 2;
    double sr[GEMV1_ROWS], si[GEMV1_ROWS];
    for (int q = 0; q < GEMV1_ROWS; q++) sr[q] = si[q] = 0.0;
    int64_t c0 = 0;
    for (; c0 + 512 <= n4; c0 += 512) {
        fvec4 v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) v[u] = x4[c0 + u * 64 + lane];
#pragma unroll
        for (int q = 0; q < GEMV1_ROWS; q++) {
            fvec4 a[8];
#pragma unroll
            for (int u = 0; u < 8; u++) a[u] = __builtin_nontemporal_load(b4[q] + c0 + u * 64 + lane);
            float pr = 0.f, pi = 0.f;
#pragma unroll
            for (int u = 0; u < 8; u++) {
                pr += a[u].x * v[u].x - a[u].y * v[u].y;
                pi += a[u].x * v[u].y + a[u].y * v[u].x;
                pr += a[u].z * v[u].z - a[u].w * v[u].w;
                pi += a[u].z * v[u].w + a[u].w * v[u].z;
            }
            sr[q] += pr;
            si[q] += pi;
        }
    }
    for (int q = 0; q < GEMV1_ROWS; q++) {
        float pr = 0.f, pi = 0.f;
        for (int64_t c = c0 + lane; c < n4; c += 64) {
            const fvec4 a = __builtin_nontemporal_load(b4[q] + c);
            const fvec4 v = x4[c];
            pr += a.x * v.x - a.y * v.y;
            pi += a.x * v.y + a.y * v.x;
            pr += a.z * v.z - a.w * v.w;
            pi += a.z * v.w + a.w * v.z;
        }
        sr[q] += pr;
        si[q] += pi;
    }
    for (int q = 0; q < GEMV1_ROWS; q++)
        for (int o = 32; o > 0; o >>= 1) {
            sr[q] += __shfl_xor(sr[q], o, 64);
            si[q] += __shfl_xor(si[q], o, 64);
        }
    if (lane == 0)
        for (int q = 0; q < nrow; q++) y[row0 + q] = make_double2(sr[q], si[q]);
}

// ------------------------------------------------ multi-RHS product on MFMA
// Y = B X for n_rhs right-hand sides as one real FP32 GEMM: B is read as a
// real [M][Kp] matrix (M = 2N rows, Kp = 4N: re/im interleaved), X as the
// transposed real columns XT[Np][Kp] of mx_prep_kernel (2r: Re, -Im; 2r + 1: Im,
// Re interleaved), so that columns 2r and 2r+1 of the product are Re and Im of
// column r of B X.
constexpr int GM = 128, GN = 128, GK = 32;   // block tile and K step
constexpr int GKC = 4096;                    // largest split-K chunk (FP32 MFMA accumulation)
constexpr int GLD = GK + 4;                  // padded rows: 16 lanes of a read in distinct banks

typedef float floatx16 __attribute__((ext_vector_type(16)));

// partial products of K chunk blockIdx.z: Yp[z][M][Np]; 4 waves, 64 x 64 each.
// Bound by the FP32 matrix cores.  The next K step's tiles are loaded into
// registers (16-byte loads) while the current one is multiplied from LDS, then
// stored to the other LDS buffer: one barrier per K step.  Both tiles are kept by
// rows along K, and a lane reads four consecutive k of its row at once: the two
// k-slots of v_mfma_f32_32x32x2 may hold any k as long as A and X agree, so
// instruction e of a group of 8 takes k = 4 (lane / 32) + e.  Four reads per 16
// matrix instructions, issued a group ahead (single values of both operands read
// right before their use: 2.42 ms a product of 64 vectors at 10 242 vertices, 94
// TFLOP/s in this kernel; now 1.88).  Kp is a multiple of 4, chunk ends of 32.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void gemm_mfma_kernel(
    const float *__restrict__ A, const float *__restrict__ XT, float *__restrict__ Yp, int64_t M,
    int64_t Kp, int Np, int kchunk) {
    __shared__ fvec4 As[2][GM * GLD / 4];
    __shared__ fvec4 Bs[2][GN * GLD / 4];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t m0 = (int64_t)blockIdx.x * GM;
    const int n0 = blockIdx.y * GN;
    const int64_t kbeg = (int64_t)blockIdx.z * kchunk;
    const int64_t kend = kbeg + kchunk < Kp ? kbeg + kchunk : Kp;
    const int wr = (wave >> 1) * 64, wc = (wave & 1) * 64;
    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;
    // per thread: 4 float4 of either tile (rows i 32 + t / 8, columns 4 (t % 8))
    const int tr = t >> 3, tc = t & 7;
    const fvec4 zero4 = fvec4{0.f, 0.f, 0.f, 0.f};
    fvec4 ra[4], rb[4];
    auto gload = [&](int64_t k0) {
        const int64_t k = k0 + 4 * tc;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int64_t row = m0 + 32 * i + tr;
            ra[i] = row < M && k < kend ? *(const fvec4 *)(A + row * Kp + k) : zero4;
            rb[i] = k < kend ? *(const fvec4 *)(XT + (int64_t)(n0 + 32 * i + tr) * Kp + k) : zero4;
        }
    };
    auto lstore = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            As[buf][(32 * i + tr) * (GLD / 4) + tc] = ra[i];
            Bs[buf][(32 * i + tr) * (GLD / 4) + tc] = rb[i];
        }
    };
    gload(kbeg);
    lstore(0);
    __syncthreads();
    int cur = 0;
    const int ra0 = (wr + (lane & 31)) * (GLD / 4) + (lane >> 5),
              rb0 = (wc + (lane & 31)) * (GLD / 4) + (lane >> 5);
    for (int64_t k0 = kbeg; k0 < kend; k0 += GK) {
        const bool more = k0 + GK < kend;
        if (more) gload(k0 + GK);
        fvec4 va[2][2], vb[2][2];   // [group parity][tile]
        auto read = [&](int gp, int p) {
#pragma unroll
            for (int i = 0; i < 2; i++) {
                va[p][i] = As[cur][ra0 + 32 * i * (GLD / 4) + 2 * gp];
                vb[p][i] = Bs[cur][rb0 + 32 * i * (GLD / 4) + 2 * gp];
            }
        };
        read(0, 0);
#pragma unroll
        for (int gp = 0; gp < GK / 8; gp++) {
            const int p = gp & 1;
            if (gp + 1 < GK / 8) read(gp + 1, p ^ 1);
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
                for (int i = 0; i < 2; i++)
#pragma unroll
                    for (int j = 0; j < 2; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[p][i][e], vb[p][j][e],
                                                                         acc[i][j], 0, 0, 0);
            // the next group's reads before this group's products
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 16, 0);
        }
        if (more) lstore(cur ^ 1);
        __syncthreads();
        cur ^= 1;
    }
    float *Y = Yp + (int64_t)blockIdx.z * M * Np;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int v = 0; v < 16; v++) {
                // 32x32 accumulator layout: column lane % 32, row
                // 8 (v / 4) + 4 (lane / 32) + v % 4
                const int64_t row = m0 + wr + 32 * i + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                const int col = n0 + wc + 32 * j + (lane & 31);
                if (row < M) Y[row * Np + col] = acc[i][j][v];
            }
}

// y[r][m] = sum over K chunks (fixed order, FP64) of (Yp[.][m][2r], Yp[.][m][2r+1]);
// 32 rows and 32 vectors per workgroup, turned through LDS so that both the
// partial products (by rows) and y (by vectors) are read and written along lines
__global__ __launch_bounds__(256) void gemm_reduce_kernel(const float *__restrict__ Yp,
                                                          int nchunks, int64_t M, int Np, int R,
                                                          double2 *__restrict__ y) {
    __shared__ double2 tile[32][33];
    const int64_t m0 = (int64_t)blockIdx.y * 32;
    const int r0 = blockIdx.x * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int q = ty; q < 32; q += 8) {
        const int64_t m = m0 + q;
        double2 v = make_double2(0.0, 0.0);
        if (m < M && r0 + tx < R) {
            const float2 *p = reinterpret_cast<const float2 *>(Yp) + m * (Np / 2) + r0 + tx;
#pragma unroll 4
            for (int c = 0; c < nchunks; c++) {
                const float2 f = p[(int64_t)c * M * (Np / 2)];
                v.x += f.x;
                v.y += f.y;
            }
        }
        tile[q][tx] = v;
    }
    __syncthreads();
    for (int q = ty; q < 32; q += 8)
        if (m0 + tx < M && r0 + q < R) y[(int64_t)(r0 + q) * M + m0 + tx] = tile[tx][q];
}

// ----------------------------- up to 32 right-hand sides: skinny MFMA product
// The same real product with 16 NT columns (8 NT complex right-hand sides) on
// v_mfma_f32_16x16x4 / v_mfma_f64_16x16x4, for the complex64 and the complex128
// operator.  Up to 8 vectors bound by HBM (every entry of B once per launch): at
// 10 242 vertices the FP64 matrix cores need 0.37 ms for 8 vectors, at the 72 TFLOP/s
// of a large product, and B 0.52 ms at the rate of the one-vector product; 9 to 16
// vectors are bound by the matrix cores (0.75 ms, measured 1.00).  A wavefront
// streams 16 RT rows over its range of K with 16-byte loads of 256 or 512 contiguous
// bytes a row, the next step's loads in flight, and turns them through LDS (loads in
// the operand's own order read 64 bytes a row, 20 % slower; 8 vectors on the vector
// units took 1.10 ms, complex128 one by one 8.3 ms, here 0.74 and 1.24); the columns
// come from XT[16 NT][Kp] through the caches.  The 4 k-slots of a matrix instruction
// may hold any 4 values of k as long as A and XT agree: lane (i, q) = (lane % 16,
// lane / 16) holds VE values of row i from k = kb + VE (4 c + q) on, and instruction
// (c, e) takes the e-th.
template <class R> struct MxOp;
template <> struct MxOp<float> {
    typedef float Vec __attribute__((ext_vector_type(4)));
    typedef float Acc __attribute__((ext_vector_type(4)));
    static constexpr int VE = 4;
    static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};
template <> struct MxOp<double> {
    typedef double Vec __attribute__((ext_vector_type(2)));
    typedef double Acc __attribute__((ext_vector_type(4)));
    static constexpr int VE = 2;
    static __device__ __forceinline__ Acc mma(double a, double b, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};
// lanes along a row per load: 16 for the complex64 operator (10 242 vertices, 8
// and 32 vectors: 0.735 and 1.23 ms, with 32 lanes 0.762 and 1.47), 32 for the
// complex128 one while the columns leave room (8 vectors 1.24 against 1.30 ms)
template <class R, int NT> constexpr int mx_lpr() {
    return std::is_same<R, double>::value && NT <= 2 ? 32 : 16;
}
// waves per SIMD asked for (registers)
template <class R, int NT> constexpr int mx_waves() {
    return NT > 2 ? 1 : std::is_same<R, double>::value ? 2 : 3;
}
// Type of the products and sums.  The complex64 operator's up to 16 vectors are
// FP64 (exact products of FP32 values): FP32 matrix instructions add four products
// into the sum each, and even sums of 8 products had an error above that of the
// vector units (1.4e-7 against 1.3e-7, 1.9e-7 for sums of 64); FP64 gives
// 1.2e-7, and for 8 vectors B still costs more than the matrix cores.  Beyond, FP32
// in sums of 64 added in FP64, as against 8.6e-7 of the MFMA GEMM it took over from.
template <class R, int NT>
using MxWork = std::conditional_t<std::is_same<R, double>::value || NT <= 2, double, float>;
template <class R, int NT> constexpr int mx_step() { return MxOp<R>::VE * mx_lpr<R, NT>(); }   // of K

// XT[2r][2k], XT[2r][2k+1] = Re, -Im and XT[2r+1][..] = Im, Re of x[r][k]; zeros
// for r >= nr (r < 8 NT)
template <class R>
__global__ __launch_bounds__(256) void mx_prep_kernel(const double2 *__restrict__ x, int nr,
                                                      int64_t K, R *__restrict__ XT) {
    // (vectors along x: their number is not bounded by a grid's y extent)
    const int64_t k = (int64_t)blockIdx.y * 256 + threadIdx.x;
    const int r = blockIdx.x;
    if (k >= K) return;
    const double2 v = r < nr ? x[(int64_t)r * K + k] : make_double2(0.0, 0.0);
    R *re = XT + (int64_t)(2 * r) * 2 * K, *im = re + 2 * K;
    re[2 * k] = (R)v.x;
    re[2 * k + 1] = (R)(-v.y);
    im[2 * k] = (R)v.y;
    im[2 * k + 1] = (R)v.x;
}

// part[blockIdx.y][M][16 NT]; grid (ceil(M / (64 RT)), ranges of klen)
template <class R, int RT, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(mx_waves<R, NT>()))) void mx_gemv_kernel(const R *__restrict__ A,
                                                      const R *__restrict__ XT,
                                                      double *__restrict__ part, int64_t M,
                                                      int64_t Kp, int64_t klen) {
    using WT = MxWork<R, NT>;
    using O = MxOp<WT>;
    using Vec = typename MxOp<R>::Vec;
    constexpr int VE = MxOp<R>::VE, STEP = mx_step<R, NT>();
    constexpr int LPR = mx_lpr<R, NT>(), UC = LPR / 4;   // UC loads per tile and step
    constexpr bool F32 = std::is_same<WT, float>::value;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, q = lane >> 4;
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * 16 * RT;
    const int64_t kbeg = (int64_t)blockIdx.y * klen;
    const int64_t kend = kbeg + klen < Kp ? kbeg + klen : Kp;
    if (row0 >= M) return;
    // this wavefront's 16 RT rows of one step, padded: the 16 lanes of a read (one
    // value of q) fall in distinct banks
    constexpr int LDR = LPR * VE + 16 / (int)sizeof(R);
    __shared__ R stage[4][RT * 16 * LDR];
    R *st = stage[wave];
    const R *xrow[NT];
    for (int n = 0; n < NT; n++) xrow[n] = XT + (int64_t)(16 * n + i) * Kp;
    const Vec zero = (Vec)(R)0;
    // load c of tile t: rows (64 / LPR) c + lr, LPR lanes of 16 bytes along each
    const int lv = lane % LPR, lr = lane / LPR;
    auto load_a = [&](int64_t kb, Vec (&v)[RT][UC]) {
        const int64_t k = kb + VE * lv;   // (K is a multiple of VE)
#pragma unroll
        for (int t = 0; t < RT; t++)
#pragma unroll
            for (int c = 0; c < UC; c++) {
                const int64_t r = row0 + 16 * t + 64 / LPR * c + lr;   // (rows beyond the end are not stored)
                v[t][c] = k < kend ? *(const Vec *)(A + (r < M ? r : M - 1) * Kp + k) : zero;
            }
    };
    typename O::Acc acc[RT][NT];
    double sum[RT][NT][4];
    for (int t = 0; t < RT; t++)
        for (int n = 0; n < NT; n++)
            for (int v = 0; v < 4; v++) acc[t][n][v] = (WT)0, sum[t][n][v] = 0.0;
    auto flush = [&]() {   // FP32 sums into the FP64 ones
        if constexpr (F32) {
#pragma unroll
            for (int t = 0; t < RT; t++)
#pragma unroll
                for (int n = 0; n < NT; n++)
#pragma unroll
                    for (int v = 0; v < 4; v++) {
                        sum[t][n][v] += (double)acc[t][n][v];
                        acc[t][n][v] = (WT)0;
                    }
        }
    };
    Vec an[RT][UC];
    load_a(kbeg, an);
    for (int64_t kb = kbeg; kb < kend; kb += STEP) {
        const bool more = kb + STEP < kend;
#pragma unroll
        for (int t = 0; t < RT; t++)
#pragma unroll
            for (int c = 0; c < UC; c++)
                *(Vec *)(st + (16 * t + 64 / LPR * c + lr) * LDR + VE * lv) = an[t][c];
        // (only this wavefront's lanes read them: LDS serves a wavefront in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (more) load_a(kb + STEP, an);
#pragma unroll
        for (int c0 = 0; c0 < UC; c0 += 4) {
            Vec av[RT][4], bv[NT][4];
#pragma unroll
            for (int n = 0; n < NT; n++)
#pragma unroll
                for (int c = 0; c < 4; c++) {
                    const int64_t k = kb + VE * (4 * (c0 + c) + q);
                    bv[n][c] = k < kend ? *(const Vec *)(xrow[n] + k) : zero;
                }
#pragma unroll
            for (int t = 0; t < RT; t++)
#pragma unroll
                for (int c = 0; c < 4; c++)
                    av[t][c] = *(const Vec *)(st + (16 * t + i) * LDR + VE * (4 * (c0 + c) + q));
#pragma unroll
            for (int c = 0; c < 4; c++) {
#pragma unroll
                for (int e = 0; e < VE; e++) {
#pragma unroll
                    for (int t = 0; t < RT; t++)
#pragma unroll
                        for (int n = 0; n < NT; n++)
                            acc[t][n] = O::mma((WT)av[t][c][e], (WT)bv[n][c][e], acc[t][n]);
                }
            }
            flush();
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    double *out = part + (int64_t)blockIdx.y * M * 16 * NT;
    for (int t = 0; t < RT; t++)
        for (int v = 0; v < 4; v++) {
            const int64_t r = row0 + 16 * t + O::row(lane, v);
            if (r >= M) continue;
            for (int n = 0; n < NT; n++)
                out[r * 16 * NT + 16 * n + i] = F32 ? sum[t][n][v] : (double)acc[t][n][v];
        }
}

// y[r][m] = sum over the ranges, in order, of part[.][m][2r], [2r + 1]
__global__ __launch_bounds__(256) void mx_reduce_kernel(const double2 *__restrict__ part, int nsplit,
                                                        int64_t M, int half, int nr,
                                                        double2 *__restrict__ y) {
    const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t m = id / half;
    const int r = (int)(id - m * half);
    if (m >= M || r >= nr) return;
    double2 v = make_double2(0.0, 0.0);
    for (int sp = 0; sp < nsplit; sp++) {
        const double2 p = part[(int64_t)sp * M * half + id];
        v.x += p.x;
        v.y += p.y;
    }
    y[(int64_t)r * M + m] = v;
}

__global__ __launch_bounds__(256) void to_c64_kernel(const double2 *__restrict__ x,
                                                     float2 *__restrict__ o, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) o[i] = make_float2((float)x[i].x, (float)x[i].y);
}

struct RankOrder {
    DevBuf<int32_t> rank, byrank, order;   // [N], [N], [T]
    std::vector<int32_t> minrank_sorted;   // [T]
    explicit RankOrder(const bem_mesh *m);
    int count_below(int r) const;
};

template <class R, bool A, bool B, bool C>
void launch_pairs(dim3 grid, hipStream_t s, bem_mesh *m, const RankOrder &ro, int n_tau, int r0,
                  DCoefT<R> cf, const DIntT<R> *itab, typename DM<R>::C *Q) {
    const R *geo;
    if constexpr (std::is_same<R, float>::value) geo = m->geo32.p;
    else geo = m->geo64.p;
    hipLaunchKernelGGL((dense_pairs_kernel<R, A, B, C>), grid, dim3(256), 0, s, geo, m->tst.p,
                       m->tobj_d.p, m->tri_d.p, m->star_ptr.p, m->star_idx.p, ro.order.p, n_tau,
                       ro.rank.p, ro.byrank.p, (int)m->T, r0, m->N, cf, itab, Q);
}

// Vertex ranks in Morton order of the coordinates (10 bits per axis over the
// bounding box, ties by index) and the triangles in ascending order of their
// smallest vertex rank; minrank_sorted[k] is that rank for order[k].
RankOrder::RankOrder(const bem_mesh *m) {
    const int64_t N = m->N, T = m->T;
    double lo[3] = {1e300, 1e300, 1e300}, hi[3] = {-1e300, -1e300, -1e300};
    for (int64_t v = 0; v < N; v++)
        for (int a = 0; a < 3; a++) {
            lo[a] = std::min(lo[a], m->P[3 * v + a]);
            hi[a] = std::max(hi[a], m->P[3 * v + a]);
        }
    std::vector<uint64_t> code(N);
    for (int64_t v = 0; v < N; v++) {
        uint64_t c = 0;
        for (int a = 0; a < 3; a++) {
            const double ext = hi[a] - lo[a];
            const double u = ext > 0 ? (m->P[3 * v + a] - lo[a]) / ext : 0.0;
            const uint64_t q = (uint64_t)std::min(1023.0, std::max(0.0, u * 1023.0));
            for (int b = 0; b < 10; b++) c |= ((q >> b) & 1u) << (3 * b + a);
        }
        code[v] = c;
    }
    std::vector<int32_t> by(N), rk(N);
    for (int64_t v = 0; v < N; v++) by[v] = (int32_t)v;
    std::stable_sort(by.begin(), by.end(), [&](int32_t a, int32_t b) { return code[a] < code[b]; });
    for (int64_t r = 0; r < N; r++) rk[by[r]] = (int32_t)r;
    std::vector<int32_t> mr(T), ord(T);
    for (int64_t t = 0; t < T; t++) {
        mr[t] = std::min(rk[m->tri[3 * t]], std::min(rk[m->tri[3 * t + 1]], rk[m->tri[3 * t + 2]]));
        ord[t] = (int32_t)t;
    }
    std::stable_sort(ord.begin(), ord.end(), [&](int32_t a, int32_t b) { return mr[a] < mr[b]; });
    minrank_sorted.resize(T);
    for (int64_t k = 0; k < T; k++) minrank_sorted[k] = mr[ord[k]];
    rank.upload(rk);
    byrank.upload(by);
    order.upload(ord);
}

// number of triangles whose smallest vertex rank is below r
int RankOrder::count_below(int r) const {
    return (int)(std::lower_bound(minrank_sorted.begin(), minrank_sorted.end(), r) -
                 minrank_sorted.begin());
}

// assembly of the operator in precision R into B ([2N][2N], row-major)
template <class R>
void assemble_into(bem_mesh *m, const NearOperator &nf, double2 k0, typename DM<R>::C *B,
                   hipStream_t s) {
    using C = typename DM<R>::C;
    const int64_t N = m->N;
    DevBuf<C> Q((size_t)m->T * JT * 12);
    const DCoefT<R> cf = make_dcoef<R>(k0, nf);
    DevBuf<R> itab;   // per-object interior parts (several objects)
    if (m->nobj > 1) {
        constexpr size_t W = sizeof(DIntT<R>) / sizeof(R);
        std::vector<R> h((size_t)m->nobj * W);
        for (int o = 0; o < m->nobj; o++) {
            const DIntT<R> c = make_dint<R>(k0, nf.k1o[o], nf.rhoo[o], nf.s1);
            std::memcpy(h.data() + (size_t)o * W, &c, sizeof(c));
        }
        itab.upload(h);
    }
    const DIntT<R> *it = (const DIntT<R> *)itab.p;
    const int code = (k0.y != 0 ? 4 : 0) | (nf.k1_plan.y != 0 ? 2 : 0) | (m->nobj > 1 ? 1 : 0);
    const RankOrder ro(m);
    for (int64_t r0 = 0; r0 < N; r0 += JT) {
        const int jt = (int)std::min<int64_t>(JT, N - r0);
        // test triangles with a vertex ranked below the tile's end
        const int n_tau = ro.count_below((int)(r0 + jt));
        if (n_tau > 0) {
            dim3 grid((unsigned)((n_tau + 255) / 256), jt);
            const int r = (int)r0;
            switch (code) {
            case 0: launch_pairs<R, false, false, false>(grid, s, m, ro, n_tau, r, cf, it, Q.p); break;
            case 1: launch_pairs<R, false, false, true>(grid, s, m, ro, n_tau, r, cf, it, Q.p); break;
            case 2: launch_pairs<R, false, true, false>(grid, s, m, ro, n_tau, r, cf, it, Q.p); break;
            case 3: launch_pairs<R, false, true, true>(grid, s, m, ro, n_tau, r, cf, it, Q.p); break;
            case 4: launch_pairs<R, true, false, false>(grid, s, m, ro, n_tau, r, cf, it, Q.p); break;
            case 5: launch_pairs<R, true, false, true>(grid, s, m, ro, n_tau, r, cf, it, Q.p); break;
            case 6: launch_pairs<R, true, true, false>(grid, s, m, ro, n_tau, r, cf, it, Q.p); break;
            default: launch_pairs<R, true, true, true>(grid, s, m, ro, n_tau, r, cf, it, Q.p); break;
            }
            BEM_LAUNCH_CHECK();
        }
        hipLaunchKernelGGL(dense_gather_kernel<C>, dim3((unsigned)N, (jt + 255) / 256), dim3(256),
                           0, s, Q.p, m->star_ptr.p, m->star_idx.p, ro.rank.p, ro.byrank.p, N,
                           (int)r0, jt, B);
        BEM_LAUNCH_CHECK();
    }
    {
        const unsigned nt = (unsigned)((N + 31) / 32);
        hipLaunchKernelGGL(dense_mirror_kernel<C>, dim3(nt, nt, 4), dim3(256), 0, s, ro.rank.p, N,
                           B);
        BEM_LAUNCH_CHECK();
    }
    if constexpr (std::is_same<R, float>::value)
        hipLaunchKernelGGL(dense_add_near_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256), 0,
                           s, m->nf_rowptr.p, m->nf_col.p, (const double2 *)nf.vals.p, m->nf_nnz,
                           N, B);
    else
        hipLaunchKernelGGL(dense_add_near64_kernel, dim3((unsigned)((N + 255) / 256)), dim3(256),
                           0, s, m->nf_rowptr.p, m->nf_col.p, (const double2 *)nf.vals.p,
                           m->nf_nnz, N, B);
    BEM_LAUNCH_CHECK();
    BEM_HIP(hipStreamSynchronize(s));   // Q and the table are released on return
}

}   // namespace

int64_t dense_bytes(const bem_mesh *m, bool fp64) {
    return 4 * m->N * m->N * (int64_t)(fp64 ? sizeof(double2) : sizeof(float2));
}
int64_t dense_assembly_scratch_bytes(const bem_mesh *m, bool fp64) {
    return dense_need_bytes(m->N, m->T, fp64) - dense_bytes(m, fp64);
}
int64_t dense_need_bytes(int64_t N, int64_t T, bool fp64) {
    const int64_t c = fp64 ? sizeof(double2) : sizeof(float2);
    return 4 * N * N * c + T * (int64_t)JT * 12 * c + 2 * N * (int64_t)sizeof(float2) +
           (2 * N + T) * (int64_t)sizeof(int32_t);   // vertex ranks, triangle order
}

void dense_assemble_into(bem_mesh *m, const NearOperator &nf, double2 k0, hipStream_t s,
                         bool fp64, DenseOperator &op) {
    const int64_t n2 = 2 * m->N;
    op.n2 = n2;
    op.T = m->T;
    op.fp64 = fp64;
    Timer tm(fp64 ? "dense_assemble_fp64" : "dense_assemble", s);
    if (fp64) {
        op.B.release();
        if (op.B64.n != (size_t)(n2 * n2)) op.B64.alloc((size_t)(n2 * n2));
        assemble_into<double>(m, nf, k0, op.B64.p, s);
    } else {
        op.B64.release();
        if (op.B.n != (size_t)(n2 * n2)) op.B.alloc((size_t)(n2 * n2));
        assemble_into<float>(m, nf, k0, op.B.p, s);
    }
}

std::unique_ptr<DenseOperator> dense_assemble(bem_mesh *m, const NearOperator &nf, double2 k0,
                                              double2 k1, double rho, hipStream_t s, bool fp64) {
    (void)k1;
    (void)rho;
    auto op = std::make_unique<DenseOperator>();
    dense_assemble_into(m, nf, k0, s, fp64, *op);
    return op;
}

namespace {

constexpr int MX_MAX_RHS = 32;   // right-hand sides per launch of the skinny product

constexpr int MX_RT = 2;        // 16-row tiles per wavefront
constexpr int MX_SPLITS = 32;   // ranges of K at most

// Ranges of K: all workgroups cost the same, so their number just fills whole
// rounds of resident ones (a last round of a few cannot draw the memory's rate;
// fixed ranges took 107 instead of 98 us on the 5 124-row complex128 operator).
template <class R, int NT> int64_t mx_range(int64_t M, int64_t Kp) {
    static std::mutex mu;
    static std::map<int, int> cache;   // device -> resident workgroups
    int dev = 0, slots = 0;
    BEM_HIP(hipGetDevice(&dev));
    {
        std::lock_guard<std::mutex> g(mu);
        int &c = cache[dev];
        if (c == 0) {
            int cus = 0, per = 0;
            BEM_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
            BEM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &per, (const void *)mx_gemv_kernel<R, MX_RT, NT>, 256, 0));
            c = std::max(1, cus * per);
        }
        slots = c;
    }
    constexpr int64_t STEP = mx_step<R, NT>();
    const int64_t rows = (M + 64 * MX_RT - 1) / (64 * MX_RT);
    int64_t best = Kp;
    double best_cost = 1e300;
    for (int ns = 1; ns <= MX_SPLITS; ns++) {
        const int64_t len = ((Kp + ns - 1) / ns + STEP - 1) / STEP * STEP;
        const double rounds = std::ceil((double)rows * ((Kp + len - 1) / len) / slots);
        const double cost = rounds * (len + 4.0 * STEP);   // + first loads and output
        if (cost < best_cost * (1 - 1e-9)) {
            best_cost = cost;
            best = len;
        }
    }
    return best;
}

// Scratch of a launch: prepared columns, then the partial sums of the ranges.
template <class R, int NT> int64_t mx_scratch(int64_t n2, int64_t klen) {
    const int64_t Kp = 2 * n2, nsplit = (Kp + klen - 1) / klen;
    return 16 * NT * (Kp * (int64_t)sizeof(R) + nsplit * n2 * (int64_t)sizeof(double));
}
template <class R, int NT> int64_t mx_scratch(int64_t n2) {
    return mx_scratch<R, NT>(n2, mx_range<R, NT>(n2, 2 * n2));
}

// nr <= 8 NT right-hand sides in one launch
template <class R, int NT>
void mx_launch(const R *B, int64_t n2, const double2 *x, double2 *y, int nr, DenseScratch &sc,
               hipStream_t s) {
    const int64_t M = n2, Kp = 2 * n2;
    const int64_t klen = mx_range<R, NT>(M, Kp);
    const int nsplit = (int)((Kp + klen - 1) / klen);
    DevBuf<float2> &buf = std::is_same<R, double>::value ? sc.wide[NT / 2] : sc.xs;
    const size_t need = (size_t)mx_scratch<R, NT>(n2, klen) / sizeof(float2);
    if (buf.n < need) buf.alloc(need);
    char *scratch = (char *)buf.p;
    R *XT = (R *)scratch;
    double *part = (double *)(scratch + 16 * NT * Kp * (int64_t)sizeof(R));
    hipLaunchKernelGGL(mx_prep_kernel<R>, dim3(8 * NT, (unsigned)((n2 + 255) / 256)), dim3(256), 0, s, x,
                       nr, n2, XT);
    BEM_LAUNCH_CHECK();
    {
        Timer tm(std::is_same<R, float>::value ? "dense_skinny_mfma" : "dense_skinny_mfma64", s);
        hipLaunchKernelGGL((mx_gemv_kernel<R, MX_RT, NT>),
                           dim3((unsigned)((M + 64 * MX_RT - 1) / (64 * MX_RT)), nsplit), dim3(256), 0, s,
                           B, XT, part, M, Kp, klen);
        BEM_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(mx_reduce_kernel, dim3((unsigned)((M * 8 * NT + 255) / 256)), dim3(256), 0, s,
                       (const double2 *)part, nsplit, M, 8 * NT, nr, y);
    BEM_LAUNCH_CHECK();
}

// nr <= MX_MAX_RHS right-hand sides
template <class T>
void mx_apply(const T *B, int64_t n2, const double2 *x, double2 *y, int nr, DenseScratch &sc,
              hipStream_t s) {
    if (nr <= 8) mx_launch<T, 1>(B, n2, x, y, nr, sc, s);
    else if (nr <= 16) mx_launch<T, 2>(B, n2, x, y, nr, sc, s);
    else mx_launch<T, 4>(B, n2, x, y, nr, sc, s);
}

// right-hand sides of the next launch when `left` remain: 24 to 32 share one (four
// column tiles), below, 16 and the rest apart keep the FP64 sums (20 vectors at 10 242
// vertices 1.67 ms, against 1.22 for 24 to 32 together)
int mx_group(int left) { return left >= 24 ? std::min(left, MX_MAX_RHS) : std::min(left, 16); }

}   // namespace

int64_t dense_mx_scratch_bytes(int64_t N, int R, bool fp64) {
    const int64_t n2 = 2 * N;
    if (R < 2) return 0;
    if (fp64)
        return mx_scratch<double, 1>(n2) + (R > 8 ? mx_scratch<double, 2>(n2) : 0) +
               (R >= 24 ? mx_scratch<double, 4>(n2) : 0);
    int64_t b = mx_scratch<float, 1>(n2);
    if (R > 8) b = std::max(b, mx_scratch<float, 2>(n2));
    if (R >= 24) b = std::max(b, mx_scratch<float, 4>(n2));
    return b;
}

namespace {

template <int NR>
void launch_gemv(const DenseOperator &op, const float2 *xs, double2 *y, hipStream_t s) {
    const int64_t rows = (int64_t)gv_waves<NR>() * GV_RW;   // per workgroup
    hipLaunchKernelGGL(dense_gemv_kernel<NR>, dim3((unsigned)((op.n2 + rows - 1) / rows)),
                       dim3(64 * gv_waves<NR>()), 0, s, op.B.p, op.n2, xs, y, op.n2);
}

// Small operators are bound by their launches: the product on the vector units has
// one less than that on the matrix units (two against three).  us for 6, 7 and 8
// vectors, vector and matrix units: 324 rows 13.5 13.9 15.3 and 16.5; 504 rows 13.5
// 14.1 15.6 and 16.5; 724 rows 15.4 16.9 18.8 and 16.4.  complex128, two vectors, two
// single products against one on the matrix units: 324 rows 24.0 and 25.5, 504 rows
// 28.8 and 25.4.
constexpr int64_t GEMV_SMALL_ROWS = 600, GEMV64_SMALL_ROWS = 400;

// Vectors up to which the complex64 product runs on the vector units: all eight of a
// launch on small operators, else five, or seven on 11 000 rows and more.  The matrix
// units take the same time for any number up to 8.  us, vector units for 5, 6, 7 and
// 8 vectors, and matrix units: 5 124 rows 51 66 70 113 and 61; 8 824 rows 137 170 182
// 255 and 147; 10 584 rows 179 202 215 298 and 204; 11 524 rows 212 225 239 329 and
// 244; 12 504 rows 275 262 279 452 and 277; 16 824 rows 422 480 511 738 and 502; 20 484
// rows 643 637 693 1 051 and 733.  (Six and seven run in rounds of 8 192 rows: on
// 5 784 to 8 004 rows, just below a round, they are the faster form as well, 106 and
// 111 against 128 us on 8 004.)
int gemv_max_rhs(int64_t n2) {
    const int line = tuning().dense_skinny_min_rhs;
    if (line != DENSE_SKINNY_BY_COUNT) return line - 1;   // the caller's choice
    return n2 <= GEMV_SMALL_ROWS ? 8 : n2 >= 11000 ? 7 : 5;
}
constexpr int GEMV_RHS = 8;   // vectors of a launch on the vector units at most

}   // namespace

void dense_gemv(const DenseOperator &op, const double2 *x, double2 *y, int R, DenseScratch &sc,
                hipStream_t s) {
    const int64_t n2 = op.n2;
    for (int r0 = 0; r0 < R;) {
        const double2 *xr = x + r0 * n2;
        double2 *yr = y + r0 * n2;
        int nr = R - r0;
        if (nr > gemv_max_rhs(n2)) {
            nr = mx_group(nr);
            mx_apply((const float *)op.B.p, n2, xr, yr, nr, sc, s);
        } else {
            nr = std::min(nr, GEMV_RHS);
            const int64_t cnt = nr * n2;
            DevBuf<float2> &xs = sc.xs;
            if (xs.n < (size_t)cnt) xs.alloc((size_t)cnt);
            hipLaunchKernelGGL(to_c64_kernel, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, s, xr,
                               xs.p, cnt);
            BEM_LAUNCH_CHECK();
            Timer tm("dense_gemv", s);
            switch (nr) {
            case 1:
                hipLaunchKernelGGL(dense_gemv1_kernel,
                                   dim3((unsigned)((n2 + 4 * GEMV1_ROWS - 1) / (4 * GEMV1_ROWS))),
                                   dim3(256), 0, s, op.B.p, n2, xs.p, yr);
                break;
            case 2: launch_gemv<2>(op, xs.p, yr, s); break;
            case 3: launch_gemv<3>(op, xs.p, yr, s); break;
            case 4: launch_gemv<4>(op, xs.p, yr, s); break;
            case 5: launch_gemv<5>(op, xs.p, yr, s); break;
            case 6: launch_gemv<6>(op, xs.p, yr, s); break;
            case 7: launch_gemv<7>(op, xs.p, yr, s); break;
            default: launch_gemv<8>(op, xs.p, yr, s); break;
            }
            BEM_LAUNCH_CHECK();
        }
        r0 += nr;
    }
}

// smallest split-K chunk: at most about 40 partial products, none below 256 k
static int gemm_kmin(int64_t Kp) {
    return (int)std::min<int64_t>(1024, std::max<int64_t>(256, (Kp / 40 + GK - 1) / GK * GK));
}

int64_t dense_gemm_scratch_bytes(const bem_mesh *m, int R) {
    const int64_t M = 2 * m->N, Kp = 2 * M;
    const int64_t Np = 2 * (((int64_t)R + 63) / 64) * 64, kmin = gemm_kmin(Kp),
                  nchunks = (Kp + kmin - 1) / kmin;
    return (Kp * Np + nchunks * M * Np) * (int64_t)sizeof(float);
}

namespace {

// Split-K chunk of the MFMA product: all workgroups cost the same, so the chunk
// (a multiple of the K step) that makes rounds of resident workgroups times its
// length, with three steps for the first loads and the output, least; longer
// chunks at equal cost.
int gemm_kchunk(int64_t mtiles, int64_t Kp) {
    static int slots = 0;
    if (slots == 0) {
        int dev = 0, cus = 0, per = 0;
        BEM_HIP(hipGetDevice(&dev));
        BEM_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        BEM_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, gemm_mfma_kernel, 256, 0));
        slots = std::max(1, cus * std::max(per, 1));
    }
    int best = GKC;
    double best_cost = 1e300;
    for (int kc = GKC; kc >= gemm_kmin(Kp); kc -= GK) {
        const int64_t nch = (Kp + kc - 1) / kc;
        const double cost = std::ceil((double)(mtiles * nch) / slots) * (std::min<int64_t>(kc, Kp) + 3 * GK);
        if (cost < best_cost * (1 - 1e-9)) {
            best_cost = cost;
            best = kc;
        }
    }
    return best;
}

}   // namespace

void dense_apply(const DenseOperator &op, const double2 *x, double2 *y, int R,
                 DenseScratch &sc, hipStream_t s, const TuneEntry *forced) {
    if (op.fp64) {
        for (int r0 = 0; r0 < R;) {
            int nr = mx_group(R - r0);
            if (nr == 2 && op.n2 <= GEMV64_SMALL_ROWS) nr = 1;
            const double2 *xr = x + r0 * op.n2;
            double2 *yr = y + r0 * op.n2;
            if (nr > 1) {
                mx_apply((const double *)op.B64.p, op.n2, xr, yr, nr, sc, s);
            } else {
                Timer tm("dense_gemv_fp64", s);
                hipLaunchKernelGGL(dense_gemv64_kernel,
                                   dim3((unsigned)((op.n2 + 4 * G64_RW - 1) / (4 * G64_RW))), dim3(256),
                                   0, s, op.B64.p, op.n2, xr, yr);
                BEM_LAUNCH_CHECK();
            }
            r0 += nr;
        }
        return;
    }
    const TuneEntry te = forced ? *forced : tune_lookup(op.T, R);
    if (R >= te.gemm_min) dense_gemm(op, x, y, R, s);
    else dense_gemv(op, x, y, R, sc, s);
}

void dense_gemm(const DenseOperator &op, const double2 *x, double2 *y, int R, hipStream_t s) {
    const int64_t M = op.n2, K = op.n2, Kp = 2 * K;
    const int Rp = ((R + 63) / 64) * 64, Np = 2 * Rp;
    const int kchunk = gemm_kchunk(((M + GM - 1) / GM) * (Np / GN), Kp);
    const int nchunks = (int)((Kp + kchunk - 1) / kchunk);
    const size_t nx = (size_t)(Kp * Np), ny = (size_t)nchunks * M * Np;
    // the operator's workspace when no other call holds it, else our own
    DenseOperator::GemmWork &w = *op.gw;
    std::unique_lock<std::mutex> lk(w.mu, std::try_to_lock);
    DevBuf<float> own_x, own_y;
    float *Xp, *Yp;
    if (lk.owns_lock()) {
        if (w.Xp.n < nx) w.Xp.alloc(nx);
        if (w.Yp.n < ny) w.Yp.alloc(ny);
        w.held = w.Xp.bytes() + w.Yp.bytes();
        Xp = w.Xp.p;
        Yp = w.Yp.p;
    } else {
        own_x.alloc(nx);
        own_y.alloc(ny);
        Xp = own_x.p;
        Yp = own_y.p;
    }
    hipLaunchKernelGGL(mx_prep_kernel<float>, dim3(Rp, (unsigned)((K + 255) / 256)), dim3(256), 0, s, x, R,
                       K, Xp);
    BEM_LAUNCH_CHECK();
    {
        Timer tm("dense_gemm_mfma", s);
        hipLaunchKernelGGL(gemm_mfma_kernel,
                           dim3((unsigned)((M + GM - 1) / GM), Np / GN, nchunks), dim3(256), 0, s,
                           (const float *)op.B.p, Xp, Yp, M, Kp, Np, kchunk);
        BEM_LAUNCH_CHECK();
    }
    hipLaunchKernelGGL(gemm_reduce_kernel, dim3((R + 31) / 32, (unsigned)((M + 31) / 32)), dim3(256), 0, s,
                       Yp, nchunks, M, Np, R, y);
    BEM_LAUNCH_CHECK();
    BEM_HIP(hipStreamSynchronize(s));   // the workspace is free again, or released
}

namespace {
std::atomic<uint64_t> g_share_tick{0};   // last-use stamps comparable across meshes
}

int64_t DenseShare::bytes() {
    std::lock_guard<std::mutex> g(mu);
    int64_t b = 0;
    for (const auto &kv : ops) b += kv.second.op->bytes();
    return b;
}

int64_t DenseShare::idle_bytes() {
    std::lock_guard<std::mutex> g(mu);
    int64_t b = 0;
    for (const auto &kv : ops)
        if (kv.second.op.use_count() == 1) b += kv.second.op->bytes();
    return b;
}

uint64_t DenseShare::oldest_idle() {
    std::lock_guard<std::mutex> g(mu);
    uint64_t t = UINT64_MAX;
    for (const auto &kv : ops)
        if (kv.second.op.use_count() == 1) t = std::min(t, kv.second.last);
    return t;
}

int64_t DenseShare::evict_idle_lru() {
    std::shared_ptr<DenseOperator> drop;   // freed outside the lock
    {
        std::lock_guard<std::mutex> g(mu);
        auto victim = ops.end();
        for (auto it = ops.begin(); it != ops.end(); ++it)
            if (it->second.op.use_count() == 1 &&
                (victim == ops.end() || it->second.last < victim->second.last))
                victim = it;
        if (victim == ops.end()) return 0;
        drop = std::move(victim->second.op);
        ops.erase(victim);
    }
    return drop->bytes();
}

namespace {

__global__ __launch_bounds__(256) void dense_round_kernel(const double2 *__restrict__ a,
                                                          float2 *__restrict__ b, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * 256)
        b[i] = make_float2((float)a[i].x, (float)a[i].y);
}

// into `op` (its complex64 buffer reused when it has the size)
void dense_round_into(const DenseOperator &d64, DenseOperator &o, hipStream_t s) {
    DenseOperator *op = &o;
    op->n2 = d64.n2;
    op->T = d64.T;
    op->fp64 = false;
    op->B64.release();
    const int64_t n = d64.n2 * d64.n2;
    if (op->B.n != (size_t)n) op->B.alloc((size_t)n);
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 16384);
    hipLaunchKernelGGL(dense_round_kernel, dim3((unsigned)blocks), dim3(256), 0, s, d64.B64.p,
                       op->B.p, n);
    BEM_LAUNCH_CHECK();
}

std::unique_ptr<DenseOperator> dense_round(const DenseOperator &d64, hipStream_t s) {
    auto op = std::make_unique<DenseOperator>();
    dense_round_into(d64, *op, s);
    return op;
}

}   // namespace

const DenseOperator &dense_get_rounded(bem_mesh *m, double2 k0, double2 k1, double rho,
                                       hipStream_t s, int s1, const ObjMaterials *om) {
    const NearKey key = near_key(m, k0, k1, rho, s1, om);
    auto it = m->dense_rounded_cache.find(key);
    if (it != m->dense_rounded_cache.end()) return *it->second;
    const DenseOperator &d64 = dense_get(m, k0, k1, rho, s, s1, om, true);
    if (!m->dense_rounded_cache.empty()) m->dense_rounded_cache.clear();   // one at a time
    auto op = dense_round(d64, s);
    auto &ref = *op;
    m->dense_rounded_cache.emplace(key, std::move(op));
    return ref;
}

std::shared_ptr<const DenseOperator> dense_share_get(bem_mesh *m, double2 k0, double2 k1,
                                                     double rho, hipStream_t s, int s1,
                                                     const ObjMaterials *om, int kind) {
    DenseShare &sh = *m->dense_share;
    const DenseShare::Key key{near_key(m, k0, k1, rho, s1, om), kind};
    {
        std::unique_lock<std::mutex> lk(sh.mu);
        for (;;) {
            auto it = sh.ops.find(key);
            if (it != sh.ops.end()) {
                it->second.last = ++g_share_tick;
                return it->second.op;
            }
            if (!sh.building.count(key)) break;
            sh.cv.wait(lk);   // another replica assembles it
        }
        sh.building.insert(key);
    }
    // an idle operator of the same kind that the `keep` rule would drop gives
    // its buffer to the new one (no device free and allocation per new
    // wavenumber)
    std::shared_ptr<DenseOperator> op;
    {
        std::lock_guard<std::mutex> g(sh.mu);
        int idle = 0;
        auto victim = sh.ops.end();
        for (auto it = sh.ops.begin(); it != sh.ops.end(); ++it)
            if (it->second.op.use_count() == 1) {
                idle++;
                if (it->first.second == kind &&
                    (victim == sh.ops.end() || it->second.last < victim->second.last))
                    victim = it;
            }
        if (idle >= sh.keep && victim != sh.ops.end()) {
            op = std::move(victim->second.op);
            sh.ops.erase(victim);
        }
    }
    try {
        if (!op) op = std::make_shared<DenseOperator>();
        if (kind == DENSE_C64_ROUNDED) {
            // from the shared complex128 operator (held until rounded)
            const auto d64 = dense_share_get(m, k0, k1, rho, s, s1, om, DENSE_C128);
            dense_round_into(*d64, *op, s);
            BEM_HIP(hipStreamSynchronize(s));
        } else {
            const NearOperator &nf = nearfield_get(m, k0, k1, rho, s, s1, om);
            dense_assemble_into(m, nf, k0, s, kind == DENSE_C128, *op);
        }
    } catch (...) {
        std::lock_guard<std::mutex> g(sh.mu);
        sh.building.erase(key);
        sh.cv.notify_all();
        throw;
    }
    std::vector<std::shared_ptr<DenseOperator>> drop;   // freed outside the lock
    {
        std::lock_guard<std::mutex> g(sh.mu);
        sh.building.erase(key);
        sh.ops[key] = DenseShare::Entry{op, ++g_share_tick};
        // keep at most `keep` operators beside those in use
        for (;;) {
            int idle = 0;
            auto victim = sh.ops.end();
            for (auto it = sh.ops.begin(); it != sh.ops.end(); ++it)
                if (it->second.op.use_count() == 1) {   // the new one is held by `op`
                    idle++;
                    if (victim == sh.ops.end() || it->second.last < victim->second.last)
                        victim = it;
                }
            if (idle < sh.keep || victim == sh.ops.end()) break;
            drop.push_back(std::move(victim->second.op));
            sh.ops.erase(victim);
        }
        sh.cv.notify_all();
    }
    return op;
}

const DenseOperator &dense_get(bem_mesh *m, double2 k0, double2 k1, double rho, hipStream_t s,
                               int s1, const ObjMaterials *om, bool fp64) {
    const NearKey key = near_key(m, k0, k1, rho, s1, om);
    auto &cache = fp64 ? m->dense64_cache : m->dense_cache;
    auto it = cache.find(key);
    if (it != cache.end()) return *it->second;
    const NearOperator &nf = nearfield_get(m, k0, k1, rho, s, s1, om);
    // one resident dense operator per mesh unless memory allows more
    const int64_t need = dense_bytes(m, fp64) + dense_assembly_scratch_bytes(m, fp64) +
                         (int64_t)(1ll << 30);
    size_t free_b = 0, total_b = 0;
    BEM_HIP(hipMemGetInfo(&free_b, &total_b));
    while ((!m->dense_cache.empty() || !m->dense64_cache.empty()) && (int64_t)free_b < need) {
        auto &victim = m->dense64_cache.empty() ? m->dense_cache : m->dense64_cache;
        victim.erase(victim.begin());
        BEM_HIP(hipMemGetInfo(&free_b, &total_b));
    }
    if ((int64_t)free_b < need)
        fail(BEM_E_NOMEM, "dense operator of " + std::to_string(dense_bytes(m, fp64)) +
                              " bytes does not fit in device memory");
    auto op = dense_assemble(m, nf, k0, k1, rho, s, fp64);
    auto &ref = *op;
    cache.emplace(key, std::move(op));
    return ref;
}

}   // namespace bem
