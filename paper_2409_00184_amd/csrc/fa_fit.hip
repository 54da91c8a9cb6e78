// Least-squares fit of micro-models to grid samples and its error map
// (the model(NCP, degree) step of the adaptive encoding, Sec. 4.2.1 and
// Alg. 1; Error(NCP) of Eq. 4).
//
// The design matrix of a block is the Kronecker product of the per-axis
// collocation matrices B_a[i][j] = N_j(u_i) on the decode grid, so the
// least-squares lattice is P = y x_1 X_x x_2 X_y x_3 X_z with the
// pseudo-inverses X_a = B_a^+ = (B_a^T B_a)^{-1} B_a^T (n_a x R_a).  Each X_a
// is built in FP64: the basis at the
// grid points in FP64 (same spans as the decode), the band Gram matrix
// B_a^T B_a (half-bandwidth p), its band Cholesky factor, and one
// forward/backward solve per grid point.  Forming X_a first and applying it
// as a dense contraction keeps the error proportional to the condition
// number of B_a, where solving the normal equations on B^T y would square
// it (the collocation matrix of NCP close to R on the uniform grid is
// badly conditioned).  Three kernels, FP64 throughout:
//   fit_pinv: X_a of every (block, axis), one wave each, into the caller's
//           workspace,
//   fit_zy: U[b][x] = X_y y[b][x] X_z^T for every x slice (one wave per slice,
//           both products in registers, U in the workspace),
//   fit_x:  P[b] = X_x U[b], a product over the lattice's contiguous (j, k),
// the dense products on the FP64 matrix cores (v_mfma_f64_16x16x4f64), and
// the lattice rounded to FP32 once.
// residual kernel: one workgroup per block reduces y - f to (max |r|,
// sqrt(mean r^2)) in a fixed order (deterministic).
#include <algorithm>

#include "fa_device.hpp"
#include "fa_internal.hpp"

namespace fa {
namespace {

constexpr int kFitThreads = 256;
constexpr int kFitR = 64;  // grid points per axis a fit supports
constexpr int kFitN = FA_MAX_NCP;

// FP64 basis of degree p <= 3 on span s: N[r] = N_{s-p+r,p}(u), triangular
// form of the de Boor recursion.
__device__ __forceinline__ void basis64(const float *t, int s, double u, int p, double (&N)[4]) {
    double left[4] = {0, 0, 0, 0}, right[4] = {0, 0, 0, 0};
    N[0] = 1.0;
    N[1] = N[2] = N[3] = 0.0;
#pragma unroll
    for (int k = 1; k <= 3; ++k) {
        if (k > p) break;
        left[k] = u - (double)t[s + 1 - k];
        right[k] = (double)t[s + k] - u;
        double saved = 0.0;
#pragma unroll
        for (int r = 0; r < k; ++r) {
            const double q = N[r] / (right[r + 1] + left[k - r]);
            N[r] = saved + right[r + 1] * q;
            saved = left[k - r] * q;
        }
        N[k] = saved;
    }
}

// One wave per pseudo-inverse, lane i solving for grid point i, so the
// build needs no barrier and four of them share a CU.  What bounds it is the
// serial chain of the band factorisation and of the two substitutions along
// j: the factor keeps reciprocal diagonals (one product a step where a
// division stood), and the last p values of a recursion stay in registers.
struct PinvSmem {
    double N[kFitR][4];
    int first[kFitN + 8];    // first grid point on span s or a later one
    double G[kFitN + 1][4];  // G[j][d] = G(j, j + d)
    double L[kFitN + 3][4];  // L[j][d] = L(j, j - d), L[j][0] = 1 / L(j, j); zero rows after n
    double Z[kFitN][kFitR];  // forward substitution, column i
};

// X = B^+ of one axis (n functions of degree p, knots t, R grid points) as
// X[j * kFitR + i], j < n; columns i >= R are zero.
__device__ void build_pinv(PinvSmem &w, const float *t, int n, int p, int R, double *X) {
    const int i = threadIdx.x;  // one wave
    double Nv[4] = {0.0, 0.0, 0.0, 0.0};
    int s = 0;
    if (i < R) {
        const float uf = grid_pos(i, R);
        s = span_search(n, p, t, uf);
        basis64(t, s, (double)uf, p, Nv);
    }
    // first[t] = i for the spans t after the previous point's up to this one's
    const int before = __shfl_up(s, 1);
    if (i < R)
        for (int t = i == 0 ? 0 : before + 1; t <= s; ++t) w.first[t] = i;
    if (i == R - 1)
        for (int t = s + 1; t <= n + p; ++t) w.first[t] = R;
#pragma unroll
    for (int r = 0; r < 4; ++r) w.N[i][r] = Nv[r];
    if (i < 3)
#pragma unroll
        for (int d = 0; d < 4; ++d) w.L[n + i][d] = 0.0;
    __syncthreads();
    for (int e = i; e < n * 4; e += kWave) {
        const int j = e >> 2, d = e & 3;
        double g = 0.0;
        // points on spans j + d .. j + p, in order: on span t, function j is
        // N[j - t + p]
        if (d <= p)
            for (int t = j + d; t <= j + p; ++t)
                for (int q = w.first[t]; q < w.first[t + 1]; ++q)
                    g += w.N[q][j - t + p] * w.N[q][j - t + p + d];
        w.G[j][d] = g;
    }
    __syncthreads();
    {  // band Cholesky G = L L^T: row j from rows j - 1 .. j - 3, every lane the same
        double a1[4] = {0, 0, 0, 0}, a2[4] = {0, 0, 0, 0}, a3[4] = {0, 0, 0, 0};  // L rows j-1, j-2, j-3
        for (int j = 0; j < n; ++j) {
            double c[4] = {0.0, 0.0, 0.0, 0.0};
            if (p >= 3 && j >= 3) c[3] = w.G[j - 3][3] * a3[0];
            if (p >= 2 && j >= 2) c[2] = (w.G[j - 2][2] - c[3] * a2[1]) * a2[0];
            if (j >= 1) c[1] = (w.G[j - 1][1] - c[3] * a1[2] - c[2] * a1[1]) * a1[0];
            c[0] = rsqrt(w.G[j][0] - c[3] * c[3] - c[2] * c[2] - c[1] * c[1]);
            if (i < 4) w.L[j][i] = i == 0 ? c[0] : (i == 1 ? c[1] : (i == 2 ? c[2] : c[3]));
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                a3[d] = a2[d];
                a2[d] = a1[d];
                a1[d] = c[d];
            }
        }
    }
    __syncthreads();
    // column i of X solves G x = B[i, :]^T (non-zero at s_i - p .. s_i)
    const int j0 = s - p;
    double z1 = 0.0, z2 = 0.0, z3 = 0.0;
#pragma unroll 4
    for (int j = 0; j < n; ++j) {  // forward: L z = rhs
        const int r = j - j0;
        double v = r == 0 ? Nv[0] : (r == 1 ? Nv[1] : (r == 2 ? Nv[2] : (r == 3 ? Nv[3] : 0.0)));
        v = v - w.L[j][3] * z3 - w.L[j][2] * z2 - w.L[j][1] * z1;
        v = (i < R && r >= 0) ? v * w.L[j][0] : 0.0;
        w.Z[j][i] = v;
        z3 = z2;
        z2 = z1;
        z1 = v;
    }
    double x1 = 0.0, x2 = 0.0, x3 = 0.0;
#pragma unroll 4
    for (int j = n - 1; j >= 0; --j) {  // backward: L^T x = z
        double v = w.Z[j][i] - w.L[j + 3][3] * x3 - w.L[j + 2][2] * x2 - w.L[j + 1][1] * x1;
        v = i < R ? v * w.L[j][0] : 0.0;
        X[j * kFitR + i] = v;
        x3 = x2;
        x2 = x1;
        x1 = v;
    }
}

__device__ __forceinline__ const float *axis_knots(const float *knots, const fa_block &b, int a) {
    const float *t = knots + b.knot_off;
    if (a >= 1) t += b.ncp[0] + b.degree[0] + 1;
    if (a >= 2) t += b.ncp[1] + b.degree[1] + 1;
    return t;
}

constexpr int64_t kPinvStride = (int64_t)kFitN * kFitR;  // doubles per (block, axis)

__device__ __forceinline__ int uni32(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Xg[(b * 3 + a) * kPinvStride + j * kFitR + i] = X_a[j][i]
__global__ __launch_bounds__(kWave) void fit_pinv_kernel(const fa_block *blocks, int nblocks,
                                                         const float *knots, int r0, int r1,
                                                         int r2, double *Xg) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    PinvSmem &sm = *reinterpret_cast<PinvSmem *>(smem_raw);
    for (int64_t item = blockIdx.x; item < (int64_t)nblocks * 3; item += gridDim.x) {
        const int bi = (int)(item / 3), a = (int)(item - (int64_t)bi * 3);
        const fa_block b = blocks[bi];
        const int n = a == 0 ? b.ncp[0] : (a == 1 ? b.ncp[1] : b.ncp[2]);
        const int Ra = a == 0 ? r0 : (a == 1 ? r1 : r2);
        build_pinv(sm, axis_knots(knots, b, a), n, b.degree[0], Ra, Xg + item * kPinvStride);
        __syncthreads();
    }
}

// knot j of a clamped uniform vector: t_j = 0 (j <= p), 1 (j >= n), else
// fl32((j - p) / (n - p))
__device__ __forceinline__ float candidate_knot(int j, int n, int p) {
    if (j <= p) return 0.0f;
    if (j >= n) return 1.0f;
    return (float)(j - p) / (float)(n - p);
}

// The search's candidates share one knot vector per NCP (every block, every
// axis), so their pseudo-inverses are built once per (candidate, axis), all
// candidates in one launch: knots of candidate c (n = ncp_lo + c) at
// kall + c * kstride (x, y, z vectors back to back), X_a at
// xall + (c * 3 + a) * kPinvStride.
__global__ __launch_bounds__(kWave) void pinv_candidates_kernel(float *kall, int ncp_lo, int ncand,
                                                                int p, int kstride, int r0, int r1,
                                                                int r2, double *xall) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    PinvSmem &sm = *reinterpret_cast<PinvSmem *>(smem_raw);
    for (int item = blockIdx.x; item < ncand * 3; item += gridDim.x) {
        const int c = item / 3, a = item - 3 * c, n = ncp_lo + c, nk = n + p + 1;
        float *t = kall + (int64_t)c * kstride + a * nk;
        for (int j = threadIdx.x; j < nk; j += kWave) t[j] = candidate_knot(j, n, p);
        __syncthreads();
        const int Ra = a == 0 ? r0 : (a == 1 ? r1 : r2);
        build_pinv(sm, t, n, p, Ra, xall + (int64_t)item * kPinvStride);
        __syncthreads();
    }
}

// FP64 matrix-core contraction tiles: v_mfma_f64_16x16x4f64 takes
// A[l%16][l/16] and B[l/16][l%16] from lane l and returns D[4r + l/16][l%16]
// in component r (layout checked on the device).
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Arguments of the two products of a fit.  Entry e of `blocks` is fitted to
// the samples of block e % nsrc; its pseudo-inverses start at X + (e / nsrc)
// * xcand + (e % nsrc) * xstride, its intermediate at T + e * tstride.
struct FitArgs {
    const fa_block *blocks;
    int nblocks, nsrc;
    int r0, r1, r2, max_n;
    const float *y;
    const double *X;
    int64_t xcand, xstride;
    double *T;
    int64_t tstride;
    float *ctrl;
};

__device__ __forceinline__ const double *fit_x_of(const FitArgs &a, int bi) {
    return a.X + (bi / a.nsrc) * a.xcand + (bi % a.nsrc) * a.xstride;
}

constexpr uint32_t kDeadFit = 0x40000000u;      // offset beyond every buffer (also two or three times)
constexpr int kZyWaves = 4;                     // waves per fit_zy workgroup
constexpr int kOpSteps = kFitR / 4;             // K steps of a 64-long contraction
constexpr int kOpTile = kOpSteps * kWave;       // doubles of one 16-row operand table

// U[x][j][k] = sum_y X_y[j][y] sum_z X_z[k][z] y[x][y][z] of one x slice,
// both products on the FP64 matrix cores without leaving the wave's
// registers: the z product of a 16-row band of the slice leaves Z[yy][k] in
// exactly the B operand of four K steps of the y product (component r of
// band t: row 16t + 4r + l/16, column l%16).  A lane reads four consecutive
// samples of its rows with one 16-byte load (the K order of the z product
// is permuted to z = 16q + 4(l/16) + j), so a slice goes from memory to U
// without LDS or a barrier; the operands of X_z and X_y sit in LDS in lane
// order.
//
// Bound by the FP64 matrix cores (64 cycles per product, n_z / 16 tiles of
// 16 NT + 16 NJ products a slice), busy 61% of the time: 260 us for 512
// blocks of 64^3 at NCP 32, where a pair of kernels that kept T[k][x][y]
// between the products (64 / n times larger than U) and staged the operands
// of both through LDS between barriers took 850 us with the x product in it
// (now 108 us, fit_x below).
template <int NT, int NJ>
__device__ __forceinline__ void fit_zy_slice(const double *oz, const double *oy, u32x4 (&s)[4][4],
                                             int nq, int nk, int ny, int nz, int lane,
                                             __amdgpu_buffer_rsrc_t U, uint32_t u0) {
    for (int kt = 0; kt < nk; ++kt) {
        // opaque to the compiler, so that it keeps neither the y operands nor
        // (below) the converted samples in registers from k tile to k tile
        asm volatile("" : "+v"(lane));
        const double *bz = oz + kt * kOpTile + lane;
        f64x4 Z[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) Z[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q >= nq) break;  // uniform: no samples there
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double b = bz[(4 * q + j) * kWave];
#pragma unroll
                for (int t = 0; t < NT; ++t)  // independent chains
                    Z[t] = mfma64((double)__uint_as_float(s[t][q][j]), b, Z[t]);
            }
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(s[t][q]));
        f64x4 Y[NJ];
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt) Y[jt] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int jt = 0; jt < NJ; ++jt)
                    Y[jt] = mfma64(oy[jt * kOpTile + (4 * t + r) * kWave + lane], Z[t][r], Y[jt]);
        const int j = lane >> 4, k = 16 * kt + (lane & 15);
        const uint32_t at = k < nz ? (uint32_t)(j * nz + k) * 8u : kDeadFit;
#pragma unroll
        for (int jt = 0; jt < NJ; ++jt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                __builtin_amdgcn_raw_buffer_store_b64(
                    __builtin_bit_cast(u32x2, (double)Y[jt][r]), U,
                    16 * jt + 4 * r + j < ny ? at : kDeadFit,
                    u0 + (uint32_t)((16 * jt + 4 * r) * nz) * 8u, 0);
            }
    }
}

template <int NT, int NJ>
__device__ __forceinline__ void fit_zy_block(const FitArgs &a, int bi, int x0, int x1, int ny, int nz,
                                             const double *oz, const double *oy) {
    const int wave = uni32(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int gq = lane >> 4, l16 = lane & 15;
    const int r1 = a.r1, r2 = a.r2;
    const uint32_t slice = (uint32_t)r1 * (uint32_t)r2 * 4u;
    // rows and columns outside the slice load at a vector offset beyond the
    // resource and read as zero (the range check need not see the scalar
    // offset, so nothing relies on that one leaving the resource)
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(
        a.y + (int64_t)(bi % a.nsrc) * a.r0 * r1 * r2, (uint32_t)a.r0 * slice);
    uint32_t row[4], col[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        row[t] = 16 * t + l16 < r1 ? (uint32_t)((16 * t + l16) * r2) * 4u : kDeadFit;
        col[t] = 16 * t + 4 * gq < r2 ? (uint32_t)(16 * t + 4 * gq) * 4u : kDeadFit;
    }
    const bool ragged = (r2 & 3) != 0;
    auto load = [&](uint32_t at, u32x4(&s)[4][4]) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                s[t][q] = __builtin_amdgcn_raw_buffer_load_b128(rs, row[t] + col[q] + at, 0, 0);
            }
    };
    auto trim = [&](u32x4(&s)[4][4]) {  // the part of the last load past its row's end
        if (!ragged) return;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (16 * q + 4 * gq + j >= r2) s[t][q][j] = 0u;
    };
    const int nq = (r2 + 15) >> 4, nk = (nz + 15) >> 4;
    const uint32_t ub = (uint32_t)(ny * nz) * 8u;  // bytes of U of a slice
    const __amdgpu_buffer_rsrc_t U = make_rsrc(a.T + (int64_t)bi * a.tstride, (uint32_t)a.r0 * ub);
    u32x4 cur[4][4], nxt[4][4];
    int x = x0 + wave;
    if (x < x1) load((uint32_t)x * slice, cur);
    for (; x < x1; x += kZyWaves) {
        // the next slice, in flight during all of this one (after the last one
        // nothing: the vector offset is dead)
        load(x + kZyWaves < x1 ? (uint32_t)(x + kZyWaves) * slice : kDeadFit, nxt);
        trim(cur);
        fit_zy_slice<NT, NJ>(oz, oy, cur, nq, nk, ny, nz, lane, U, (uint32_t)x * ub);
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) cur[t][q] = nxt[t][q];
    }
}

// One workgroup per (block, group of x slices); wave w takes slices w, w + 4, ...
template <int NT>
__global__ __launch_bounds__(kZyWaves * 64, 2) void fit_zy_kernel(FitArgs a, int xgroup) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tid = threadIdx.x;
    const int groups = (a.r0 + xgroup - 1) / xgroup;
    // a block's groups on one XCD: its L2 then holds their pseudo-inverses
    const int wg = xcd_order(blockIdx.x, gridDim.x), bi = wg / groups;
    const int x0 = (wg - bi * groups) * xgroup;
    const int x1 = min(a.r0, x0 + xgroup);
    const fa_block &b = a.blocks[bi];
    const int ny = uni32(b.ncp[1]), nz = uni32(b.ncp[2]);
    // the workspace has no room for it (the lattice is left as is), or the
    // Gram matrix is singular (fit_x_kernel writes the lattice)
    if (nz > a.max_n || ny > a.r1) return;
    const int nk = (nz + 15) >> 4, nj = (ny + 15) >> 4;
    double *oz = reinterpret_cast<double *>(smem_raw), *oy = oz + nk * kOpTile;
    const double *X = fit_x_of(a, bi);
    // X_z[k][z] to the z product's B operand (step (q, j), lane), X_y[j][y]
    // to the y product's A operand (step (t, r), lane); zero outside
    for (int e = tid; e < (nk + nj) * kOpTile; e += kZyWaves * 64) {
        const bool isz = e < nk * kOpTile;
        const int f = isz ? e : e - nk * kOpTile;
        const int step = (f >> 6) & (kOpSteps - 1), g = (f >> 4) & 3;
        const int row = (f / kOpTile) * 16 + (f & 15);
        const int c = isz ? 16 * (step >> 2) + 4 * g + (step & 3) : 4 * step + g;
        const bool in = isz ? (row < nz && c < a.r2) : (row < ny && c < a.r1);
        oz[e] = in ? X[(isz ? 2 : 1) * kPinvStride + row * kFitR + c] : 0.0;
    }
    __syncthreads();
    if (nj == 4) fit_zy_block<NT, 4>(a, bi, x0, x1, ny, nz, oz, oy);
    else if (nj == 3) fit_zy_block<NT, 3>(a, bi, x0, x1, ny, nz, oz, oy);
    else if (nj == 2) fit_zy_block<NT, 2>(a, bi, x0, x1, ny, nz, oz, oy);
    else fit_zy_block<NT, 1>(a, bi, x0, x1, ny, nz, oz, oy);
}

// P[i][e] = sum_x X_x[i][x] U[x][e], e = j n_z + k: the lattice is
// contiguous in e, so both sides stream.  A wave takes 16-wide tiles of e and
// all of i; the next tile's U is in flight during a tile's products.  Bound by
// the stream of U (512 blocks of 32^3: 335 MB in 108 us); 32-wide tiles (two
// columns per lane, half the waves) took 118 us.
constexpr int kFxWaves = 4;

template <int NI>
__device__ __forceinline__ void fit_x_tiles(const FitArgs &a, int t0, int t1, int nx, int ne,
                                            const double *U, const double *ox, float *P) {
    const int wave = uni32(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int gq = lane >> 4, l16 = lane & 15;
    // rows x >= r0 and i >= n_x and tiles past the last are at a dead vector
    // offset: the loop issues the same accesses every time
    const uint32_t ub = (uint32_t)ne * 8u, pb = (uint32_t)ne * 4u;
    const __amdgpu_buffer_rsrc_t ur = make_rsrc(U, (uint32_t)a.r0 * ub);
    const __amdgpu_buffer_rsrc_t pr = make_rsrc(P, (uint32_t)nx * pb);
    auto load = [&](int t, double(&u)[kOpSteps]) {
        const int e = 16 * t + l16;
        const uint32_t at = t < t1 && e < ne ? (uint32_t)gq * ub + (uint32_t)e * 8u : kDeadFit;
#pragma unroll
        for (int ks = 0; ks < kOpSteps; ++ks)
            u[ks] = __builtin_bit_cast(
                double, __builtin_amdgcn_raw_buffer_load_b64(ur, 4 * ks + gq < a.r0 ? at : kDeadFit,
                                                             (uint32_t)(4 * ks) * ub, 0));
    };
    double cur[kOpSteps], nxt[kOpSteps];
    int t = t0 + wave;
    load(t, cur);
    for (; t < t1; t += kFxWaves) {
        load(t + kFxWaves, nxt);
        int ol = lane;
        asm volatile("" : "+v"(ol));  // the operands stay in LDS from tile to tile
        f64x4 acc[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[i] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < kOpSteps; ++ks)
#pragma unroll
            for (int i = 0; i < NI; ++i)
                acc[i] = mfma64(ox[i * kOpTile + ks * kWave + ol], cur[ks], acc[i]);
        const int e = 16 * t + l16;
        const uint32_t at = e < ne ? (uint32_t)gq * pb + (uint32_t)e * 4u : kDeadFit;
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint((float)acc[i][r]), pr,
                                                      16 * i + 4 * r + gq < nx ? at : kDeadFit,
                                                      (uint32_t)(16 * i + 4 * r) * pb, 0);
#pragma unroll
        for (int ks = 0; ks < kOpSteps; ++ks) cur[ks] = nxt[ks];
    }
}

__global__ __launch_bounds__(kFxWaves * 64) void fit_x_kernel(FitArgs a, int echunks, int tchunk) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tid = threadIdx.x;
    const int wg = xcd_order(blockIdx.x, gridDim.x), bi = wg / echunks;
    const int t0 = (wg - bi * echunks) * tchunk;
    const fa_block &b = a.blocks[bi];
    const int nx = uni32(b.ncp[0]), ny = uni32(b.ncp[1]), nz = uni32(b.ncp[2]);
    const int ne = ny * nz, t1 = min(t0 + tchunk, (ne + 15) >> 4);
    if (nz > a.max_n || t0 >= t1) return;
    float *P = a.ctrl + b.ctrl_off;
    if (ny > a.r1) {  // more functions than samples: no least-squares lattice
        for (int64_t e = tid; e < (int64_t)nx * ne; e += kFxWaves * 64) P[e] = __builtin_nanf("");
        return;
    }
    double *ox = reinterpret_cast<double *>(smem_raw);
    const double *X = fit_x_of(a, bi);
    const int ni = (nx + 15) >> 4;
    for (int f = tid; f < ni * kOpTile; f += kFxWaves * 64) {
        const int c = 4 * ((f >> 6) & (kOpSteps - 1)) + ((f >> 4) & 3);
        const int row = (f / kOpTile) * 16 + (f & 15);
        ox[f] = (row < nx && c < a.r0) ? X[row * kFitR + c] : 0.0;
    }
    __syncthreads();
    const double *U = a.T + (int64_t)bi * a.tstride;
    if (ni == 4) fit_x_tiles<4>(a, t0, t1, nx, ne, U, ox, P);
    else if (ni == 3) fit_x_tiles<3>(a, t0, t1, nx, ne, U, ox, P);
    else if (ni == 2) fit_x_tiles<2>(a, t0, t1, nx, ne, U, ox, P);
    else fit_x_tiles<1>(a, t0, t1, nx, ne, U, ox, P);
}

// errs[b * stride + 0] = max |y - f|, errs[b * stride + 1] = sqrt(mean (y-f)^2).
// With chunks > 1 a block's voxels are split into `chunks` equal ranges,
// each reduced by its own workgroup into part[(b * chunks + c) * 2 + {0,1}]
// (max, sum of squares), and combine_kernel finishes the block in a fixed
// order (deterministic either way).
__global__ __launch_bounds__(kFitThreads) void residual_kernel(const float *y, const float *f,
                                                                int64_t vox, int nblocks,
                                                                int chunks, double *part,
                                                                float *errs, int64_t stride) {
    __shared__ float smax[kFitThreads];
    __shared__ double ssum[kFitThreads];
    const int tid = threadIdx.x;
    const int64_t cv = (vox / chunks + 3) / 4 * 4;  // voxels per chunk, a multiple of 4
    for (int64_t item = blockIdx.x; item < (int64_t)nblocks * chunks; item += gridDim.x) {
        const int bi = (int)(item / chunks), c = (int)(item - (int64_t)bi * chunks);
        const int64_t v0 = (int64_t)c * cv;
        const int64_t v1 = c == chunks - 1 ? vox : (v0 + cv < vox ? v0 + cv : vox);
        const float *yb = y + (int64_t)bi * vox;
        const float *fb = f + (int64_t)bi * vox;
        float m = 0.0f;
        double s = 0.0;
        if ((vox & 3) == 0) {
            const float4 *y4 = reinterpret_cast<const float4 *>(yb);
            const float4 *f4 = reinterpret_cast<const float4 *>(fb);
            for (int64_t i = v0 / 4 + tid; i < v1 / 4; i += kFitThreads) {
                const float4 a = y4[i], cc = f4[i];
                const float r0 = a.x - cc.x, r1 = a.y - cc.y, r2 = a.z - cc.z, r3 = a.w - cc.w;
                m = fmaxf(m, fmaxf(fmaxf(fabsf(r0), fabsf(r1)), fmaxf(fabsf(r2), fabsf(r3))));
                s += (double)r0 * r0 + (double)r1 * r1 + (double)r2 * r2 + (double)r3 * r3;
            }
        } else {
            for (int64_t i = v0 + tid; i < v1; i += kFitThreads) {
                const float r = yb[i] - fb[i];
                m = fmaxf(m, fabsf(r));
                s += (double)r * r;
            }
        }
        smax[tid] = m;
        ssum[tid] = s;
        __syncthreads();
        for (int w = kFitThreads / 2; w > 0; w >>= 1) {
            if (tid < w) {
                smax[tid] = fmaxf(smax[tid], smax[tid + w]);
                ssum[tid] += ssum[tid + w];
            }
            __syncthreads();
        }
        if (tid == 0) {
            if (chunks == 1) {
                errs[(int64_t)bi * stride] = smax[0];
                errs[(int64_t)bi * stride + 1] = (float)sqrt(ssum[0] / (double)vox);
            } else {
                part[item * 2] = (double)smax[0];
                part[item * 2 + 1] = ssum[0];
            }
        }
        __syncthreads();
    }
}

__global__ void combine_kernel(const double *part, int chunks, int64_t vox, int nblocks,
                               float *errs, int64_t stride) {
    const int bi = blockIdx.x * blockDim.x + threadIdx.x;
    if (bi >= nblocks) return;
    double m = 0.0, s = 0.0;
    for (int c = 0; c < chunks; ++c) {
        m = fmax(m, part[((int64_t)bi * chunks + c) * 2]);
        s += part[((int64_t)bi * chunks + c) * 2 + 1];
    }
    errs[(int64_t)bi * stride] = (float)m;
    errs[(int64_t)bi * stride + 1] = (float)sqrt(s / (double)vox);
}

// Least-squares loss of a fit and its cotangent in one pass (the residual
// step between the forward decode and the adjoint): per block b,
//   grad[b][v] = scale * (f[b][v] - y[b][v]),  sumsq[b] = sum_v (f - y)^2
// (FP64 sum, fixed order).
__global__ __launch_bounds__(kFitThreads) void mse_grad_kernel(const float *f, const float *y,
                                                                int64_t vox, int nblocks,
                                                                float scale, float *grad,
                                                                double *sumsq) {
    __shared__ double ssum[kFitThreads];
    const int tid = threadIdx.x;
    for (int bi = blockIdx.x; bi < nblocks; bi += gridDim.x) {
        const int64_t o = (int64_t)bi * vox;
        double acc = 0.0;
        if ((vox & 3) == 0) {
            const f32x4 *f4 = reinterpret_cast<const f32x4 *>(f + o);
            const f32x4 *y4 = reinterpret_cast<const f32x4 *>(y + o);
            f32x4 *g4 = reinterpret_cast<f32x4 *>(grad + o);
            for (int64_t i = tid; i < vox / 4; i += kFitThreads) {
                const f32x4 a = __builtin_nontemporal_load(f4 + i);
                const f32x4 c = __builtin_nontemporal_load(y4 + i);
                const f32x4 r = a - c;
                acc += (double)r.x * r.x + (double)r.y * r.y + (double)r.z * r.z +
                       (double)r.w * r.w;
                g4[i] = r * scale;
            }
        } else {
            for (int64_t i = tid; i < vox; i += kFitThreads) {
                const float r = f[o + i] - y[o + i];
                acc += (double)r * r;
                grad[o + i] = r * scale;
            }
        }
        ssum[tid] = acc;
        __syncthreads();
        for (int w = kFitThreads / 2; w > 0; w >>= 1) {
            if (tid < w) ssum[tid] += ssum[tid + w];
            __syncthreads();
        }
        if (tid == 0) sumsq[bi] = ssum[0];
        __syncthreads();
    }
}

// Descriptors of `ncand` candidate NCPs n = n0, n0 - 1, ... of a search (same
// n and p on every axis, knots of n at (n - ncp_lo) * kstride): entry c *
// nblocks + b, its lattice at (c % g * nblocks + b) * cstride (g candidates
// are fitted at a time).
__global__ void candidate_kernel(fa_block *desc, int nblocks, int ncand, int n0, int ncp_lo, int p,
                                 int g, int kstride, int64_t cstride) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nblocks * ncand) return;
    const int c = i / nblocks, n = n0 - c;
    fa_block d{};
    d.ncp[0] = d.ncp[1] = d.ncp[2] = n;
    d.degree[0] = d.degree[1] = d.degree[2] = p;
    d.knot_off = (int64_t)(n - ncp_lo) * kstride;
    d.ctrl_off = (int64_t)(c % g * nblocks + i % nblocks) * cstride;
    d.scale = 1.0f;
    d.flags = FA_FLAG_UNIFORM_X | FA_FLAG_UNIFORM_Y | FA_FLAG_UNIFORM_Z;
    desc[i] = d;
}

}  // namespace

int64_t fit_workspace_bytes(int nblocks, int rx, int ry, int max_n) {
    return ((int64_t)nblocks * max_n * rx * ry + (int64_t)nblocks * 3 * kPinvStride) *
           (int64_t)sizeof(double);
}

namespace {
// raise the dynamic LDS limits of the fit kernels once per process
hipError_t fit_attributes() {
    static const hipError_t attr = [] {
        const void *ks[7] = {reinterpret_cast<const void *>(&fit_zy_kernel<1>),
                             reinterpret_cast<const void *>(&fit_zy_kernel<2>),
                             reinterpret_cast<const void *>(&fit_zy_kernel<3>),
                             reinterpret_cast<const void *>(&fit_zy_kernel<4>),
                             reinterpret_cast<const void *>(&fit_x_kernel),
                             reinterpret_cast<const void *>(&fit_pinv_kernel),
                             reinterpret_cast<const void *>(&pinv_candidates_kernel)};
        const int zy = 8 * kOpTile * (int)sizeof(double);
        const int bytes[7] = {zy, zy, zy, zy, zy / 2, (int)sizeof(PinvSmem), (int)sizeof(PinvSmem)};
        hipError_t r = hipSuccess;
        for (int i = 0; i < 7; ++i) {
            const hipError_t e =
                hipFuncSetAttribute(ks[i], hipFuncAttributeMaxDynamicSharedMemorySize, bytes[i]);
            if (e != hipSuccess) r = e;
        }
        return r;
    }();
    return attr;
}

// the two products of a fit given the pseudo-inverses; max_y >= NCP_y of
// every entry that has no more functions than samples along y
hipError_t launch_fit_products(const FitArgs &a, int max_y, hipStream_t s) {
    // slices per workgroup (a multiple of its waves): as many as leave two
    // workgroups per CU, both resident (one's set-up hides behind the other's
    // products)
    const int64_t rounds = (int64_t)a.nblocks * ((a.r0 + kZyWaves - 1) / kZyWaves);
    const int xgroup = kZyWaves * (int)std::max<int64_t>(1, std::min<int64_t>(16, rounds / 512));
    const int64_t groups = (a.r0 + xgroup - 1) / xgroup;
    const int nk = (a.max_n + 15) / 16, nj = (std::min(max_y, a.r1) + 15) / 16;
    const size_t lds = (size_t)(nk + nj) * kOpTile * sizeof(double);
    const dim3 gz((unsigned)(a.nblocks * groups)), tz(kZyWaves * 64);
    switch ((a.r1 + 15) / 16) {
    case 1: hipLaunchKernelGGL(fit_zy_kernel<1>, gz, tz, lds, s, a, xgroup); break;
    case 2: hipLaunchKernelGGL(fit_zy_kernel<2>, gz, tz, lds, s, a, xgroup); break;
    case 3: hipLaunchKernelGGL(fit_zy_kernel<3>, gz, tz, lds, s, a, xgroup); break;
    default: hipLaunchKernelGGL(fit_zy_kernel<4>, gz, tz, lds, s, a, xgroup); break;
    }
    // tiles per workgroup: as many as leave eight workgroups per CU
    const int tiles = (std::min(max_y, a.r1) * a.max_n + 15) / 16;
    const int64_t quads = (int64_t)a.nblocks * ((tiles + kFxWaves - 1) / kFxWaves);
    const int tchunk = kFxWaves * (int)std::max<int64_t>(1, std::min<int64_t>(8, quads / 2048));
    const int echunks = (tiles + tchunk - 1) / tchunk;
    hipLaunchKernelGGL(fit_x_kernel, dim3((unsigned)((int64_t)a.nblocks * echunks)),
                       dim3(kFxWaves * 64), 4 * kOpTile * sizeof(double), s, a, echunks, tchunk);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_fit(const fa_block *blocks, int nblocks, const float *knots, int rx, int ry,
                      int rz, int max_n, const float *samples, double *T, float *ctrl,
                      hipStream_t s) {
    const hipError_t attr = fit_attributes();
    if (attr != hipSuccess) return attr;
    double *Xg = T + (int64_t)nblocks * max_n * rx * ry;
    const int gp = (int)std::min<int64_t>((int64_t)nblocks * 3, 1 << 20);
    hipLaunchKernelGGL(fit_pinv_kernel, dim3(gp), dim3(kWave), sizeof(PinvSmem), s, blocks,
                       nblocks, knots, rx, ry, rz, Xg);
    const FitArgs a{blocks, nblocks, nblocks, rx, ry, rz, max_n, samples, Xg, 0, 3 * kPinvStride,
                    T, (int64_t)max_n * rx * ry, ctrl};
    return launch_fit_products(a, kFitN, s);
}

int64_t pinv_doubles() { return kPinvStride; }

hipError_t launch_pinv_candidates(float *kall, int ncp_lo, int ncand, int p, int kstride, int rx,
                                  int ry, int rz, double *xall, hipStream_t s) {
    const hipError_t attr = fit_attributes();
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(pinv_candidates_kernel, dim3(ncand * 3), dim3(kWave), sizeof(PinvSmem), s,
                       kall, ncp_lo, ncand, p, kstride, rx, ry, rz, xall);
    return hipGetLastError();
}

hipError_t launch_fit_candidates(const fa_block *desc, int nblocks, int ncand, int rx, int ry,
                                 int rz, int max_n, const float *samples, const double *X,
                                 double *T, float *ctrl, hipStream_t s) {
    const hipError_t attr = fit_attributes();
    if (attr != hipSuccess) return attr;
    const FitArgs a{desc, nblocks * ncand, nblocks, rx, ry, rz, max_n, samples, X,
                    -3 * kPinvStride, 0, T, (int64_t)rx * max_n * max_n, ctrl};
    return launch_fit_products(a, max_n, s);
}

hipError_t launch_residual(const float *y, const float *f, int64_t vox, int nblocks, float *errs,
                           int64_t stride, hipStream_t s, int chunks, double *part) {
    if (chunks < 1 || !part) chunks = 1;
    const int64_t items = (int64_t)nblocks * chunks;
    const int grid = (int)(items < 65536 ? items : 65536);
    hipLaunchKernelGGL(residual_kernel, dim3(grid), dim3(kFitThreads), 0, s, y, f, vox, nblocks,
                       chunks, part, errs, stride);
    if (chunks > 1)
        hipLaunchKernelGGL(combine_kernel, dim3((nblocks + 255) / 256), dim3(256), 0, s, part,
                           chunks, vox, nblocks, errs, stride);
    return hipGetLastError();
}

hipError_t launch_mse_grad(const float *f, const float *y, int64_t vox, int nblocks, float scale,
                           float *grad, double *sumsq, hipStream_t s) {
    const int grid = nblocks < 65536 ? nblocks : 65536;
    hipLaunchKernelGGL(mse_grad_kernel, dim3(grid), dim3(kFitThreads), 0, s, f, y, vox, nblocks,
                       scale, grad, sumsq);
    return hipGetLastError();
}

hipError_t launch_candidates(fa_block *desc, int nblocks, int ncand, int n0, int ncp_lo, int p, int g,
                             int kstride, int64_t cstride, hipStream_t s) {
    hipLaunchKernelGGL(candidate_kernel, dim3((nblocks * ncand + 255) / 256), dim3(256), 0, s, desc,
                       nblocks, ncand, n0, ncp_lo, p, g, kstride, cstride);
    return hipGetLastError();
}

}  // namespace fa
