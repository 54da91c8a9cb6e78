// Adjoint of the grid decode on the FP32 matrix cores (row a7): G = B^T g.
// With a cotangent of the values alone it is the least-squares fit's
// gradient (2/M) B^T r that the fit of control points needs; with cotangents
// of the derivative channels, that of a loss on gradients too.
//
// The transposed tensor-product contraction is ordered per x slice u of the
// cotangent block; for the values
//     Z_u[v][k] = sum_w g[u][v][w] Bz[w][k]        (z, dense product)
//     Y_u[j][k] = sum_v By[v][j] Z_u[v][k]         (y, dense product)
//     G[i][j][k] += Bx[u][i] Y_u[j][k]             (x, p+1 planes per slice)
// and with all four channels
//     Z0 = g_0 Bz + g_3 Dz,  Z1 = g_1 Bz,  Z2 = g_2 Bz
//     G[i] += Bx[u][i] (By^T Z0 + Dy^T Z2) + Dx[u][i] By^T Z1.
// The products run on v_mfma_f32_16x16x4f32 and never leave the wave's
// registers: the z product of a 16-row band of the slice leaves its 16 x 16
// tile of Z_u in exactly the operand layout of four K steps of the y
// product, so a wave contracts its slices from HBM to Y_u without LDS or
// barriers.  A wave owns one 16-wide k tile and up to two 16-wide j tiles
// of the output and a chunk of consecutive x slices; it keeps the p+1
// control planes its current slice touches in a register ring (plane i in
// slot i mod (p+1)) and stores a plane once when the span along x moves
// past it.  The waves of a workgroup split its x slices into chunks
// whose plane ranges overlap only with their neighbours' (at most p+1
// planes per boundary): the chunk to the right of a boundary leaves its
// partial planes there in LDS, and the chunk to the left adds them to its
// own after the workgroup's one barrier.  The z product's K steps cover the
// 16-column groups of w inside the basis band of the wave's k tile; the y
// product runs over all row bands of the slice, one, two or four by the
// resolution (its y basis operands are zero outside each j tile's band).  The
// slice body is straight-line code, one instance per (row bands, band width,
// one or two j tiles), so that the z chains (one per row band), the loads of the next slice and the y chains of a
// slice are scheduled together.  Fixed summation order, no floating-point
// atomics: the result is deterministic.
//
// Values only: the basis operands of both products stay in registers for
// the whole block.  All channels: they sit in LDS in lane order (16 reads of
// 1 KB per channel and slice against 64 products), and two buffers hold the
// channel in use and the one in flight.
//
// With two or more channels a segment whose lattice has few planes for its slices, or
// more columns than two tiles hold, is summed along x first on the vector ALUs
// (adj_planes): one set of y and z sums per plane instead of products per slice.
//
// A micro-model is split between `nseg` workgroups when there are fewer
// micro-models than CUs: a segment owns the control planes [i0, i1), streams
// the slices whose basis touches them (neighbours re-read an overlap of p
// spans) and stores its own planes only.
//
// Bound by the matrix cores of the busiest SIMD and the cotangent's reads:
// values of 256 blocks of 64^3, NCP 16..32, 84 us (3.2 TB/s); all channels of
// 128 blocks, NCP 8..32, 167 us (3.2 TB/s), 195 with every block on the matrix
// cores, 914 with every block on the vector ALUs and one workgroup of 16 waves each.
//
// Operand layout of v_mfma_f32_16x16x4f32 (checked on the device): lane l
// holds A[l%16][l/16] and B[l/16][l%16] and receives D[4(l/16)+r][l%16].
// The z product sums w in the order w = 16 q + 4 (l/16) + j (step (q, j)),
// so each lane reads four consecutive w of its row with one 16-byte load;
// the y product sums v = 16 m + 4 (l/16) + r (step (m, r)), which is the
// row that lane's result register r of band m's Z tile holds.
#include "fa_device.hpp"
#include "fa_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace fa {
namespace {

typedef float f32x4a __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kAW = 8;           // waves per workgroup
constexpr int kAT = kAW * 64;    // threads per workgroup
constexpr int kAM = 64;          // res[1], res[2] and NCP_y, NCP_z limit
constexpr int kJT = 2;           // j tiles per wave
constexpr int kCUs = 256;
constexpr int kMaxSegs = 8;      // segments of a micro-model
// micro-models of one launch: a launch holds fewer than 2^32 threads
constexpr int kMostGroups = 1 << 20;
// partial planes of the chunk boundaries: at most (X - 1) (p + 1) NCP_y
// NCP_z floats, X <= kAW / (k tiles x j tile pairs), which is below
// (p + 1) * 4096 for every shape
constexpr int kLB = 4 * 4096;

template <bool DER>
struct AmSmem;

template <>
struct AmSmem<false> {
    float kn[kMaxKnotsPerBlock + 4];
    float4 xB[kMaxRes];  // x basis of each slice in ring order
    int xS[kMaxRes];     // span along x of each slice
    float4 yN[kAM];      // y basis of each v (entries beyond p zero)
    float4 zN[kAM];
    int ys[kAM];         // span along y of each v
    int zs[kAM];
    int tw[2][kAM / 16];  // first and last w with a basis entry in each k tile
    float lb[kLB];        // left partial planes of chunks 1..X-1
    uint32_t bad[2];      // planes in which a wave holds a value that is not finite
};

template <>
struct AmSmem<true> : AmSmem<false> {
    float4 xD[kMaxRes], yD[kAM], zD[kAM];  // derivatives beside xB, yN, zN
    // operands in lane order, basis then derivative: the z product's of k
    // tile t and columns 16q + 4(l/16) + (x, y, z, w), the y product's of j
    // tile t and rows 16m + 4(l/16) + (x, y, z, w)
    float4 op[2][2][kAM / 16][4][kWave];  // z product, y product
};

__device__ __forceinline__ f32x4a mma4(float a, float b, const f32x4a &c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float pick4(const float4 &v, int d) {
    return d == 0 ? v.x : (d == 1 ? v.y : (d == 2 ? v.z : v.w));
}

template <int P>
__device__ __forceinline__ float4 row4(const float (&v)[P + 1]) {
    float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int r = 0; r <= P; ++r) c[r] = v[r];
    return make_float4(c[0], c[1], c[2], c[3]);
}

// v[0..P] moved to ring order: plane s - P + r in slot (s - P + r) mod (P + 1)
template <int P>
__device__ __forceinline__ float4 ring4(const float (&v)[P + 1], int s) {
    constexpr int R = P + 1;
    const int base = (s - P) % R;
    float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int m = 0; m < R; ++m) {
        const int r = (m - base + R) % R;
#pragma unroll
        for (int q = 0; q < R; ++q) c[m] = r == q ? v[q] : c[m];
    }
    return make_float4(c[0], c[1], c[2], c[3]);
}

// First position whose span, in the non-decreasing s[0..n), is at least t.
__device__ __forceinline__ int first_at(const int *s, int n, int t) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s[mid] < t) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Component d of entry i of a table in LDS, read as one dword: a choice between
// the components of the entry (pick4) is compiled to branches over addresses
// where it stands in a divergent loop, and clang 22 forms the one of component 3
// under the wrong execution mask there.
__device__ __forceinline__ float entry(const float4 *tab, int i, int d) {
    return reinterpret_cast<const float *>(tab)[4 * i + d];
}

// The planes of the set `bad` once more with every sum over its window alone,
// by the slices of [slo, shi) that touch them: a slice's channels into LDS, their
// z sums into LDS, y and x by the thread that owns (j, k).  The products of the
// matrix cores include zero weights, so an infinite or NaN cotangent value turns
// whole tiles into NaN there; here it reaches the p + 1 lattice indices of its
// window on each axis and no others.  Only workgroups that found such a value
// come here, for the marked planes.  Bound by the latency of its sums' LDS reads:
// 128 blocks of 64^3, all channels, one NaN in each, 0.55 ms at NCP 32, 1.4 at
// 8..32, 1.9 at 4 (finite 0.15, 0.17, 0.18).
template <int P, bool DER>
__device__ __forceinline__ void adj_windows(int ny, int nz, int ry, int rz, uint32_t mask,
                                            const float *g, int64_t vox, float *Gb, uint64_t bad,
                                            int slo, int shi, AmSmem<DER> &sm) {
    constexpr int R = P + 1, kS = kAM * kAM;
    const int tid = threadIdx.x, plane = ny * nz, row = ry * rz;
    float *z0 = sm.lb, *z1 = z0 + kS, *z2 = z1 + kS;  // z sums of a slice
    // channel c of the slice at c kS, row v turned by v (rows in step would meet
    // on one bank)
    float *gl;
    if constexpr (DER) gl = reinterpret_cast<float *>(sm.op);
    else gl = z1;
    static_assert(3 * kS <= kLB, "z sums of a slice");
    __syncthreads();
    for (int e = tid; e < plane; e += kAT)
        for (uint64_t m = bad; m; m &= m - 1)
            Gb[(int64_t)__builtin_ctzll(m) * plane + e] = 0.0f;
    for (int u = slo; u < shi; ++u) {
        const int s = __builtin_amdgcn_readfirstlane(sm.xS[u]);
        const uint32_t hit = (uint32_t)(bad >> (s - P)) & ((1u << R) - 1u);  // of its planes
        if (!hit) continue;
        __syncthreads();  // the previous slice's z sums are read
        const float *src = g + (int64_t)u * row;
        for (int c = 0; c < (DER ? 4 : 1); ++c) {
            const bool has = mask >> c & 1u;
#pragma unroll
            for (int q = 0; q < kS / kAT; ++q) {
                const int e = tid + q * kAT, v = e / rz, t = e - v * rz + v % rz;
                if (e < row) gl[c * kS + v * rz + (t < rz ? t : t - rz)] = has ? src[e] : 0.0f;
            }
            src += has ? vox : 0;
        }
        __syncthreads();
        for (int e = tid; e < ry * nz; e += kAT) {
            const int v = e / nz, k = e - v * nz;
            const float *gv = gl + v * rz;
            const int turn = v % rz;
            float a0 = 0.0f, a1 = 0.0f, a2 = 0.0f;
            // (a channel that is not there was staged as zeros)
            const int wb = first_at(sm.zs, rz, k), we = first_at(sm.zs, rz, k + P + 1);
#pragma unroll 4
            for (int w = wb; w < we; ++w) {
                const int d = k - (sm.zs[w] - P);
                const float n = entry(sm.zN, w, d);
                const int t = w + turn < rz ? w + turn : w + turn - rz;
                a0 = fmaf(n, gv[t], a0);
                if constexpr (DER) {
                    a1 = fmaf(n, gv[kS + t], a1);
                    a2 = fmaf(n, gv[2 * kS + t], a2);
                    a0 = fmaf(entry(sm.zD, w, d), gv[3 * kS + t], a0);
                }
            }
            z0[e] = a0;
            if constexpr (DER) {
                z1[e] = a1;
                z2[e] = a2;
            }
        }
        __syncthreads();
        for (int e = tid; e < plane; e += kAT) {
            const int j = e / nz, k = e - j * nz;
            float b0 = 0.0f, b1 = 0.0f;
            const int vb = first_at(sm.ys, ry, j), ve = first_at(sm.ys, ry, j + P + 1);
#pragma unroll 4
            for (int v = vb; v < ve; ++v) {
                const int d = j - (sm.ys[v] - P);
                const float n = entry(sm.yN, v, d);
                b0 = fmaf(n, z0[v * nz + k], b0);
                if constexpr (DER) {
                    b0 = fmaf(entry(sm.yD, v, d), z2[v * nz + k], b0);
                    b1 = fmaf(n, z1[v * nz + k], b1);
                }
            }
            float *o = Gb + (int64_t)(s - P) * plane + e, sum[R];
#pragma unroll
            for (int r = 0; r < R; ++r)  // all loads, then the stores
                sum[r] = hit >> r & 1u ? o[(int64_t)r * plane] : 0.0f;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int slot = (s - P + r) % R;
                sum[r] = fmaf(entry(sm.xB, u, slot), b0, sum[r]);
                if constexpr (DER) sum[r] = fmaf(entry(sm.xD, u, slot), b1, sum[r]);
                if (hit >> r & 1u) o[(int64_t)r * plane] = sum[r];
            }
        }
    }
}

// Whether x first (adj_planes) is the faster form for a segment: `len` slices in X
// chunks, `waves` = X * (k tiles) * (j tile pairs) in use, nq column groups and nj j
// tiles per product, np planes of r - 1 = degree.  The sums estimate the two forms'
// time in ns: a wave's products per slice at 22 ns, 40 where two waves share a SIMD;
// rows and channels per slice, y and z sums per plane.  Coefficients by least squares
// over 914 launches (NCP 4..48, cubic and not, degrees 1 to 3, 16^3 to 100 x 64 x 64,
// one to four channels), which they meet to 16% and 13%.  A wrong choice costs more
// than a missed one, so x first has to be estimated a fifth lower, with two channels
// 30%, and one channel or more planes than slices stay with the products.  800 blocks
// of 64^3, all channels, x first and matrix form: degree 1, NCP 40 1.33 and 2.69 ms,
// NCP 20 0.80 and 1.13, NCP 16 0.72 and 0.68; degree 3 1.77 and 2.69, 0.98 and 1.13,
// 0.92 and 0.75.
template <int MB>
__device__ __forceinline__ bool planes_first(int len, int X, int waves, int nq, int nj, int np,
                                             int r, int ny, int ry, int rz, uint32_t mask) {
    const int nch = __builtin_popcount(mask);
    const int nyp = !!(mask & 2u) + !!(mask & 9u) + !!(mask & 4u);  // y products
    const int products = 4 * MB * (nch * nq + nyp * nj);
    const int m = 15000 + (len + X - 1) / X * (580 + products * (waves > kAW / 2 ? 40 : 22));
    const int x = 7000 + len * (104 + MB * (42 * r + 61 * nch)) +
                  np * (1043 + 13 * ry * r + ny * rz * r / 4);
    return nch > 1 && np <= len && 10 * x < (nch > 2 ? 8 : 7) * m;
}

// The segment's planes with x first, on the vector ALUs: lane w, row wave + 8 m
// of every slice; a thread keeps the p + 1 newest x sums of its columns,
// and a plane whose last slice has passed goes to LDS, where y is summed
// over each j's rows and z over each k's columns.  An infinite or NaN value meets
// no weight outside its windows here.  Bound by the cotangent's reads where planes
// are few (4.2 TB/s at 64^3, NCP 20, degree 1), else by the LDS reads of the y sums.
// Two slices are in registers at four row bands and four below, where a slice is a
// few KB (1000 blocks of 100 x 20 x 30, NCP 4 x 16 x 32, degree 1, in a kernel of this
// form alone: 0.70 ms with two, 0.29 with four).
template <int P, int MB>
__device__ __forceinline__ void adj_planes(int ny, int nz, int ry, int rz, uint32_t mask,
                                           const float *g, int64_t vox, float *Gb, int i0, int i1,
                                           int slo, int shi, AmSmem<true> &sm) {
    constexpr int R = P + 1, kRows = 2 * MB, kP = kAM * kWave;
    constexpr int kDeep = MB == 4 ? 2 : 4;  // slices in registers
    static_assert(3 * kP + 4 * kAM <= kLB, "x sums of a plane and supports");
    static_assert(2 * kP * sizeof(float) <= sizeof(sm.op), "y sums of a plane");
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int plane = ny * nz;
    float *H0 = sm.lb, *H2 = H0 + kP, *H3 = H2 + kP;
    float *KB = reinterpret_cast<float *>(sm.op), *K3 = KB + kP;
    // first and last position of each lattice index along y and z
    int *lo = reinterpret_cast<int *>(H3 + kP), *hi = lo + 2 * kAM;
    if (tid < 2 * kAM) {
        lo[tid] = 0x7fffffff;
        hi[tid] = -1;
    }
    lds_barrier();
    for (int t = tid; t < ry + rz; t += kAT) {
        const bool isy = t < ry;
        const int pos = isy ? t : t - ry, s = (isy ? sm.ys : sm.zs)[pos];
        for (int i = s - P; i <= s; ++i) {
            atomicMin(&lo[(isy ? 0 : kAM) + i], pos);
            atomicMax(&hi[(isy ? 0 : kAM) + i], pos);
        }
    }
    const float *gw = g + min(lane, rz - 1);
    const int64_t slice = (int64_t)ry * rz;
    int row[kRows];
#pragma unroll
    for (int m = 0; m < kRows; ++m) row[m] = min(wave + kAW * m, ry - 1) * rz;
    float hB[kRows][R], h2[kRows][R], h3[kRows][R];
#pragma unroll
    for (int m = 0; m < kRows; ++m)
#pragma unroll
        for (int r = 0; r < R; ++r) hB[m][r] = h2[m][r] = h3[m][r] = 0.0f;

    auto emit = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < kRows; ++m) {
            const int v = wave + kAW * m;
            if (v < ry) {
                H0[v * kWave + lane] = hB[m][0];
                H2[v * kWave + lane] = h2[m][0];
                H3[v * kWave + lane] = h3[m][0];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                hB[m][r] = r < P ? hB[m][r + 1] : 0.0f;
                h2[m][r] = r < P ? h2[m][r + 1] : 0.0f;
                h3[m][r] = r < P ? h3[m][r + 1] : 0.0f;
            }
        }
        if (i < i0) return;  // uniform: a neighbour's plane
        lds_barrier();
        for (int e = tid; e < ny * kWave; e += kAT) {
            const int j = e >> 6, w = e & 63;
            float kb = 0.0f, k3 = 0.0f;
            for (int v = lo[j]; v <= hi[j]; ++v) {
                const int r = j - (sm.ys[v] - P);
                const float cb = entry(sm.yN, v, r);
                kb = fmaf(cb, H0[v * kWave + w], kb);
                kb = fmaf(entry(sm.yD, v, r), H2[v * kWave + w], kb);
                k3 = fmaf(cb, H3[v * kWave + w], k3);
            }
            KB[e] = kb;
            K3[e] = k3;
        }
        lds_barrier();
        for (int e = tid; e < plane; e += kAT) {
            const int j = e / nz, k = e - j * nz;
            float acc = 0.0f;
            for (int w = lo[kAM + k]; w <= hi[kAM + k]; ++w) {
                const int r = k - (sm.zs[w] - P);
                acc = fmaf(entry(sm.zN, w, r), KB[j * kWave + w], acc);
                acc = fmaf(entry(sm.zD, w, r), K3[j * kWave + w], acc);
            }
            Gb[(int64_t)i * plane + e] = acc;
        }
        lds_barrier();
    };

    float f[kDeep][4][kRows];  // the slice in use and the next ones
    auto fetch = [&](int u, float(&x)[4][kRows]) __attribute__((always_inline)) {
        int c = 0;
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) {
            if (mask >> ch & 1u) {
                const float *gu = gw + (int64_t)c * vox + (int64_t)u * slice;
#pragma unroll
                for (int m = 0; m < kRows; ++m) x[ch][m] = gu[row[m]];
                ++c;
            } else {
#pragma unroll
                for (int m = 0; m < kRows; ++m) x[ch][m] = 0.0f;
            }
        }
    };
    int nxt = i0;  // the next plane to leave: window slot 0
    auto use = [&](int u, const float(&x)[4][kRows]) __attribute__((always_inline)) {
        const int s = __builtin_amdgcn_readfirstlane(sm.xS[u]);
        for (; nxt < s - P; ++nxt) emit(nxt);
        float cf[R], ef[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            cf[r] = entry(sm.xB, u, (s - P + r) % R);
            ef[r] = entry(sm.xD, u, (s - P + r) % R);
        }
#pragma unroll
        for (int m = 0; m < kRows; ++m)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                hB[m][r] = fmaf(cf[r], x[0][m], fmaf(ef[r], x[1][m], hB[m][r]));
                h2[m][r] = fmaf(cf[r], x[2][m], h2[m][r]);
                h3[m][r] = fmaf(cf[r], x[3][m], h3[m][r]);
            }
    };
    if (slo < shi) {
        nxt = min(nxt, __builtin_amdgcn_readfirstlane(sm.xS[slo]) - P);
#pragma unroll
        for (int d = 0; d < kDeep; ++d) fetch(min(slo + d, shi - 1), f[d]);
        for (int u = slo; u < shi; u += kDeep)
#pragma unroll
            for (int d = 0; d < kDeep; ++d) {
                if (u + d >= shi) break;  // uniform
                use(u + d, f[d]);
                fetch(min(u + d + kDeep, shi - 1), f[d]);
            }
    }
    for (; nxt < i1; ++nxt) emit(nxt);
}

// RAG: the rows of the cotangent are not whole 16-byte vectors (the values a
// load takes from past its row's end are replaced by zeros).  MB: the 16-row bands
// of a slice, ry <= 16 MB
template <int P, bool DER, bool RAG, int MB>
__device__ __forceinline__ void adj_block(const fa_block &B, const float *knots, int rx, int ry,
                                          int rz, uint32_t mask, const float *g, float *G, int b,
                                          int seg, int nseg, AmSmem<DER> &sm) {
    constexpr int R = P + 1;  // ring slots
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int gq = lane >> 4, l16 = lane & 15;
    const int nx = B.ncp[0], ny = B.ncp[1], nz = B.ncp[2];
    const int i0 = seg * nx / nseg, i1 = (seg + 1) * nx / nseg;  // planes stored here
    if (i0 >= i1) return;

    // knots; span and basis tables of the y and z positions and the x slices
    const int nkn = nx + ny + nz + 3 * R;
    for (int e = tid; e < nkn; e += kAT) sm.kn[e] = knots[B.knot_off + e];
    if (tid < kAM / 16) {
        sm.tw[0][tid] = 0x7fffffff;
        sm.tw[1][tid] = -1;
    }
    if (tid < 2) sm.bad[tid] = 0u;
    lds_barrier();
    const float *tx = sm.kn, *ty = tx + nx + R, *tz = ty + ny + R;
    for (int t = tid; t < ry + rz; t += kAT) {
        const bool isy = t < ry;
        const int pos = isy ? t : t - ry;
        const int n = isy ? ny : nz;
        const float *tk = isy ? ty : tz;
        const float x = grid_pos(pos, isy ? ry : rz);
        const int s = span_search(n, P, tk, x);
        float N[R], D[R];
        basis_ders<P>(tk, s, x, N, D);
        (isy ? sm.yN : sm.zN)[pos] = row4<P>(N);
        if constexpr (DER) (isy ? sm.yD : sm.zD)[pos] = row4<P>(D);
        (isy ? sm.ys : sm.zs)[pos] = s;
        // the k tiles of 16 lattice indices this w position's window touches
        if (!isy) {
            for (int tt = (s - P) >> 4; tt <= s >> 4; ++tt) {
                atomicMin(&sm.tw[0][tt], pos);
                atomicMax(&sm.tw[1][tt], pos);
            }
        }
    }
    for (int u = tid; u < rx; u += kAT) {
        const float x = grid_pos(u, rx);
        const int s = span_search(nx, P, tx, x);
        float N[R], D[R];
        basis_ders<P>(tx, s, x, N, D);
        sm.xB[u] = ring4<P>(N, s);
        if constexpr (DER) sm.xD[u] = ring4<P>(D, s);
        sm.xS[u] = s;
    }
    lds_barrier();

    // entry (position pos, lattice index i) of the basis along z or y
    auto zval = [&](int w, int k, const float4 *tab) {
        if (w >= rz || k >= nz) return 0.0f;
        const int d = k - (sm.zs[w] - P);
        return d >= 0 && d <= P ? pick4(tab[w], d) : 0.0f;
    };
    auto yval = [&](int v, int j, const float4 *tab) {
        if (v >= ry || j >= ny) return 0.0f;
        const int d = j - (sm.ys[v] - P);
        return d >= 0 && d <= P ? pick4(tab[v], d) : 0.0f;
    };
    // waves: (chunk, j tile pair, k tile).  The segment's slices [slo, shi)
    // are split into X chunks of consecutive slices; each chunk after the
    // first starts at the first change of the span along x at or after slo +
    // c (shi - slo) / X, when there is
    // one (neighbouring chunks then share fewer control planes), and X is
    // as large as the waves allow with every chunk non-empty and no control
    // plane touched by three chunks.  (Values read from LDS that are the
    // same in every lane go through readfirstlane, so the control flow they
    // decide stays scalar.)
    const int njt = (ny + 15) >> 4, nkt = (nz + 15) >> 4;
    const int njp = (njt + 1) >> 1;
    const int W1 = nkt * njp;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int cw = wv / W1, wr = wv % W1;
    uint64_t first[4];  // bit u % 64 of word u / 64: slice u starts a span
    int slo = 0, shi = 0;  // spans are non-decreasing along x
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int u = 64 * w + lane;
        first[w] = 0;
        if (64 * w >= rx) continue;  // uniform
        first[w] = __ballot(u < rx && u > 0 && sm.xS[u] != sm.xS[u - 1]);
        slo += __builtin_popcountll(__ballot(u < rx && sm.xS[u] < i0));
        shi += __builtin_popcountll(__ballot(u < rx && sm.xS[u] - P < i1));
    }
    const int plane = ny * nz;
    float *Gb = G + B.ctrl_off;
    if (slo >= shi) {  // no slice touches the segment's planes
        for (int e = tid; e < (i1 - i0) * plane; e += kAT) Gb[(int64_t)i0 * plane + e] = 0.0f;
        return;
    }
    auto next_start = [&](int u) -> int {  // the first span start >= u, else rx
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            if (w < (u >> 6)) continue;
            uint64_t m = first[w];
            if (w == (u >> 6)) m &= ~0ull << (u & 63);
            if (m) return min(64 * w + __builtin_ctzll(m), rx);
        }
        return rx;
    };
    const int len = shi - slo;
    int X = min(kAW / W1, len), ua = slo, ue = shi;  // this wave's chunk [ua, ue)
    for (;; --X) {
        bool ok = true;
        int prev = slo;
        ua = slo;
        ue = shi;
        for (int c = 1; c < X && ok; ++c) {
            const int u0 = max(slo + c * len / X, prev + 1);
            int u = next_start(u0);
            if (u >= shi) u = u0;
            ok = u < shi && (c < 2 || sm.xS[prev - 1] < sm.xS[u] - P);
            if (c == cw) ua = u;
            if (c == cw + 1) ue = u;
            prev = u;
        }
        if (ok || X == 1) break;
    }
    // Small lattices, where X so chosen leaves two thirds of the waves idle: X
    // as the waves allow with equal chunks, if every chunk's own copy of the
    // planes it touches fits in LDS; each chunk leaves all of its planes there
    // and the sums over the chunks follow the barrier (128 blocks of 8^3, all
    // channels: 211 -> 151 us).  At half the waves idle the copies cost more
    // than they give (128 blocks of 16..32, values: 51 us without, 59 with), and
    // so they do for the values in chunks of fewer than three slices (50000 blocks
    // of 8^3 on 8^3: 2.70 ms without, 3.19 with; all channels 5.09, 4.12).
    const int XO = min(kAW / W1, len);
    int lbase = 0;
    bool open = false;
    if (3 * X <= XO && (DER || len >= 3 * XO)) {
        int total = 0;
        for (int c = 0; c < XO; ++c) {
            if (c == cw) lbase = total;
            total += (sm.xS[slo + (c + 1) * len / XO - 1] - sm.xS[slo + c * len / XO] + R) * plane;
        }
        open = __builtin_amdgcn_readfirstlane(total) <= kLB;
        lbase = __builtin_amdgcn_readfirstlane(lbase);
        if (open) {
            X = XO;
            ua = slo + cw * len / XO;
            ue = slo + (cw + 1) * len / XO;
        }
    }
    X = __builtin_amdgcn_readfirstlane(X);
    if constexpr (DER) {
        int nqm = 1;  // 16-column groups of the widest k tile's band
        for (int t = 0; t < nkt; ++t) nqm = max(nqm, (sm.tw[1][t] >> 4) - (sm.tw[0][t] >> 4) + 1);
        if (__builtin_amdgcn_readfirstlane(planes_first<MB>(
                len, X, X * W1, nqm, min(2, njt), i1 - i0, P + 1, ny, ry, rz, mask))) {
            const int64_t vox = (int64_t)rx * ry * rz;
            adj_planes<P, MB>(ny, nz, ry, rz, mask, g + (int64_t)b * __builtin_popcount(mask) * vox,
                              vox, G + B.ctrl_off, i0, i1, slo, shi, sm);
            return;
        }
        for (int e = tid; e < 4 * (kAM / 16) * 4 * kWave; e += kAT) {
            const int l = e & (kWave - 1), q = (e >> 6) & 3, t = (e >> 8) & 3, d = (e >> 10) & 1;
            const int p0 = 16 * q + 4 * (l >> 4), i = 16 * t + (l & 15);
            float f[4];
            if (e >> 11) {
#pragma unroll
                for (int r = 0; r < 4; ++r) f[r] = yval(p0 + r, i, d ? sm.yD : sm.yN);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) f[r] = zval(p0 + r, i, d ? sm.zD : sm.zN);
            }
            sm.op[e >> 11][d][t][q][l] = make_float4(f[0], f[1], f[2], f[3]);
        }
        lds_barrier();
    }
    ua = __builtin_amdgcn_readfirstlane(ua);
    ue = __builtin_amdgcn_readfirstlane(ue);
    const int c = cw;
    const bool active = c < X;
    const int nt = wr % nkt, jp = wr / nkt;
    const int ub = ue - 1;
    const int Lc = __builtin_amdgcn_readfirstlane(sm.xS[active ? ua : slo] - P);
    // last plane of chunk c-1, first plane of chunk c+1
    const int Hprev = c > 0 && active ? __builtin_amdgcn_readfirstlane(sm.xS[ua - 1]) : -1;
    const int Lnext = c + 1 < X ? __builtin_amdgcn_readfirstlane(sm.xS[ue] - P) : nx;
    const int k = 16 * nt + l16;

    f32x4a ring[kJT][R];
#pragma unroll
    for (int jj = 0; jj < kJT; ++jj)
#pragma unroll
        for (int m = 0; m < R; ++m) ring[jj][m] = f32x4a{0.0f, 0.0f, 0.0f, 0.0f};
    // plane i of the wave's tiles: into G, or (dst != null) into a partial
    // plane buffer; with add, the buffer's values are added first.  Element
    // (j, k) of a plane is lane_e + (16 jt + r) nz; G is written through a
    // buffer resource, the plane and row in the scalar offset.
    const __amdgpu_buffer_rsrc_t gs = make_rsrc(Gb, (uint32_t)((int64_t)nx * plane * 4));
    const int lane_e = 4 * gq * nz + k;
    // the planes that hold a value which is not finite are marked: such a value,
    // or an overflow of the z product, is in every j of its tile column (the y
    // product's zero weights turn it into NaN), so one j per lane shows it.  With
    // derivatives plane by plane as they leave the ring; for the values by a sum
    // that turns NaN and stands for all of the chunk's planes, cheaper where chunks
    // are short (50000 blocks of 8^3: 2.82 ms, 2.86 plane by plane; 256 of 64^3:
    // 97 us either way).  All channels of 128 blocks of 64^3: 267 us either way, but
    // with NaN in the data the planes of the sum take 0.76 ms, single planes 0.55
    float chk = 0.0f;
    auto mark = [&](uint64_t set) __attribute__((always_inline)) {
        if ((uint32_t)set) atomicOr(&sm.bad[0], (uint32_t)set);
        if ((uint32_t)(set >> 32)) atomicOr(&sm.bad[1], (uint32_t)(set >> 32));
    };
    auto check = [&](float v, int i) __attribute__((always_inline)) {
        if constexpr (!DER) chk = fmaf(0.0f, v, chk);
        else if (!(fabsf(v) <= 3.402823466e38f)) atomicOr(&sm.bad[i >> 5], 1u << (i & 31));
    };
    const int lplane = open ? lbase : (c - 1) * R * plane;  // this chunk's planes in LDS
    auto put_plane = [&](int slot, float *dst, int i, const float *add)
        __attribute__((always_inline)) {
        const bool mine = i >= i0 && i < i1;
        // opaque, so that the masks below are formed here and not kept in
        // scalar registers through the slice loop
        int j0 = 4 * gq, kk = k;
        asm volatile("" : "+v"(j0), "+v"(kk));
#pragma unroll
        for (int jj = 0; jj < kJT; ++jj) {
            const int jt = 2 * jp + jj;
            if (jt >= njt) continue;
#pragma unroll
            for (int m = 0; m < R; ++m) {
                if (m != slot) continue;
                if (jj == 0) check(ring[jj][m][0], i);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = (16 * jt + r) * nz;  // uniform
                    if ((dst || mine) && 16 * jt + j0 + r < ny && kk < nz) {
                        float v = ring[jj][m][r];
                        if (add) v = add[lane_e + row] + v;
                        if (dst) dst[lane_e + row] = v;
                        else
                            __builtin_amdgcn_raw_buffer_store_b32(
                                __float_as_uint(v), gs, (uint32_t)lane_e * 4u,
                                (uint32_t)(i * plane + row) * 4u, 0);
                    }
                }
                ring[jj][m] = f32x4a{0.0f, 0.0f, 0.0f, 0.0f};
            }
        }
    };
    // a completed plane of this chunk: shared with the chunk to the left
    // (its partial goes to LDS) or this chunk's alone (stored)
    auto flush = [&](int i) __attribute__((always_inline)) {
        if (open || i <= Hprev)
            put_plane(i % R, sm.lb + lplane + (i - Lc) * plane, i, nullptr);
        else
            put_plane(i % R, nullptr, i, nullptr);
    };

    int top = Lc - 1;  // newest plane in the ring
    if (active) {
        // the k tile's z band: the 16-column groups q = q0 + q', q' < nq, in
        // which some w has a basis entry for one of the tile's k (a tile no
        // position touches takes one group of zero weights)
        const int qlo = __builtin_amdgcn_readfirstlane(sm.tw[0][nt] >> 4);
        const int qhi = __builtin_amdgcn_readfirstlane(sm.tw[1][nt] >> 4);
        const int nq = qhi >= qlo ? qhi - qlo + 1 : 1;
        const int q0 = qhi >= qlo ? qlo : 0;
        // values only: operands held for the whole block, the z basis at the
        // lane's w = 16 (q0 + q') + 4 gq + j for its k, the y basis at its 16
        // v positions for its j (zero outside each j tile's band, so the y
        // product runs over all row bands)
        float bzs[4][4], by[MB][4][kJT];
        if constexpr (!DER) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    bzs[q][j] = zval(16 * (q0 + q) + 4 * gq + j, k, sm.zN);
#pragma unroll
            for (int mt = 0; mt < MB; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int jj = 0; jj < kJT; ++jj)
                        by[mt][r][jj] = yval(16 * mt + 4 * gq + r, 16 * (2 * jp + jj) + l16, sm.yN);
        }

        // slice loads: 16 bytes of row 16 m + l16 at w = 16 q + 4 gq, rows
        // and columns clamped into the slice (the bases are zero there, so
        // the values read have no weight; every lane issues the same loads):
        // a buffer resource over the block, the lane's row and column in
        // one 32-bit offset, the channel and slice in the scalar offset.  In
        // rows that are not whole vectors the last load of a row runs past
        // its end (past the block's end it reads zeros), and the values of
        // no column are zeroed before use.
        const int64_t vox = (int64_t)rx * ry * rz;
        const int nch = __builtin_popcount(mask);
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(g + (int64_t)b * nch * vox,
                                                    (uint32_t)(nch * vox * 4));
        uint32_t roff[MB], coff[4];
#pragma unroll
        for (int t = 0; t < MB; ++t) roff[t] = (uint32_t)(min(16 * t + l16, ry - 1) * rz * 4);
#pragma unroll
        for (int t = 0; t < 4; ++t)
            coff[t] = (uint32_t)(min(16 * t + 4 * gq, (rz - 1) & ~3) * 4);
        const uint32_t sbytes = (uint32_t)(ry * rz * 4);
        // (the range check need not see the scalar offset: where a load may
        // leave the block, all of its offset is in the vector part)
        auto load = [&](uint32_t at, uint32_t dead, int mt, int q) -> float4 {
            const uint32_t in = roff[mt] + coff[q];
            const u32x4 x = RAG || DER ? __builtin_amdgcn_raw_buffer_load_b128(rs, in + (at + dead), 0, 0)
                                : __builtin_amdgcn_raw_buffer_load_b128(rs, in + dead, at, 0);
            return make_float4(__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]),
                               __uint_as_float(x[3]));
        };
        const int nj = min(2, njt - 2 * jp);
        // the slice loop, straight-line code for each (nq, one or two j tiles)
        auto slices = [&](auto NQc, auto NJc) __attribute__((always_inline)) {
            constexpr int NQ = decltype(NQc)::value, NJ = decltype(NJc)::value;
            auto loads = [&](uint32_t at, uint32_t dead, float4(&f)[MB][NQ]) {
#pragma unroll
                for (int mt = 0; mt < MB; ++mt)
#pragma unroll
                    for (int q = 0; q < NQ; ++q) f[mt][q] = load(at, dead, mt, min(q0 + q, 3));
            };
            // value j of a load of column group q, zero past the row's end
            auto val = [&](const float4 &f, int q, int j) {
                const float x = j == 0 ? f.x : (j == 1 ? f.y : (j == 2 ? f.z : f.w));
                return RAG && 16 * min(q0 + q, 3) + 4 * gq + j >= rz ? 0.0f : x;
            };
            // advance the ring to slice u's span
            auto advance = [&](int u) __attribute__((always_inline)) {
                const int s = __builtin_amdgcn_readfirstlane(sm.xS[u]);
                while (top < s) {  // uniform: plane top+1 enters, plane top-P leaves
                    ++top;
                    if (top - R >= Lc) flush(top - R);
                }
            };
          if constexpr (!DER) {
            float4 ga[MB][NQ];
            loads((uint32_t)ua * sbytes, 0u, ga);
            for (int u = ua; u <= ub; ++u) {
                const int un = u < ub ? u + 1 : u;  // the next slice (the last one again at the end)
                // z: independent chains, one per 16-row band
                f32x4a Z[MB];
#pragma unroll
                for (int mt = 0; mt < MB; ++mt) Z[mt] = f32x4a{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int mt = 0; mt < MB; ++mt)
                            Z[mt] = mma4(val(ga[mt][q], q, j), bzs[q][j], Z[mt]);
                // the next slice, in flight during the rest of this one
                loads((uint32_t)un * sbytes, 0u, ga);
                // y: the y basis is zero outside each j tile's band
                f32x4a Y[kJT], Yo[kJT];
#pragma unroll
                for (int jj = 0; jj < kJT; ++jj) Y[jj] = Yo[jj] = f32x4a{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int mt = 0; mt < MB; ++mt)
#pragma unroll
                    for (int jj = 0; jj < NJ; ++jj) {
                        Y[jj] = mma4(by[mt][0][jj], Z[mt][0], Y[jj]);
                        Yo[jj] = mma4(by[mt][1][jj], Z[mt][1], Yo[jj]);
                        Y[jj] = mma4(by[mt][2][jj], Z[mt][2], Y[jj]);
                        Yo[jj] = mma4(by[mt][3][jj], Z[mt][3], Yo[jj]);
                    }
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) Y[jj] += Yo[jj];
                // x contraction: advance the ring to this slice's span, then
                // add its contributions to the p+1 planes it touches
                advance(u);
                const float4 cx = sm.xB[u];
                const float cf[4] = {cx.x, cx.y, cx.z, cx.w};
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
                    for (int m = 0; m < R; ++m)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            ring[jj][m][r] = fmaf(cf[m], Y[jj][r], ring[jj][m][r]);
            }
          } else {
            // channels 1, 0, 3, 2 of a slice in turn, two buffers, each
            // reloaded two channels ahead once its z product has read it; one
            // Z tile set is live at a time
            const uint32_t vb = (uint32_t)(vox * 4);
            // a channel that is not there reads zeros past the resource's end
            auto fetch = [&](int u, int ch, float4(&f)[MB][NQ]) __attribute__((always_inline)) {
                const bool has = mask & (1u << ch);
                const uint32_t c = (uint32_t)__builtin_popcount(mask & ((1u << ch) - 1u));
                loads(has ? c * vb + (uint32_t)u * sbytes : 0u, has ? 0u : 0x40000000u, f);
            };
            float4 ga[MB][NQ], gb[MB][NQ];
            fetch(ua, 1, ga);
            fetch(ua, 0, gb);
            for (int u = ua; u <= ub; ++u) {
                const int un = u < ub ? u + 1 : u;
                int ln = lane;  // opaque: the operands stay in LDS
                asm volatile("" : "+v"(ln));
                f32x4a Z[MB];
                auto zero = [&](f32x4a *f, int n) __attribute__((always_inline)) {
#pragma unroll
                    for (int m = 0; m < n; ++m) f[m] = f32x4a{0.0f, 0.0f, 0.0f, 0.0f};
                };
                auto zmul = [&](const float4(&f)[MB][NQ], int d) __attribute__((always_inline)) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        const float4 o = sm.op[0][d][nt][min(q0 + q, 3)][ln];
                        const float ov[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
                        for (int j = 0; j < 4; ++j)
#pragma unroll
                            for (int mt = 0; mt < MB; ++mt)
                                Z[mt] = mma4(val(f[mt][q], q, j), ov[j], Z[mt]);
                    }
                };
                // two chains per j tile (even and odd K steps)
                f32x4a Yb[kJT], Yo[kJT], Yd[kJT];
                auto ymul = [&](int d, f32x4a(&Y)[kJT]) __attribute__((always_inline)) {
#pragma unroll
                    for (int mt = 0; mt < MB; ++mt)
#pragma unroll
                        for (int jj = 0; jj < NJ; ++jj) {
                            const float4 o = sm.op[1][d][2 * jp + jj][mt][ln];
                            Y[jj] = mma4(o.x, Z[mt][0], Y[jj]);
                            Yo[jj] = mma4(o.y, Z[mt][1], Yo[jj]);
                            Y[jj] = mma4(o.z, Z[mt][2], Y[jj]);
                            Yo[jj] = mma4(o.w, Z[mt][3], Yo[jj]);
                        }
                };
                zero(Yd, kJT);
                zero(Yo, kJT);
                zero(Z, MB);
                if (mask & 2u) zmul(ga, 0);
                fetch(u, 3, ga);
                if (mask & 2u) ymul(0, Yd);
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) Yd[jj] += Yo[jj];
                zero(Yb, kJT);
                zero(Yo, kJT);
                zero(Z, MB);
                if (mask & 1u) zmul(gb, 0);
                fetch(u, 2, gb);
                if (mask & 8u) zmul(ga, 1);
                fetch(un, 1, ga);
                if (mask & 9u) ymul(0, Yb);
                zero(Z, MB);
                if (mask & 4u) zmul(gb, 0);
                fetch(un, 0, gb);
                if (mask & 4u) ymul(1, Yb);
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) Yb[jj] += Yo[jj];
                advance(u);
                const float4 cx = sm.xB[u], ex = sm.xD[u];
                const float cf[4] = {cx.x, cx.y, cx.z, cx.w}, ef[4] = {ex.x, ex.y, ex.z, ex.w};
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
                    for (int m = 0; m < R; ++m)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            ring[jj][m][r] = fmaf(cf[m], Yb[jj][r],
                                                  fmaf(ef[m], Yd[jj][r], ring[jj][m][r]));
            }
          }
        };
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        using I3 = std::integral_constant<int, 3>;
        using I4 = std::integral_constant<int, 4>;
        if (nj == 2) {
            if (nq == 4) slices(I4{}, I2{});
            else if (nq == 3) slices(I3{}, I2{});
            else if (nq == 2) slices(I2{}, I2{});
            else slices(I1{}, I2{});
        } else {
            if (nq == 4) slices(I4{}, I1{});
            else if (nq == 3) slices(I3{}, I1{});
            else if (nq == 2) slices(I2{}, I1{});
            else slices(I1{}, I1{});
        }
        // planes between this chunk's last and the next chunk's first (no
        // slice touches them when the x span jumps by more than p+1 between
        // neighbouring slices) leave the ring as zeros
        while (!open && c + 1 < X && top < Lnext - 1) {
            ++top;
            if (top - R >= Lc) flush(top - R);
        }
        // planes still in the ring that no chunk to the right shares
        for (int i = max(Lc, top - P); i <= top && (open || i < Lnext); ++i) flush(i);
#pragma unroll
        for (int m = 0; m < R; ++m)  // those still shared: slot m holds plane top - (top - m) mod R
            check(ring[0][m][0], max(top - (top - m + R) % R, 0));
        if (chk != chk) mark((~0ull >> (63 - top)) & (~0ull << Lc));
    }
    lds_barrier();  // left partial planes of every chunk in LDS
    const uint32_t bad_lo = sm.bad[0], bad_hi = sm.bad[1];
    if (open) {
        // every plane of the segment: the chunks that touch it, in order
        for (int e = tid; e < (i1 - i0) * plane; e += kAT) {
            const int i = i0 + e / plane, r = e - (i - i0) * plane;
            float sum = 0.0f;
            int at = 0;
            for (int c = 0; c < X; ++c) {
                const int lo = sm.xS[slo + c * len / X] - P;
                const int hi = sm.xS[slo + (c + 1) * len / X - 1];
                if (i >= lo && i <= hi) sum += sm.lb[at + (i - lo) * plane + r];
                at += (hi - lo + 1) * plane;
            }
            Gb[(int64_t)i * plane + r] = sum;
        }
    }
    if (!open && active && c + 1 < X) {
        // planes shared with the chunk to the right: its partial + this one
        for (int i = Lnext; i <= top; ++i)
            put_plane(i % R, nullptr, i, sm.lb + (c * R + (i - Lnext)) * plane);
    }
    // planes of the segment that no slice touches, before its first slice's
    // and after its last one's
    const int lo = __builtin_amdgcn_readfirstlane(sm.xS[slo]) - P;
    const int hl = max(__builtin_amdgcn_readfirstlane(sm.xS[shi - 1]) + 1, i0);
    if (!open) {
        for (int e = tid; e < (min(lo, i1) - i0) * plane; e += kAT) Gb[(int64_t)i0 * plane + e] = 0.0f;
        for (int e = tid; e < (i1 - hl) * plane; e += kAT) Gb[(int64_t)hl * plane + e] = 0.0f;
    }
    const uint64_t bad =
        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)bad_hi) << 32 |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)bad_lo)) &
        (~0ull >> (64 - i1)) & (~0ull << i0);  // of this segment
    if (bad) {
        const int64_t vox = (int64_t)rx * ry * rz;
        adj_windows<P, DER>(ny, nz, ry, rz, mask, g + (int64_t)b * __builtin_popcount(mask) * vox,
                            vox, Gb, bad, slo, shi, sm);
    }
}

template <bool DER, bool RAG, int MB>
__global__ __launch_bounds__(kAT) void adjoint_kernel(const fa_block *blocks, int nseg,
                                                      const float *knots, int rx, int ry, int rz,
                                                      uint32_t mask, const float *g, float *G) {
    extern __shared__ float4 dyn_lds[];
    AmSmem<DER> &sm = *reinterpret_cast<AmSmem<DER> *>(dyn_lds);
    // one workgroup per (micro-model, segment)
    const int b = blockIdx.x / nseg, seg = blockIdx.x - b * nseg;
    const fa_block &B = blocks[b];
    const int p = B.degree[0];
    if (p == 3) adj_block<3, DER, RAG, MB>(B, knots, rx, ry, rz, mask, g, G, b, seg, nseg, sm);
    else if (p == 2) adj_block<2, DER, RAG, MB>(B, knots, rx, ry, rz, mask, g, G, b, seg, nseg, sm);
    else adj_block<1, DER, RAG, MB>(B, knots, rx, ry, rz, mask, g, G, b, seg, nseg, sm);
}

template <bool DER, bool RAG, int MB>
hipError_t launch(const fa_block *blocks, int nblocks, const float *knots, int rx, int ry, int rz,
                  uint32_t mask, const float *g, float *G, hipStream_t s) {
    // raise the dynamic LDS limit once per process (before any graph capture)
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void *>(&adjoint_kernel<DER, RAG, MB>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(AmSmem<DER>));
    if (attr != hipSuccess) return attr;
    // one workgroup fits a CU: segments while a CU would be without one
    const int nseg = std::max(1, std::min(kMaxSegs, kCUs / nblocks));
    const int64_t values = (int64_t)__builtin_popcount(mask) * rx * ry * rz;
    for (int b0 = 0; b0 < nblocks; b0 += kMostGroups) {
        const int n = std::min(nblocks - b0, kMostGroups);
        hipLaunchKernelGGL((adjoint_kernel<DER, RAG, MB>), dim3((unsigned)n * nseg), dim3(kAT),
                           sizeof(AmSmem<DER>), s, blocks + b0, nseg, knots, rx, ry, rz, mask,
                           g + b0 * values, G);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int MB>
hipError_t launch_rows(const fa_block *blocks, int nblocks, const float *knots, int rx, int ry,
                       int rz, uint32_t mask, const float *g, float *G, hipStream_t s) {
    const bool rag = (rz & 3) != 0;
    if (mask == 1u)
        return rag ? launch<false, true, MB>(blocks, nblocks, knots, rx, ry, rz, mask, g, G, s)
                   : launch<false, false, MB>(blocks, nblocks, knots, rx, ry, rz, mask, g, G, s);
    return rag ? launch<true, true, MB>(blocks, nblocks, knots, rx, ry, rz, mask, g, G, s)
               : launch<true, false, MB>(blocks, nblocks, knots, rx, ry, rz, mask, g, G, s);
}

}  // namespace

hipError_t launch_adjoint(const fa_block *blocks, int nblocks, const float *knots, int rx, int ry,
                          int rz, uint32_t mask, const float *g, float *G, hipStream_t s) {
    if (ry > kAM || rz > kAM) return hipErrorNotSupported;
    if (nblocks <= 0) return hipSuccess;
    mask &= 15u;
    // 16-row bands of the cotangent's slices that hold rows: products over the
    // rows of no band are zeros.  Four at any resolution cost (20000 blocks of
    // 16^3, mixed NCP and degree) values 1.41 ms, all channels 2.62; two 1.21 and
    // 2.00; one 1.07 and 1.73.  4000 of 32^3: four 0.455 and 1.14, two 0.356, 0.746
    return ry <= 16   ? launch_rows<1>(blocks, nblocks, knots, rx, ry, rz, mask, g, G, s)
           : ry <= 32 ? launch_rows<2>(blocks, nblocks, knots, rx, ry, rz, mask, g, G, s)
                      : launch_rows<4>(blocks, nblocks, knots, rx, ry, rz, mask, g, G, s);
}

}  // namespace fa
