// Grid decode of batched micro-models on gfx950 (FP32 VALU forms).
//
// decode_sep: the batched, persistent, separable form (rows a0-a6).
//   The tensor-product sum over the (p+1)^3 window factorises per axis, so
//   one column (v, w) of a work item is decoded as
//     T_B[j] = sum_k Bz[w][k] P[i][j][k],   T_D[j] = sum_k Dz[w][k] P[i][j][k]
//     U_BB[i] = sum_j By[v][j] T_B[j],  U_DB[i] = sum_j Dy[v][j] T_B[j],
//     U_BD[i] = sum_j By[v][j] T_D[j]
//     value = sum_i Bx[u][i] U_BB[i], d/du = sum_i Dx[u][i] U_BB[i],
//     d/dv  = sum_i Bx[u][i] U_DB[i], d/dw = sum_i Bx[u][i] U_BD[i]
//   with every sum banded to the p+1 non-zero basis functions.  A lane owns
//   one (v, w) column (lanes along z, so every store is a contiguous 256 B
//   row) and walks u = 0..Rx-1 keeping the p+1 newest U values in
//   registers; U[i] is built on the fly from a lattice slab staged once per
//   work item in LDS.  The x-axis basis (span + p+1 values + p+1
//   derivatives per u) is tabulated in LDS once per item and read as
//   broadcasts.  Work items are (block, y-row range, 64-wide z chunk); a
//   workgroup runs the items a host plan assigned to it, or a grid-stride
//   share of the default order.
//
// The residual form (MODE 1) decodes the value channel only and, instead of
//   the value f, stores gscale * (f - samples) for a fit's loss, summing
//   (f - samples)^2 in FP64 per lane (x order), per wave (fixed shuffle
//   tree) and per work item (waves in order) into one partial per item; a
//   second kernel adds each block's partials in item order.  The samples
//   are read four x positions ahead through a buffer resource, and dead lanes
//   load and store at an offset outside every resource (no branch), so the
//   x walk issues a fixed number of memory operations per step.
// The error form (MODE 2) reads the samples the same way and stores nothing per
//   voxel: each item leaves max |f - samples| and the FP64 sum of squares,
//   and a second kernel turns them into each block's (max, rms) error, the
//   error-map entry of the adaptive NCP search, without the decode ever
//   reaching memory.
//
// decode_plain: the baseline -- one thread per voxel, one launch per block,
//   each thread doing its own span searches, basis evaluation and (p+1)^3
//   window sum straight from global memory.
#include "fa_sep.hpp"

namespace fa {
namespace {

// The x positions [ua, ub) that segment seg of an item of micro-model B walks,
// none if ua == ub.  A segment forms p + 1 control planes of its own before its
// first position, (p + 1)^2 products a column each; where the planes of an
// item's segments cost a.xcost or more, segment 0 walks the whole item and the
// others do nothing.  Segments are then dealt to an item's workgroups from one
// that a hash of the tile picks: always from the first, the working ones of
// whole items would meet on a quarter of the CUs (1024 blocks of 64^3, NCP 32,
// four workgroups an item: 1540 us; hashed 812; whole items from the outset 806).
__device__ __forceinline__ void item_range(const DecodeLaunch &a, const fa_block &B, int64_t tile,
                                           int seg, int &ua, int &ub) {
    const int p = B.degree[0], segs = a.xsegs;
    seg = (seg + (int)(((uint32_t)tile * 0x9e3779b1u) >> 16)) % segs;
    const bool whole = (B.ncp[0] - p + segs * (p + 1)) * (p + 1) * (p + 1) >= a.xcost;
    ua = whole ? 0 : seg * a.rx / segs;
    ub = whole ? (seg == 0 ? a.rx : 0) : (seg + 1) * a.rx / segs;
}

template <int WAVES, bool NT, int MODE>
__global__ __launch_bounds__(WAVES * 64) void decode_sep_kernel(DecodeLaunch a) {
    extern __shared__ float4 dyn_lds[];
    SepSmem sm = carve(dyn_lds, a.rx, a.slab);
    const int wg = xcd_order(blockIdx.x, gridDim.x);
    int64_t beg, end, step;
    int seg = 0;
    if (a.work) {  // xsegs workgroups run a plan's group, one x segment each
        const int group = wg / a.xsegs;
        seg = wg - group * a.xsegs;
        beg = a.wg_off[group];
        end = a.wg_off[group + 1];
        step = 1;
    } else {
        beg = wg;
        end = a.nitems;
        step = gridDim.x;
    }
    const int64_t per = (int64_t)a.nrowt * a.ncolt;
    for (int64_t it = beg; it < end; it += step) {
        int b, row0, nrows, col0;
        int64_t tile = it;
        if (a.work) {
            const fa_work wk = a.work[it];
            b = wk.block;
            row0 = wk.row0;
            nrows = wk.nrows;
            col0 = wk.col0;
        } else {
            // a tile's x segments in a row (a block's tiles of one segment in a
            // row: 270 us against 260 for 384 uneven blocks, records)
            tile = it / a.xsegs;
            seg = (int)(it - tile * a.xsegs);
            b = (int)(tile / per);
            const int r = (int)(tile - (int64_t)b * per);
            row0 = (r / a.ncolt) * a.rows;
            nrows = min(a.rows, a.ry - row0);
            col0 = (r % a.ncolt) * kWave;
        }
        int ua = seg * a.rx / a.xsegs, ub = (seg + 1) * a.rx / a.xsegs;
        if constexpr (MODE == 0 || MODE == 3) {  // (all four channels)
            if (a.xcost != 0) item_range(a, a.blocks[b], tile, seg, ua, ub);
            if (ua == ub) continue;  // uniform over the workgroup
        }
        // the item's index in the default order, whatever order runs it
        const int64_t item = (int64_t)b * per + (row0 / a.rows) * a.ncolt + col0 / kWave;
        const int p = a.blocks[b].degree[0];
        if (p == 3) sep_item<3, NT, MODE>(a, b, row0, nrows, col0, ua, ub, item, sm);
        else if (p == 2) sep_item<2, NT, MODE>(a, b, row0, nrows, col0, ua, ub, item, sm);
        else sep_item<1, NT, MODE>(a, b, row0, nrows, col0, ua, ub, item, sm);
    }
}

// ------------------------------------------------------------------ plain

template <int P>
__device__ __forceinline__ void plain_voxel(const fa_block &B, const float *knots,
                                            const float *ctrl, int u, int v, int w, int rx,
                                            int ry, int rz, float (&res)[4]) {
    const int nx = B.ncp[0], ny = B.ncp[1], nz = B.ncp[2];
    const float *tx = knots + B.knot_off;
    const float *ty = tx + nx + P + 1;
    const float *tz = ty + ny + P + 1;
    const float pu = grid_pos(u, rx), pv = grid_pos(v, ry), pw = grid_pos(w, rz);
    const int su = span_search(nx, P, tx, pu);
    const int sv = span_search(ny, P, ty, pv);
    const int sw = span_search(nz, P, tz, pw);
    float xB[P + 1], xD[P + 1], yB[P + 1], yD[P + 1], zB[P + 1], zD[P + 1];
    basis_ders<P>(tx, su, pu, xB, xD);
    basis_ders<P>(ty, sv, pv, yB, yD);
    basis_ders<P>(tz, sw, pw, zB, zD);
    float f = 0.0f, fx = 0.0f, fy = 0.0f, fz = 0.0f;
    const float *base = ctrl + B.ctrl_off;
    for (int i = 0; i <= P; ++i) {
        for (int j = 0; j <= P; ++j) {
            for (int k = 0; k <= P; ++k) {
                const float c = base[((int64_t)(su - P + i) * ny + (sv - P + j)) * nz + (sw - P + k)];
                f += xB[i] * yB[j] * zB[k] * c;
                fx += xD[i] * yB[j] * zB[k] * c;
                fy += xB[i] * yD[j] * zB[k] * c;
                fz += xB[i] * yB[j] * zD[k] * c;
            }
        }
    }
    res[0] = f;
    res[1] = fx;
    res[2] = fy;
    res[3] = fz;
}

__global__ __launch_bounds__(256) void decode_plain_kernel(const fa_block *blocks, int b,
                                                           const float *knots,
                                                           const float *ctrl, int rx, int ry,
                                                           int rz, uint32_t mask, int nch,
                                                           float *out) {
    const int64_t vox = (int64_t)rx * ry * rz;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= vox) return;
    const int w = (int)(idx % rz);
    const int v = (int)((idx / rz) % ry);
    const int u = (int)(idx / ((int64_t)ry * rz));
    const fa_block &B = blocks[b];
    float res[4];
    const int p = B.degree[0];
    if (p == 3) plain_voxel<3>(B, knots, ctrl, u, v, w, rx, ry, rz, res);
    else if (p == 2) plain_voxel<2>(B, knots, ctrl, u, v, w, rx, ry, rz, res);
    else plain_voxel<1>(B, knots, ctrl, u, v, w, rx, ry, rz, res);
    float *o = out + (int64_t)b * nch * vox + idx;
    int c = 0;
    for (int ch = 0; ch < 4; ++ch) {
        if ((mask >> ch) & 1u) {
            o[(int64_t)c * vox] = res[ch];
            ++c;
        }
    }
}

// sumsq[b] = sum of block b's per-item partials, in item order
__global__ void residual_combine_kernel(const double *partials, int nblocks, int per,
                                        double *sumsq) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nblocks) return;
    double t = 0.0;
    for (int k = 0; k < per; ++k) t += partials[(int64_t)b * per + k];
    sumsq[b] = t;
}

// errs[b * stride - 2 c + {0, 1}] = (max, sqrt(sum / vox)) of block b under
// candidate c from its per-item (max, sum of squares) partials, in item order
__global__ void errors_combine_kernel(const double *partials, int nblocks, int ncand, int per,
                                      int64_t vox, float *errs, int64_t stride) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= nblocks * ncand) return;
    double m = 0.0, t = 0.0;
    for (int k = 0; k < per; ++k) {
        m = fmax(m, partials[2 * ((int64_t)e * per + k)]);
        t += partials[2 * ((int64_t)e * per + k) + 1];
    }
    float *o = errs + (int64_t)(e % nblocks) * stride - 2 * (e / nblocks);
    o[0] = (float)m;
    o[1] = (float)sqrt(t / (double)vox);
}

}  // namespace

template <bool NT, int MODE>
hipError_t launch_sep(const DecodeLaunch &a, int waves, int grid, hipStream_t s) {
    const size_t lds = sep_lds_bytes(a.rx, a.slab);
    // raise the dynamic LDS limit once per process to the largest layout
    static const hipError_t attr = [] {
        const int most = (int)sep_lds_bytes(kMaxRes, kSlabMax);
        hipError_t r = hipSuccess, e;
        const void *ks[4] = {reinterpret_cast<const void *>(&decode_sep_kernel<1, NT, MODE>),
                             reinterpret_cast<const void *>(&decode_sep_kernel<2, NT, MODE>),
                             reinterpret_cast<const void *>(&decode_sep_kernel<4, NT, MODE>),
                             reinterpret_cast<const void *>(&decode_sep_kernel<8, NT, MODE>)};
        for (const void *k : ks)
            if ((e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, most)) !=
                hipSuccess)
                r = e;
        return r;
    }();
    if (attr != hipSuccess) return attr;
    switch (waves) {
    case 2: hipLaunchKernelGGL((decode_sep_kernel<2, NT, MODE>), dim3(grid), dim3(128), lds, s, a); break;
    case 4: hipLaunchKernelGGL((decode_sep_kernel<4, NT, MODE>), dim3(grid), dim3(256), lds, s, a); break;
    case 8: hipLaunchKernelGGL((decode_sep_kernel<8, NT, MODE>), dim3(grid), dim3(512), lds, s, a); break;
    default: hipLaunchKernelGGL((decode_sep_kernel<1, NT, MODE>), dim3(grid), dim3(64), lds, s, a); break;
    }
    return hipGetLastError();
}

hipError_t launch_decode_sep(const DecodeLaunch &a, int waves, int grid, hipStream_t s) {
    if (a.samples && a.error_form) return launch_sep<false, 2>(a, waves, grid, s);
    if (a.interleave)
        return a.nt_store ? launch_sep<true, 3>(a, waves, grid, s)
                          : launch_sep<false, 3>(a, waves, grid, s);
    if (!a.samples && a.mask == 1u)
        return a.nt_store ? launch_sep<true, 4>(a, waves, grid, s)
                          : launch_sep<false, 4>(a, waves, grid, s);
    if (a.samples)
        return a.nt_store ? launch_sep<true, 1>(a, waves, grid, s)
                          : launch_sep<false, 1>(a, waves, grid, s);
    return a.nt_store ? launch_sep<true, 0>(a, waves, grid, s)
                      : launch_sep<false, 0>(a, waves, grid, s);
}

hipError_t launch_residual_combine(const double *partials, int nblocks, int per, double *sumsq,
                                   hipStream_t s) {
    hipLaunchKernelGGL(residual_combine_kernel, dim3((nblocks + 255) / 256), dim3(256), 0, s,
                       partials, nblocks, per, sumsq);
    return hipGetLastError();
}

hipError_t launch_errors_combine(const double *partials, int nblocks, int ncand, int per,
                                 int64_t vox, float *errs, int64_t stride, hipStream_t s) {
    hipLaunchKernelGGL(errors_combine_kernel, dim3((nblocks * ncand + 255) / 256), dim3(256), 0, s,
                       partials, nblocks, ncand, per, vox, errs, stride);
    return hipGetLastError();
}

hipError_t launch_decode_plain(const fa_block *blocks, int nblocks, const float *knots,
                               const float *ctrl, int rx, int ry, int rz, uint32_t mask,
                               float *out, hipStream_t s) {
    const int64_t vox = (int64_t)rx * ry * rz;
    const int nch = __builtin_popcount(mask & 15u);
    const int grid = (int)((vox + 255) / 256);
    for (int b = 0; b < nblocks; ++b) {
        hipLaunchKernelGGL(decode_plain_kernel, dim3(grid), dim3(256), 0, s, blocks, b, knots,
                           ctrl, rx, ry, rz, mask, nch, out);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace fa
