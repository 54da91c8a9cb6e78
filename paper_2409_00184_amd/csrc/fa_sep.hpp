// One work item of the separable grid decode (FP32 on the vector ALUs): shared
// by the batched decode and, for items that its tile does not take, by the
// matrix-core decode.  The scheme is described in fa_decode.hip.
#pragma once

#include <type_traits>

#include "fa_device.hpp"
#include "fa_internal.hpp"

namespace fa {
namespace {

// Dynamic LDS of the separable decode: x table (rx rows), knots, slab.
struct SepSmem {
    float4 *xB;
    float4 *xD;
    int *xS;
    float *kn;
    float *slab;
    int slab_floats;
};

__device__ __forceinline__ SepSmem carve(void *base, int rx, int slab) {
    SepSmem s;
    char *p = static_cast<char *>(base);
    s.xB = reinterpret_cast<float4 *>(p);
    p += sizeof(float4) * rx;
    s.xD = reinterpret_cast<float4 *>(p);
    p += sizeof(float4) * rx;
    s.kn = reinterpret_cast<float *>(p);
    p += sizeof(float) * (kMaxKnotsPerBlock + 4);
    s.xS = reinterpret_cast<int *>(p);
    p += sizeof(int) * ((rx + 3) & ~3);
    s.slab = reinterpret_cast<float *>(p);
    s.slab_floats = slab;
    return s;
}

__host__ __device__ size_t sep_lds_bytes(int rx, int slab) {
    return sizeof(float4) * 2 * rx + sizeof(float) * (kMaxKnotsPerBlock + 4) +
           sizeof(int) * ((rx + 3) & ~3) + sizeof(float) * slab;
}

template <int P>
__device__ __forceinline__ float4 pack4(const float (&v)[P + 1]) {
    float4 r;
    r.x = v[0];
    r.y = P >= 1 ? v[P >= 1 ? 1 : 0] : 0.0f;
    r.z = P >= 2 ? v[P >= 2 ? 2 : 0] : 0.0f;
    r.w = P >= 3 ? v[P >= 3 ? 3 : 0] : 0.0f;
    return r;
}

__device__ __forceinline__ float comp(const float4 &v, int r) {
    return r == 0 ? v.x : (r == 1 ? v.y : (r == 2 ? v.z : v.w));
}

// MODE 0: decode, 1: residual form, 2: error form, 3: decode of all four
// channels stored interleaved (one 16-byte record per voxel), 4: decode of
// the values alone
//
// The item's nrows x ncols columns are dealt to the lanes back to back, so
// that narrow grids (ncols < 64) leave no lane idle but the last wave's.  The
// walk covers x positions [ua, ub).  Every access of the walk goes through a
// buffer resource with the lane's column in the vector offset (beyond the
// resource for a lane without a column) and the x position and channel, always
// inside, in the scalar offset, so a step spends no vector instruction on addresses: the
// error form of 256 blocks of 64^3 went from 115 to 95 us.
template <int P, bool NT, int MODE>
__device__ void sep_item(const DecodeLaunch &a, int b, int row0, int nrows, int col0, int ua, int ub,
                         int64_t item, SepSmem &sm) {
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, nwaves = nthr >> 6;
    const fa_block &B = a.blocks[b];
    const int nx = B.ncp[0], ny = B.ncp[1], nz = B.ncp[2];
    const int64_t koff = B.knot_off, coff = B.ctrl_off;
    const float scale = B.scale;
    const int nkn = nx + ny + nz + 3 * (P + 1);
    constexpr bool RESID = MODE == 1 || MODE == 2;  // reads the samples
    constexpr bool GRAD = MODE == 1;   // stores the scaled residual
    constexpr int kCpol = NT ? 2 : 0;  // buffer accesses: non-temporal
    constexpr uint32_t kDead = 0x80000000u;  // beyond every resource

    lds_barrier();  // the previous item is done with the shared buffers
    for (int e = tid; e < nkn; e += nthr) sm.kn[e] = a.knots[koff + e];
    lds_barrier();
    const float *tx = sm.kn;
    const float *ty = tx + nx + P + 1;
    const float *tz = ty + ny + P + 1;

    // control planes [i0, i1) cover the x windows of the item, lattice rows j
    // in [jlo, jhi] its y windows
    const int i0 = span_search(nx, P, tx, grid_pos(ua, a.rx)) - P;
    const int i1 = span_search(nx, P, tx, grid_pos(ub - 1, a.rx)) + 1;
    const int jlo = span_search(ny, P, ty, grid_pos(row0, a.ry)) - P;
    const int jhi = span_search(ny, P, ty, grid_pos(row0 + nrows - 1, a.ry));
    const int plane = (jhi - jlo + 1) * nz;  // slab floats per x plane
    const int ic = min(i1 - i0, sm.slab_floats / plane);
    const bool single = (ic == i1 - i0);

    // Slab element e = ii * plane + r is value r of control plane c0 + ii's
    // rows jlo..jhi, which lie back to back in the lattice.  A thread walks
    // its elements (stride nthr) with (ii, r) kept incrementally, and issues
    // four loads before their four LDS writes.
    const int nynz = ny * nz;
    const int dii = nthr / plane, dr = nthr - dii * plane;
    const int ii0 = tid / plane, r0 = tid - ii0 * plane;
    auto stage = [&](int c0, int c1) {
        const int cnt = (c1 - c0) * plane;
        const int64_t base = coff + (int64_t)(c0 * ny + jlo) * nz;
        int ii = ii0, r = r0;
        for (int e0 = tid; e0 < cnt; e0 += 4 * nthr) {
            float v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[q] = e0 + q * nthr < cnt
                           ? load_ctrl(a.ctrl, a.dtype, base + (ii * nynz + r), scale)
                           : 0.0f;
                r += dr;
                ii += dii;
                if (r >= plane) {
                    r -= plane;
                    ++ii;
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (e0 + q * nthr < cnt) sm.slab[e0 + q * nthr] = v[q];
        }
    };
    if (single) stage(i0, i1);

    // x table: span and basis of the item's positions along x
    for (int u = ua + tid; u < ub; u += nthr) {
        const float uu = grid_pos(u, a.rx);
        const int s = span_search(nx, P, tx, uu);
        float N[P + 1], D[P + 1];
        basis_ders<P>(tx, s, uu, N, D);
        sm.xB[u] = pack4<P>(N);
        if (!RESID && MODE != 4) sm.xD[u] = pack4<P>(D);
        sm.xS[u] = s;
    }
    lds_barrier();  // x table and slab visible

    const int64_t vox = (int64_t)a.rx * a.ry * a.rz;
    const uint32_t vb = (uint32_t)vox * 4u;
    constexpr uint32_t rec = MODE == 3 ? 16u : 4u;  // bytes of a column's store
    const uint32_t pstep = (uint32_t)(a.ry * a.rz) * rec;
    double acc = 0.0;
    float amax = 0.0f;
    // this block's samples (residual and error form), and its output: the
    // channels of the mask one after the other, or records
    const __amdgpu_buffer_rsrc_t yr = make_rsrc(
        RESID ? a.samples + (int64_t)(MODE == 2 ? b % a.nsrc : b) * vox : a.out, RESID ? vb : 0u);
    const int nch = RESID || MODE == 4 ? 1 : a.nch;
    const __amdgpu_buffer_rsrc_t orc =
        make_rsrc(MODE == 2 ? nullptr : a.out + (int64_t)b * nch * vox,
                  MODE == 2 ? 0u : (uint32_t)nch * vb);
    uint32_t choff[4];
    {
        uint32_t c = 0;
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) {
            choff[ch] = c;
            c += (a.mask >> ch) & 1u ? vb : 0u;
        }
    }

    const int ncols = min(kWave, a.rz - col0), total = nrows * ncols;
    for (int rb = kWave * wave; rb < (single ? total : ((total - 1) / (kWave * nwaves) + 1) * kWave * nwaves);
         rb += kWave * nwaves) {
        // this lane's column; a lane past the end repeats the last one, stores
        // nothing and adds nothing
        const bool live = rb + lane < total;
        const int id = live ? rb + lane : total - 1;
        const int rr = id / ncols;
        const int v = row0 + rr, w = col0 + id - rr * ncols;
        const float zw = grid_pos(w, a.rz), yv = grid_pos(v, a.ry);
        const int sz = span_search(nz, P, tz, zw), sy = span_search(ny, P, ty, yv);
        float zB[P + 1], zD[P + 1], yB[P + 1], yD[P + 1];
        basis_ders<P>(tz, sz, zw, zB, zD);
        basis_ders<P>(ty, sy, yv, yB, yD);
        const int sl0 = (sy - P - jlo) * nz + sz - P;
        const uint32_t col = live ? ((uint32_t)v * (uint32_t)a.rz + (uint32_t)w) * rec : kDead;

      // the x walk, specialised on whether the slab holds every control
      // plane (then it stages nothing inside the walk)
      auto walk = [&](auto single_c) {
        constexpr bool SINGLE = decltype(single_c)::value;
        int clo = i0, chi = SINGLE ? i1 : i0 + ic;
        if (!SINGLE) {
            lds_barrier();
            stage(clo, chi);
            lds_barrier();
        }

        float wBB[P + 1], wDB[P + 1], wBD[P + 1];
#pragma unroll
        for (int r = 0; r <= P; ++r) wBB[r] = wDB[r] = wBD[r] = 0.0f;
        int top = i0 - 1;
        // the sample of x position u (the last one again past the end), loaded
        // four positions ahead into one of four registers used in turn (no
        // register copy waits for a load in flight)
        auto yload = [&](int u) {
            return RESID ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                         yr, col, (uint32_t)min(u, ub - 1) * pstep, 0))
                         : 0.0f;
        };
        // issue order load, store, load, store as in every step, so the
        // counter wait at a step is the same on entry as in the loop (the
        // stores go beyond the resource and are dropped)
        auto ydummy = [&]() {
            if (GRAD) __builtin_amdgcn_raw_buffer_store_b32(0u, orc, kDead, 0, 0);
        };
        float y0 = 0.0f, y1 = 0.0f, y2 = 0.0f, y3 = 0.0f;
        if constexpr (RESID) {
            y0 = yload(ua);
            ydummy();
            y1 = yload(ua + 1);
            ydummy();
            y2 = yload(ua + 2);
            ydummy();
            y3 = yload(ua + 3);
            ydummy();
        }

        auto step = [&](int u, float &ycur) {
            const int s = __builtin_amdgcn_readfirstlane(sm.xS[u]);
            while (top < s) {  // uniform over the workgroup
                ++top;
                if (!SINGLE && top >= chi) {
                    lds_barrier();
                    clo = chi;
                    chi = min(clo + ic, i1);
                    stage(clo, chi);
                    lds_barrier();
                }
                const float *sl = sm.slab + (top - clo) * plane + sl0;
                float tB[P + 1], tD[P + 1];
#pragma unroll
                for (int jj = 0; jj <= P; ++jj) {
                    float x = 0.0f, y = 0.0f;
#pragma unroll
                    for (int kk = 0; kk <= P; ++kk) {
                        const float c = sl[jj * nz + kk];
                        x = fmaf(zB[kk], c, x);
                        y = fmaf(zD[kk], c, y);
                    }
                    tB[jj] = x;
                    tD[jj] = y;
                }
                float uBB = 0.0f, uDB = 0.0f, uBD = 0.0f;
#pragma unroll
                for (int jj = 0; jj <= P; ++jj) {
                    uBB = fmaf(yB[jj], tB[jj], uBB);
                    uDB = fmaf(yD[jj], tB[jj], uDB);
                    uBD = fmaf(yB[jj], tD[jj], uBD);
                }
#pragma unroll
                for (int r = 0; r < P; ++r) {
                    wBB[r] = wBB[r + 1];
                    wDB[r] = wDB[r + 1];
                    wBD[r] = wBD[r + 1];
                }
                wBB[P] = uBB;
                wDB[P] = uDB;
                wBD[P] = uBD;
            }
            const float4 bx = sm.xB[u];
            const float4 dx = RESID || MODE == 4 ? bx : sm.xD[u];
            float val = 0.0f, gx = 0.0f, gy = 0.0f, gz = 0.0f;
#pragma unroll
            for (int r = 0; r <= P; ++r) {
                const float cb = comp(bx, r), cd = comp(dx, r);
                val = fmaf(cb, wBB[r], val);
                gx = fmaf(cd, wBB[r], gx);
                gy = fmaf(cb, wDB[r], gy);
                gz = fmaf(cb, wBD[r], gz);
            }
            const uint32_t at = (uint32_t)u * pstep;
            auto put = [&](float x, uint32_t ch) {
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), orc, col, at + ch, kCpol);
            };
            if (RESID) {
                // use the sample before the register is reloaded, so the
                // old and new values never live at once (no copy)
                const float r = live ? val - ycur : 0.0f;
                ycur = yload(u + 4);
                acc = fma((double)r, (double)r, acc);
                if (GRAD) put(r * a.gscale, 0);
                else amax = fmaxf(amax, fabsf(r));
            } else if (MODE == 3) {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                const u32x4 d = {__float_as_uint(val), __float_as_uint(gx), __float_as_uint(gy),
                                 __float_as_uint(gz)};
                __builtin_amdgcn_raw_buffer_store_b128(d, orc, col, at, kCpol);
            } else if (MODE == 4) {
                put(val, 0);
            } else {
                if (a.mask & 1u) put(val, choff[0]);
                if (a.mask & 2u) put(gx, choff[1]);
                if (a.mask & 4u) put(gy, choff[2]);
                if (a.mask & 8u) put(gz, choff[3]);
            }
        };
        int u = ua;
        if constexpr (RESID) {
            for (; u + 3 < ub; u += 4) {
                step(u, y0);
                step(u + 1, y1);
                step(u + 2, y2);
                step(u + 3, y3);
            }
            if (u < ub) step(u, y0);
            if (u + 1 < ub) step(u + 1, y1);
            if (u + 2 < ub) step(u + 2, y2);
        } else {  // no samples: two steps per iteration keep the code small
            for (; u + 1 < ub; u += 2) {
                step(u, y0);
                step(u + 1, y1);
            }
            if (u < ub) step(u, y0);
        }
      };
        if (single) walk(std::true_type{});
        else walk(std::false_type{});
    }

    if (RESID) {
        // fixed-order sum of the item: lanes by a shuffle tree (lane 0's
        // result), then waves in order
        __shared__ double wsum[8];
        __shared__ float wmax[8];
        for (int off = 32; off >= 1; off >>= 1) {
            acc += __shfl_xor(acc, off);
            if (!GRAD) amax = fmaxf(amax, __shfl_xor(amax, off));
        }
        if (lane == 0) {
            wsum[wave] = acc;
            wmax[wave] = amax;
        }
        lds_barrier();
        if (tid == 0) {
            double t = 0.0;
            float m = 0.0f;
            for (int q = 0; q < nwaves; ++q) {
                t += wsum[q];
                m = fmaxf(m, wmax[q]);
            }
            if (GRAD) {
                a.partials[item] = t;
            } else {
                a.partials[2 * item] = (double)m;
                a.partials[2 * item + 1] = t;
            }
        }
    }
}

}  // namespace
}  // namespace fa
