// Two time steps per pass for D3Q19 in columns of whole 64-node lines
// (3-term polynomials; walls on z or periodic).
//
// k_sweep2_3d gives a wave the 62 nodes of a row that its halo lanes leave, so
// an axis of 64 m nodes, the common size, takes one column more than it needs
// (128: three of 62 instead of two, half again the work; 256: five instead of
// four) and every row starts and ends inside a cache line.  Here a row of the
// column is 64 own nodes, one per lane, and the nodes beside it belong to one
// further wave, whose lanes take the left and the right neighbour of every
// row.  The halo wave runs phase 1 only.
//
// The schedule is that of k_sweep2_3d: a workgroup marches up a chunk of zc
// planes; phase 1 runs step t on plane i of the column and its halo into an
// LDS ring (38 values per node), phase 2 step t + 1 on plane i - 1 from it.
// Every node update is the single-sweep arithmetic on the same inputs, rounded
// to the storage type as a store would round it: the result equals two single
// sweeps bit for bit.
//
// One workgroup fills a CU's LDS, so its barriers and loads are exposed; large
// grids are bound by memory (256^3 FP32 4.8 TB/s of its own bytes, 0.85 of a plain
// copy).  us per step 62-node columns -> lines: 256^3 FP32 325 -> 267, FP64 728 ->
// 590; 128^3 FP32 49 -> 41, FP64 with a source 113 -> 90.
#pragma once

#include "lbm_kernels.h"

namespace lbm {

// Anti-bounce-back of the populations with c_z = CZ at a wall: own[k] holds the
// node's own population opp(k).
template <int CZ, typename TC>
__device__ __forceinline__ void wall_fix(const Coefs<TC> *__restrict__ cf, const TC *own, TC *h) {
#pragma unroll
    for (int k = 0; k < 19; ++k)
        if (Lattice<19>::cz(k) == CZ) h[k] = -own[k] + cf->ew[CZ == 1 ? 0 : 1][k];
}

template <typename TS, typename TC, bool KVAR, bool WALL, int NP, int TY, bool SB, bool SRC, int EQ>
__global__ void __launch_bounds__(64 * (TY + 3))
k_sweep2_3dw(const Geom g, const Coefs<TC> *__restrict__ cfa, const TS *__restrict__ fin, TS *__restrict__ fout,
             const typename HistType<TS>::T *__restrict__ pin, typename HistType<TS>::T *__restrict__ pout,
             uint32_t tiles_x, uint32_t tiles_y, uint32_t zc, int *flag) {
    using L = Lattice<19>;
    using TP = typename HistType<TS>::T;
    constexpr int TX = 64, TR = TY + 2, TW = TX + 2;
    // The loads of the next plane are issued before phase 1 in FP32, after it
    // otherwise: FP64 then needs no second copy of 19 values in registers, and
    // both gained (256^3 FP64 with a source 786 -> 758 us per step, FP16 215 ->
    // 213; FP32 277 -> 282).
    constexpr bool LATE = sizeof(TS) != 4;
    // Next to a wall the node's own opposite replaces what would come from
    // beyond it.  The choice is the same for a whole plane: selects of the
    // address in general, a scalar branch around five further loads in FP64
    // with a source, whose 168 registers have no room for the selects (256^3
    // 758 -> 719 us per step; without a source 596 -> 615, FP32 277 -> 280).
    constexpr bool BRANCH = SRC && sizeof(TC) == 8;
    static_assert(TR <= 32 && std::is_same<TP, TC>::value, "the halo wave holds both neighbours of every row");
    __shared__ TS rp[2][5][TR][TW], r0[2][9][TR][TW], rm[2][5][TR][TW];
    const uint32_t blk = block_index(blockIdx.x, gridDim.x, g.remap);
    const uint32_t per_z = tiles_x * tiles_y;
    const uint32_t tz = blk / per_z, rem = blk - tz * per_z;
    const uint32_t tyi = rem / tiles_x, txi = rem - tyi * tiles_x;
    const int nx = (int)g.nx, ny = (int)g.ny, nz = (int)g.nz;
    const int x0 = (int)(txi * TX), y0 = (int)(tyi * TY), z0 = (int)(tz * zc);
    const int zend = min(z0 + (int)zc, nz);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // row and column of the lane's node in the region (TR rows, TW columns);
    // spare lanes of the halo wave repeat its last row
    const bool halo = wv == TR;
    const int row = halo ? min(lane & 31, TR - 1) : wv;
    const int col = halo ? (lane < 32 ? 0 : TW - 1) : lane + 1;
    const int xg = wrap_coord(x0 - 1 + col, nx), yg = wrap_coord(y0 - 1 + row, ny);
    // byte offsets in a z plane of the source nodes (x - c_x, y - c_y), index
    // [1 - c_y][1 - c_x]; every load is a scalar plane base plus one of them
    uint32_t vo[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const int y = b == 1 ? yg : (b == 0 ? (yg == 0 ? ny - 1 : yg - 1) : (yg == ny - 1 ? 0 : yg + 1));
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int x = a == 1 ? xg : (a == 0 ? (xg == 0 ? nx - 1 : xg - 1) : (xg == nx - 1 ? 0 : xg + 1));
            vo[b][a] = ((uint32_t)y * g.nx + (uint32_t)x) * (uint32_t)sizeof(TS);
        }
    }
    const uint64_t nxy = (uint64_t)g.nx * g.ny;
    bool bad = false;
    const int nplanes = zend - z0 + 2;
    // raw values of the phase-1 gather of logical plane i: population k from
    // its source node, or at a wall the own node's opposite
    auto load = [&](int i, TS (&dst)[19], TP &pdst) {
        const int zl = z0 - 1 + i;
        if (WALL && (zl < 0 || zl >= nz)) return;
        const int zg = WALL ? zl : wrap_coord(zl, nz);
        const uint64_t zs[3] = {nxy * (uint64_t)(zg == nz - 1 ? 0 : zg + 1), nxy * (uint64_t)zg,
                                nxy * (uint64_t)(zg == 0 ? nz - 1 : zg - 1)};   // z - c_z, c_z = -1, 0, 1
#pragma unroll
        for (int k = 0; k < 19; ++k) {
            const int cx = L::cx(k), cy = L::cy(k), cz = L::cz(k);
            if constexpr (BRANCH) {
                dst[k] = *row_elem(fin + (uint64_t)k * g.plane + zs[1 + cz], 0u, vo[1 - cy][1 - cx]);
            } else {
                const bool wl = WALL && ((cz == 1 && zg == 0) || (cz == -1 && zg == nz - 1));
                const TS *base = fin + (uint64_t)(wl ? L::opp(k) : k) * g.plane + (wl ? zs[1] : zs[1 + cz]);
                uint32_t o = WALL && cz && wl ? vo[1][1] : vo[1 - cy][1 - cx];
                dst[k] = *row_elem(base, 0u, o);
            }
        }
        if (BRANCH && WALL && zg == 0) {
#pragma unroll
            for (int k = 0; k < 19; ++k)
                if (L::cz(k) == 1) dst[k] = *row_elem(fin + (uint64_t)L::opp(k) * g.plane + zs[1], 0u, vo[1][1]);
        }
        if (BRANCH && WALL && zg == nz - 1) {
#pragma unroll
            for (int k = 0; k < 19; ++k)
                if (L::cz(k) == -1) dst[k] = *row_elem(fin + (uint64_t)L::opp(k) * g.plane + zs[1], 0u, vo[1][1]);
        }
        if (SRC) pdst = pin[nxy * (uint64_t)zg + vo[1][1] / (uint32_t)sizeof(TS)];
    };
    SrcLevel<TC> lev1, lev0;   // source terms of planes i - 1 and i (this lane's node)
    TP ph1, ph0;               // phi - phi_ref of them
    TS hn[19];
    TP pn;
    load(0, hn, pn);
    for (int i = 0; i < nplanes; ++i) {
        const int zl = z0 - 1 + i;
        const int s1 = i & 1, s0 = s1 ^ 1;          // slots of plane i and of plane i - 1
        const bool p1 = WALL ? (zl >= 0 && zl < nz) : true;
        TS hc[19];
        const TP pc = pn;
#pragma unroll
        for (int k = 0; k < 19; ++k) hc[k] = hn[k];
        if (!LATE && i + 1 < nplanes) load(i + 1, hn, pn);
        // phase 1: plane zl (skipped beyond a wall)
        TS keep[5];
        if (p1) {
            const int zg = WALL ? zl : wrap_coord(zl, nz);
            const Coefs<TC> *cf = cfa + opaque_zero();
            TC h[19], out[19];
#pragma unroll
            for (int k = 0; k < 19; ++k) h[k] = (TC)hc[k];
            if (WALL && zg == 0) wall_fix<1>(cf, h, h);
            if (WALL && zg == nz - 1) wall_fix<-1>(cf, h, h);
            const TC phio = collide_node<19, TC, EQ, SRC, KVAR, NP, SB, exact_mass<19, TS>>(cf, h, SRC ? (TC)pc : TC(0), 0u, nullptr, nullptr,
                                                                         false, out, SRC ? &lev0 : nullptr);
            bad |= !__builtin_isfinite(phio);
            if (SRC) ph0 = (TP)phio;
#pragma unroll
            for (int c = 0; c < 9; ++c) r0[s1][c][row][col] = to_store<TS>(out[Zc3::z[c]]);
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                rm[s1][c][row][col] = to_store<TS>(out[Zc3::m[c]]);
                keep[c] = to_store<TS>(out[Zc3::p[c]]);
            }
        }
        if (LATE && i + 1 < nplanes) load(i + 1, hn, pn);
        __syncthreads();
        // phase 2: plane zl - 1 of the column's own nodes, the wave's row
        if (i >= 2 && wv >= 1 && wv <= TY) {
            const int zc2 = zl - 1;
            const Coefs<TC> *cf = cfa + opaque_zero();
            TC h[19], out[19];
#pragma unroll
            for (int k = 0; k < 19; ++k) {
                const int cx = L::cx(k), cy = L::cy(k), cz = L::cz(k), q = Zc3::pos(k);
                h[k] = (TC)(cz == 1 ? rp[s1][q][wv - cy][col - cx]
                                    : (cz == -1 ? rm[s1][q][wv - cy][col - cx] : r0[s0][q][wv - cy][col - cx]));
            }
            if (WALL && (zc2 == 0 || zc2 == nz - 1)) {
                // the node's own populations of its plane, beyond whose wall side
                // nothing was computed
                TC own[19];
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    own[L::opp(Zc3::m[c])] = (TC)rm[s0][c][wv][col];
                    own[L::opp(Zc3::p[c])] = (TC)rp[s0][c][wv][col];
                }
                if (zc2 == 0) wall_fix<1>(cf, own, h);
                if (zc2 == nz - 1) wall_fix<-1>(cf, own, h);
            }
            const TC phio = collide_node<19, TC, EQ, SRC, KVAR, NP, SB, exact_mass<19, TS>>(cf, h, SRC ? (TC)ph1 : TC(0), 0u, nullptr, nullptr,
                                                                         false, out, nullptr, SRC ? &lev1 : nullptr);
            bad |= !__builtin_isfinite(phio);
            if (x0 + lane < nx && y0 + wv - 1 < ny) {
                const uint32_t m = ((uint32_t)zc2 * g.ny + (uint32_t)(y0 + wv - 1)) * g.nx + (uint32_t)(x0 + lane);
                store_planes<19, false>(fout, g.plane, m, out);
                if (SRC) *at<true>(pout, m) = (TP)phio;
            }
        }
        if (SRC) { lev1 = lev0; ph1 = ph0; }
        __syncthreads();
        // the c_z = +1 populations of plane i, now that plane i - 2's are read
        if (p1) {
#pragma unroll
            for (int c = 0; c < 5; ++c) rp[s1][c][row][col] = keep[c];
        }
    }
    if (bad) *flag = 1;
}

}  // namespace lbm
