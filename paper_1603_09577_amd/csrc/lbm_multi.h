// T time steps per pass for D2Q9 (T even; 3-term polynomials): the state
// crosses memory once per T steps and a pass costs one launch.
//
// A workgroup owns a tile of (TX - 2H) x (TR - 2H) nodes, H = T - 1, and keeps
// a region of TX x TR nodes (TX = 64: a row per wave, or 32: two rows), the tile
// and H nodes around it, in LDS.  Step 0
// gathers the region from the stored state; step s runs on the rows and
// columns at least s inside the region, so that after T steps the tile is
// complete, and the last step stores it.  Every node update is the
// single-sweep arithmetic on the same inputs, with populations rounded to the
// storage type in LDS as a store would round them, so the result equals T
// single sweeps bit for bit.
//
// One LDS copy serves all steps: the A-A pattern of in-place streaming (Bailey et
// al., 2009), on a tile instead of the grid.  Slot k of a cell holds, before an odd step,
// the population the cell gathers from direction k; an odd step reads its own
// cell's nine slots and leaves population k in its own slot opp(k); an even
// step s > 0 gathers population k from slot opp(k) of the cell at -c_k and
// leaves its own population k in slot k of the cell at +c_k, which is where it
// read population opp(k).  Every step thus writes exactly the slots the same
// node has read, so no second copy is needed and one barrier separates steps.
// At a wall the node's own slot takes the place of the one beyond it: the
// reader negates it and adds the wall term (the anti-bounce-back gather).
// Lanes and rows that are no longer inside hold values nobody uses: a write
// of a boundary lane that leaves its row of LDS reaches only column 0 or 63 of
// another slot, which no step reads any more at that point.
//
// What it buys: a two-step pass on 1024^2 FP32 (16.0 us) is as long as moving
// its 84 MB through the Infinity Cache takes with the ramp of a launch, and on
// a small grid most of a pass is launch, first loads and last stores.  With
// six steps the bytes per step fall to a third and what is left is vector
// issue (97 operations per node and step with rates 1, 106 with equal and 133 with
// unequal rates, 1.45 times that with the halo) and the barriers.  us per step before -> after, FP32 with K(phi) and a
// source unless noted: 64^2 FP64 unequal rates 2.41 -> 1.14, 32-wide 0.89;
// 256^2 3.5 -> 1.23; 1024^2 8.0 -> 5.8, FP64 14.3 -> 12.0; 1000 x 723 channel with
// unequal rates 7.9 -> 5.1; 2048^2 44 -> 18.9, FP64 80 -> 48; 4000 x 2500 FP16 54 ->
// 41.7.
//
// A Scheme-A run reads phi(t - 1) of the region from pin, hands each node's
// source terms to the next step in the registers of the wave that owns its
// row, and writes phi(t + T - 1) of the tile to pout (not pin: neighbouring
// tiles still read it at their halo).
#pragma once

#include "lbm_kernels.h"

namespace lbm {

// REC: every step's state of the tile is stored, step s at fout + s fstep and
// its history at pout + s pstep (elements): a run that needs all states (the
// adjoint's recomputation) then reads one state per pass instead of one per step.
template <typename TS, typename TC, bool SRC, bool KVAR, int T, int TR, int NW, bool SB, bool WALL, int EQ,
          bool REC = false, int TX = 64>
__device__ __forceinline__ void sweep_multi_tile(const Geom &g, const Coefs<TC> *__restrict__ cf,
                                                 const TS *__restrict__ fin, TS *__restrict__ fout,
                                                 const typename HistType<TS>::T *__restrict__ pin,
                                                 typename HistType<TS>::T *__restrict__ pout, uint32_t tx,
                                                 uint32_t ty, int *flag, uint64_t fstep = 0, uint64_t pstep = 0) {
    using L = Lattice<9>;
    using TP = typename HistType<TS>::T;
    constexpr bool HALF = TX == 32;   // two region rows per wave
    constexpr int H = T - 1, TH = TR - 2 * H, NR = TR / NW / (HALF ? 2 : 1), PAD = HALF ? 1 : 0;
    static_assert(T % 2 == 0 && NR * NW * (HALF ? 2 : 1) == TR && std::is_same<TP, TC>::value, "whole rows per wave");
    __shared__ TS raw[(TR + 2 * PAD) * 9 * TX + 2];
    const int lane = threadIdx.x & (TX - 1);               // column of the region
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    TS *const cell = raw + 1 + lane + PAD * 9 * TX;        // slot k of region row r: cell[(r * 9 + k) * TX]
    // Row i of this wave: r0 = wv + i NW, in half-width regions the upper half
    // of the wave takes TR - 1 - r0, so that both halves leave the shrinking
    // region at the same step.
    auto row_of = [&](int r0) {
        if constexpr (HALF) return (threadIdx.x & 32) ? TR - 1 - r0 : r0;
        else return r0;
    };
    const int nx = (int)g.nx, ny = (int)g.ny;
    const int x0 = (int)(tx * (TX - 2 * H)), y0 = (int)(ty * TH);
    const int xg = wrap_coord(x0 - H + lane, nx);
    uint32_t cb[3] = {(uint32_t)(xg == 0 ? nx - 1 : xg - 1) * (uint32_t)sizeof(TS),    // c_x = 1
                      (uint32_t)xg * (uint32_t)sizeof(TS),                              // c_x = 0
                      (uint32_t)(xg == nx - 1 ? 0 : xg + 1) * (uint32_t)sizeof(TS)};   // c_x = -1
    const uint32_t row_bytes = g.nx * (uint32_t)sizeof(TS);
    const bool own = lane >= H && lane < TX - H && x0 - H + lane < nx;
    SrcLevel<TC> lev[SRC ? NR : 1];
    bool bad = false;
    auto store = [&](int s, int yl, const TC *out, TC phio) {
        const uint32_t m = (uint32_t)yl * g.nx + (uint32_t)(x0 - H + lane);
        store_planes<9, false>(fout + (REC ? (uint64_t)s * fstep : 0), g.plane, m, out);
        if (SRC) *at<true>(pout + (REC ? (uint64_t)s * pstep : 0), m) = (TP)phio;
    };
    // step 0: scalar row base plus one of three column offsets per load
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int r = row_of(wv + i * NW), yl = y0 - H + r;
        if (WALL && (yl < 0 || yl >= ny)) continue;        // beyond a wall
        const int yg = WALL ? yl : wrap_coord(yl, ny);
        const int ym = yg == 0 ? ny - 1 : yg - 1, yp = yg == ny - 1 ? 0 : yg + 1;
        TC h[9], out[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int cy = L::cy(k);
            const bool wl = WALL && ((cy == 1 && yg == 0) || (cy == -1 && yg == ny - 1));
            const uint32_t row = (uint32_t)(wl ? yg : (cy == 1 ? ym : (cy == -1 ? yp : yg)));
            const TS *pl = fin + (uint64_t)(wl ? L::opp(k) : k) * g.plane;
            const TC v = HALF ? (TC)*reinterpret_cast<const TS *>(reinterpret_cast<const char *>(pl) +
                                                                  (row * row_bytes + cb[wl ? 1 : 1 - L::cx(k)]))
                              : (TC)*row_elem(pl, row * row_bytes, cb[wl ? 1 : 1 - L::cx(k)]);
            h[k] = wl ? -v + cf->ew[cy == 1 ? 0 : 1][k] : v;
        }
        const TC pp = SRC ? (TC)*at<true>(pin, (uint32_t)yg * g.nx + (uint32_t)xg) : TC(0);
        const TC phi0 = collide_node<9, TC, EQ, SRC, KVAR, 3, SB, exact_mass<9, TS>>(cf, h, pp, 0u, nullptr, nullptr, false, out,
                                                                  SRC ? &lev[SRC ? i : 0] : nullptr);
        if (REC && own && r >= H && r < TR - H && yl < ny) store(0, yl, out, phi0);
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int cy = L::cy(k), cx = L::cx(k);
            const bool wl = WALL && ((cy == -1 && yg == 0) || (cy == 1 && yg == ny - 1));
            if (wl) cell[(r * 9 + L::opp(k)) * TX] = to_store<TS>(out[k]);
            else if (HALF || (r + cy >= 0 && r + cy < TR)) cell[((r + cy) * 9 + k) * TX + cx] = to_store<TS>(out[k]);
        }
    }
    // Steps 1 .. T - 2 in pairs (odd, even), then the last, odd one.  The pair
    // loop stays rolled: unrolled, the source terms of T = 6 and 8 went to
    // scratch memory.
    auto step = [&](int s, auto odd, auto last) {
        constexpr bool ODD = decltype(odd)::value, LAST = decltype(last)::value;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int r0 = wv + i * NW, r = row_of(r0), yl = y0 - H + r;
            if (r0 < s || (!HALF && r0 >= TR - s) || (WALL && (yl < 0 || yl >= ny))) continue;
            TC h[9], out[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const int cy = L::cy(k), cx = L::cx(k);
                const bool wl = WALL && ((cy == 1 && yl == 0) || (cy == -1 && yl == ny - 1));
                const int idx = ODD || wl ? (r * 9 + k) * TX : ((r - cy) * 9 + L::opp(k)) * TX - cx;
                const TC v = (TC)cell[idx];
                h[k] = wl ? -v + cf->ew[cy == 1 ? 0 : 1][k] : v;
            }
            SrcLevel<TC> *lv = SRC ? &lev[SRC ? i : 0] : nullptr;
            const TC phio = collide_node<9, TC, EQ, SRC, KVAR, 3, SB, exact_mass<9, TS>>(cf, h, TC(0), 0u, nullptr, nullptr, false, out,
                                                                      LAST ? nullptr : lv, lv);
            if constexpr (!LAST) {
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    const int cy = L::cy(k), cx = L::cx(k);
                    const bool wl = WALL && ((cy == -1 && yl == 0) || (cy == 1 && yl == ny - 1));
                    const int idx = ODD || wl ? (r * 9 + L::opp(k)) * TX : ((r + cy) * 9 + k) * TX + cx;
                    cell[idx] = to_store<TS>(out[k]);
                }
                if (REC && own && r >= H && r < TR - H && yl < ny) store(s, yl, out, phio);
            } else if (own && yl < ny) {
                // a non-finite phi of an earlier step reaches the same node's
                // later ones through its rest population
                bad |= !__builtin_isfinite(phio);
                store(T - 1, yl, out, phio);
            }
        }
    };
#pragma nounroll
    for (int s = 1; s < T - 1; s += 2) {
        __syncthreads();
        step(s, std::true_type{}, std::false_type{});
        __syncthreads();
        step(s + 1, std::false_type{}, std::false_type{});
    }
    __syncthreads();
    step(T - 1, std::true_type{}, std::true_type{});
    if (bad) *flag = 1;
}

// FP32 arithmetic with at most two rows per wave fits 64 vector registers, so
// that LDS decides the waves per CU; the attribute keeps the scalar registers
// within 8 waves per SIMD too (one more would cost a whole workgroup).
template <typename TS, typename TC, bool SRC, bool KVAR, int T, int TR, int NW, bool SB, bool WALL, int EQ, int TX>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(sizeof(TC) == 4 ? 8 : 1, 8)))
k_sweep_multi(const Geom g, const Coefs<TC> *__restrict__ cf, const TS *__restrict__ fin, TS *__restrict__ fout,
              const typename HistType<TS>::T *__restrict__ pin, typename HistType<TS>::T *__restrict__ pout,
              uint32_t tiles_x, int *flag) {
    const uint32_t tile = block_index(blockIdx.x, gridDim.x, g.remap);
    const uint32_t ty = tile / tiles_x, tx = tile - ty * tiles_x;
    sweep_multi_tile<TS, TC, SRC, KVAR, T, TR, NW, SB, WALL, EQ, false, TX>(g, cf, fin, fout, pin, pout, tx, ty,
                                                                                    flag);
}

template <typename TS, typename TC, bool SRC, bool KVAR, int T, int TR, int NW, bool WALL, int EQ>
__global__ void __launch_bounds__(64 * NW)
k_sweep_record(const Geom g, const Coefs<TC> *__restrict__ cf, const TS *__restrict__ fin, TS *__restrict__ fout,
               uint64_t fstep, const typename HistType<TS>::T *__restrict__ pin,
               typename HistType<TS>::T *__restrict__ pout, uint64_t pstep, uint32_t tiles_x, int *flag) {
    const uint32_t tile = block_index(blockIdx.x, gridDim.x, g.remap);
    const uint32_t ty = tile / tiles_x, tx = tile - ty * tiles_x;
    sweep_multi_tile<TS, TC, SRC, KVAR, T, TR, NW, false, WALL, EQ, true>(g, cf, fin, fout, pin, pout, tx, ty, flag,
                                                                           fstep, pstep);
}

}  // namespace lbm
