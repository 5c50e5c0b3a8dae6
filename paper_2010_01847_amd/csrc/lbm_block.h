// Kernels of small lattices (included by lbm_device.hip): several time steps per launch of whole thread
// blocks, the populations held on the chip in between.  A small lattice's
// single-step launches last as long as a launch takes (3 to 5 us on MI355X),
// whatever they compute, and the marching kernel needs
// thousands of wavefronts to be fast; here a launch holds few wavefronts, and
// the nodes recomputed around each block's outputs cost time that the chip
// would otherwise spend idle.
//
// Per node and step the arithmetic is the single-step kernels' (lbm_node.h),
// every step rounded to the storage type as a stored step is, so the results
// are the same bits for any number of steps per launch.
#pragma once

#include "lbm_node.h"

#include <stdint.h>
#include <type_traits>

namespace plbm {

// Kept values of a node: rounded as a stored step, and read back.
template <class S, int SR, int SPLIT>
__device__ __forceinline__ void store_node(S* base, const InstDesc& d, int x, int y, const S o[8], float E,
                                           int nontemporal) {
    S* row = base + d.off + (int64_t)y * d.row;
    const int64_t c = col_off(d, x);
#pragma unroll
    for (int i = 0; i < 8; ++i)
        store_raw<S>(reinterpret_cast<char*>(row + c + (int64_t)i * d.plane), o[i], nontemporal);
    if (SPLIT) store_one<float, 0>(reinterpret_cast<char*>(row) + e_off(d, x), E, 0u, nontemporal);
}

template <class S, int SPLIT>
__device__ __forceinline__ void load_node(const S* base, const InstDesc& d, int x, int y, S v[8], float& E) {
    const S* row = base + d.off + (int64_t)y * d.row;
    const int64_t c = col_off(d, x);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = row[(int64_t)i * d.plane + c];
    E = SPLIT ? *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + e_off(d, x)) : 0.0f;
}

__device__ __forceinline__ bool x_walled(const InstDesc& d) { return d.bc_x == 1 || d.bc_x == 2 || d.bc_x == 4; }

// ------------------------------------------------------------------ tiles

// K <= halo steps of one tile.  The block's window is 64 columns by waves * R
// rows (each position a periodic image of a node, mapped as the single-step
// pull wraps): wavefront w holds rows w R .. w R + R - 1 in registers, one
// column per lane.  A step pulls along x from the adjacent lanes (DPP), along
// y from the wavefront's own rows, and at its first and last row from the
// neighbouring wavefronts through LDS (three populations each way, written
// before and read after the step's one barrier; two slots in turn, so the
// next step's writes need no second barrier).  Step s is valid one node
// further inside the window than step s - 1; rows that no output needs any
// more are skipped.
// a.ctr_out gets the step count after the launch from tile 0.  b.prev (may be
// null): the state after step K - 1 as a stored step, for readouts at time n.
// Measured (MI355X, FP32, us per step, single-step launches / this): 401 x 301
// 4.1 / 1.46, 1024 x 256 4.9 / 1.95, 1024^2 11.2 / 4.7, 2048^2 39 / 15.7 (the
// marching kernel 17.8).  Bound by VALU issue and the barrier's latency at
// few blocks per CU, by the windows' loads (one third of 1024 x 256's time) at
// many.  Rows are worked through one by one: interleaving them (or holding the
// steps in separate code for the last two) took 91-103 VGPRs instead of 73 and
// ran 1024^2 in 5.3 us.  Launches that end on a check step need 110-121 VGPRs for
// the FP64 moments, so one block of 12 wavefronts runs per CU instead of two.
template <class S, int SR, int SPLIT, int R, int END>
__global__ __launch_bounds__(1024) void tile_kernel(BlockArgs b, int xcd, int nontemporal) {
    extern __shared__ float edges[];          // [2][waves][6][64]
    const StepArgs& a = b.s;
    int t = blockIdx.x;
    if (xcd) {
        const int nb = a.ntiles, q = nb >> 3, r = nb & 7, k = t & 7, j = t >> 3;
        t = k * q + (k < r ? k : r) + j;
    }
    const int tg = t + a.tile_base;
    const int inst = a.tile_inst[tg];
    const InstDesc d = a.desc[inst];
    const RefView rv = ref_view(a.ref[inst]);
    const double q_ref = END == kEndCheck ? a.ref[inst].q_ref : 0.0;
    const int K = b.steps, H = b.halo, NW = b.waves;
    const int rows = NW * R;
    const int W = 64 - 2 * H, HO = rows - 2 * H;
    const int local = tg - d.b_tile_begin;
    const int ty = local / d.b_tiles_x;
    const int tx = local - ty * d.b_tiles_x;
    const int x0 = tx * W, y0 = ty * HO;
    const int nx = d.nx, ny = d.ny;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int gx = wrapm(x0 - H + lane, nx, 64);
    const int wr0 = wv * R;
    const int top = H + min(HO, ny - y0);     // window row after the last output row
    const uint32_t step = a.ctr_in[0];
    const S* src = reinterpret_cast<const S*>(a.src);
    uint32_t colw[4] = {0u, 0u, 0u, 0u};
    if (SR) {
#pragma unroll
        for (int k = 0; k < 4; ++k) colw[k] = sr_col_word((uint32_t)gx, k, a.seed);
    }
    const bool xw = x_walled(d) && (gx == 0 || gx == nx - 1);
    const int ox = x0 + lane - H;
    const bool out_lane = lane >= H && lane < 64 - H && ox < nx;

    S raw[R][8];
    float rawE[R];
    int gy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        gy[r] = wrapm(y0 - H + wr0 + r, ny, rows);
        load_node<S, SPLIT>(src, d, gx, gy[r], raw[r], rawE[r]);
    }
    float f[R][8];
#pragma unroll
    for (int r = 0; r < R; ++r) reload<S, SPLIT>(raw[r], rawE[r], f[r]);
    double pm[R][3];
    DD acc[kPartials] = {dd_zero(), dd_zero(), dd_zero(), dd_zero(), dd_zero()};

    // One loop for all steps and a branch per row (uniform: on the row and the
    // step): rows are worked through one by one, in few registers.
    for (int s = 1; s <= K; ++s) {
        float* slot = edges + (s & 1) * NW * 384;
        float* mine = slot + wv * 384 + lane;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            mine[k * 64] = f[R - 1][yup(k)];                   // the row above pulls these
            mine[(3 + k) * 64] = f[0][ydown(k)];               // the row below pulls these
        }
        __syncthreads();
        // the window's first and last rows are never pulled into a row that is
        // still needed: any value will do there
        const float* below = slot + (wv > 0 ? wv - 1 : 0) * 384 + lane;
        const float* above = slot + (wv + 1 < NW ? wv + 1 : wv) * 384 + lane;
        float up[3], dn_edge[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            up[k] = below[k * 64];
            dn_edge[k] = above[(3 + k) * 64];
        }
        const int lo = H - K + s, hi = top + K - s;            // rows some output still needs
        S* out = s == K ? reinterpret_cast<S*>(a.dst) : (s == K - 1 ? reinterpret_cast<S*>(b.prev) : nullptr);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float dn[8];
#pragma unroll
            for (int k = 0; k < 3; ++k)
                dn[ydown(k)] = r + 1 < R ? f[r + 1 < R ? r + 1 : 0][ydown(k)] : dn_edge[k];
            const float keep[3] = {f[r][yup(0)], f[r][yup(1)], f[r][yup(2)]};
            const int wr = wr0 + r;
            if (wr >= lo && wr < hi) {
                const float mid[2] = {f[r][ymid(0)], f[r][ymid(1)]};
                float g[8];
                march_gather(dn, mid, up, g);
                if (s == 1 && a.apply_shift) {
                    asm volatile("");                          // a branch, not selects
                    apply_shift(g, rv);
                }
                const int y = gy[r];
                if (xw || (d.bc_y != 0 && (y == 0 || y == ny - 1))) boundary<1>(g, d, rv.wall_kd, gx, y);
                if constexpr (END == kEndCheck) {
                    if (s == K - 1) {
                        double E;
                        node_moments_f64(g, d, q_ref, E, pm[r][0], pm[r][1], pm[r][2]);
                    } else if (s == K && out_lane) {
                        double E, dT, qx, qy;
                        node_moments_f64(g, d, q_ref, E, dT, qx, qy);
                        check_sums(acc, d.s * E, qx, qy, dT, pm[r][0], pm[r][1], pm[r][2]);
                    }
                }
                uint32_t w[4] = {0u, 0u, 0u, 0u};
                if (SR)
                    sr_words(w, colw, sr_row_word((uint32_t)(d.node_off + (int64_t)y * nx), step + (uint32_t)(s - 1),
                                                  a.seed));
                S o[8];
                float E;
                relax_round<S, SR, SPLIT>(g, d, rv, w, o, E);
                reload<S, SPLIT>(o, E, f[r]);
                if (out && wr >= H && wr < top && out_lane) store_node<S, SR, SPLIT>(out, d, ox, y, o, E, nontemporal);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) up[k] = keep[k];
        }
    }
    if (t == 0 && threadIdx.x == 0) a.ctr_out[0] = step + (uint32_t)K;
    if constexpr (END == kEndCheck) block_partials(acc, a.partials + (int64_t)tg * kPartials);
}

// ------------------------------------------------------------------ windows in LDS

// K steps of a window of at most M * 1024 nodes held in one block's LDS (M
// nodes per thread: window node n = thread + m * threads, row by row).  WHOLE:
// the window is the whole lattice (halo 0), every node's sources lie in it, any
// K.  Otherwise the window is a tile with a halo of b.halo >= K nodes on each
// side, as in tile_kernel; sources beyond the window's edge are replaced by
// the node itself (their results are never used), and wavefronts whose rows
// no output needs any more skip the step.  Two copies of the window in turn,
// one barrier per step.
// Measured (MI355X, FP32, us per step, single-step launches / this): 20 x 20
// 3.4 / 0.31, 401 x 3 3.5 / 0.67 (whole), 128 x 64 3.5 / 0.70, 201^2 3.6 /
// 1.07 (windows).  A step's latency bounds it: a wavefront alone on its SIMD
// issues a VALU instruction every 5.9 cycles (four of them one every 2.6), so
// about 75 of them, the LDS round trip and the barrier take 0.3-0.45 us whatever
// the window; a launch adds 3.4 us.
template <class S, int SR, int SPLIT, int M, int END, int WHOLE>
__global__ __launch_bounds__(1024) void patch_kernel(BlockArgs b) {
    __shared__ float pop[2][8][M * 1024];
    const StepArgs& a = b.s;
    const int tg = (int)blockIdx.x + a.tile_base;
    const int inst = a.tile_inst[tg];
    const InstDesc d = a.desc[inst];
    const int K = b.steps, H = WHOLE ? 0 : b.halo;
    const int nx = d.nx, ny = d.ny;
    const int WX = WHOLE ? nx : b.win_x, WY = WHOLE ? ny : b.win_y, n = WX * WY;
    int x0 = 0, y0 = 0, top = ny;
    if (!WHOLE) {
        const int local = tg - d.b_tile_begin;
        const int ty = local / d.b_tiles_x;
        x0 = (local - ty * d.b_tiles_x) * (WX - 2 * H);
        y0 = ty * (WY - 2 * H);
        top = H + min(WY - 2 * H, ny - y0);   // window row after the last output row
    }
    int node[M], x[M], y[M], row[M], from[M][8];
    bool out_node[M];
    uint32_t colw[M][4];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        node[m] = (int)threadIdx.x + m * (int)blockDim.x;
        const bool live = node[m] < n;
        const int wy = live ? node[m] / WX : 0;
        const int wx = live ? node[m] - wy * WX : 0;
        row[m] = live ? wy : -1;
        x[m] = WHOLE ? wx : wrapm(x0 - H + wx, nx, WX);
        y[m] = WHOLE ? wy : wrapm(y0 - H + wy, ny, WY);
        out_node[m] = live && (WHOLE || (wx >= H && wx < WX - H && x0 + wx - H < nx && wy >= H && wy < top));
        const int xs[3] = {wx, wx == 0 ? (WHOLE ? WX - 1 : 0) : wx - 1, wx == WX - 1 ? (WHOLE ? 0 : wx) : wx + 1};
        const int ys[3] = {wy, wy == 0 ? (WHOLE ? WY - 1 : 0) : wy - 1, wy == WY - 1 ? (WHOLE ? 0 : wy) : wy + 1};
#pragma unroll
        for (int i = 0; i < 8; ++i) from[m][i] = ys[src_row(i)] * WX + xs[src_dx(i) == 0 ? 0 : (src_dx(i) < 0 ? 1 : 2)];
        if (SR) {
#pragma unroll
            for (int k = 0; k < 4; ++k) colw[m][k] = sr_col_word((uint32_t)x[m], k, a.seed);
        }
    }
    S raw[M][8];
    float rawE[M];
#pragma unroll
    for (int m = 0; m < M; ++m) load_node<S, SPLIT>(reinterpret_cast<const S*>(a.src), d, x[m], y[m], raw[m], rawE[m]);
    const RefView rv = ref_view(a.ref[inst]);
    const double q_ref = END == kEndCheck ? a.ref[inst].q_ref : 0.0;
    const uint32_t step = a.ctr_in[0];
    bool wall[M], walled = false;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        float f[8];
        reload<S, SPLIT>(raw[m], rawE[m], f);
        // the pending reference shift of the first step's pulled values is the
        // same for every node: added before the pull, the same bits
        if (a.apply_shift) apply_shift(f, rv);
        // (a thread past the window's last node writes its own, unread slot)
#pragma unroll
        for (int i = 0; i < 8; ++i) pop[0][i][node[m]] = f[i];
        wall[m] = row[m] >= 0 && on_wall(d, x[m], y[m]);
        walled = walled || __any(wall[m]);
    }
    // window rows of this wavefront (tiles hold one node per thread)
    const int r_lo = __builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u) / WX);
    const int r_hi = __builtin_amdgcn_readfirstlane((int)(threadIdx.x | 63u) / WX);
    double pm[M][3];
    DD acc[kPartials] = {dd_zero(), dd_zero(), dd_zero(), dd_zero(), dd_zero()};

    // Step s, from copy CUR to the other; AT: 0 an earlier one, 1 step K - 1
    // (also stored in b.prev; the check launch forms its moments), 2 step K.
    auto advance = [&](const int s, auto cur, auto at) {
        constexpr int CUR = decltype(cur)::value, AT = decltype(at)::value;
        __syncthreads();
        if (!WHOLE && (r_hi < H - K + s || r_lo >= top + K - s)) return;
        float g[M][8];
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int i = 0; i < 8; ++i) g[m][i] = pop[CUR][i][from[m][i]];
        if (walled) {
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (wall[m]) boundary<1>(g[m], d, rv.wall_kd, x[m], y[m]);
        }
#pragma unroll
        for (int m = 0; m < M; ++m) {
            if constexpr (END == kEndCheck && AT == 1) {
                double E;
                node_moments_f64(g[m], d, q_ref, E, pm[m][0], pm[m][1], pm[m][2]);
            }
            if constexpr (END == kEndCheck && AT == 2) {
                if (out_node[m]) {
                    double E, dT, qx, qy;
                    node_moments_f64(g[m], d, q_ref, E, dT, qx, qy);
                    check_sums(acc, d.s * E, qx, qy, dT, pm[m][0], pm[m][1], pm[m][2]);
                }
            }
            uint32_t w[4] = {0u, 0u, 0u, 0u};
            if (SR)
                sr_words(w, colw[m], sr_row_word((uint32_t)(d.node_off + (int64_t)y[m] * nx),
                                                 step + (uint32_t)(s - 1), a.seed));
            S o[8];
            float E, f[8];
            relax_round<S, SR, SPLIT>(g[m], d, rv, w, o, E);
            if (AT < 2) {
                reload<S, SPLIT>(o, E, f);
#pragma unroll
                for (int i = 0; i < 8; ++i) pop[1 - CUR][i][node[m]] = f[i];
            }
            if (AT > 0 && out_node[m]) {
                S* out = reinterpret_cast<S*>(AT == 2 ? a.dst : b.prev);
                if (out) store_node<S, SR, SPLIT>(out, d, x[m], y[m], o, E, 0);
            }
        }
    };
    typedef std::integral_constant<int, 0> C0;
    typedef std::integral_constant<int, 1> C1;
    typedef std::integral_constant<int, 2> C2;
    int s = 1;
    for (; s + 1 <= K - 2; s += 2) {
        advance(s, C0{}, C0{});
        advance(s + 1, C1{}, C0{});
    }
    // one to three steps are left; the last two are kept apart
    if (s == K - 2) {
        advance(s, C0{}, C0{});
        advance(s + 1, C1{}, C1{});
        advance(s + 2, C0{}, C2{});
    } else if (s == K - 1) {
        advance(s, C0{}, C1{});
        advance(s + 1, C1{}, C2{});
    } else {
        advance(s, C0{}, C2{});
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr_out[0] = step + (uint32_t)K;
    if constexpr (END == kEndCheck) block_partials(acc, a.partials + (int64_t)tg * kPartials);
}

// ------------------------------------------------------------------ launches

template <class S, int SR, int SPLIT, int END>
static hipError_t launch_block_e(const BlockPlan& p, const Shape& sh, const BlockArgs& b, hipStream_t st) {
    const dim3 grid(b.s.ntiles), block(p.waves * 64);
    if (p.kind == kBlockWhole) {
        if (p.rows == 1) hipLaunchKernelGGL((patch_kernel<S, SR, SPLIT, 1, END, 1>), grid, block, 0, st, b);
        else hipLaunchKernelGGL((patch_kernel<S, SR, SPLIT, 2, END, 1>), grid, block, 0, st, b);
    } else if (p.kind == kBlockPatch) {
        hipLaunchKernelGGL((patch_kernel<S, SR, SPLIT, 1, END, 0>), grid, block, 0, st, b);
    } else {
        const size_t lds = (size_t)2 * p.waves * 6 * 64 * sizeof(float);
        if (p.rows == 3)
            hipLaunchKernelGGL((tile_kernel<S, SR, SPLIT, 3, END>), grid, block, lds, st, b, sh.xcd, sh.nt);
        else
            hipLaunchKernelGGL((tile_kernel<S, SR, SPLIT, 4, END>), grid, block, lds, st, b, sh.xcd, sh.nt);
    }
    return hipGetLastError();
}

template <class S, int SPLIT>
static hipError_t launch_block_s(const BlockPlan& p, const Shape& sh, const BlockArgs& b, int end, hipStream_t st) {
    if (end == kEndCheck)
        return b.s.sr ? launch_block_e<S, 1, SPLIT, kEndCheck>(p, sh, b, st)
                      : launch_block_e<S, 0, SPLIT, kEndCheck>(p, sh, b, st);
    return b.s.sr ? launch_block_e<S, 1, SPLIT, kEndPlain>(p, sh, b, st)
                  : launch_block_e<S, 0, SPLIT, kEndPlain>(p, sh, b, st);
}

hipError_t launch_block(int storage, const BlockPlan& p, const Shape& sh, const BlockArgs& b, int end,
                        hipStream_t st) {
    if (b.s.ntiles <= 0) return hipSuccess;
    // what the kernels' indexing assumes
    if (end != kEndPlain && end != kEndCheck) return hipErrorInvalidValue;
    if (b.steps < (end == kEndCheck ? 2 : 1) || p.waves < 1 || p.waves > 16) return hipErrorInvalidValue;
    if (end == kEndCheck && !b.s.partials) return hipErrorInvalidValue;
    if (p.kind == kBlockWhole) {
        if (p.rows != 1 && p.rows != 2) return hipErrorInvalidValue;
    } else {
        if (b.halo != p.halo || b.steps > p.halo) return hipErrorInvalidValue;
        if (p.out_x() < 1 || p.out_y() < 1) return hipErrorInvalidValue;
        if (p.kind == kBlockPatch) {
            if (b.win_x != p.win_x() || b.win_y != p.win_y() || p.win_x() * p.win_y() > p.waves * 64)
                return hipErrorInvalidValue;
        } else if (p.kind != kBlockTiles || (p.rows != 3 && p.rows != 4) || b.waves != p.waves) {
            return hipErrorInvalidValue;
        }
    }
    switch (storage) {
        case 0: return launch_block_s<float, 0>(p, sh, b, end, st);
        case 1: return launch_block_s<_Float16, 0>(p, sh, b, end, st);
        case 2: return launch_block_s<bf16_bits, 0>(p, sh, b, end, st);
        case 3: return launch_block_s<_Float16, 1>(p, sh, b, end, st);
        case 4: return launch_block_s<bf16_bits, 1>(p, sh, b, end, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace plbm
