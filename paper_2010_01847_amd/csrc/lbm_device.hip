// Device code of the phonon lattice Boltzmann library for gfx950 (CDNA4, wave64).
//
// One fused kernel performs a whole time step of Eq. 13 per node: it pulls the
// eight populations along the velocities of Eq. 14 from the previous step's
// post-relaxation buffer, applies the boundary treatment of Sec. 2.5 to the
// unknown ones, forms the moments of Eqs. 53-54 in registers, relaxes toward
// the equilibrium of Eq. 15 with the source of Eq. 16, and stores the result
// into the other buffer.  The path is a bandwidth-bound stencil (about 40
// flop per 64 bytes in FP32), so there is no matrix-core work: the design
// goals are coalesced, wide HBM accesses and enough bytes in flight.
//
// Stored quantity: g_i = (e_i - R_i(x)) / s, the deviation from a reference
// state R (RefState) that one step (advection, then relaxation) maps onto
// itself up to a uniform forcing: the ramp T_ref = t0 - G x of the gradient
// seam of Eqs. 59-60 (G = 0 without it) with a uniform x-flux J and the
// non-equilibrium share that the ramp sustains.  The scheme is affine in e,
// so the update of g is the bare relaxation with plain periodic wrap (the
// seam disappears) plus that forcing.  J follows the lattice's mean flux
// (updated at check steps), so the stored values are the small departures
// from the current state's own bulk part, which is what keeps FP32 accurate
// when tau_R is large, in transients and at steady state.
//
// Layout (see InstDesc): either eight direction planes of ny rows each, x
// contiguous, or "chunked": each 64-node row segment stores its eight
// direction runs back to back, so the eight loads of a wavefront fall in one
// contiguous 2 KB (FP32) region instead of eight streams a plane apart.  Two
// such buffers, ping-pong.
#include "lbm_node.h"
#include "lbm_block.h"

#include <stdint.h>
#include <type_traits>

namespace plbm {

// ------------------------------------------------------------------ step

template <class S, int V, int MODE>
__global__ __launch_bounds__(kMaxBlock) void step_kernel(StepArgs a, int64_t snap_stride,
                                                          int xcd, int nontemporal) {
    // tile of this block; with xcd != 0, consecutive tiles go to the same XCD
    // (workgroups are dealt to the 8 XCDs round robin)
    const int b = blockIdx.x;
    int t = b;
    if (xcd) {
        const int nb = a.ntiles, q = nb >> 3, r = nb & 7, k = b & 7, j = b >> 3;
        t = k * q + (k < r ? k : r) + j;
    }
    // the first tile of the launch advances the step counter
    if (t == 0 && threadIdx.x == 0 && threadIdx.y == 0) a.ctr_out[0] = a.ctr_in[0] + 1u;
    t += a.tile_base;
    const int inst = a.tile_inst[t];
    const InstDesc& d = a.desc[inst];
    const RefState& ref = a.ref[inst];
    const RefView rv = ref_view(ref);
    const int local = t - d.tile_begin;
    const int ty = local / d.tiles_x;
    const int tx = local - ty * d.tiles_x;
    const int x0 = tx * (V * blockDim.x) + threadIdx.x * V;
    const int y = ty * blockDim.y + threadIdx.y;
    const int nx = d.nx, ny = d.ny;
    const bool live = (y < ny) && (x0 < nx);

    DD acc[kPartials] = {dd_zero(), dd_zero(), dd_zero(), dd_zero(), dd_zero()};
    if (live) {
        const S* __restrict__ src = reinterpret_cast<const S*>(a.src) + d.off;
        S* __restrict__ dst = reinterpret_cast<S*>(a.dst) + d.off;
        const int ym = (y == 0) ? ny - 1 : y - 1;
        const int yp = (y == ny - 1) ? 0 : y + 1;
        const int64_t rows[3] = {(int64_t)y * d.row, (int64_t)ym * d.row, (int64_t)yp * d.row};
        const int64_t xo = col_off(d, x0);
        const bool full = (x0 + V <= nx);
        const int cs = d.cshift;
        float g[V][8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int dx = src_dx(i);
            const S* base = src + (int64_t)i * d.plane + rows[src_row(i)];
            float v[V];
            // elements the fast path touches: contiguous only within a chunk
            const int lo = (sizeof(S) == 2 && V > 1 && dx < 0) ? x0 - 2 : (dx < 0 ? x0 + dx : x0);
            const int hi = (sizeof(S) == 2 && V > 1 && dx > 0) ? x0 + V + 1 : x0 + V - 1 + (dx > 0 ? dx : 0);
            if (full && lo >= 0 && hi < nx && (lo >> cs) == (hi >> cs)) {
                load_shifted<S, V>(base + xo, dx, v);
            } else {
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    const int xs = wrapx(x0 + k + dx, nx);
                    v[k] = (x0 + k < nx) ? Cvt<S>::ld(base[col_off(d, xs)]) : 0.0f;
                }
            }
#pragma unroll
            for (int k = 0; k < V; ++k) g[k][i] = v[k];
        }
        if (a.apply_shift) {
#pragma unroll
            for (int k = 0; k < V; ++k) apply_shift(g[k], rv);
        }
        const bool edge_y = (d.bc_y != 0) && (y == 0 || y == ny - 1);
        const bool edge_x = (d.bc_x == 1 || d.bc_x == 2 || d.bc_x == 4) && (x0 == 0 || x0 + V > nx - 1);
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (edge_y || edge_x) boundary(g[k], d, rv.wall_kd, x0 + k, y);
        }
        if (MODE != kPlain) {
            const int64_t nbase = d.node_off + (int64_t)y * nx;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                if (x0 + k >= nx) continue;
                double E, dT, qx, qy;
                node_moments_f64(g[k], d, ref.q_ref, E, dT, qx, qy);
                const int64_t n = nbase + x0 + k;
                if (MODE == kSnap) {
                    a.snap[n] = dT;
                    a.snap[n + snap_stride] = qx;
                    a.snap[n + 2 * snap_stride] = qy;
                } else {
                    const double p0 = a.snap[n], p1 = a.snap[n + snap_stride],
                                 p2 = a.snap[n + 2 * snap_stride];
                    check_sums(acc, d.s * E, qx, qy, dT, p0, p1, p2);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < V; ++k) relax(g[k], d, rv);
        // a V-aligned run never crosses a 64-node chunk
        S* out = dst + rows[0] + xo;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float v[V];
#pragma unroll
            for (int k = 0; k < V; ++k) v[k] = g[k][i];
            S* p = out + (int64_t)i * d.plane;
            if (full) {
                store_run<S, V>(p, v, nontemporal);
            } else {
#pragma unroll
                for (int k = 0; k < V; ++k)
                    if (x0 + k < nx) p[k] = Cvt<S>::st(v[k]);
            }
        }
    }
    if (MODE == kCheck) block_partials(acc, a.partials + (int64_t)t * kPartials);
}

// Wavefront-centric step for one node per lane.  Each wave owns one 64-node
// row segment (chunk cx of row y), so the row, chunk and plane bases are
// wave-uniform scalars and every load is a scalar base plus a 32-bit lane
// offset; the boundary branches are taken per wave, not per lane.
// Same per-node arithmetic as step_kernel, hence the same bits.  SPLIT: the
// populations are rebuilt as h_i + omega_i E from the source node's 16-bit
// h_i and FP32 E, and stored back in that form.
template <class S, int MODE, int SR, int SPLIT>
__global__ __launch_bounds__(kMaxBlock) void wave_kernel(StepArgs a, int64_t snap_stride, int xcd,
                                                          int nontemporal) {
    const int b = blockIdx.x;
    int t = b;
    if (xcd) {
        const int nb = a.ntiles, q = nb >> 3, r = nb & 7, k = b & 7, j = b >> 3;
        t = k * q + (k < r ? k : r) + j;
    }
    t += a.tile_base;
    const int inst = a.tile_inst[t];
    const InstDesc& d = a.desc[inst];
    const RefState& ref = a.ref[inst];
    const int local = t - d.tile_begin;
    const int ty = local / d.tiles_x;
    const int tx = local - ty * d.tiles_x;
    const int wpx = blockDim.x >> 6;                                   // waves per block along x
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wy = __builtin_amdgcn_readfirstlane(threadIdx.y);
    const int lane = threadIdx.x & 63;
    const int cx = tx * wpx + wid;                                     // chunk index (uniform)
    const int y = ty * blockDim.y + wy;                                // row (uniform)
    const int nx = d.nx, ny = d.ny;
    const int xc = cx * 64;                                            // first node of the chunk
    const int x = xc + lane;
    const bool wave_live = (y < ny) && (xc < nx);
    // step counter: every block reads the count before this step; the block of
    // global tile 0 publishes count + 1 in the other slot for the next step
    // (at the end, so no store precedes the kernel's loads)
    const uint32_t step = a.ctr_in[0];

    DD acc[kPartials] = {dd_zero(), dd_zero(), dd_zero(), dd_zero(), dd_zero()};
    if (wave_live && x < nx) {
        const RefView rv = ref_view(ref);
        const int ym = (y == 0) ? ny - 1 : y - 1;
        const int yp = (y == ny - 1) ? 0 : y + 1;
        // wave-uniform row bases; per-lane 32-bit byte offsets within a row
        // (a row of one instance is far below 4 GB), so each access is the
        // scalar-base + vector-offset form of the global load/store
        const char* src = reinterpret_cast<const char*>(a.src) + d.off * (int64_t)sizeof(S);
        const int64_t rb = d.row * (int64_t)sizeof(S);
        const char* rows[3] = {src + (int64_t)y * rb, src + (int64_t)ym * rb, src + (int64_t)yp * rb};
        const int64_t pb = d.plane * (int64_t)sizeof(S);
        const uint32_t es = sizeof(S);
        // column offsets of x, x - 1 and x + 1 (periodic wrap at the row ends)
        const int xm_edge = xc == 0 ? nx - 1 : xc - 1;
        const int xp_edge = xc + 64 < nx ? xc + 64 : 0;
        const bool in_m = lane > 0, in_p = lane < 63 && x + 1 < nx;
        const uint32_t c0 = ((uint32_t)col_off(d, xc) + lane) * es;
        const uint32_t cm = in_m ? c0 - es : (uint32_t)col_off(d, xm_edge) * es;
        const uint32_t cp = in_p ? c0 + es : (x + 1 == nx ? 0u : (uint32_t)col_off(d, xp_edge) * es);
        float g[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int dx = src_dx(i);
            g[i] = Cvt<S>::ld(*reinterpret_cast<const S*>(rows[src_row(i)] + i * pb + (dx < 0 ? cm : (dx > 0 ? cp : c0))));
        }
        const uint32_t e0 = SPLIT ? e_off(d, x) : 0u;
        if (SPLIT) {
            // energies of the source nodes: rows y, y - 1, y + 1 at x - 1, x, x + 1
            float El[3], Ec[3], Er[3];
            if (xc + 64 <= nx) {
                // full chunk: one load per row, neighbours by lane shifts; lanes 0
                // and 63 load the energies beyond the chunk ends in the same
                // instruction (every other lane repeats lane 63's address)
                const uint32_t eo = lane == 0 ? e_off(d, xm_edge) : e_off(d, xp_edge);
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    Ec[r] = *reinterpret_cast<const float*>(rows[r] + e0);
                    const float Eb = *reinterpret_cast<const float*>(rows[r] + eo);
                    El[r] = from_left(Ec[r], Eb);
                    Er[r] = from_right(Ec[r], Eb);
                }
            } else {
                const uint32_t em = in_m ? e0 - 4u : e_off(d, xm_edge);
                const uint32_t ep = in_p ? e0 + 4u : e_off(d, x + 1 == nx ? 0 : xp_edge);
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    Ec[r] = *reinterpret_cast<const float*>(rows[r] + e0);
                    El[r] = *reinterpret_cast<const float*>(rows[r] + em);
                    Er[r] = *reinterpret_cast<const float*>(rows[r] + ep);
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int dx = src_dx(i), r = src_row(i);
                g[i] = g[i] + omega_e(i, dx < 0 ? El[r] : (dx > 0 ? Er[r] : Ec[r]));
            }
        }
        if (a.apply_shift) apply_shift(g, rv);
        const bool edge_y = (d.bc_y != 0) && (y == 0 || y == ny - 1);
        const bool edge_x = (d.bc_x == 1 || d.bc_x == 2 || d.bc_x == 4) && (xc == 0 || xc + 64 >= nx);
        if (edge_y || edge_x) boundary(g, d, rv.wall_kd, x, y);
        if (MODE != kPlain) {
            double E, dT, qx, qy;
            node_moments_f64(g, d, ref.q_ref, E, dT, qx, qy);
            const int64_t n = d.node_off + (int64_t)y * nx + x;
            if (MODE == kSnap) {
                a.snap[n] = dT;
                a.snap[n + snap_stride] = qx;
                a.snap[n + 2 * snap_stride] = qy;
            } else {
                const double p0 = a.snap[n], p1 = a.snap[n + snap_stride], p2 = a.snap[n + 2 * snap_stride];
                acc[0].hi = d.s * E;
                acc[1].hi = qx;
                acc[2].hi = qy;
                acc[3].hi = (dT - p0) * (dT - p0) + (qx - p1) * (qx - p1) + (qy - p2) * (qy - p2);
                acc[4].hi = dT * dT + qx * qx + qy * qy;
            }
        }
        char* out = reinterpret_cast<char*>(a.dst) + d.off * (int64_t)sizeof(S) + (int64_t)y * rb;
        // four 32-bit random words per node and step (SR), as in sr_words
        uint32_t r[4] = {0u, 0u, 0u, 0u};
        if (SR) {
            uint32_t colw[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) colw[k] = sr_col_word((uint32_t)x, k, a.seed);
            sr_words(r, colw, sr_row_word((uint32_t)(d.node_off + (int64_t)y * nx), step, a.seed));
        }
        if (SPLIT) {
            // h*_i = (g_i - omega_i E) + delta_i; the collision keeps E (the
            // FP32 sum of the populations before relaxation).  The rounding
            // residual of the eight h is added to the stored E, so the node's
            // stored populations still sum to E: 16-bit rounding moves energy
            // between directions but creates or destroys none.
            float delta[8], e[8], hv[8];
            S o[8];
            relax_delta(g, d, rv, delta, e);
            const float E = ((g[0] + g[2]) + (g[1] + g[3])) + ((g[4] + g[6]) + (g[5] + g[7]));
#pragma unroll
            for (int i = 0; i < 8; ++i) hv[i] = (g[i] - e[i]) + delta[i];
            round_pairs<S, SR, 8>(hv, r, o);
            float res = 0.0f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                res = res + (hv[i] - Cvt<S>::ld(o[i]));
                store_raw<S>(out + i * pb + c0, o[i], nontemporal);
            }
            store_one<float, 0>(out + e0, E + res, 0u, nontemporal);
        } else if (SR && sizeof(S) == 4) {
            float o[8];
            relax_sr_f32(g, d, rv, r, o);
#pragma unroll
            for (int i = 0; i < 8; ++i) store_one<S, 0>(out + i * pb + c0, o[i], 0u, nontemporal);
        } else {
            // 16-bit SR narrows the round-to-nearest FP32 result stochastically
            relax(g, d, rv);
            S o[8];
            round_pairs<S, SR, 8>(g, r, o);
#pragma unroll
            for (int i = 0; i < 8; ++i) store_raw<S>(out + i * pb + c0, o[i], nontemporal);
        }
    }
    if (t == a.tile_base && threadIdx.x == 0 && threadIdx.y == 0) a.ctr_out[0] = step + 1u;
    if (MODE == kCheck) block_partials(acc, a.partials + (int64_t)t * kPartials);
}

template <class S, int V>
static hipError_t launch_step_v(const Shape& sh, int mode, const StepArgs& a, int64_t snap_stride,
                                hipStream_t st) {
    dim3 grid(a.ntiles), block(sh.bx, sh.by);
    if (mode == kPlain)
        hipLaunchKernelGGL((step_kernel<S, V, kPlain>), grid, block, 0, st, a, snap_stride, sh.xcd, sh.nt);
    else if (mode == kSnap)
        hipLaunchKernelGGL((step_kernel<S, V, kSnap>), grid, block, 0, st, a, snap_stride, sh.xcd, sh.nt);
    else
        hipLaunchKernelGGL((step_kernel<S, V, kCheck>), grid, block, 0, st, a, snap_stride, sh.xcd, sh.nt);
    return hipGetLastError();
}

template <class S, int SR, int SPLIT>
static hipError_t launch_wave_sr(const Shape& sh, int mode, const StepArgs& a, int64_t snap_stride,
                                 hipStream_t st) {
    dim3 grid(a.ntiles), block(sh.bx, sh.by);
    if (mode == kPlain)
        hipLaunchKernelGGL((wave_kernel<S, kPlain, SR, SPLIT>), grid, block, 0, st, a, snap_stride, sh.xcd, sh.nt);
    else if (mode == kSnap)
        hipLaunchKernelGGL((wave_kernel<S, kSnap, SR, SPLIT>), grid, block, 0, st, a, snap_stride, sh.xcd, sh.nt);
    else
        hipLaunchKernelGGL((wave_kernel<S, kCheck, SR, SPLIT>), grid, block, 0, st, a, snap_stride, sh.xcd, sh.nt);
    return hipGetLastError();
}

template <class S, int SPLIT>
static hipError_t launch_wave(const Shape& sh, int mode, const StepArgs& a, int64_t snap_stride,
                              hipStream_t st) {
    return a.sr ? launch_wave_sr<S, 1, SPLIT>(sh, mode, a, snap_stride, st)
                : launch_wave_sr<S, 0, SPLIT>(sh, mode, a, snap_stride, st);
}

template <class S>
static hipError_t launch_step_s(const Shape& sh, int mode, const StepArgs& a, int64_t ss, hipStream_t st) {
    if (a.sr && sh.vec != 1) return hipErrorInvalidValue;
    switch (sh.vec) {
        case 1: return launch_wave<S, 0>(sh, mode, a, ss, st);
        case 2: return launch_step_v<S, 2>(sh, mode, a, ss, st);
        case 4: return launch_step_v<S, 4>(sh, mode, a, ss, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step(int storage, const Shape& sh, int mode, const StepArgs& a, int64_t snap_stride,
                       hipStream_t st) {
    if (a.ntiles <= 0) return hipSuccess;
    if (storage >= 3 && sh.vec != 1) return hipErrorInvalidValue;
    switch (storage) {
        case 0: return launch_step_s<float>(sh, mode, a, snap_stride, st);
        case 1: return launch_step_s<_Float16>(sh, mode, a, snap_stride, st);
        case 2: return launch_step_s<bf16_bits>(sh, mode, a, snap_stride, st);
        case 3: return launch_wave<_Float16, 1>(sh, mode, a, snap_stride, st);
        case 4: return launch_wave<bf16_bits, 1>(sh, mode, a, snap_stride, st);
        default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------------ moments

// Population i of node (x, y) as stored in the instance's buffer (`base`
// points at its first element); SPLIT rebuilds it as h_i + omega_i E.
template <class S, int SPLIT>
__device__ __forceinline__ float load_pop(const S* base, const InstDesc& d, int i, int x, int y) {
    const S* row = base + (int64_t)y * d.row;
    float v = Cvt<S>::ld(row[(int64_t)i * d.plane + col_off(d, x)]);
    if (SPLIT) v = v + omega_e(i, *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + e_off(d, x)));
    return v;
}

// Store the relaxation of the populations g of node (x, y), rounded to
// nearest: as in the step kernels, SPLIT stores h*_i = (g_i - omega_i E) +
// delta_i and E.
template <class S, int SPLIT>
__device__ __forceinline__ void relax_store(S* base, const InstDesc& d, const RefView& rv, float g[8], int x,
                                            int y) {
    S* row = base + (int64_t)y * d.row;
    S* p = row + col_off(d, x);
    if (SPLIT) {
        float delta[8], e[8];
        relax_delta(g, d, rv, delta, e);
        const float E = ((g[0] + g[2]) + (g[1] + g[3])) + ((g[4] + g[6]) + (g[5] + g[7]));
        float res = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float hv = (g[i] - e[i]) + delta[i];
            const S o = Cvt<S>::st(hv);
            res = res + (hv - Cvt<S>::ld(o));
            p[(int64_t)i * d.plane] = o;
        }
        *reinterpret_cast<float*>(reinterpret_cast<char*>(row) + e_off(d, x)) = E + res;
    } else {
        relax(g, d, rv);
#pragma unroll
        for (int i = 0; i < 8; ++i) p[(int64_t)i * d.plane] = Cvt<S>::st(g[i]);
    }
}

// One node per thread, 256 threads along x, one row per block row.
template <class S, int SPLIT>
__global__ __launch_bounds__(256) void moments_kernel(const InstDesc* __restrict__ descs,
                                                      const RefState* __restrict__ refs, int inst,
                                                      const void* buf, int pull, int pending_shift,
                                                      int out_kind, void* T, void* qx, void* qy,
                                                      double t0, double grad, DD* partials) {
    const InstDesc& d = descs[inst];
    const RefState& ref = refs[inst];
    const RefView rv = ref_view(ref);
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    const int nx = d.nx, ny = d.ny;
    DD acc[kPartials] = {dd_zero(), dd_zero(), dd_zero(), dd_zero(), dd_zero()};
    if (x < nx) {
        const S* src = reinterpret_cast<const S*>(buf) + d.off;
        float g[8];
        if (pull) {
            const int ym = (y == 0) ? ny - 1 : y - 1;
            const int yp = (y == ny - 1) ? 0 : y + 1;
            const int rows[3] = {y, ym, yp};
#pragma unroll
            for (int i = 0; i < 8; ++i) g[i] = load_pop<S, SPLIT>(src, d, i, wrapx(x + src_dx(i), nx), rows[src_row(i)]);
            if (pending_shift) apply_shift(g, rv);
            boundary(g, d, rv.wall_kd, x, y);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) g[i] = load_pop<S, SPLIT>(src, d, i, x, y);
        }
        double E = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) E += (double)g[i];
        const double jx = ((double)g[0] - (double)g[2]) + ((double)g[4] - (double)g[6])
                        + ((double)g[7] - (double)g[5]);
        const double jy = ((double)g[1] - (double)g[3]) + ((double)g[4] - (double)g[6])
                        + ((double)g[5] - (double)g[7]);
        const double dT = d.s_cv * E, vx = ref.q_ref + d.s_beta * jx, vy = d.s_beta * jy;
        const int64_t n = (int64_t)y * nx + x;
        if (out_kind == 0) {
            const double tref = t0 - grad * (double)x;
            if (T) reinterpret_cast<float*>(T)[n] = (float)(tref + dT);
            if (qx) reinterpret_cast<float*>(qx)[n] = (float)vx;
            if (qy) reinterpret_cast<float*>(qy)[n] = (float)vy;
        } else {
            if (T) reinterpret_cast<double*>(T)[n] = dT;
            if (qx) reinterpret_cast<double*>(qx)[n] = vx;
            if (qy) reinterpret_cast<double*>(qy)[n] = vy;
        }
        acc[0].hi = d.s * E;
        acc[1].hi = vx;
        acc[2].hi = vy;
    }
    if (partials) block_partials(acc, partials + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kPartials);
}

hipError_t launch_moments(int storage, const InstDesc* d_desc, const RefState* d_ref, int inst,
                          const InstDesc& h, const void* buf, int pull, int pending_shift, int out_kind,
                          void* T, void* qx, void* qy, double t0, double grad, DD* partials,
                          hipStream_t st) {
    dim3 grid((h.nx + 255) / 256, h.ny), block(256);
    switch (storage) {
#define PLBM_MOMENTS(S, SPLIT)                                                                         \
    hipLaunchKernelGGL((moments_kernel<S, SPLIT>), grid, block, 0, st, d_desc, d_ref, inst, buf, pull,  \
                       pending_shift, out_kind, T, qx, qy, t0, grad, partials)
        case 0: PLBM_MOMENTS(float, 0); break;
        case 1: PLBM_MOMENTS(_Float16, 0); break;
        case 2: PLBM_MOMENTS(bf16_bits, 0); break;
        case 3: PLBM_MOMENTS(_Float16, 1); break;
        case 4: PLBM_MOMENTS(bf16_bits, 1); break;
#undef PLBM_MOMENTS
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Moments of one instance from FP64 (dT, qx, qy) planes indexed like the
// snapshot (node_off + y nx + x, `stride` between the planes), written in the
// form moments_kernel writes them; the partials carry s E as dT C_V.
__global__ __launch_bounds__(256) void plane_moments_kernel(const InstDesc* __restrict__ descs, int inst,
                                                            const double* __restrict__ planes, int64_t stride,
                                                            int out_kind, void* T, void* qx, void* qy, double t0,
                                                            double grad, DD* partials) {
    const InstDesc& d = descs[inst];
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    const int nx = d.nx;
    DD acc[kPartials] = {dd_zero(), dd_zero(), dd_zero(), dd_zero(), dd_zero()};
    if (x < nx) {
        const int64_t n = (int64_t)y * nx + x;
        const int64_t m = d.node_off + n;
        const double dT = planes[m], vx = planes[m + stride], vy = planes[m + 2 * stride];
        if (out_kind == 0) {
            const double tref = t0 - grad * (double)x;
            if (T) reinterpret_cast<float*>(T)[n] = (float)(tref + dT);
            if (qx) reinterpret_cast<float*>(qx)[n] = (float)vx;
            if (qy) reinterpret_cast<float*>(qy)[n] = (float)vy;
        } else {
            if (T) reinterpret_cast<double*>(T)[n] = dT;
            if (qx) reinterpret_cast<double*>(qx)[n] = vx;
            if (qy) reinterpret_cast<double*>(qy)[n] = vy;
        }
        acc[0].hi = dT * d.cv;
        acc[1].hi = vx;
        acc[2].hi = vy;
    }
    if (partials) block_partials(acc, partials + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kPartials);
}

hipError_t launch_plane_moments(const InstDesc* d_desc, int inst, const InstDesc& h, const double* planes,
                                int64_t stride, int out_kind, void* T, void* qx, void* qy, double t0, double grad,
                                DD* partials, hipStream_t st) {
    dim3 grid((h.nx + 255) / 256, h.ny), block(256);
    hipLaunchKernelGGL(plane_moments_kernel, grid, block, 0, st, d_desc, inst, planes, stride, out_kind, T, qx,
                       qy, t0, grad, partials);
    return hipGetLastError();
}

// ------------------------------------------------------------------ K steps per launch, y-marching
//
// Temporal blocking without barriers: K time steps per pass over HBM.
// A wavefront owns a 64-column window (W = 64 - 2 KMAX output columns and a
// KMAX-node halo on each side, periodic images) of a chunk of march_rows
// output rows and marches along y.  Iteration `it` loads input row
// yi = y0 - K + it and runs K stages: stage s advances row yi - s from the
// rows of level s - 1 (level 0: loaded, level s: advanced s steps), on lanes
// s..63-s (its pulls stay inside the window); stage K stores its output
// lanes.  A node pulls direction i from row y - c_iy, so of a level's newest
// row the c_y = -1 movers are used at once, the c_y = 0 movers one iteration
// later and the c_y = +1 movers two iterations later (kept in registers, in
// launches of many steps partly in LDS: MarchForm), and the x neighbours come
// from the adjacent lanes by DPP.  Per node and step the arithmetic is the
// single-step kernels' (same functions, same order, same random bits).  RM
// (FusedRounding) says which levels are rounded exactly as a stored step: all of
// them (kRoundEvery, then the result equals K single steps bit for bit), or for
// 16-bit storage only the last (kRoundLast), the others keeping the FP32 result
// of the relaxation: the state a 16-bit launch leaves in HBM then carries one
// rounding to 16 bits, not K.

// K <= KMAX: the window geometry depends on KMAX only, so launches of fewer
// steps (before a check step or at the end of a call) use the same tile table.
// END (how the launch ends):
//   kEndPlain: K plain steps;
//   kEndSnap : the last step is the snapshot step before a check step; its
//              stage also writes the FP64 moments of its pulled nodes, as the
//              single-step kernels do on that step;
//   kEndCheck: the last step is the check step.  Stage K - 1 forms the FP64
//              moments of its nodes (the state at time n - 1) and keeps them
//              in registers for one iteration, until stage K reaches the same
//              row; stage K forms the moments at time n and accumulates, per
//              output node, the check-step sums (energy, heat flux, squared
//              change and squared size of m = (dT, qx, qy)); each wavefront
//              writes its five FP64 sums to a.partials at its tile index.  No
//              snapshot goes through HBM;
//   kEndMoments: (readouts of 16-bit storage, kRoundLast) stage K writes the
//              FP64 moments of its pulled nodes as kEndSnap does and stores
//              no populations.
// CH: chunked layout, whose direction runs are kChunkPlane elements apart, so
// that the eight loads or stores of a row share one address and differ by
// immediate offsets.
// In launches of many steps the first kDelayLevels levels keep their c_y = +1
// movers (two rows of three values) in LDS, 1.5 KB per level and wavefront, the
// others in registers.  These launches are bound by VALU issue, which more
// wavefronts per SIMD fill better: 73-96 VGPRs (the stochastic split kinds spill
// 4 to 7 of theirs at six steps) instead of 114-128 allow five instead of four,
// whose LDS (120 KB of a CU's 160) four levels leave room for.
// Reading a level back at the neighbouring lanes' addresses also saves its two
// diagonal DPP pulls and six moves.  Measured (8192^2, us per step, all in
// registers / this): FP16-SR 159.5 / 145.6, FP16 154.6 / 139.6, BF16-SR 163 /
// 156, F16_SPLIT 167 / 153, BF16_SPLIT 168 / 154, FP32 179.4 / 177.2 (bound by
// its HBM traffic there; 3000 x 2500: 27.3 / 23.9).  At four wavefronts per SIMD
// the LDS form is 1 to 4% slower than registers (see kMidRows); five levels leave LDS for four
// (FP16-SR 164); all five delayed movers of three levels 145.7, of two 163 (105
// VGPRs).
// Launches of fewer steps wait for memory, and more wavefronts in flight or LDS
// in their chain only cost: registers / LDS, us per step as a call of that many
// steps, FP32 two steps 608 / 652, four 308 / 326, five 219 / 267, six 202 / 201;
// FP16-SR two 289 / 347, four on 3000 x 2500 22.0 / 24.8, five 171 / 159;
// F16_SPLIT four 198 / 221, five 190 / 177; rounding every step, FP16-SR four on
// 3000 x 2500 30.7 / 34.0.  So FP32 takes it from seven steps on, 16-bit storage
// from five.  Launches ending on a check step (four wavefronts per SIMD instead
// of three): FP16-SR six steps 8192^2 211 / 180, 3000 x 2500 30.8 / 32.0; FP32
// to nearest, seven, 232 / 224 and 32.4 / 35.6, so in registers; FP32-SR 538 /
// 465 and 76.7 / 75.3.
constexpr int kDelayLevels = 4;
template <class S, int SR, int K, int END>
struct MarchForm {
    static constexpr bool lds = sizeof(S) == 4 ? K >= 7 && (SR || END == kEndPlain) : K >= 5;
    static constexpr int levels = lds ? kDelayLevels : 0;
    // waves per SIMD the register allocation must leave room for (1: no constraint)
    static constexpr int waves = levels && END == kEndPlain ? 5 : 1;
};

template <class S, int SR, int SPLIT, int K, int KMAX, int END, int CH, int RM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MarchForm<S, SR, K, END>::waves)))
void march_kernel(StepArgs a, int xcd, int nontemporal, int64_t snap_stride) {
    static_assert(K >= 2 && K <= KMAX, "stages per launch");
    static_assert(RM == kRoundEvery || sizeof(S) == 2, "FP32 storage rounds every step");
    static_assert(END != kEndMoments || RM == kRoundLast, "the readout replay rounds the last step only");
    // input rows loaded ahead: one iteration's stages must cover a row load's
    // latency, so launches of few plain steps load further ahead (8 VGPRs per
    // FP32 row).  Measured on MI355X (8192^2, us per launch, ahead 1 / more):
    // FP32 three steps 1269 / 1186 (two ahead), two steps 1188 / 1247 (three);
    // FP16 two steps 656 / 603 (three), three 632 / 607 (two), four 745 / 788
    // (two); the check launches' FP64 work covers the latency by itself.
    constexpr int PF = END == kEndCheck ? 1
                     : (K == 3 ? 2 : ((K == 2 && sizeof(S) == 2) ? 3 : 1));
    static_assert(PF >= 1 && PF <= 2 * K + 1, "the first PF rows are all input rows");
    constexpr int W = 64 - 2 * KMAX;
    const int lane = threadIdx.x & 63;
    int b = blockIdx.x;
    if (xcd) {
        const int nb = gridDim.x, q = nb >> 3, r = nb & 7, k = b & 7, j = b >> 3;
        b = k * q + (k < r ? k : r) + j;
    }
    const int t = b * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (t >= a.ntiles) return;                // whole wavefront: no lane is left behind a DPP move
    const int tg = t + a.tile_base;
    // halved (few-step launches of a handle with kTallRows strips): the launch's
    // tiles are strips of half the table's height, two for each of the table's
    constexpr bool HALVES = sizeof(S) == 2 && K < kTallSteps && END != kEndCheck;
    const int halved = HALVES ? a.halved : 0;
    // a private copy of the descriptor, read once before the first store (the
    // compiler cannot keep fields of device memory in registers across stores)
    const int inst = __builtin_amdgcn_readfirstlane(a.tile_inst[tg >> halved]);
    const InstDesc d = a.desc[inst];
    const RefView rv = ref_view(a.ref[inst]);
    const double q_ref = END != kEndPlain ? a.ref[inst].q_ref : 0.0;
    const int local = tg - (d.p_tile_begin << halved);
    const int ty = local / d.p_tiles_x;
    const int tx = local - ty * d.p_tiles_x;
    // FP32 storage always takes kMarchRows, as a constant: with the count read
    // from the arguments launches of two and three steps ran 6% slower on 8192^2
    // (us per launch, argument / constant: 1295 / 1217, 1320 / 1241), with the
    // same loop and 14% more HBM reads; reading it earlier did not help
    const int rows = sizeof(S) == 4 ? kMarchRows : a.march_rows;
    const int x0 = tx * W, y0 = ty * rows;
    const int nx = d.nx, ny = d.ny;
    if (HALVES && y0 >= ny) return;           // the last strip of the table may fill one half only
    const int gx = wrapm(x0 - KMAX + lane, nx, 64);
    const int iters = min(rows, ny - y0) + 2 * K;
    const uint32_t step = a.ctr_in[0];
    const S* __restrict__ src = reinterpret_cast<const S*>(a.src) + d.off;
    S* __restrict__ dst = reinterpret_cast<S*>(a.dst) + d.off;
    const int64_t col = col_off(d, gx);
    const int64_t plane = CH ? (int64_t)kChunkPlane : d.plane;
    uint32_t colw[4] = {0u, 0u, 0u, 0u};
    if (SR) {
#pragma unroll
        for (int k = 0; k < 4; ++k) colw[k] = sr_col_word((uint32_t)gx, k, a.seed);
    }

    // raw loads of input row yi (converted only where the row is used, so
    // the loads stay in flight across the iterations in between)
    auto fetch_row = [&](int yi, S v[8], float& E) {
        const int gy = wrapm(yi, ny, rows + 2 * K + PF);
        const S* row = src + (int64_t)gy * d.row;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = row[(int64_t)i * plane + col];
        E = SPLIT ? *reinterpret_cast<const float*>(reinterpret_cast<const char*>(row) + e_off(d, gx)) : 0.0f;
    };

    // per level l (0: loaded rows, l: results of stage l), the c_y = 0 movers of
    // the previous row and the c_y = +1 movers of the two previous rows
    // (levels below DL keep the c_y = +1 movers in LDS, in the slots of the
    // last two rows; `par`: the slot this iteration reads and refills.  A
    // wavefront touches its own part only, and the hardware executes its LDS
    // accesses in the order they are issued, so no barrier is needed.  The
    // compiler sees one lane, whose reads of its neighbours' slots never meet its
    // own refills, and might move one past the other; the empty asm takes away
    // what it knows of the neighbours' addresses, so that each of them may be any
    // address a refill writes and every read keeps its place among the refills.
    // (Wavefront-scope fences before every refill do the same, but also hold back
    // everything else: FP16-SR 8192^2 at six steps 854 -> 864 us per launch.)
    constexpr int DL = MarchForm<S, SR, K, END>::levels;
    __shared__ float delay[4][DL ? DL : 1][2][3][64];
    const uint32_t mine = (threadIdx.x >> 6) * (uint32_t)sizeof(delay[0]);
    const uint32_t at_c = mine + (uint32_t)lane * 4u;
    uint32_t at_l = mine + (uint32_t)((lane - 1) & 63) * 4u, at_r = mine + (uint32_t)((lane + 1) & 63) * 4u;
    if constexpr (DL > 0) asm volatile("" : "+v"(at_l), "+v"(at_r));
    uint32_t par = 0u;
    auto delayed = [&](uint32_t at) -> float& {
        return *reinterpret_cast<float*>(reinterpret_cast<char*>(&delay[0][0][0][0][0]) + at);
    };
    float mid[K][2], up1[K][3], up2[K][3];
#pragma unroll
    for (int l = 0; l < K; ++l) {
        mid[l][0] = mid[l][1] = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) up1[l][k] = up2[l][k] = 0.0f;
    }
    // check launch: moments of the stage K - 1 nodes of this iteration (new)
    // and of the previous one (old, the row stage K reaches now), and the
    // output nodes' check sums
    double pm_new[3] = {0.0, 0.0, 0.0}, pm_old[3] = {0.0, 0.0, 0.0};
    DD acc[kPartials] = {dd_zero(), dd_zero(), dd_zero(), dd_zero(), dd_zero()};
    // rows yi .. yi + PF - 1 of the coming iterations, in flight
    S ring[PF][8];
    float ringE[PF];
#pragma unroll
    for (int j = 0; j < PF; ++j) fetch_row(y0 - K + j, ring[j], ringE[j]);
    // One iteration: take row yi from the ring and load row yi + PF into it,
    // then every stage whose input rows exist; WARM (the first 2 K
    // iterations) tests that per stage, later iterations run all K stages.
    auto iteration = [&](const int it, auto warm) {
        constexpr bool WARM = decltype(warm)::value;
        const int yi = y0 - K + it;
        float cur[8];
        reload<S, SPLIT>(ring[0], ringE[0], cur);
#pragma unroll
        for (int j = 0; j + 1 < PF; ++j) {
#pragma unroll
            for (int i = 0; i < 8; ++i) ring[j][i] = ring[j + 1][i];
            ringE[j] = ringE[j + 1];
        }
        if (it + PF < iters) fetch_row(yi + PF, ring[PF - 1], ringE[PF - 1]);
#pragma unroll
        for (int s = 1; s <= K; ++s) {
            // stage s: row yi - s from level s - 1 (valid once it >= 2 s)
            float out[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
            if (!WARM || it >= 2 * s) {
                float g[8];
                if (s - 1 < DL) {
                    const uint32_t o = (uint32_t)((s - 1) * sizeof(delay[0][0])) + par;
                    float up[3] = {delayed(at_c + o), delayed(at_l + o + 256), delayed(at_r + o + 512)};
                    march_gather<1>(cur, mid[s - 1], up, g);
                } else {
                    march_gather<0>(cur, mid[s - 1], up2[s - 1], g);
                }
                if (s < K) {
                    const int gy = wrapm(yi - s, ny, rows + 2 * K + PF);
                    if (s == 1 && a.apply_shift) {
                        // the empty asm keeps this a branch: as selects the
                        // shift would run on every row of every lattice
                        asm volatile("");
                        apply_shift(g, rv);
                    }
                    if (on_wall(d, gx, gy)) boundary(g, d, rv.wall_kd, gx, gy);
                    if constexpr (END == kEndCheck) {
                        if (s == K - 1) {
                            double E;
                            node_moments_f64(g, d, q_ref, E, pm_new[0], pm_new[1], pm_new[2]);
                        }
                    }
                    // 16-bit storage, kRoundLast: the result stays in FP32
                    // (round to nearest), as FP32 storage would keep it
                    if (RM == kRoundLast) {
                        relax_folded(g, d, rv);
#pragma unroll
                        for (int i = 0; i < 8; ++i) out[i] = g[i];
                    } else {
                        uint32_t r[4] = {0u, 0u, 0u, 0u};
                        if (SR)
                            sr_words(r, colw, sr_row_word((uint32_t)(d.node_off + (int64_t)gy * nx),
                                                          step + (uint32_t)(s - 1), a.seed));
                        S o[8];
                        float E;
                        relax_round<S, SR, SPLIT>(g, d, rv, r, o, E);
                        reload<S, SPLIT>(o, E, out);
                    }
                } else {
                    const int ox = x0 + lane - KMAX, oy = yi - s;
                    if (lane >= KMAX && lane < KMAX + W && ox < nx) {
                        if (on_wall(d, ox, oy)) boundary(g, d, rv.wall_kd, ox, oy);
                        if constexpr (END == kEndSnap || END == kEndMoments) {
                            double E, dT, qx, qy;
                            node_moments_f64(g, d, q_ref, E, dT, qx, qy);
                            const int64_t n = d.node_off + (int64_t)oy * nx + ox;
                            a.snap[n] = dT;
                            a.snap[n + snap_stride] = qx;
                            a.snap[n + 2 * snap_stride] = qy;
                            if constexpr (END == kEndMoments) {
                                // the caller's arrays in the same pass, not in
                                // a second one that copies them: 16384^2 split
                                // 6.2 -> 4.8 ms, 8192^2 1.29 -> 1.18 ms
                                if (inst == a.out_inst) {
                                    const int64_t m = (int64_t)oy * nx + ox;
                                    if (a.out[0]) a.out[0][m] = dT;
                                    if (a.out[1]) a.out[1][m] = qx;
                                    if (a.out[2]) a.out[2][m] = qy;
                                }
                            }
                        } else if constexpr (END == kEndCheck) {
                            // the same sums, in the same per-node form, as the
                            // single-step check kernels
                            double E, dT, qx, qy;
                            node_moments_f64(g, d, q_ref, E, dT, qx, qy);
                            const double p0 = pm_old[0], p1 = pm_old[1], p2 = pm_old[2];
                            check_sums(acc, d.s * E, qx, qy, dT, p0, p1, p2);
                        }
                        if constexpr (END != kEndMoments) {
                            uint32_t r[4] = {0u, 0u, 0u, 0u};
                            if (SR)
                                sr_words(r, colw, sr_row_word((uint32_t)(d.node_off + (int64_t)oy * nx),
                                                              step + (uint32_t)(s - 1), a.seed));
                            S o[8];
                            float E;
                            relax_round<S, SR, SPLIT>(g, d, rv, r, o, E);
                            S* row = dst + (int64_t)oy * d.row;
                            const int64_t c = col_off(d, ox);
#pragma unroll
                            for (int i = 0; i < 8; ++i)
                                store_raw<S>(reinterpret_cast<char*>(row + c + (int64_t)i * plane), o[i], nontemporal);
                            if (SPLIT)
                                store_one<float, 0>(reinterpret_cast<char*>(row) + e_off(d, ox), E, 0u, nontemporal);
                        }
                    }
                }
            }
            // level s - 1 moves one row on (its values are valid whenever a later stage reads them)
            if (s - 1 < DL) {
                const uint32_t o = (uint32_t)((s - 1) * sizeof(delay[0][0])) + par;
#pragma unroll
                for (int k = 0; k < 3; ++k) delayed(at_c + o + 256 * k) = cur[yup(k)];
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    up2[s - 1][k] = up1[s - 1][k];
                    up1[s - 1][k] = cur[yup(k)];
                }
            }
#pragma unroll
            for (int k = 0; k < 2; ++k) mid[s - 1][k] = cur[ymid(k)];
            if (s < K) {
#pragma unroll
                for (int i = 0; i < 8; ++i) cur[i] = out[i];
            } else if constexpr (END == kEndCheck) {
                // stage K has used the moments stage K - 1 formed one iteration ago
#pragma unroll
                for (int c = 0; c < 3; ++c) pm_old[c] = pm_new[c];
            }
        }
    };
    // iters >= 2 K + 1: the warm-up always completes
    int it = 0;
    for (; it < 2 * K; ++it, par ^= (uint32_t)sizeof(delay[0][0][0])) iteration(it, std::true_type{});
    for (; it < iters; ++it, par ^= (uint32_t)sizeof(delay[0][0][0])) iteration(it, std::false_type{});
    if (t == 0 && lane == 0) a.ctr_out[0] = step + (uint32_t)K;
    if constexpr (END == kEndCheck) {
        // fixed-order wavefront sums; one record per tile (all 64 lanes are
        // active here: a wavefront leaves early only as a whole)
        wave_sums(acc);
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < kPartials; ++c) a.partials[(int64_t)tg * kPartials + c] = acc[c];
        }
    }
}

template <class S, int SR, int SPLIT, int K, int KMAX, int END, int RM>
static void launch_march_ch(const Shape& sh, const StepArgs& a, int chunked, int64_t snap_stride, hipStream_t st) {
    dim3 grid((a.ntiles + 3) / 4), block(256);
    if (chunked)
        hipLaunchKernelGGL((march_kernel<S, SR, SPLIT, K, KMAX, END, 1, RM>), grid, block, 0, st, a, sh.xcd, sh.nt,
                           snap_stride);
    else
        hipLaunchKernelGGL((march_kernel<S, SR, SPLIT, K, KMAX, END, 0, RM>), grid, block, 0, st, a, sh.xcd, sh.nt,
                           snap_stride);
}

template <class S, int SR, int SPLIT, int K, int KMAX, int RM>
static void launch_march_e(const Shape& sh, const StepArgs& a, int end, int chunked, int64_t snap_stride,
                           hipStream_t st) {
    if (end == kEndSnap) launch_march_ch<S, SR, SPLIT, K, KMAX, kEndSnap, RM>(sh, a, chunked, snap_stride, st);
    else if (end == kEndCheck) launch_march_ch<S, SR, SPLIT, K, KMAX, kEndCheck, RM>(sh, a, chunked, snap_stride, st);
    else if (end == kEndPlain) launch_march_ch<S, SR, SPLIT, K, KMAX, kEndPlain, RM>(sh, a, chunked, snap_stride, st);
    else if constexpr (RM == kRoundLast)
        launch_march_ch<S, SR, SPLIT, K, KMAX, kEndMoments, RM>(sh, a, chunked, snap_stride, st);
}

template <class S, int SPLIT, int K, int KMAX, int RM>
static hipError_t launch_march_s(const Shape& sh, const StepArgs& a, int end, int chunked, int64_t snap_stride,
                                 hipStream_t st) {
    if (a.sr) launch_march_e<S, 1, SPLIT, K, KMAX, RM>(sh, a, end, chunked, snap_stride, st);
    else launch_march_e<S, 0, SPLIT, K, KMAX, RM>(sh, a, end, chunked, snap_stride, st);
    return hipGetLastError();
}

// Whether a variant of k = K steps, step rounding rm and end is built.
template <class S, int K>
constexpr bool march_built(int rm, int end) {
    if (rm == kRoundLast) return sizeof(S) == 2;
    if (rm != kRoundEvery || end == kEndMoments) return false;
    return sizeof(S) == 4 || K <= kFuseEveryStep;
}

template <class S, int SPLIT, int K, int KMAX>
static hipError_t launch_march_k(const Shape& sh, const StepArgs& a, int k, int end, int chunked, int rm,
                                 int64_t snap_stride, hipStream_t st) {
    if constexpr (K > KMAX) {
        return hipErrorInvalidValue;
    } else {
        if (k != K) return launch_march_k<S, SPLIT, K + 1, KMAX>(sh, a, k, end, chunked, rm, snap_stride, st);
        if (!march_built<S, K>(rm, end)) return hipErrorInvalidValue;
        if constexpr (sizeof(S) == 2) {
            if (rm == kRoundLast)
                return launch_march_s<S, SPLIT, K, KMAX, kRoundLast>(sh, a, end, chunked, snap_stride, st);
        }
        if constexpr (sizeof(S) == 4 || K <= kFuseEveryStep)
            return launch_march_s<S, SPLIT, K, KMAX, kRoundEvery>(sh, a, end, chunked, snap_stride, st);
        return hipErrorInvalidValue;
    }
}

// Launch every fused-kernel variant a handle may use (its storage kind,
// rounding, layout and step rounding; 2 .. fuse_max steps; each end) once with
// no tiles: each wavefront returns at its first test, touching no memory.
// The runtime does its once-per-kernel work (loading the code; for a kernel
// that spills, setting up scratch memory) at a kernel's first launch, which
// would otherwise land in the first real launch of each variant.
template <class S, int SR, int SPLIT, int K, int KMAX, int END, int RM>
static hipError_t preload_one(int chunked, hipStream_t st) {
    StepArgs a{};
    a.ntiles = 0;
    const dim3 grid(1), block(256);
    if (chunked)
        hipLaunchKernelGGL((march_kernel<S, SR, SPLIT, K, KMAX, END, 1, RM>), grid, block, 0, st, a, 0, 0, 0);
    else
        hipLaunchKernelGGL((march_kernel<S, SR, SPLIT, K, KMAX, END, 0, RM>), grid, block, 0, st, a, 0, 0, 0);
    return hipGetLastError();
}

template <class S, int SR, int SPLIT, int K, int KMAX, int RM>
static hipError_t preload_ends(int chunked, hipStream_t st) {
    hipError_t e = preload_one<S, SR, SPLIT, K, KMAX, kEndPlain, RM>(chunked, st);
    if (e == hipSuccess) e = preload_one<S, SR, SPLIT, K, KMAX, kEndSnap, RM>(chunked, st);
    if (e == hipSuccess) e = preload_one<S, SR, SPLIT, K, KMAX, kEndCheck, RM>(chunked, st);
    if constexpr (RM == kRoundLast) {
        if (e == hipSuccess) e = preload_one<S, SR, SPLIT, K, KMAX, kEndMoments, RM>(chunked, st);
    }
    return e;
}

template <class S, int SR, int SPLIT, int K, int KMAX>
static hipError_t preload_march_k(int chunked, int every_step, hipStream_t st) {
    if constexpr (K > KMAX) {
        return hipSuccess;
    } else {
        hipError_t e = hipSuccess;
        if constexpr (sizeof(S) == 2) {
            if (!every_step) e = preload_ends<S, SR, SPLIT, K, KMAX, kRoundLast>(chunked, st);
        }
        if constexpr (sizeof(S) == 4 || K <= kFuseEveryStep) {
            if (every_step || sizeof(S) == 4) e = preload_ends<S, SR, SPLIT, K, KMAX, kRoundEvery>(chunked, st);
        }
        if (e != hipSuccess) return e;
        return preload_march_k<S, SR, SPLIT, K + 1, KMAX>(chunked, every_step, st);
    }
}

template <class S, int SPLIT, int STORAGE>
static hipError_t preload_fused_s(int sr, int chunked, int every_step, hipStream_t st) {
    return sr ? preload_march_k<S, 1, SPLIT, 2, fuse_max(STORAGE)>(chunked, every_step, st)
              : preload_march_k<S, 0, SPLIT, 2, fuse_max(STORAGE)>(chunked, every_step, st);
}

hipError_t preload_fused(int storage, int sr, int chunked, int every_step, hipStream_t st) {
    switch (storage) {
        case 0: return preload_fused_s<float, 0, 0>(sr, chunked, 1, st);
        case 1: return preload_fused_s<_Float16, 0, 1>(sr, chunked, every_step, st);
        case 2: return preload_fused_s<bf16_bits, 0, 2>(sr, chunked, every_step, st);
        case 3: return preload_fused_s<_Float16, 1, 3>(sr, chunked, every_step, st);
        case 4: return preload_fused_s<bf16_bits, 1, 4>(sr, chunked, every_step, st);
        default: return hipErrorInvalidValue;
    }
}

template <class S, int SPLIT, int STORAGE>
static hipError_t launch_fused_s(const Shape& sh, const StepArgs& a, int k, int end, int chunked, int rm,
                                 int64_t snap_stride, hipStream_t st) {
    return launch_march_k<S, SPLIT, 2, fuse_max(STORAGE)>(sh, a, k, end, chunked, rm, snap_stride, st);
}

hipError_t launch_fused(int storage, const Shape& sh, const StepArgs& a, int k, int end, int chunked,
                        int rounding, int64_t snap_stride, hipStream_t st) {
    if (a.ntiles <= 0) return hipSuccess;
    if (a.halved && (storage == 0 || k >= kTallSteps || end == kEndCheck)) return hipErrorInvalidValue;
    if (storage == 0 && a.march_rows != kMarchRows) return hipErrorInvalidValue;
    if ((end == kEndSnap || end == kEndMoments) && !a.snap) return hipErrorInvalidValue;
    if (end == kEndCheck && !a.partials) return hipErrorInvalidValue;
    if (end < kEndPlain || end > kEndMoments) return hipErrorInvalidValue;
    switch (storage) {
        case 0: return launch_fused_s<float, 0, 0>(sh, a, k, end, chunked, rounding, snap_stride, st);
        case 1: return launch_fused_s<_Float16, 0, 1>(sh, a, k, end, chunked, rounding, snap_stride, st);
        case 2: return launch_fused_s<bf16_bits, 0, 2>(sh, a, k, end, chunked, rounding, snap_stride, st);
        case 3: return launch_fused_s<_Float16, 1, 3>(sh, a, k, end, chunked, rounding, snap_stride, st);
        case 4: return launch_fused_s<bf16_bits, 1, 4>(sh, a, k, end, chunked, rounding, snap_stride, st);
        default: return hipErrorInvalidValue;
    }
}

// ------------------------------------------------------------------ scratch contents

// Words of a timing scratch pattern: each 16-bit half is a random sign, the
// exponent pattern 0x3a and eight random mantissa bits, so the buffer reads as
// moderate finite values in FP32 (about 1e-3), FP16 (0.75 .. 0.88) and BF16
// (about 1e-3) with bits that change from element to element, as real data
// do (zero-filled buffers run faster than real contents and bias timings).
__global__ __launch_bounds__(256) void fill_kernel(uint32_t* __restrict__ p, int64_t nwords, uint32_t seed) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= nwords) return;
    const uint32_t h = mix32((uint32_t)i ^ mix32((uint32_t)(i >> 32) + seed));
    const uint32_t lo = (h & 0x8000u) | 0x3a00u | (h & 0xffu);
    const uint32_t hi = ((h >> 16) & 0x8000u) | 0x3a00u | ((h >> 8) & 0xffu);
    p[i] = (hi << 16) | lo;
}

hipError_t launch_fill(void* buf, size_t bytes, uint32_t seed, hipStream_t st) {
    const int64_t n = (int64_t)(bytes / 4);
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<uint32_t*>(buf), n, seed);
    return hipGetLastError();
}

// ------------------------------------------------------------------ init

// Pre-relaxation state at n = 0 (equilibrium of Eq. 15 with j = q / beta, wall
// nodes at their Eq. 55 equilibrium), stored rounded to `pre`; its relaxation,
// computed from the rounded values exactly as a step would, goes to `post`.
// The instance's descriptor and initial reference state come with the kernel's
// arguments and are written to their device tables here, and the step counters
// are cleared: one launch instead of three copies and a memset around it.  256
// initialisations of a sweep from device fields: 8.2 -> 4.1 ms.
template <class S, int SPLIT>
__global__ __launch_bounds__(256) void init_kernel(InstDesc d, RefState ref, InitTables t, int inst,
                                                   void* pre, void* post, const double* __restrict__ T,
                                                   const double* __restrict__ qx,
                                                   const double* __restrict__ qy, double t0,
                                                   double grad, double beta) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        t.desc[inst] = d;
        t.ref[inst] = ref;
        t.ref_prev[inst] = ref;
        t.ctr[0] = t.ctr[1] = 0u;
    }
    const RefView rv = ref_view(ref);
    const int x = blockIdx.x * 256 + threadIdx.x;
    const int y = blockIdx.y;
    if (x >= d.nx) return;
    const int64_t n = (int64_t)y * d.nx + x;
    const double dT = T[n] - (t0 - grad * (double)x);
    const double jx = qx ? qx[n] / beta : 0.0, jy = qy ? qy[n] / beta : 0.0;
    const double inv_s = 1.0 / d.s;
    const double ea = (2.0 / 9.0) * d.cv * dT, ed = (1.0 / 36.0) * d.cv * dT;
    // minus the reference state's shares c_ix p_i
    const double pa = ref.p_axis, pd = ref.p_diag;
    float g[8];
    g[0] = (float)((ea + jx / 3.0 - pa) * inv_s);
    g[1] = (float)((ea + jy / 3.0) * inv_s);
    g[2] = (float)((ea - jx / 3.0 + pa) * inv_s);
    g[3] = (float)((ea - jy / 3.0) * inv_s);
    g[4] = (float)((ed + (jx + jy) / 12.0 - pd) * inv_s);
    g[5] = (float)((ed + (-jx + jy) / 12.0 + pd) * inv_s);
    g[6] = (float)((ed - (jx + jy) / 12.0 + pd) * inv_s);
    g[7] = (float)((ed + (jx - jy) / 12.0 - pd) * inv_s);
    const bool wall = (x == 0 && d.wk[0] == 1) || (x == d.nx - 1 && d.wk[1] == 1) ||
                      (y == 0 && d.wk[2] == 1) || (y == d.ny - 1 && d.wk[3] == 1);
    if (wall) boundary(g, d, rv.wall_kd, x, y);
    S* pb = reinterpret_cast<S*>(pre) + d.off;
    S* row = pb + (int64_t)y * d.row;
    S* p = row + col_off(d, x);
    if (SPLIT) {
        const float E = ((g[0] + g[2]) + (g[1] + g[3])) + ((g[4] + g[6]) + (g[5] + g[7]));
        float hq[8], res = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float hv = g[i] - omega_e(i, E);
            const S v = Cvt<S>::st(hv);
            p[(int64_t)i * d.plane] = v;
            hq[i] = Cvt<S>::ld(v);
            res = res + (hv - hq[i]);
        }
        const float Es = E + res;
        *reinterpret_cast<float*>(reinterpret_cast<char*>(row) + e_off(d, x)) = Es;
        // the populations as the next read will rebuild them
#pragma unroll
        for (int i = 0; i < 8; ++i) g[i] = hq[i] + omega_e(i, Es);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const S v = Cvt<S>::st(g[i]);
            p[(int64_t)i * d.plane] = v;
            g[i] = Cvt<S>::ld(v);
        }
    }
    relax_store<S, SPLIT>(reinterpret_cast<S*>(post) + d.off, d, rv, g, x, y);
}

hipError_t launch_init(int storage, const InitTables& t, int inst, const InstDesc& h, const RefState& ref, void* pre, void* post, const double* T, const double* qx,
                       const double* qy, double t0, double grad, double beta, hipStream_t st) {
    dim3 grid((h.nx + 255) / 256, h.ny), block(256);
    switch (storage) {
#define PLBM_INIT(S, SPLIT)                                                                            \
    hipLaunchKernelGGL((init_kernel<S, SPLIT>), grid, block, 0, st, h, ref, t, inst, pre, post, T, qx, \
                       qy, t0, grad, beta)
        case 0: PLBM_INIT(float, 0); break;
        case 1: PLBM_INIT(_Float16, 0); break;
        case 2: PLBM_INIT(bf16_bits, 0); break;
        case 3: PLBM_INIT(_Float16, 1); break;
        case 4: PLBM_INIT(bf16_bits, 1); break;
#undef PLBM_INIT
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ reductions

// Fixed-order compensated sum of `count` partial records starting at
// `first`: thread t adds records t, t + 256, ... in order, then a fixed tree
// over the block.
__device__ void reduce_records(const DD* __restrict__ partials, int64_t first, int count, DD* __restrict__ out) {
    __shared__ DD red[256][kPartials];
    const int t = threadIdx.x;
    DD s[kPartials] = {dd_zero(), dd_zero(), dd_zero(), dd_zero(), dd_zero()};
    for (int j = t; j < count; j += 256)
#pragma unroll
        for (int c = 0; c < kPartials; ++c) s[c] = dd_add(s[c], partials[(first + j) * kPartials + c]);
#pragma unroll
    for (int c = 0; c < kPartials; ++c) red[t][c] = s[c];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w)
#pragma unroll
            for (int c = 0; c < kPartials; ++c) red[t][c] = dd_add(red[t][c], red[t + w][c]);
        __syncthreads();
    }
    if (t == 0)
#pragma unroll
        for (int c = 0; c < kPartials; ++c) out[c] = red[0][c];
}

// First stage: group b = g0 + blockIdx.x of the tile records of its
// instance.  fused != 0: records of the fused kernel's tiles (strips), else of
// the single-step tiles.
__global__ __launch_bounds__(256) void group_reduce_kernel(const InstDesc* __restrict__ descs,
                                                           const int32_t* __restrict__ group_inst,
                                                           const DD* __restrict__ partials,
                                                           DD* __restrict__ gpart, int fused, int g0) {
    const int b = g0 + (int)blockIdx.x;
    const InstDesc& d = descs[group_inst[b]];
    const int gb = fused == 2 ? d.b_group_begin : (fused ? d.p_group_begin : d.group_begin);
    const int tb = fused == 2 ? d.b_tile_begin : (fused ? d.p_tile_begin : d.tile_begin);
    const int nt = fused == 2 ? d.b_ntiles : (fused ? d.p_ntiles : d.ntiles);
    const int j = b - gb;
    const int rest = nt - j * kGroup;
    reduce_records(partials, (int64_t)tb + (int64_t)j * kGroup, rest < kGroup ? rest : kGroup,
                   gpart + (int64_t)b * kPartials);
}

// Second stage, per instance (i0 + blockIdx.x): the check-step totals, then (adaptive
// instances) the move of the reference flux to the mean flux of the state just
// checked.  The shift is rounded to FP32 first and J is moved by the rounded
// amount (in FP64), so J and the stored populations stay consistent;
// shift_d = shift_a / 4 is exact.  The reference state in force before the
// move is kept in refs_prev (the steps up to the check step ran with it).
__global__ __launch_bounds__(256) void finalize_kernel(const InstDesc* __restrict__ descs,
                                                       RefState* __restrict__ refs,
                                                       RefState* __restrict__ refs_prev,
                                                       const DD* __restrict__ records,
                                                       double* __restrict__ results, int fused, int i0, int grouped) {
    const int inst = i0 + (int)blockIdx.x;
    const InstDesc& d = descs[inst];
    __shared__ DD sum[kPartials];
    const int gb = fused == 2 ? d.b_group_begin : (fused ? d.p_group_begin : d.group_begin);
    const int ng = fused == 2 ? d.b_ngroups : (fused ? d.p_ngroups : d.ngroups);
    const int tb = fused == 2 ? d.b_tile_begin : (fused ? d.p_tile_begin : d.tile_begin);
    const int nt = fused == 2 ? d.b_ntiles : (fused ? d.p_ntiles : d.ntiles);
    reduce_records(records, grouped ? gb : tb, grouped ? ng : nt, sum);
    if (threadIdx.x != 0) return;
    double* out = results + (int64_t)inst * kPartials;
#pragma unroll
    for (int c = 0; c < kPartials; ++c) out[c] = sum[c].hi;
    RefState& r = refs[inst];
    refs_prev[inst] = r;
    if (!r.adapt) return;
    // mean heat flux = beta (mean first moment); reference's first moment J + j_b
    const double target = out[1] * r.inv_nodes / r.beta - r.jb;
    float sa = 0.0f;
    double J = r.J;
    if (isfinite(target)) {
        sa = (float)((r.J - target) / (3.0 * r.s));
        J = r.J - 3.0 * r.s * (double)sa;
    }
    r.shift_a = sa;
    r.shift_d = 0.25f * sa;
    ref_set_flux(r, J);
}

// Block b reduces records [b * span, min((b + 1) * span, count)).
__global__ __launch_bounds__(256) void range_reduce_kernel(const DD* __restrict__ partials, int count,
                                                           int span, DD* __restrict__ out) {
    const int64_t first = (int64_t)blockIdx.x * span;
    const int64_t rest = count - first;
    reduce_records(partials, first, (int)(rest < span ? rest : span), out + (int64_t)blockIdx.x * kPartials);
}

hipError_t launch_finalize(const InstDesc* d_desc, const int32_t* group_inst, int g0, int ngroups, RefState* d_ref,
                           RefState* d_ref_prev, int i0, int ninst, const DD* partials, DD* gpart,
                           double* results, int fused, hipStream_t st) {
    if (ngroups <= 0 || ninst <= 0) return hipSuccess;
    // one group per instance: its tile records are the second stage's input
    // (the same order of additions, one launch less)
    const int grouped = ngroups > ninst;
    if (grouped)
        hipLaunchKernelGGL(group_reduce_kernel, dim3(ngroups), dim3(256), 0, st, d_desc, group_inst, partials, gpart,
                           fused, g0);
    hipLaunchKernelGGL(finalize_kernel, dim3(ninst), dim3(256), 0, st, d_desc, d_ref, d_ref_prev,
                       grouped ? gpart : partials, results, fused, i0, grouped);
    return hipGetLastError();
}

__global__ void set_float_kernel(float* dst, float v) { *dst = v; }

__global__ void copy_u32_kernel(uint32_t* dst, const uint32_t* src, int n) {
    if ((int)threadIdx.x < n) dst[threadIdx.x] = src[threadIdx.x];
}

hipError_t launch_copy_u32(uint32_t* dst, const uint32_t* src, int n, hipStream_t st) {
    if (n <= 0 || n > 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(copy_u32_kernel, dim3(1), dim3(64), 0, st, dst, src, n);
    return hipGetLastError();
}

hipError_t launch_set_float(float* dst, float v, hipStream_t st) {
    hipLaunchKernelGGL(set_float_kernel, dim3(1), dim3(1), 0, st, dst, v);
    return hipGetLastError();
}

hipError_t launch_finalize_range(const DD* partials, int nparts, DD* gpart, DD* result, hipStream_t st) {
    const int ng = (nparts + kGroup - 1) / kGroup;
    hipLaunchKernelGGL(range_reduce_kernel, dim3(ng), dim3(256), 0, st, partials, nparts, kGroup, gpart);
    hipLaunchKernelGGL(range_reduce_kernel, dim3(1), dim3(256), 0, st, gpart, ng, ng, result);
    return hipGetLastError();
}

}  // namespace plbm
