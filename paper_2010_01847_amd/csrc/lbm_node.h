// One lattice node in device code: loads and stores of its populations, the
// relaxation (Eq. 13 with Eqs. 15-16), the boundary treatment (Sec. 2.5), the
// FP64 moments (Eqs. 53-54), rounding to the storage type, and the compensated
// sums of the check steps.  Shared by every D2Q8 kernel, so that they all
// compute the same bits.
#pragma once

#include "lbm_internal.h"
#include "lbm_numeric.h"

#include <stdint.h>

namespace plbm {

template <int BYTES> struct RawT;
template <> struct RawT<2> { typedef uint16_t T; };
template <> struct RawT<4> { typedef uint32_t T; };
template <> struct RawT<8> { typedef uint32_t T __attribute__((ext_vector_type(2))); };
template <> struct RawT<16> { typedef uint32_t T __attribute__((ext_vector_type(4))); };

// V consecutive elements from an element-aligned address (one wide load; the
// gfx9 memory path accepts dword-unaligned vector accesses).
template <class S, int V>
__device__ __forceinline__ void load_run(const S* __restrict__ p, float* out) {
    S tmp[V];
    __builtin_memcpy(tmp, p, sizeof(S) * V);
#pragma unroll
    for (int k = 0; k < V; ++k) out[k] = Cvt<S>::ld(tmp[k]);
}

// V consecutive elements to a V-element-aligned address.
template <class S, int V>
__device__ __forceinline__ void store_run(S* __restrict__ p, const float* v, int nontemporal) {
    S tmp[V];
#pragma unroll
    for (int k = 0; k < V; ++k) tmp[k] = Cvt<S>::st(v[k]);
    typedef typename RawT<sizeof(S) * V>::T R;
    R raw;
    __builtin_memcpy(&raw, tmp, sizeof(R));
    R* q = reinterpret_cast<R*>(p);
    if (nontemporal)
        __builtin_nontemporal_store(raw, q);
    else
        *q = raw;
}

// ------------------------------------------------------------------ physics

// Weights of Eq. 17 in FP32.
#define W_AXIS 0.222222222222222222f   // 2/9
#define W_DIAG 0.027777777777777778f   // 1/36

// Relaxation of one node (Eq. 13 right-hand side with Eqs. 15-16, dt = c = 1)
// in g-form, applied in the operator's eigen-decomposition.  With
// E = sum g, j = sum c_i g (Eqs. 53-54 up to the factor beta), the flux share
// f_i = (5 a_i / 3) c_i . j and the remainder h_i = g_i - omega_i E - f_i,
// Eqs. 13, 15 and 16 give
//     g*_i = omega_i E + rho f_i + (1 - 1/tau) h_i
//          = g_i - (1/tau) h_i - (1 - rho) f_i,
// rho = (2 tau_r - 1)/(2 tau_r + 1): energy is kept, the heat flux decays by
// rho per step, everything else by 1 - 1/tau.  Writing it this way keeps the
// small per-step flux decay 1 - rho = 2/(2 tau_r + 1) as its own coefficient
// (rounded once): forming it as the difference of two FP32 coefficients of
// order 1 loses ~5 digits when tau_r ~ 1e3.  The equilibrium energy share is
// split so that 4 ea + 4 ed == E holds exactly (E - 4 ea is exact by
// Sterbenz' lemma).  The library is built with contraction off and the fused
// multiply-adds are written out, so every kernel instance produces the same
// bits.
#define W_FA 0.333333333333333333f      // 5 a_i / 3, axis directions
#define W_FD 0.083333333333333333f      // 5 a_i / 3, diagonal directions

__device__ __forceinline__ void relax_parts(const float g[8], float e[8], float fl[8]) {
    const float E = ((g[0] + g[2]) + (g[1] + g[3])) + ((g[4] + g[6]) + (g[5] + g[7]));
    // (g5 - g7) = -(g7 - g5) and 4 ea is exact, so the shared difference and
    // the fused form below round exactly as the plain expressions
    const float d46 = g[4] - g[6], d75 = g[7] - g[5];
    const float jx = ((g[0] - g[2]) + d46) + d75;
    const float jy = ((g[1] - g[3]) + d46) - d75;
    const float ea = W_AXIS * E;
    const float ed = __builtin_fmaf(-4.0f, ea, E) * 0.25f;
    const float fx = W_FA * jx, fy = W_FA * jy;
    const float fp = W_FD * (jx + jy), fm = W_FD * (jx - jy);
    fl[0] = fx;  fl[1] = fy;  fl[2] = -fx;  fl[3] = -fy;
    fl[4] = fp;  fl[5] = -fm; fl[6] = -fp;  fl[7] = fm;
#pragma unroll
    for (int i = 0; i < 8; ++i) e[i] = i < 4 ? ea : ed;
}

// x component of velocity i (directions 0..7 are the paper's 1..8 of Eq. 14).
__device__ __forceinline__ constexpr int vel_x(int i) {
    return (i == 0 || i == 4 || i == 7) ? 1 : ((i == 2 || i == 5 || i == 6) ? -1 : 0);
}

// c_ix times a per-class value (axis / diagonal); a compile-time select once
// the direction loop is unrolled, so directions with c_ix = 0 get an exact 0.
__device__ __forceinline__ float cx_times(int i, float va, float vd) {
    const float v = i < 4 ? va : vd;
    return vel_x(i) > 0 ? v : (vel_x(i) < 0 ? -v : 0.0f);
}

// Reference-state values a kernel needs per instance (see RefState).
struct RefView {
    float force_a, force_d, shift_a, shift_d, wall_kd;
};
__device__ __forceinline__ RefView ref_view(const RefState& r) {
    return RefView{r.force_a, r.force_d, r.shift_a, r.shift_d, r.wall_kd};
}

// Per-step change of population i: -(1/tau) h_i - (1 - rho) f_i plus the
// reference state's forcing, formed at the size of the change itself and
// added to g once.
__device__ __forceinline__ void relax_delta(const float g[8], const InstDesc& d, const RefView& rv,
                                            float delta[8], float e[8]) {
    float fl[8];
    relax_parts(g, e, fl);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        // h_i = (g_i - omega_i E) - f_i: the first difference nearly cancels,
        // so h_i carries the rounding of f_i, not of the energy share
        const float force = cx_times(i, rv.force_a, rv.force_d);
        delta[i] = __builtin_fmaf(-d.sigma, fl[i], __builtin_fmaf(-d.inv_tau, (g[i] - e[i]) - fl[i], force));
    }
}
__device__ __forceinline__ void relax_delta(const float g[8], const InstDesc& d, const RefView& rv,
                                            float delta[8]) {
    float e[8];
    relax_delta(g, d, rv, delta, e);
}

__device__ __forceinline__ void relax(float g[8], const InstDesc& d, const RefView& rv) {
    float delta[8];
    relax_delta(g, d, rv, delta);
#pragma unroll
    for (int i = 0; i < 8; ++i) g[i] = g[i] + delta[i];
}

// The same relaxation with the flux decay and the forcing folded into one
// term per opposite pair: g_i + fma(-1/tau, g_i - omega_i E, k_i), k_i =
// (1/tau - (1 - rho)) f_i + forcing_i.  Fewer operations (about a fifth of a
// stage's), but k_i is rounded at the scale of the flux share, not of the
// change, so the small flux decay 1 - rho loses digits when tau_r is large:
// used only for the steps a 16-bit launch keeps in FP32 registers, where that
// error is far below the 16-bit rounding of the state it stores.
__device__ __forceinline__ void relax_folded(float g[8], const InstDesc& d, const RefView& rv) {
    const float E = ((g[0] + g[2]) + (g[1] + g[3])) + ((g[4] + g[6]) + (g[5] + g[7]));
    const float d46 = g[4] - g[6], d75 = g[7] - g[5];
    const float jx = ((g[0] - g[2]) + d46) + d75;
    const float jy = ((g[1] - g[3]) + d46) - d75;
    const float ea = W_AXIS * E;
    const float ed = __builtin_fmaf(-4.0f, ea, E) * 0.25f;
    const float k0 = __builtin_fmaf(d.flux_a, jx, rv.force_a);
    const float k1 = d.flux_a * jy;
    const float k4 = __builtin_fmaf(d.flux_d, jx + jy, rv.force_d);
    const float k7 = __builtin_fmaf(d.flux_d, jx - jy, rv.force_d);
    const float k[8] = {k0, k1, -k0, -k1, k4, -k7, -k4, k7};
#pragma unroll
    for (int i = 0; i < 8; ++i) g[i] = g[i] + __builtin_fmaf(-d.inv_tau, g[i] - (i < 4 ? ea : ed), k[i]);
}

// Pending change of reference flux: the pulled values are re-expressed
// against the new reference (a uniform c_ix w_i (J_old - J_new) / s).
__device__ __forceinline__ void apply_shift(float g[8], const RefView& rv) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if (vel_x(i) != 0) g[i] = g[i] + cx_times(i, rv.shift_a, rv.shift_d);
}

// FP64 moments of a pulled node (Eqs. 53-54) for the check-step snapshot and
// residual: E = sum g, dT = s E / C_V, q = q_ref + s beta j.
__device__ __forceinline__ void node_moments_f64(const float g[8], const InstDesc& d, double q_ref, double& E,
                                                 double& dT, double& qx, double& qy) {
    E = 0.0;
#pragma unroll
    for (int i = 0; i < 8; ++i) E += (double)g[i];
    const double jx = ((double)g[0] - (double)g[2]) + ((double)g[4] - (double)g[6]) + ((double)g[7] - (double)g[5]);
    const double jy = ((double)g[1] - (double)g[3]) + ((double)g[4] - (double)g[6]) + ((double)g[5] - (double)g[7]);
    dT = d.s_cv * E;
    qx = q_ref + d.s_beta * jx;
    qy = d.s_beta * jy;
}

// Relaxation with stochastic rounding of the stored result (FP32 storage):
// the change is added to g_i with sr_add_f32.  16-bit storage narrows the
// round-to-nearest FP32 result of relax() stochastically instead.
__device__ __forceinline__ void relax_sr_f32(const float g[8], const InstDesc& d, const RefView& rv,
                                             const uint32_t r[4], float out[8]) {
    float delta[8];
    relax_delta(g, d, rv, delta);
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = sr_add_f32(g[i], delta[i], bits16(r, i));
}

// Boundary treatment after advection (Sec. 2.5) on one node, given its
// position and the reference's diagonal offset kd = p_diag / s.  Directions 0..7 are the paper's 1..8.  Written with selects only:
// every write has a fixed index, so the eight values stay in registers.
//   diffuse (Eq. 58): the three populations leaving a wall get 4/5, 1/10, 1/10
//     (omega_i over the sum of the leaving omegas) of the incident sum S; the
//     axis share is formed as S - 2 (S/10) so the three add up to S;
//   heat flux (Eq. 57): the same with S raised by q_0 / beta (wall_q, 0 for a
//     diffuse wall);
//   isothermal (Eq. 55): all eight take omega_i C_V (T_s - T_ref) / s.
// BRANCH: branch over the treatments that neither wall of an axis needs (the
// kinds are the same for every node); the block kernels gain 8% on isothermal
// walls, the marching kernel's register allocation does not take the branches.
// Each wall has its own kind (InstDesc::wk); walls on both axes occur only
// with isothermal x walls, which own the corner nodes.
template <int BRANCH = 0>
__device__ __forceinline__ void boundary(float g[8], const InstDesc& d, float kd, int x, int y) {
    if (d.bc_y != 0) {
        // walls y = 0 and y = ny-1, each of its own kind (wk[2], wk[3])
        const bool lo = (y == 0), hi = (y == d.ny - 1);
        const int kl = d.wk[2], kh = d.wk[3];
        if (!BRANCH || kl > 1 || kh > 1) {
            const bool rl = lo && (kl == 2 || kl == 4), rh = hi && (kh == 2 || kh == 4);
            const float Sl = (g[3] + g[6] + g[7]) + d.wall_q[2];      // incident at y = 0: 4, 7, 8
            const float Sh = (g[1] + g[4] + g[5]) + d.wall_q[3];      // incident at y = ny-1: 2, 5, 6
            const float dl = 0.1f * Sl, dh = 0.1f * Sh;
            const float al = Sl - dl - dl, ah = Sh - dh - dh;
            // the reference state's diagonal shares (c_ix p_diag) are not part of
            // the reflected energy: the leaving diagonals carry -c_ix p_diag / s
            const float k = kd;
            g[1] = rl ? al : g[1];  g[4] = rl ? dl - k : g[4];  g[5] = rl ? dl + k : g[5];
            g[3] = rh ? ah : g[3];  g[6] = rh ? dh + k : g[6];  g[7] = rh ? dh - k : g[7];
        }
        if (!BRANCH || kl == 1 || kh == 1) {
            const bool w = (lo && kl == 1) || (hi && kh == 1);
            const float t = lo ? d.wall_g[2] : d.wall_g[3];
            const float a = W_AXIS * t, b = W_DIAG * t;
#pragma unroll
            for (int i = 0; i < 8; ++i) g[i] = w ? (i < 4 ? a : b) : g[i];
        }
    }
    if (d.bc_x == 1 || d.bc_x == 2 || d.bc_x == 4) {
        // walls x = 0 and x = nx-1 (wk[0], wk[1]); applied after the y walls,
        // so isothermal x walls own the corner nodes
        const bool lo = (x == 0), hi = (x == d.nx - 1);
        const int kl = d.wk[0], kh = d.wk[1];
        if (!BRANCH || kl > 1 || kh > 1) {
            const bool rl = lo && (kl == 2 || kl == 4), rh = hi && (kh == 2 || kh == 4);
            const float Sl = (g[2] + g[5] + g[6]) + d.wall_q[0];      // incident at x = 0: 3, 6, 7
            const float Sh = (g[0] + g[4] + g[7]) + d.wall_q[1];      // incident at x = nx-1: 1, 5, 8
            const float dl = 0.1f * Sl, dh = 0.1f * Sh;
            const float al = Sl - dl - dl, ah = Sh - dh - dh;
            g[0] = rl ? al : g[0];  g[4] = rl ? dl : g[4];  g[7] = rl ? dl : g[7];
            g[2] = rh ? ah : g[2];  g[5] = rh ? dh : g[5];  g[6] = rh ? dh : g[6];
        }
        if (!BRANCH || kl == 1 || kh == 1) {
            const bool w = (lo && kl == 1) || (hi && kh == 1);
            const float t = lo ? d.wall_g[0] : d.wall_g[1];
            const float a = W_AXIS * t, b = W_DIAG * t;
#pragma unroll
            for (int i = 0; i < 8; ++i) g[i] = w ? (i < 4 ? a : b) : g[i];
        }
    }
}


// x shift of the source of direction i (pull from x - c_ix), and the row of the
// source: 0 = y, 1 = y - 1 (c_iy = +1), 2 = y + 1 (c_iy = -1).  Compile-time
// functions, so unrolled loops fold them into immediates.
__device__ __forceinline__ constexpr int src_dx(int i) {
    return (i == 0 || i == 4 || i == 7) ? -1 : ((i == 2 || i == 5 || i == 6) ? 1 : 0);
}
__device__ __forceinline__ constexpr int src_row(int i) {
    return (i == 1 || i == 4 || i == 5) ? 1 : ((i == 3 || i == 6 || i == 7) ? 2 : 0);
}

// V elements starting at x0 + dx, given p0 = the address of x0 (V-aligned,
// so the dx == 0 run is V-element aligned).  FP32: one wide load, dword
// aligned.  16-bit storage: the aligned run at x0 plus one aligned pair on
// the side the shift reaches into, so no access is below dword alignment.
// Caller guarantees the touched elements are in range and in one chunk:
// [x0 + dx, x0 + V - 1 + dx] (FP32), [x0 - 2, x0 + V - 1] or [x0, x0 + V + 1]
// (16-bit, dx = -1 / +1).
template <class S, int V>
__device__ __forceinline__ void load_shifted(const S* __restrict__ p0, int dx, float* out) {
    if (dx == 0 || sizeof(S) == 4 || V == 1) {
        load_run<S, V>(p0 + dx, out);
        return;
    }
    float a[V], b[2];
    load_run<S, V>(p0, a);
    if (dx < 0) {
        load_run<S, 2>(p0 - 2, b);
        out[0] = b[1];
#pragma unroll
        for (int k = 1; k < V; ++k) out[k] = a[k - 1];
    } else {
        load_run<S, 2>(p0 + V, b);
#pragma unroll
        for (int k = 0; k < V - 1; ++k) out[k] = a[k + 1];
        out[V - 1] = b[0];
    }
}

// Offset of column x within a row (layout-independent).
__device__ __forceinline__ int64_t col_off(const InstDesc& d, int x) {
    return (int64_t)(x >> d.cshift) * d.chunk + (x & d.cmask);
}

// Periodic wrap of a column index that is at most one period out of range.
__device__ __forceinline__ int wrapx(int x, int nx) {
    return x < 0 ? x + nx : (x >= nx ? x - nx : x);
}

// Compensated additions (see DD): the exact rounding error of hi + b (Knuth's
// two-sum, exact with contraction off) is carried into lo, then the pair is
// renormalised.  dd_add(a, b) == dd_add(b, a).
__device__ __forceinline__ DD dd_renorm(double s, double t) {
    const double hi = s + t;
    return DD{hi, t - (hi - s)};
}
__device__ __forceinline__ DD dd_add(DD a, double b) {
    const double s = a.hi + b;
    const double bp = s - a.hi;
    const double e = (a.hi - (s - bp)) + (b - bp);
    return dd_renorm(s, e + a.lo);
}
__device__ __forceinline__ DD dd_add(DD a, DD b) {
    const double s = a.hi + b.hi;
    const double bp = s - a.hi;
    const double e = (a.hi - (s - bp)) + (b.hi - bp);
    return dd_renorm(s, e + (a.lo + b.lo));
}
__device__ __forceinline__ DD dd_zero() { return DD{0.0, 0.0}; }

// Add one node's check-step values (energy, heat flux, squared change and
// squared size of m = (dT, qx, qy) against the previous step's p) to a lane's
// sums.  The x-flux total decides the reference-flux rebase and is summed
// compensated from the first node on; the others, only reported, are plain
// FP64 per lane (lo stays 0) and compensated from the lane sums on.
__device__ __forceinline__ void check_sums(DD acc[kPartials], double e, double qx, double qy, double dT, double p0,
                                           double p1, double p2) {
    acc[0].hi += e;
    acc[1] = dd_add(acc[1], qx);
    acc[2].hi += qy;
    acc[3].hi += (dT - p0) * (dT - p0) + (qx - p1) * (qx - p1) + (qy - p2) * (qy - p2);
    acc[4].hi += dT * dT + qx * qx + qy * qy;
}

// Sums of kPartials values over the wavefront's lanes (a butterfly, the same
// order on every lane): the values' additions are independent, so each
// round's lane exchanges and dependent FP64 chains overlap.
__device__ __forceinline__ void wave_sums(DD v[kPartials]) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        DD o[kPartials];
#pragma unroll
        for (int c = 0; c < kPartials; ++c) o[c] = DD{__shfl_xor(v[c].hi, off, 64), __shfl_xor(v[c].lo, off, 64)};
#pragma unroll
        for (int c = 0; c < kPartials; ++c) v[c] = dd_add(v[c], o[c]);
    }
}

// Sum kPartials compensated values over the block in a fixed order; thread c
// adds up and writes value c (one thread for all of them took 3 us of a check
// launch of 16 wavefronts: dependent FP64 additions).
__device__ __forceinline__ void block_partials(DD v[kPartials], DD* out) {
    __shared__ DD red[1024 / 64][kPartials];
    const int tid = threadIdx.y * blockDim.x + threadIdx.x;
    const int lane = tid & 63, wid = tid >> 6;
    const int nw = (blockDim.x * blockDim.y + 63) >> 6;
    wave_sums(v);
    if (lane == 0) {
#pragma unroll
        for (int c = 0; c < kPartials; ++c) red[wid][c] = v[c];
    }
    __syncthreads();
    if (tid < kPartials) {
        DD s = dd_zero();
        for (int w = 0; w < nw; ++w) s = dd_add(s, red[w][tid]);
        out[tid] = s;
    }
}

// Split storage (16-bit h_i = g_i - omega_i E plus FP32 E per node): within a
// 64-node chunk the eight h runs come first, then the E run, at this element
// offset (elements of the 16-bit type).
constexpr int kSplitE = 512;

// omega_i E with the energy-exact split used by the relaxation (4 ea + 4 ed
// equals E exactly): the equilibrium part of population i at energy E.
__device__ __forceinline__ float omega_e(int i, float E) {
    const float ea = W_AXIS * E;
    return i < 4 ? ea : (E - 4.0f * ea) * 0.25f;
}

// Byte offset, within a row, of the FP32 energy of node x (split storage).
__device__ __forceinline__ uint32_t e_off(const InstDesc& d, int x) {
    return (uint32_t)(((x >> 6) * d.chunk + kSplitE) * 2 + (x & 63) * 4);
}

// Whole-wave lane shifts (DPP wave_shr:1 / wave_shl:1): lane i receives v of
// lane i - 1 (from_left) or i + 1 (from_right); the lane with no source (0,
// resp. 63) keeps `edge`.  All 64 lanes must be active.
__device__ __forceinline__ float from_left(float v, float edge) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_right(float v, float edge) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xf, 0xf, false));
}

// v rounded to S: to nearest, or (SR, 16-bit) stochastically with 16 random bits.
template <class S, int SR>
__device__ __forceinline__ S round_to(float v, uint32_t r16) {
    if constexpr (SR && __is_same(S, _Float16)) return sr_f16(v, r16);
    else if constexpr (SR && __is_same(S, bf16_bits)) return sr_bf16(v, r16);
    else return Cvt<S>::st(v);
}

template <class S>
__device__ __forceinline__ void store_raw(char* p, S o, int nontemporal) {
    typedef typename RawT<sizeof(S)>::T R;
    R raw;
    __builtin_memcpy(&raw, &o, sizeof(R));
    R* q = reinterpret_cast<R*>(p);
    if (nontemporal) __builtin_nontemporal_store(raw, q);
    else *q = raw;
}

// Random words of the stochastic-rounding stores.  Word k (16 bits for each
// of directions 2k and 2k + 1) of node (x, y) at step n is
//     col_word_k(x) ^ (row_word(y, n) * m_k),
// col_word_k a hash of the column keyed by (k, seed), row_word a hash of the
// global index of the row's first node keyed by (n, seed), m_k fixed odd
// multipliers (m_0 = 1, a bijection of the row word).  Every word is uniform
// and independent of the value it rounds (each rounding stays unbiased) and of
// the words of other rows and steps; in one row and step, two columns' words
// differ by a fixed pattern.  A pure function of (x, y, n, seed): every kernel
// and schedule draws the same bits.  A wavefront that marches along y hashes
// its columns once and each row once on the scalar unit.
__device__ __forceinline__ uint32_t sr_col_word(uint32_t x, int k, uint32_t seed) {
    return mix32(x ^ mix32(seed * 0x9e3779b9u + 0x632be5abu * (uint32_t)(k + 1)));
}
__device__ __forceinline__ uint32_t sr_row_word(uint32_t row_node, uint32_t step, uint32_t seed) {
    return mix32(row_node ^ mix32(step * 0x85ebca6bu + seed * 0x9e3779b9u));
}
__device__ __forceinline__ void sr_words(uint32_t r[4], const uint32_t colw[4], uint32_t roww) {
    r[0] = colw[0] ^ roww;
    r[1] = colw[1] ^ (roww * 0x2c1b3c6du);
    r[2] = colw[2] ^ (roww * 0x297a2d39u);
    r[3] = colw[3] ^ (roww * 0x846ca68bu);
}

template <class S, int SR>
__device__ __forceinline__ void store_one(char* p, float v, uint32_t r16, int nontemporal) {
    store_raw<S>(p, round_to<S, SR>(v, r16), nontemporal);
}

// y component of velocity i.
__device__ __forceinline__ constexpr int vel_y(int i) {
    return (i == 1 || i == 4 || i == 5) ? 1 : ((i == 3 || i == 6 || i == 7) ? -1 : 0);
}

// Periodic image of v on 0..n-1; v is at most one period outside when
// n >= span (the window's extent), else it may wrap several times.
__device__ __forceinline__ int wrapm(int v, int n, int span) {
    if (n >= span) return v < 0 ? v + n : (v >= n ? v - n : v);
    const int r = v % n;
    return r < 0 ? r + n : r;
}

// Relaxation of node g and its rounding to the storage type, exactly as the
// single-step kernels store it: o (raw values), E (FP32 energy, split only).
template <class S, int SR, int SPLIT>
__device__ __forceinline__ void relax_round(float g[8], const InstDesc& d, const RefView& rv, const uint32_t r[4],
                                            S o[8], float& E_out) {
    if constexpr (SPLIT) {
        float delta[8], e[8], hv[8];
        relax_delta(g, d, rv, delta, e);
        const float E = ((g[0] + g[2]) + (g[1] + g[3])) + ((g[4] + g[6]) + (g[5] + g[7]));
#pragma unroll
        for (int i = 0; i < 8; ++i) hv[i] = (g[i] - e[i]) + delta[i];
        round_pairs<S, SR, 8>(hv, r, o);
        float res = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; ++i) res = res + (hv[i] - Cvt<S>::ld(o[i]));
        E_out = E + res;
    } else if constexpr (SR && sizeof(S) == 4) {
        float f[8];
        relax_sr_f32(g, d, rv, r, f);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = Cvt<S>::st(f[i]);
        E_out = 0.0f;
    } else {
        relax(g, d, rv);
        if constexpr (SR && __is_same(S, bf16_bits)) {
            // one finiteness test per node (the sum of the eight is finite only
            // if all are) instead of a NaN select per value; same bits
            const float t = ((g[0] + g[1]) + (g[2] + g[3])) + ((g[4] + g[5]) + (g[6] + g[7]));
            if (fabsf(t) <= 3.402823466e38f) {
#pragma unroll
                for (int i = 0; i < 8; ++i) o[i].b = (uint16_t)((__float_as_uint(g[i]) + bits16(r, i)) >> 16);
            } else {
                round_pairs<S, SR, 8>(g, r, o);
            }
        } else {
            round_pairs<S, SR, 8>(g, r, o);
        }
        E_out = 0.0f;
    }
}

// The populations the next step reads back from a stored node.
template <class S, int SPLIT>
__device__ __forceinline__ void reload(const S o[8], float E, float out[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = SPLIT ? Cvt<S>::ld(o[i]) + omega_e(i, E) : Cvt<S>::ld(o[i]);
}

__device__ __forceinline__ bool on_wall(const InstDesc& d, int x, int y) {
    return ((d.bc_y != 0) && (y == 0 || y == d.ny - 1)) ||
           ((d.bc_x == 1 || d.bc_x == 2 || d.bc_x == 4) && (x == 0 || x == d.nx - 1));
}

// Directions by c_y: -1 {3, 6, 7}, 0 {0, 2}, +1 {1, 4, 5}.
__device__ __forceinline__ constexpr int ymid(int k) { return 2 * k; }
__device__ __forceinline__ constexpr int yup(int k) { return k == 0 ? 1 : 3 + k; }
__device__ __forceinline__ constexpr int ydown(int k) { return k == 0 ? 3 : 5 + k; }

// v of the lane at x - c_ix (the pull along x); all 64 lanes active.
template <int I>
__device__ __forceinline__ float xpull(float v) {
    if constexpr (vel_x(I) > 0) return from_left(v, v);
    else if constexpr (vel_x(I) < 0) return from_right(v, v);
    else return v;
}

// Pulled populations of one stage: direction i from the row at y - c_iy
// (dn: the newest row, mid: one row back, up: two rows back), shifted by c_ix
// (UP_SHIFTED: up is given shifted).
template <int UP_SHIFTED = 0>
__device__ __forceinline__ void march_gather(const float dn_row[8], const float mid[2], const float up[3], float g[8]) {
    g[0] = xpull<0>(mid[0]);
    g[2] = xpull<2>(mid[1]);
    g[1] = up[0];
    g[4] = UP_SHIFTED ? up[1] : xpull<4>(up[1]);
    g[5] = UP_SHIFTED ? up[2] : xpull<5>(up[2]);
    g[3] = dn_row[3];
    g[6] = xpull<6>(dn_row[6]);
    g[7] = xpull<7>(dn_row[7]);
}

}  // namespace plbm
