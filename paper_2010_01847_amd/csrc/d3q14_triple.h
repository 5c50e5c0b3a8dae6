// Three FP32 steps per launch (included by the D3Q14 device file, which holds
// the node functions).
#pragma once

// Temporal blocking of three steps in one pass over HBM.  A block of kDeepWaves
// wavefronts owns a window of 64 x (kDeepWaves * kDeepRows) nodes of every
// plane of a z range (a halo of three nodes in x and y around its outputs, each
// position mapped to its periodic image) and marches along z.  Wavefront w
// holds kDeepRows adjacent rows, one column per lane.  Iteration `it` loads
// input plane zi = z0 - 3 + it and runs three stages: stage s advances plane
// zi - s from the planes of level s - 1 (level 0: loaded planes, level s:
// planes advanced s steps); stage 3 stores its outputs.  A node pulls
// direction i from the plane z - c_iz, so of a level's newest plane the movers
// with c_z = -1 are needed at once, those with c_z = 0 one iteration later and
// those with c_z = +1 two iterations later: delay lines in registers.  Along x
// the pull comes from the adjacent lanes (DPP); along y from the wavefront's
// own rows and, at its first and last, from the neighbouring wavefronts through
// LDS: five populations each way and stage, two slots in turn, so one barrier
// per stage.  Level s is valid s nodes inside the window from iteration 2 s on.
// Per node and step the arithmetic is the single-step kernel's (same functions,
// same order, same random bits), so the result equals three single steps bit
// for bit.
//
// Why not the two-step kernel's way (the whole window in LDS): a window row
// costs 14 words of LDS per stage there, so three stages of it leave too few
// output rows; here LDS holds only the rows that cross wavefronts, and two rows
// per wavefront halve those (12 waves, 60 KB of LDS, all 168 VGPRs that three
// waves per SIMD leave; four of them spill in the chunked layout, ten in planes,
// 14 and 19 with stochastic rounding).  Bound by HBM and the caches (64 x 24
// nodes loaded for 58 x 18 stored): 512^3 runs 1716 us per step against 1884 in launches of
// two and 2670 in single steps, on another card 1622 against 1745.  16-bit
// storage stays with two steps: there this kernel's arithmetic costs more than
// the traffic it saves (512^3 at two steps per launch 1391 .. 1450 against 1251
// .. 1309 us).
constexpr int kK = kDeepSteps, kR = kDeepRows, kNW = kDeepWaves;

// Index of a direction in its delay line (c_z = 0: 0..3; c_z = +1: 4, 6, ..),
// and the directions with c_y = +1 and -1 and their index there.
__host__ __device__ constexpr int at_up(int i) { return i == 4 ? 0 : i - 5; }
__host__ __device__ constexpr int dir_yp(int k) { return k == 0 ? 2 : (k < 3 ? 5 + k : 7 + k); }
__host__ __device__ constexpr int dir_ym(int k) { return k == 0 ? 3 : (k < 3 ? 7 + k : 9 + k); }
__host__ __device__ constexpr int at_y(int i) { return i < 4 ? 0 : (i < 10 ? 1 + (i & 1) : 3 + (i & 1)); }
constexpr bool delay_tables_ok() {
    for (int k = 0; k < 5; ++k)
        if (cy(dir_yp(k)) != 1 || cy(dir_ym(k)) != -1 || at_y(dir_yp(k)) != k || at_y(dir_ym(k)) != k ||
            cz(dir_up(k)) != 1 || at_up(dir_up(k)) != k)
            return false;
    for (int k = 0; k < 4; ++k)
        if (dir_mid(k) != k || cz(k) != 0) return false;
    return true;
}
static_assert(delay_tables_ok(), "delay lines");

// v of the lane at x - c_ix (whole-wave lane shift; the lane with no source
// keeps its own value, which no output uses).
template <int I>
__device__ __forceinline__ float pull_x(float v) {
    const int u = __float_as_int(v);
    if constexpr (cx(I) > 0) return __int_as_float(__builtin_amdgcn_update_dpp(u, u, 0x138, 0xf, 0xf, false));
    else if constexpr (cx(I) < 0) return __int_as_float(__builtin_amdgcn_update_dpp(u, u, 0x130, 0xf, 0xf, false));
    else return v;
}

// A level's earlier planes held by a wavefront: the c_z = 0 movers of the one
// before the newest, and the c_z = +1 movers of the two before.
struct Level {
    float mid[kR][4], up1[kR][5], up2[kR][5];
};

// Direction I of row r of a level as the next stage pulls it.
template <int I>
__device__ __forceinline__ float level_at(const float cur[kR][kQ], const Level& l, int r) {
    if constexpr (cz(I) < 0) return cur[r][I];
    else if constexpr (cz(I) == 0) return l.mid[r][I];
    else return l.up2[r][at_up(I)];
}

template <int I>
__device__ __forceinline__ float pull_one(const float cur[kR][kQ], const Level& l, const float below[5],
                                          const float above[5], int r) {
    float v;
    if constexpr (cy(I) > 0) v = r > 0 ? level_at<I>(cur, l, r > 0 ? r - 1 : 0) : below[at_y(I)];
    else if constexpr (cy(I) < 0) v = r + 1 < kR ? level_at<I>(cur, l, r + 1 < kR ? r + 1 : r) : above[at_y(I)];
    else v = level_at<I>(cur, l, r);
    return pull_x<I>(v);
}

template <int... Is>
__device__ __forceinline__ void pull_row(const float cur[kR][kQ], const Level& l, const float below[5],
                                         const float above[5], int r, float v[kQ], std::integer_sequence<int, Is...>) {
    ((v[Is] = pull_one<Is>(cur, l, below, above, r)), ...);
}

// The level's values that the neighbouring wavefronts pull, to LDS.
template <int... Ks>
__device__ __forceinline__ void put_edges(const float cur[kR][kQ], const Level& l, float (*mine)[64], int lane,
                                          std::integer_sequence<int, Ks...>) {
    ((mine[Ks][lane] = level_at<dir_yp(Ks)>(cur, l, kR - 1)), ...);
    ((mine[5 + Ks][lane] = level_at<dir_ym(Ks)>(cur, l, 0)), ...);
}

// Direction i of row `row` = z ny + y at the lane's offset (lane_off), both in
// bytes: a wave-uniform base and a 32-bit lane offset (deep_fits), so that the
// 28 addresses of a plane cost scalar instructions.
template <int L>
__device__ __forceinline__ int64_t row_base(const Geometry& g, int64_t row, int i) {
    return (L == 0 ? (int64_t)i * g.plane + row * g.pitch : row * g.nseg * (kQ * kTileX) + i * kTileX) * 4;
}
template <int L>
__device__ __forceinline__ uint32_t lane_off(int x) {
    return (uint32_t)(L == 0 ? x : (x >> 6) * (kQ * kTileX) + (x & 63)) * 4u;
}

template <int SR, int L>
__global__ __launch_bounds__(64 * kNW) void triple_kernel(PairArgs a) {
    constexpr int XO = kDeepXO, YO = kDeepYO, WR = kR * kNW;
    __shared__ float edge[2][kNW][10][64];    // c_y = +1 movers of a wavefront's last row, -1 movers of its first
    const Geometry& g = a.g;
    const uint32_t per = (a.ntiles + 7u) >> 3;
    const uint32_t tile = (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
    if (tile >= a.ntiles) return;             // whole block: no barrier is skipped by part of it
    const uint32_t tx = tile % a.ptx;
    const uint32_t rr = tile / a.ptx;
    const uint32_t ty = rr % a.pty;
    const uint32_t tz = rr / a.pty;
    const int x0 = (int)tx * XO, y0 = (int)ty * YO, z0 = (int)tz * a.zchunk;
    const int zend = min(z0 + a.zchunk, g.nz);
    const int iters = zend - z0 + 2 * kK;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const char* __restrict__ src = reinterpret_cast<const char*>(a.src);
    char* __restrict__ dst = reinterpret_cast<char*>(a.dst);
    uint32_t slot = 0;
    const int gx = wrap_mod(x0 - kK + lane, g.nx);
    const uint32_t lo = lane_off<L>(gx);      // an output lane stores at the column it loads
    const bool out_lane = lane >= kK && lane < 64 - kK && x0 + lane - kK < g.nx;
    int gy[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) gy[r] = wrap_mod(y0 - kK + wv * kR + r, g.ny);
    uint32_t colw[7] = {0u, 0u, 0u, 0u, 0u, 0u, 0u};
    if (SR) sr_cols3(colw, (uint32_t)gx, a.seed);

    float next[kR][kQ];                       // the coming input plane, in flight
    Level lev[kK];
#pragma unroll
    for (int l = 0; l < kK; ++l)
#pragma unroll
        for (int r = 0; r < kR; ++r) {
#pragma unroll
            for (int k = 0; k < 4; ++k) lev[l].mid[r][k] = 0.0f;
#pragma unroll
            for (int k = 0; k < 5; ++k) lev[l].up1[r][k] = lev[l].up2[r][k] = 0.0f;
        }
    auto load_plane = [&](int zi) {
        const int64_t zrow = (int64_t)wrap_mod(zi, g.nz) * g.ny;
#pragma unroll
        for (int r = 0; r < kR; ++r)
#pragma unroll
            for (int i = 0; i < kQ; ++i)
                next[r][i] = *reinterpret_cast<const float*>(src + row_base<L>(g, zrow + gy[r], i) + lo);
    };
    load_plane(z0 - kK);
    for (int it = 0; it < iters; ++it) {
        const int zi = z0 - kK + it;
        float cur[kR][kQ];
#pragma unroll
        for (int r = 0; r < kR; ++r)
#pragma unroll
            for (int i = 0; i < kQ; ++i) cur[r][i] = next[r][i];
        load_plane(min(zi + 1, zend + kK - 1));
#pragma unroll
        for (int s = 1; s <= kK; ++s) {
            Level& l = lev[s - 1];
            put_edges(cur, l, edge[slot][wv], lane, std::make_integer_sequence<int, 5>{});
            __syncthreads();
            // the window's first and last rows are never pulled into a valid
            // row: any value will do there
            float below[5], above[5];
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                below[k] = edge[slot][wv > 0 ? wv - 1 : 0][k][lane];
                above[k] = edge[slot][wv + 1 < kNW ? wv + 1 : wv][5 + k][lane];
            }
            slot ^= 1u;
            float out[kR][kQ];
#pragma unroll
            for (int r = 0; r < kR; ++r)
#pragma unroll
                for (int i = 0; i < kQ; ++i) out[r][i] = 0.0f;
            if (it >= 2 * s) {
                const int zs = s < kK ? wrap_mod(zi - s, g.nz) : zi - s;
#pragma unroll
                for (int r = 0; r < kR; ++r) {
                    float v[kQ];
                    pull_row(cur, l, below, above, r, v, std::make_integer_sequence<int, kQ>{});
                    float E, jx, jy, jz;
                    moments(v, E, jx, jy, jz);
                    uint32_t w[7] = {0u, 0u, 0u, 0u, 0u, 0u, 0u};
                    if (SR)
                        sr_words3(w, colw, sr_row_word3((uint32_t)zs * (uint32_t)g.ny + (uint32_t)gy[r],
                                                        a.step + (uint32_t)(s - 1), a.seed));
                    relax_round_all<float, SR>(a.c, v, a.c.omega_axis * E, a.c.omega_corner * E, jx, jy, jz, w, out[r],
                                               std::make_integer_sequence<int, kQ>{});
                    const int wr = wv * kR + r;
                    if (s == kK && out_lane && wr >= kK && wr < WR - kK && y0 + wr - kK < g.ny) {
#pragma unroll
                        for (int i = 0; i < kQ; ++i)
                            put<float>(reinterpret_cast<float*>(dst + row_base<L>(g, (int64_t)zs * g.ny + gy[r], i) + lo),
                                       out[r][i], a.nontemporal);
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < kR; ++r) {
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    l.up2[r][k] = l.up1[r][k];
                    l.up1[r][k] = cur[r][dir_up(k)];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) l.mid[r][k] = cur[r][k];
#pragma unroll
                for (int i = 0; i < kQ; ++i) cur[r][i] = out[r][i];
            }
        }
    }
}

hipError_t launch_triple(int sr, const PairArgs& a, hipStream_t st) {
    if (a.ntiles == 0) return hipSuccess;
    const dim3 grid(8u * ((a.ntiles + 7u) / 8u)), block(64 * kNW);
    if (a.g.layout)
        if (sr) hipLaunchKernelGGL((triple_kernel<1, 1>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((triple_kernel<0, 1>), grid, block, 0, st, a);
    else if (sr) hipLaunchKernelGGL((triple_kernel<1, 0>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((triple_kernel<0, 0>), grid, block, 0, st, a);
    return hipGetLastError();
}
