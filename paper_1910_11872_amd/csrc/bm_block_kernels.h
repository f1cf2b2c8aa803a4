// Block windows (the paper's L x L moving window, Sec. 3) for gfx950.
//
// block_tile_kernel: one block of 256 lanes owns a tile of 16 x 16 pixels, one
// pixel per lane.  The (16 + L - 1)^2 samples its windows cover are staged in
// LDS once.  With R_y[i][j] = sum_k G[r+i][c+k] conj(G[r+j][c+k]) (Eq. 4, the
// window's columns as snapshots) the covariance of the window at (r, c) is a
// table look-up, R_y[i][i+d] = S_d(r+i, c), of the row-wise lag sums
//   S_d(r, c) = sum_{k<L} G[r][c+k] conj(G[r+d][c+k]),
// which the windows above and below share; likewise for omega_x with rows and
// columns exchanged, R_x[i][i+d] = sum_k G[r+k][c+i] conj(G[r+k][c+i+d]).  So
// a window costs about L sums of L products per direction instead of L (L+1)/2
// of them, and neighbouring sums share most of their terms as well (below).
// The lag sums of one direction at a time live in LDS.
//
// What bounds it: VALU issue, with the LDS reads of the lag sums (L (L+1)/2
// per window and direction) beside it at about half their rate's limit.
// Measured against summing each window's T from its own snapshots, on 20
// frames of 1024 x 1024 with 11 x 11 blocks 4.25 -> 1.58 ms, one 1850 x 700
// frame with 15 x 15 blocks and the phase 0.96 -> 0.26 (all the call's launches).
// The eigen-split's real symmetric T holds L (L+1)/2 registers, so the sizes
// above 8 x 8 keep only the common route in this kernel (power iteration, then
// the closed form of a window close to one tone, with its second expansion): at
// two to four waves per SIMD they hide the LDS latency that the one wave of the
// whole method's 512 registers cannot.  A window that this route does not prove gets a NaN of its
// own payload in its map, and block_rest_kernel, launched behind on the same
// stream, finishes exactly those with every other solver.  Up to 8 x 8 the
// whole method fits beside it and each lane finishes its window itself.
//
// With the snapshots read in increasing x (or y), omega = +arg of the selected
// root in both directions -- the paper's -arg(z_x) for its E{Gamma^H Gamma}
// form.  With both frequencies, the block phase (Eq. 15's alpha, block
// coordinates measured from the pixel) is
// arg sum_{i,j} G[i][j] e^{-j(omega_x (j-h) + omega_y (i-h))}.
#pragma once

#include "bm_rootmusic_kernels.h"

namespace bm {
namespace {

constexpr int kTile = kBlockTile;                       // pixels per side of a tile
constexpr int kTileLanes = kTile * kTile;
// NaN payload of a window left to block_rest_kernel.
constexpr unsigned kPending = 0x7FC0B10Cu;
__device__ __forceinline__ bool pending(float w) { return __float_as_uint(w) == kPending; }

template <int L>
struct BlockTile {
    static constexpr int G = kTile + L - 1;             // staged rows and columns
    static constexpr int GP = G | 1;                    // their pitch: odd, so that a column's samples
                                                        // lie on distinct LDS banks
    static constexpr int C = L >= 8 ? 8 : (L >= 4 ? 4 : 2);   // sums formed together (C <= L)
    // omega_y: lag d holds rows r < G - d, at a pitch of 17 (the lanes that
    // write run along r).  omega_x: 16 rows of G - d columns; the lags d and
    // L - 1 - d share rows of G - d + G - (L - 1 - d) = PX columns.
    static constexpr int PX = 2 * G - (L - 1);
    static constexpr int off_y(int d) { return (kTile + 1) * (d * G - d * (d - 1) / 2); }
    static constexpr int off_x(int d) {
        const int e = L - 1 - d;
        return d <= e ? d * kTile * PX : e * kTile * PX + (G - e);
    }
    static constexpr int size_x = (L + 1) / 2 * kTile * PX;
    static constexpr int size = off_y(L) > size_x ? off_y(L) : size_x;
};

// The lag sums S_d over runs of L products a_k conj(b_k), k = j .. j+L-1, for
// j = 0 .. 15: C of them at a time, each the sum of the products from its own
// start up to k = c0+L-1 (built downwards from the C-th start, which the others
// contain) and of those beyond it (built upwards): L + C - 1 products and C - 1
// additions for C sums, and no subtraction, so a sum's rounding comes from its
// own terms alone.  `a(k)`, `b(k)` return samples, `put(j, s)` stores.
template <int L, typename FA, typename FB, typename FP>
__device__ __forceinline__ void lag_runs(FA a, FB b, FP put) {
    constexpr int C = BlockTile<L>::C;
    auto add = [&](int k, float2& s) {
        const float2 p = a(k), q = b(k);
        s.x = fmaf(p.x, q.x, fmaf(p.y, q.y, s.x));
        s.y = fmaf(p.y, q.x, fmaf(-p.x, q.y, s.y));
    };
#pragma unroll
    for (int c0 = 0; c0 < kTile; c0 += C) {
        float2 low[C];
        float2 s = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = c0 + C - 1; k < c0 + L; ++k) add(k, s);
        low[C - 1] = s;
#pragma unroll
        for (int j = C - 2; j >= 0; --j) {
            add(c0 + j, s);
            low[j] = s;
        }
        float2 up = make_float2(0.f, 0.f);
        put(c0, low[0]);
#pragma unroll
        for (int j = 1; j < C; ++j) {
            add(c0 + L - 1 + j, up);
            put(c0 + j, make_float2(low[j].x + up.x, low[j].y + up.y));
        }
    }
}

// T = Q^H R_fb Q (up to the scale) from the lag sums S(d, i) = R[i][i+d] of one
// window, as build_T forms it from R: E1 = F[i][j] and E2 = F[i][L-1-j] of
// F = R + J conj(R) J give four entries of T each.  (c1r, c1i): the lag-1 sum
// sum_i conj(R[i][i+1]), whose phase starts the power iteration.
template <int L, typename FS>
__device__ __forceinline__ void T_from_lags(FS S, Sym<L>& T, float& c1r, float& c1i) {
    constexpr int m = L / 2;
    constexpr int o = L - m;
    constexpr float kSqrt2 = 1.41421356237309515f;
    c1r = 0.f;
    c1i = 0.f;
#pragma unroll
    for (int i = 0; i < m; ++i) {
#pragma unroll
        for (int j = i; j < m; ++j) {
            const float2 p = S(j - i, i), q = S(j - i, L - 1 - j);
            const float2 r = S(L - 1 - j - i, i), s = S(L - 1 - j - i, j);
            const float e1r = p.x + q.x, e1i = j == i ? 0.f : p.y + q.y;
            const float e2r = r.x + s.x, e2i = r.y + s.y;
            T.a[i][j] = e1r + e2r;
            T.a[o + i][o + j] = e1r - e2r;
            T.a[i][o + j] = e2i - e1i;
            if (j != i) T.a[j][o + i] = e2i + e1i;
            if (j == i + 1) {
                c1r += e1r;
                c1i -= e1i;
            }
            if (L - 1 - j - i == 1) {                      // even L: i = j = m - 1, the middle lag
                c1r = fmaf(0.5f, e2r, c1r);
                c1i = fmaf(-0.5f, e2i, c1i);
            }
        }
        if (L & 1) {
            const float2 p = S(m - i, i), q = S(m - i, m);
            T.a[i][m] = kSqrt2 * (p.x + q.x);
            T.a[m][o + i] = kSqrt2 * (p.y + q.y);
            if (i == m - 1) {
                c1r += p.x + q.x;
                c1i -= p.y + q.y;
            }
        }
    }
    if (L & 1) T.a[m][m] = 2.f * S(0, m).x;
}

// One direction of one window from its lag sums.  WHOLE: every solver (omega
// final); otherwise the common route alone, pending() where it does not serve.
template <int L, bool WHOLE, bool JACOBI, typename FS>
__device__ __forceinline__ void block_omega(FS S, const RootTemplate& tmpl, bool full_roots, float& omega,
                                            unsigned& flag, LaneStats& ls) {
    Sym<L> T;
    float c1r, c1i, hc, hs;
    T_from_lags<L>(S, T, c1r, c1i);
    half_angle_of(c1r, c1i, hc, hs);
    if (!trace_normalise<L>(T)) {
        flag |= BM_FLAG_UNDEFINED;
        return;
    }
    if constexpr (WHOLE) {
        window_omega_Ts<L, JACOBI>(T, hc, hs, kPowerTolBlock, tmpl, full_roots, __builtin_nanf(""), omega, flag, ls);
    } else {
        float v[L], nu, cw, sw;
        int steps = 0;
        bool ok = power_top_eigvec<L>(T, hc, hs, kPowerMinSteps, power_max_steps_big(L), kPowerTolBlock, v, steps, nu);
        if (ok) {
            guess_direction<L>(v, cw, sw);
            ok = tone_omega<L, true>(v, cw, sw, omega);
        }
        if (ok) {
            ls.counted += 1;
            ls.power += 1;
            ls.eig_its += steps;
            ls.pair_its32 += 1;
            ls.pair_its += 1;
            ls.accepted += 1;
        } else {
            omega = __uint_as_float(kPending);
        }
    }
}

// Rows i0 .. i1-1 of the block phase's sum; `at(i, j)` returns G[i][j] of the
// window, (exr, exi)[j] = e^{-j wx (j-h)}.  The hardware sine and cosine: arguments
// stay within |w| (L/2) <= 8.5 pi, where their error (~1e-6) is far below the phase
// tolerance, and the library's large-argument reduction would hold registers the
// whole kernel pays for.  The rows are not unrolled (one 1850 x 700 frame, 15 x 15:
// 295 us, 299 unrolled).
template <int L>
struct PhaseRow {
    float exr[L], exi[L];
    __device__ __forceinline__ explicit PhaseRow(float wx) {
#pragma unroll
        for (int j = 0; j < L; ++j) {
            float sn, cs;
            __sincosf(wx * (float)(j - L / 2), &sn, &cs);
            exr[j] = cs;
            exi[j] = -sn;
        }
    }
    // AHEAD: the next row's loads in flight meanwhile (samples in device memory).
    template <bool AHEAD, typename FG>
    __device__ __forceinline__ float2 sum(FG at, float wy, int i0, int i1) const {
        float ar = 0.f, ai = 0.f;
        float2 next[L];
        auto fetch = [&](int i) {
#pragma unroll
            for (int j = 0; j < L; ++j) next[j] = at(i, j);
        };
        if (AHEAD) fetch(i0);
#pragma unroll 1
        for (int i = i0; i < i1; ++i) {
            float rr = 0.f, ri = 0.f;     // sum_j G[i][j] e^{-j wx (j-h)}
            float2 row[L];
            if (!AHEAD) fetch(i);
#pragma unroll
            for (int j = 0; j < L; ++j) row[j] = next[j];
            if (AHEAD && i + 1 < i1) fetch(i + 1);
#pragma unroll
            for (int j = 0; j < L; ++j) {
                const float2 v = row[j];
                rr = fmaf(v.x, exr[j], fmaf(-v.y, exi[j], rr));
                ri = fmaf(v.x, exi[j], fmaf(v.y, exr[j], ri));
            }
            float sn, cs;
            __sincosf(wy * (float)(i - L / 2), &sn, &cs);   // times e^{-j wy (i-h)}
            ar = fmaf(rr, cs, fmaf(ri, sn, ar));
            ai = fmaf(ri, cs, fmaf(-rr, sn, ai));
        }
        return make_float2(ar, ai);
    }
};

// The block phase from the sums of the rows below L/2 and of the others: two lane
// groups may take one each, and the order is the same where one lane takes both,
// so a frame's phase does not depend on the batch that it shares a launch with.
__device__ __forceinline__ float phase_of(float2 low, float2 high) { return atan2f(low.y + high.y, low.x + high.x); }

template <int L, bool AHEAD, typename FG>
__device__ __forceinline__ float block_phase(FG at, float wx, float wy) {
    const PhaseRow<L> e(wx);
    const float2 low = e.template sum<AHEAD>(at, wy, 0, L / 2);
    return phase_of(low, e.template sum<AHEAD>(at, wy, L / 2, L));
}

// Waves per SIMD asked of the compiler: what the LDS of the blocks lets be
// resident and T's registers allow without spilling.
constexpr int block_tile_waves(int L) { return L <= 11 ? 4 : (L <= 13 ? 3 : 2); }

// Work item w: tile (w - prefix[j]) of job j, bpl tiles per row of tiles.
// BOTH: 512 lanes, 256 for each direction, each with its own lag sums in LDS;
// otherwise 256 lanes take the job's directions one after the other.
template <int L, bool STATS, bool JACOBI, bool BOTH>
__global__ __launch_bounds__(kTileLanes * (BOTH ? 2 : 1))
__attribute__((amdgpu_waves_per_eu(STATS ? (BOTH ? 2 : 1) : block_tile_waves(L))))
void block_tile_kernel(RmBatch B) {
    using BT = BlockTile<L>;
    constexpr bool kWhole = L <= kMaxL;
    constexpr int h = L / 2;
    constexpr int kLanes = kTileLanes * (BOTH ? 2 : 1);
    __shared__ float2 sg[BT::G * BT::GP];
    __shared__ float2 sS[(BOTH ? 2 : 1) * BT::size];
    const int j = find_job(B.prefix, B.njobs, blockIdx.x);
    const RmJob J = B.jobs[j];
    const int local = blockIdx.x - B.prefix[j];
    const int tr = local / J.bpl;
    const int line0 = tr * kTile, p0 = (local - tr * J.bpl) * kTile;
    const int len = J.len, nl = J.nlines;
    for (int e = threadIdx.x; e < BT::G * 32; e += kLanes) {
        const int r = e >> 5, c = e & 31;                  // G <= 32
        const int y = line0 - h + r, x = p0 - h + c;
        if (c < BT::G)
            sg[r * BT::GP + c] =
                (y >= 0 && y < nl && x >= 0 && x < len) ? J.gamma[(int64_t)y * J.gamma_ls + x] : make_float2(0.f, 0.f);
    }
    const int t = threadIdx.x & (kTileLanes - 1);
    const int ty = t >> 4, tx = t & 15;
    const int line = line0 + ty, p = p0 + tx;
    const bool inside = line < nl && p < len;
    const bool valid = inside && line >= h && line - h + L <= nl && p >= h && p - h + L <= len;
    const int u = t & 31, g = t >> 5;                      // lag sums: row (column) u, lags g, g + 8, ..
    float w2[2] = {__builtin_nanf(""), __builtin_nanf("")};   // omega_x, omega_y
    unsigned f2[2] = {0u, 0u};
    LaneStats ls;
    __syncthreads();
    // directions of this lane: its half's (BOTH), or both in turn
    auto sums = [&](int dir, float2* S) {
        if (dir == 0) {
            for (int d = g; d < L; d += 8)
                if (u < BT::G - d) {
                    const float2* s = sg + u;
                    float2* out = S + BT::off_x(d) + u;
                    lag_runs<L>([&](int k) { return s[k * BT::GP]; }, [&](int k) { return s[k * BT::GP + d]; },
                                [&](int q, float2 v) { out[q * BT::PX] = v; });
                }
        } else {
            for (int d = g; d < L; d += 8)
                if (u < BT::G - d) {
                    const float2* s = sg + u * BT::GP;
                    const float2* sd = s + d * BT::GP;
                    float2* out = S + BT::off_y(d) + u * (kTile + 1);
                    lag_runs<L>([&](int k) { return s[k]; }, [&](int k) { return sd[k]; },
                                [&](int q, float2 v) { out[q] = v; });
                }
        }
    };
    auto window = [&](int dir, const float2* S) {
        if (!valid) {
            f2[dir] = BM_FLAG_UNDEFINED;
        } else if (dir == 0) {
            const float2* s = S + ty * BT::PX + tx;
            block_omega<L, kWhole, JACOBI>([&](int d, int i) { return s[BT::off_x(d) + i]; }, B.tmpl,
                                           B.full_roots != 0, w2[0], f2[0], ls);
        } else {
            const float2* s = S + ty * (kTile + 1) + tx;
            block_omega<L, kWhole, JACOBI>([&](int d, int i) { return s[BT::off_y(d) + i * (kTile + 1)]; }, B.tmpl,
                                           B.full_roots != 0, w2[1], f2[1], ls);
        }
    };
    const bool dx = (J.bdirs & BM_DIR_X) != 0, dy = (J.bdirs & BM_DIR_Y) != 0;
    const int64_t o = (int64_t)p * J.out_es + (int64_t)line * J.out_ls;
    const int64_t fo = (int64_t)p * J.flag_es + (int64_t)line * J.flag_ls;
    if constexpr (BOTH) {
        const int half = threadIdx.x >> 8;                 // wave-uniform: omega_x or omega_y
        if (half == 0) {
            if (dx) sums(0, sS);
        } else {
            if (dy) sums(1, sS + BT::size);
        }
        __syncthreads();
        if (half == 0) {
            if (dx) window(0, sS);
            if (inside && dx) J.out[o] = w2[0];
        } else {
            if (dy) window(1, sS + BT::size);
            if (inside && dy) J.out_y[o] = w2[1];
        }
        if (J.flags || J.phase) {
            // the halves exchange their results: the lag sums are dead
            __syncthreads();
            float* xw = reinterpret_cast<float*>(sS);      // [2][256] omegas, then partial phases
            unsigned* xf = reinterpret_cast<unsigned*>(xw + 2 * kTileLanes);
            float2* xp = reinterpret_cast<float2*>(xf + kTileLanes);
            xw[half * kTileLanes + t] = half == 0 ? w2[0] : w2[1];
            if (half == 1) xf[t] = f2[1];
            __syncthreads();
            float2 sum = make_float2(0.f, 0.f);
            const float wx = xw[t], wy = xw[kTileLanes + t];
            const bool ok = J.phase && finitef(wx) && finitef(wy);
            if (ok) {
                const float2* s = sg + ty * BT::GP + tx;
                sum = PhaseRow<L>(wx).template sum<false>([&](int r, int c) { return s[r * BT::GP + c]; }, wy,
                                                         half ? L / 2 : 0, half ? L : L / 2);
            }
            if (half == 1) xp[t] = sum;
            __syncthreads();
            if (half == 0 && inside) {
                if (J.phase) J.phase[o] = ok ? phase_of(sum, xp[t]) : __builtin_nanf("");
                if (J.flags) J.flags[fo] = (uint8_t)((dx ? f2[0] : 0u) | ((dy ? xf[t] : 0u) << 4));
            }
        }
    } else {
        if (dx) {
            sums(0, sS);
            __syncthreads();
            window(0, sS);
            __syncthreads();
        }
        if (dy) {
            sums(1, sS);
            __syncthreads();
            window(1, sS);
        }
        if (inside) {
            if (dx) J.out[o] = w2[0];
            if (dy) J.out_y[o] = w2[1];
            if (J.phase) {
                float ph = __builtin_nanf("");
                if (finitef(w2[0]) && finitef(w2[1])) {
                    const float2* s = sg + ty * BT::GP + tx;
                    ph = block_phase<L, false>([&](int r, int c) { return s[r * BT::GP + c]; }, w2[0], w2[1]);
                }
                J.phase[o] = ph;
            }
            if (J.flags) J.flags[fo] = (uint8_t)(f2[0] | (f2[1] << 4));
        }
    }
    if constexpr (!kWhole) {
        const int left = __syncthreads_or(pending(w2[0]) || pending(w2[1]));
        if (threadIdx.x == 0) B.left[blockIdx.x] = (uint8_t)(left != 0);
    }
    if (STATS) flush_stats<kLanes>(ls, B.stats);
}

// The windows above 8 x 8 that block_tile_kernel left (pending() maps in the
// tiles it marked; all valid windows with full_roots), each direction of each
// window on a lane of its own, by the whole method from the signal in device
// memory: up to 512 registers, one wave per SIMD.  A block skips the unmarked
// tiles of its chunks by their byte, gathers what is pending in up to
// kRestTiles marked ones at a time into a list and works it off densely: at
// low SNR a few windows of every wave are pending, and a wave costs the same
// for one as for 64 (4 x 1024^2 at 3 dB, 9 x 9 blocks: 1.51 ms with the windows
// left on their own lanes, 0.88 gathered; where nothing is left, reading the
// maps for it instead of the bytes cost 0.34 ms of 1.16 per 10 x 1024^2).
// Where few windows are left, what a block costs is the latency of one pass
// (reads of the maps, gathering, one wave's worth of every solver), so a pass
// takes up to kRestTiles tiles, looks their places up once and reads the maps
// of kRestScan tiles together: against four tiles a pass, each looked up and
// read in turn, 20 x 1024^2 at 10 dB with 9 x 9 blocks 1.57 -> 1.46 ms, 11 x 11
// 1.80 -> 1.75, 4 x 1024^2 at 3 dB 0.97 -> 0.94, one 1850 x 700 frame 164 -> 157 us
// (with the windows that the tile kernel left before its second expansion; now the
// pass finds next to nothing in the first two and takes 4 us).
constexpr int kRestTiles = 16;
constexpr int kRestScan = 4;           // marked tiles whose maps are read together
constexpr int kRestChunk = 4;          // neighbouring tiles of a block's chunk
constexpr unsigned kListed = 0x80u;

template <int L, bool STATS>
__global__ __launch_bounds__(kTileLanes) void block_rest_kernel(RmBatch B, int chunk) {
    constexpr int h = L / 2;
    __shared__ unsigned short list[2 * kRestTiles * kTileLanes];   // slot << 9 | direction << 8 | pixel
    __shared__ unsigned char flag[2 * kRestTiles * kTileLanes];    // by the same index: BM_FLAG_*, kListed
    __shared__ int tiles[kTileLanes];                              // work items of the marked tiles
    __shared__ int tjob[kRestTiles], tline[kRestTiles], tpix[kRestTiles];   // job, first line and pixel of a listed tile
    __shared__ int ntiles, count;
    LaneStats ls;
    const int t = threadIdx.x;
    if (t == 0) ntiles = 0;
    __syncthreads();
    // lane t looks at tile t % chunk of the block's chunk t / chunk
    const int64_t w = ((int64_t)(t / chunk) * gridDim.x + blockIdx.x) * chunk + t % chunk;
    if (w < B.total && (B.full_roots || B.left[w])) tiles[atomicAdd(&ntiles, 1)] = (int)w;
    __syncthreads();
    // pixel q of listed tile k
    auto place = [&](int k, int q, int& line, int& p) {
        line = tline[k] + (q >> 4);
        p = tpix[k] + (q & 15);
    };
    const int nt = ntiles;
    for (int b0 = 0; b0 < nt; b0 += kRestTiles) {
        const int n_tiles = nt - b0 < kRestTiles ? nt - b0 : kRestTiles;
        if (t == 0) count = 0;
        if (t < n_tiles) {
            const int item = tiles[b0 + t], j = find_job(B.prefix, B.njobs, item);
            const int local = item - B.prefix[j], tr = local / B.jobs[j].bpl;
            tjob[t] = j;
            tline[t] = tr * kTile;
            tpix[t] = (local - tr * B.jobs[j].bpl) * kTile;
        }
        __syncthreads();
        for (int k0 = 0; k0 < n_tiles; k0 += kRestScan) {
            float w2[kRestScan][2];
#pragma unroll
            for (int u = 0; u < kRestScan; ++u) {
                w2[u][0] = w2[u][1] = 0.f;
                int line, p;
                if (B.full_roots || k0 + u >= n_tiles) continue;
                place(k0 + u, t, line, p);
                const RmJob& J = B.jobs[tjob[k0 + u]];
                if (line >= J.nlines || p >= J.len) continue;
                const int64_t o = (int64_t)p * J.out_es + (int64_t)line * J.out_ls;
                if (J.bdirs & BM_DIR_X) w2[u][0] = J.out[o];
                if (J.bdirs & BM_DIR_Y) w2[u][1] = J.out_y[o];
            }
#pragma unroll
            for (int u = 0; u < kRestScan; ++u) {
                const int k = k0 + u;
                int line, p;
                if (k >= n_tiles) continue;
                place(k, t, line, p);
                const RmJob& J = B.jobs[tjob[k]];
                if (line >= J.nlines || p >= J.len) continue;
                const int64_t o = (int64_t)p * J.out_es + (int64_t)line * J.out_ls;
                const bool valid = line >= h && line - h + L <= J.nlines && p >= h && p - h + L <= J.len;
#pragma unroll
                for (int dir = 0; dir < 2; ++dir) {
                    const int e = k << 9 | dir << 8 | t;
                    flag[e] = 0;
                    if (!(J.bdirs & (dir == 0 ? BM_DIR_X : BM_DIR_Y))) continue;
                    if (B.full_roots) {
                        // nothing ran before: borders are written here
                        if (!valid) {
                            (dir == 0 ? J.out : J.out_y)[o] = __builtin_nanf("");
                            flag[e] = BM_FLAG_UNDEFINED;
                            continue;
                        }
                    } else if (!pending(w2[u][dir])) {
                        continue;
                    }
                    flag[e] = (unsigned char)kListed;
                    list[atomicAdd(&count, 1)] = (unsigned short)e;
                }
                if (B.full_roots && !valid) {
                    if (J.phase) J.phase[o] = __builtin_nanf("");
                    if (J.flags)
                        J.flags[(int64_t)p * J.flag_es + (int64_t)line * J.flag_ls] =
                            (uint8_t)(flag[k << 9 | t] | flag[k << 9 | 256 | t] << 4);
                }
            }
        }
        __syncthreads();
        const int n = count;
        for (int i = t; i < n; i += kTileLanes) {
            const int e = list[i], dir = (e >> 8) & 1;
            int line, p;
            place(e >> 9, e & 255, line, p);
            const RmJob& J = B.jobs[tjob[e >> 9]];
            const float2* g = J.gamma + (int64_t)(line - h) * J.gamma_ls + (p - h);
            const int64_t sk = dir == 0 ? J.gamma_ls : 1, si = dir == 0 ? 1 : J.gamma_ls;   // s_k[i] = g[k sk + i si]
            float omega = __builtin_nanf("");
            unsigned fl = 0;
            Sym<L> T;
            float c1r, c1i, hc, hs;
            T_from_snapshots<L>(L, [&](int k, int q) { return g[k * sk + q * si]; }, T, c1r, c1i);
            half_angle_of(c1r, c1i, hc, hs);
            if (!trace_normalise<L>(T)) {
                fl |= BM_FLAG_UNDEFINED;
            } else {
                ls.counted += 1;
                // what the tile kernel leaves was not proven there or took many steps: the
                // tridiagonal solver at once (with every root wanted nothing was tried yet)
                float v[L], nu;
                int steps = 0;
                const bool have = B.full_roots && power_top_eigvec<L>(T, hc, hs, kPowerMinSteps, kPowerMaxSteps,
                                                                      kPowerTolBlock, v, steps, nu);
                if (have) {
                    ls.power += 1;
                    ls.eig_its += steps;
                }
                if (have || signal_eigvec_T<L, false>(T, v, fl, ls))
                    window_omega_v<L>(v, B.tmpl, B.full_roots != 0, __builtin_nanf(""), omega, fl, ls);
            }
            (dir == 0 ? J.out : J.out_y)[(int64_t)p * J.out_es + (int64_t)line * J.out_ls] = omega;
            flag[e] = (unsigned char)(kListed | fl);
        }
        __syncthreads();
        // flags and phase of the pixels touched, each by one lane: its omega_x
        // entry's, or its omega_y entry's when omega_x was not on the list
        for (int i = t; i < n; i += kTileLanes) {
            const int e = list[i];
            int line, p;
            place(e >> 9, e & 255, line, p);
            const RmJob& J = B.jobs[tjob[e >> 9]];
            if ((e & 256) && (flag[e ^ 256] & kListed)) continue;
            if (J.flags) {
                uint8_t* f = J.flags + (int64_t)p * J.flag_es + (int64_t)line * J.flag_ls;
                const unsigned fx = flag[e & ~256] & 15u, fy = flag[e | 256] & 15u;
                *f = (uint8_t)((B.full_roots ? 0u : (unsigned)*f) | fx | (fy << 4));
            }
            if (J.phase) {
                const int64_t o = (int64_t)p * J.out_es + (int64_t)line * J.out_ls;
                const float wx = J.out[o], wy = J.out_y[o];
                float ph = __builtin_nanf("");
                if (finitef(wx) && finitef(wy)) {
                    const float2* g = J.gamma + (int64_t)(line - h) * J.gamma_ls + (p - h);
                    const int64_t gl = J.gamma_ls;
                    ph = block_phase<L, true>([&](int r, int c) { return g[r * gl + c]; }, wx, wy);
                }
                J.phase[o] = ph;
            }
        }
        __syncthreads();
    }
    if (STATS) flush_stats<kTileLanes>(ls, B.stats);
}

template <int L, bool JACOBI, bool BOTH>
hipError_t launch_block_tiles(const RmBatch& b, hipStream_t s) {
    const dim3 grid(b.total), lanes(kTileLanes * (BOTH ? 2 : 1));
    if (b.stats) hipLaunchKernelGGL((block_tile_kernel<L, true, JACOBI, BOTH>), grid, lanes, 0, s, b);
    else hipLaunchKernelGGL((block_tile_kernel<L, false, JACOBI, BOTH>), grid, lanes, 0, s, b);
    return hipGetLastError();
}

// Tiles of one eigen solver.  Both directions at once keep twice the lanes busy
// per tile but hold two sets of lag sums, so fewer tiles fit a CU: faster where
// the tiles do not fill the chip (64 x 64 with 7 x 7 blocks 34 -> 28 us, 15 x 15
// 109 -> 80) and where two sets still leave two waves per SIMD, all that T's
// registers allow (without the phase, 4 x 1024^2: 15 x 15 1.03 -> 0.97 ms, 17 x 17 1.33 -> 1.24),
// slower otherwise (8 x 8 0.34 -> 0.38, 11 x 11 0.53 -> 0.56, 13 x 13 0.67 ->
// 0.84).
template <int L, bool JACOBI>
hipError_t launch_block_LJ(const RmBatch& b, hipStream_t s) {
    const bool both = b.both_dirs && ((L >= 15 && !b.phases) || b.total <= 512);
    return both ? launch_block_tiles<L, JACOBI, true>(b, s) : launch_block_tiles<L, JACOBI, false>(b, s);
}

// Line and block windows up to 8 x 8 of one eigen solver (JACOBI or the
// default route), one translation unit each.
template <int L, bool JACOBI>
hipError_t launch_LJ(const RmBatch& b, int block, int grid, hipStream_t s) {
    if (b.block_windows) return launch_block_LJ<L, JACOBI>(b, s);
    if (block == 128) return launch_LBJ<L, 128, JACOBI>(b, grid, s);
    return launch_LBJ<L, 256, JACOBI>(b, grid, s);
}

template <bool JACOBI>
hipError_t launch_rootmusic_J(int L, const RmBatch& b, int block, int grid, hipStream_t s) {
    switch (L) {
        case 2: return launch_LJ<2, JACOBI>(b, block, grid, s);
        case 3: return launch_LJ<3, JACOBI>(b, block, grid, s);
        case 4: return launch_LJ<4, JACOBI>(b, block, grid, s);
        case 5: return launch_LJ<5, JACOBI>(b, block, grid, s);
        case 6: return launch_LJ<6, JACOBI>(b, block, grid, s);
        case 7: return launch_LJ<7, JACOBI>(b, block, grid, s);
        case 8: return launch_LJ<8, JACOBI>(b, block, grid, s);
        default: return hipErrorInvalidValue;
    }
}

// Block windows above 8 x 8: the common route, then what it left.
template <int L>
hipError_t launch_big_block(const RmBatch& b, hipStream_t s) {
    if (!b.block_windows) return hipErrorInvalidValue;
    if (!b.full_roots) {
        const hipError_t e = launch_block_LJ<L, false>(b, s);
        if (e != hipSuccess) return e;
    }
    // kRestChunk tiles per block for dense lists, one while there are few tiles (spread over
    // the CUs), and several chunks of them (strided) above 8192 tiles, so that tiles without
    // anything left cost few blocks; a block looks at kTileLanes tiles at most
    const int chunk = b.total <= 1024 ? 1 : kRestChunk;
    const int chunks = (b.total + chunk - 1) / chunk, most = kTileLanes / chunk;
    const int g = chunks < 2048 ? chunks : 2048, least = (chunks + most - 1) / most;
    const dim3 grid(g > least ? g : least);
    if (b.stats) hipLaunchKernelGGL((block_rest_kernel<L, true>), grid, dim3(kTileLanes), 0, s, b, chunk);
    else hipLaunchKernelGGL((block_rest_kernel<L, false>), grid, dim3(kTileLanes), 0, s, b, chunk);
    return hipGetLastError();
}

}  // namespace
}  // namespace bm
