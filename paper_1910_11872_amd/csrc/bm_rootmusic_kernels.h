// Per-window root-MUSIC local-frequency kernels for gfx950 (device code and
// launch templates, shared by bm_rootmusic.hip and bm_bigblock.hip).
//
// One lane owns two windows (two output pixels of one direction).  A block of
// BLOCK lanes (128 or 256) covers 2 BLOCK - (L-1) consecutive window starts of one line; the
// overlapping windows are staged once in LDS with coalesced loads.  Steps:
//
//   lag sums    S_d(m) = sum_k g[m+k] conj(g[m+k+d]), d < L, two starts m per
//               lane, shared through LDS: the covariance of the window that
//               starts at s is R_ij = S_{j-i}(s+i)             (paper Eq. 4)
//   FB average + unitary real transform: T = Q^H R_fb Q is real symmetric
//               (Q the sparse centro-symmetric unitary matrix), built in
//               closed form from R without forming R_fb
//   eigen-split the eigenvector v of the largest eigenvalue of T gives the
//               signal subspace u1 = Q v (paper Eq. 6-11, one-dimensional
//               signal subspace).  Power iteration on T, shifted by the
//               mean of its other eigenvalues, from
//               the steering vector of the window's lag-1 phase, kept when
//               an a-posteriori bound proves it within 6e-6 rad of the top
//               eigenvector (2-3 steps at 10 dB).  Otherwise: Householder
//               reduction to tridiagonal form, Newton's
//               method from above on the characteristic polynomial
//               (monotone for real-rooted polynomials) for the largest
//               eigenvalue, one shifted inverse iteration for its
//               eigenvector, back-transformation.  The cyclic Jacobi solver
//               is kept as a selectable alternative.
//   closed-form pair  a window whose u1 is close to one tone's steering
//               vector has, by Rouche's theorem, one root pair near the
//               circle, and the derivatives of the spectrum at its peak give
//               that pair (tone_omega): nearly every window ends here.  The
//               steps below serve the others.
//   polynomial  c_k = sum_i C[i,i+k] with C = I - u1 u1^H = Un Un^H
//               (paper Eq. 12-14)
//   certified pair  Newton (FP32, then FP64) for the signal root with its mate
//               1/conj(z) divided out, started just inside the unit circle
//               at the peak of the spectrum; accepted when the polynomial divides by
//               the pair's factor and a Schur-Cohn count on the quotient
//               puts every other inner root strictly inside |z_in|: that
//               pair is the one the selection below would pick.  Windows
//               that fail this (about 1 in 10^4 at 8 dB) take the path below.
//   roots       Aberth-Ehrlich simultaneous iteration in FP32 from the roots
//               of the noise-free single-tone polynomial rotated to the
//               window's frequency guess; evaluation at 1/conj(z) for roots
//               outside the unit circle keeps Horner free of overflow
//   selection   the root nearest the unit circle and its mate nearest
//               1/conj(z_sel) (the paper's rule, Sec. 3, applied to the
//               conjugate-reciprocal root pairs)
//   polish      FP64 Newton iteration on the pair's quadratic factor
//               z^2 - r z - s (Bairstow's method with complex coefficients),
//               which is well conditioned even when the pair is a
//               near-double root
//   omega       arg(r) = arg(z_sel + z_mate)  (paper Eq. 15)
#pragma once

#include "bm_window.h"

namespace bm {
namespace {

// Line windows per lane (two window starts per lane).  For L <= 6 a lane sums
// the lags of its two starts, the second slid from the first (lag_sums_pair);
// for L >= 7 a lane pair sums the lags of four consecutive starts, one half of
// the lags each, the first start directly and the next three slid by one
// sample (lag_sums_quad), so each start costs about a quarter of a direct sum
// over all lags while the block keeps the same 2 x 256 starts in LDS.  (At
// L = 6 the quarter-cost form measured 3-6% slower: with three lags per lane
// its two LDS reads per snapshot weigh more than the FMAs it saves.)  Blocks
// start at multiples of two (four) pixels, so which window starts are summed
// directly and which are slid depends on the start alone, not on the tile
// size: results are the same for every tiling.  (Four starts per lane, each
// lane with all lags, double the lag sums a block keeps in LDS, which halves
// the blocks resident per CU: twice slower on 1024-wide lines.)
constexpr int kLineSpan = 2;

constexpr bool line_quad(int L) { return L >= 7; }
constexpr int line_windows_per_block(int L, int block) {
    return (kLineSpan * block - (L - 1)) & (line_quad(L) ? ~3 : ~1);
}

template <int L, int BLOCK>
struct LineSpan {
    static constexpr int span = kLineSpan * BLOCK;                  // window starts per block
    static constexpr int wpb = line_windows_per_block(L, BLOCK);    // output pixels per block (even; L >= 7: x4)
    static constexpr bool quad = line_quad(L);                      // lag_sums_quad (else lag_sums_pair)
    static constexpr int row = span + 8;                            // lag-sum row: >= span, 16-byte multiple
    static constexpr int quarter = sg_quarter(span + kMaxN);        // staged samples, de-interleaved
};

// One block of windows: SPAN-(L-1) consecutive pixels p0.. of one line of job J.
template <int L, int BLOCK, bool JACOBI, bool WARM>
__device__ __forceinline__ void rootmusic_block(const RmJob& J, int line, int p0, float2* sg,
                                                float2 (*sS)[LineSpan<L, BLOCK>::row], const RootTemplate& tmpl,
                                                bool full_roots, LaneStats& ls) {
    constexpr int SPAN = LineSpan<L, BLOCK>::span;
    constexpr int WPB = LineSpan<L, BLOCK>::wpb;
    const int t = threadIdx.x;
    const int N = J.N;
    const int half = N >> 1;
    const int K = N - L + 1;
    const float2* g = J.gamma + (int64_t)line * J.gamma_ls;
    const int len = J.len;

    // window of pixel p0+s starts at base+s
    const int base = p0 - half;
    // ---- lag sums S_d(base + s), s < need, d < L -----------------------------
    // (a line's last block holds fewer windows: 1024-sample lines end in one of 12-16,
    // which cost 5% of 100 x 1024^2 when it staged and summed a whole block's starts)
    const int need = min(SPAN, len - p0 + L - 1);
    if constexpr (LineSpan<L, BLOCK>::quad) {
        for (int i = t; i < min(need + 3, SPAN) + N; i += BLOCK) {   // whole quads, and one for the odd-L dummy lag
            const int q = base + i;
            sg[sg_slot(i, LineSpan<L, BLOCK>::quarter)] = (q >= 0 && q < len) ? g[q] : make_float2(0.f, 0.f);
        }
        __syncthreads();
        if (2 * (t & ~1) < need)
            lag_sums_quad<L, LineSpan<L, BLOCK>::row, LineSpan<L, BLOCK>::quarter>(sg, t, K, sS);
    } else {
        for (int i = t; i < need + N; i += BLOCK) {
            const int q = base + i;
            sg[i] = (q >= 0 && q < len) ? g[q] : make_float2(0.f, 0.f);
        }
        __syncthreads();
        if (kLineSpan * t < need) lag_sums_pair<L, LineSpan<L, BLOCK>::row>(sg, kLineSpan * t, K, sS);
    }
    __syncthreads();

#pragma unroll 1
    for (int r = 0; r < kLineSpan; ++r) {
        const int s = r * BLOCK + t;
        const int p = p0 + s;
        const bool inside_line = (s < WPB) && (p < len);
        const bool valid = inside_line && (p - half >= 0) && (p - half + N <= len);
        float omega = __builtin_nanf("");
        unsigned flag = 0;
        if (valid) {
            // covariance R_ij = S_{j-i}(s+i) (Eq. 4, up to the 1/K scale)
            Cov<L> R;
#pragma unroll
            for (int i = 0; i < L; ++i)
#pragma unroll
                for (int j = i; j < L; ++j) {
                    const float2 v = sS[j - i][s + i];
                    R.re[i][j] = v.x;
                    R.im[i][j] = (i == j) ? 0.f : v.y;
                }
            const float wprev = (WARM && J.prev) ? J.prev[(int64_t)p * J.prev_es + (int64_t)line * J.prev_ls]
                                                 : __builtin_nanf("");
            window_omega<L, JACOBI>(R, tmpl, full_roots, K, wprev, omega, flag, ls);
        } else {
            flag |= BM_FLAG_UNDEFINED;
        }
        if (inside_line) store_omega(J, line, p, omega, flag);
    }
}


template <int BLOCK>
__device__ __forceinline__ void flush_stats(const LaneStats& ls, unsigned long long* stats) {
    unsigned long long a[kStatFields] = {(unsigned long long)ls.counted, (unsigned long long)ls.eig_its,
                                         (unsigned long long)ls.iters, (unsigned long long)ls.pfail,
                                         (unsigned long long)ls.accepted, (unsigned long long)ls.rejected,
                                         (unsigned long long)ls.pair_its, (unsigned long long)ls.pair_its32,
                                         (unsigned long long)ls.power};
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int c = 0; c < kStatFields; ++c) a[c] += __shfl_xor(a[c], off);
    if ((threadIdx.x & 63) == 0) {
        // spread the counters over kStatSlots slots to avoid one hot address
        unsigned long long* sl =
            stats + kStatFields * ((blockIdx.x * (BLOCK / 64) + (threadIdx.x >> 6)) % kStatSlots);
#pragma unroll
        for (int c = 0; c < kStatFields; ++c)
            if (a[c]) atomicAdd(sl + c, a[c]);
    }
}

// Grid-stride loop over the work items of every job of one L: item w is
// block (w - prefix[j]) of job j, i.e. line (w - prefix[j]) / bpl and window
// block (w - prefix[j]) % bpl.  A grid of one block per item runs each item
// once; a smaller (persistent) grid walks the list.
// Without the statistics counters the L <= 6 line kernels fit five waves per
// SIMD (96 VGPRs, a few spilled), 1.3% faster on L = 6 than the four that 119
// VGPRs allow, and the L = 7, 8 ones four (128 VGPRs; L = 8 spills seven and
// runs 3% faster than at the three waves of its 151).
// WARM: line windows may read a previous-frame map (the other build folds the
// warm-start branch away: four fewer spilled registers at L = 8).
// LOOP = false (line windows): one block per work item (grid = total), no
// grid-stride loop; the loop keeps values live across items that cost the
// L = 6 and 8 line kernels 40-50 spilled registers.
template <int L, int BLOCK, bool STATS, bool JACOBI, bool WARM = false, bool LOOP = true>
__global__ __launch_bounds__(BLOCK)
__attribute__((amdgpu_waves_per_eu(STATS ? 1 : (L <= 6 ? 5 : 4))))
void rootmusic_kernel(RmBatch B) {
    // staged signal and lag sums
    __shared__ float2 sg[4 * LineSpan<L, BLOCK>::quarter];
    __shared__ __align__(16) float2 sS[L][LineSpan<L, BLOCK>::row];
    LaneStats ls;
    // LOOP = false: exactly one item, blockIdx.x (a trip count of one the compiler sees)
    const int wend = LOOP ? B.total : (int)blockIdx.x + 1;
    const int wstep = LOOP ? (int)gridDim.x : 1;
    for (int w = blockIdx.x; w < wend; w += wstep) {
        const int j = find_job(B.prefix, B.njobs, w);
        const RmJob J = B.jobs[j];
        const int local = w - B.prefix[j];
        const int line = local / J.bpl;
        const int bx = local - line * J.bpl;
        rootmusic_block<L, BLOCK, JACOBI, WARM>(J, line, bx * LineSpan<L, BLOCK>::wpb, sg, sS, B.tmpl,
                                                B.full_roots != 0, ls);
        __syncthreads();
    }
    if (STATS) flush_stats<BLOCK>(ls, B.stats);
}

template <int L, int BLOCK, bool JACOBI, bool WARM>
hipError_t launch_LBJW(const RmBatch& b, int grid, hipStream_t s) {
    if (b.stats)
        hipLaunchKernelGGL((rootmusic_kernel<L, BLOCK, true, JACOBI, WARM>), dim3(grid), dim3(BLOCK), 0, s, b);
    else if (grid < b.total)
        hipLaunchKernelGGL((rootmusic_kernel<L, BLOCK, false, JACOBI, WARM>), dim3(grid), dim3(BLOCK), 0, s,
                           b);
    else
        hipLaunchKernelGGL((rootmusic_kernel<L, BLOCK, false, JACOBI, WARM, false>), dim3(b.total),
                           dim3(BLOCK), 0, s, b);
    return hipGetLastError();
}

template <int L, int BLOCK, bool JACOBI>
hipError_t launch_LBJ(const RmBatch& b, int grid, hipStream_t s) {
    return b.warm ? launch_LBJW<L, BLOCK, JACOBI, true>(b, grid, s) : launch_LBJW<L, BLOCK, JACOBI, false>(b, grid, s);
}

}  // namespace
}  // namespace bm
