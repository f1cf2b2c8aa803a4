// The kernels' per-window arithmetic (bm_window.h) compiled for the host, so that
// CPU tests run the code itself.  The hardware's approximate instructions are the
// exact operations rounded to FP32 here; __sincosf is off by up to 2^-21 as the
// hardware's sine and cosine are.
#include <cmath>
#include <cstdint>
#include <cstring>

typedef unsigned short __bf16;          // named by declarations only
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_sqrtf(x) std::sqrt(x)
#define __builtin_amdgcn_rsqf(x) (1.0f / std::sqrt(x))
#define __builtin_amdgcn_rcp(x) (1.0 / (x))
#define __builtin_amdgcn_exp2f(x) std::exp2(x)
#define __builtin_amdgcn_logf(x) std::log2(x)
static void host_sincos(float x, float* s, float* c) {
    *s = (float)(std::nearbyint(std::sin((double)x) * 1048576.0) / 1048576.0);
    *c = (float)(std::nearbyint(std::cos((double)x) * 1048576.0) / 1048576.0);
}
#define __sincosf host_sincos
#define __expf(x) std::exp(x)
#include "bm_window.h"

using namespace bm;

namespace {

// tone_omega of n signal vectors from the directions (cw, sw), above L = 8 as the tile
// kernel of block windows calls it.
template <int L>
void tone(const float* v, const float* cw, const float* sw, int n, float* omega, uint8_t* ok) {
    for (int q = 0; q < n; ++q) {
        float a[L], w = NAN;
        std::memcpy(a, v + (int64_t)q * L, sizeof a);
        ok[q] = tone_omega<L, (L > kMaxL)>(a, cw[q], sw[q], w);
        omega[q] = w;
    }
}

// window_omega_v of n signal vectors with previous frequencies wprev; steps[2 q], [2 q + 1]:
// FP32 and FP64 steps counted.  No all-roots template: windows that need it are not meant.
template <int L>
void window(const float* v, const float* wprev, int n, float* omega, int* steps) {
    static const RootTemplate tmpl = {};
    for (int q = 0; q < n; ++q) {
        float a[L], w = NAN;
        unsigned flag = 0;
        LaneStats ls;
        std::memcpy(a, v + (int64_t)q * L, sizeof a);
        window_omega_v<L>(a, tmpl, false, wprev[q], w, flag, ls);
        omega[q] = w;
        steps[2 * q] = ls.pair_its32;
        steps[2 * q + 1] = ls.pair_its;
    }
}

// power_top_eigvec of n trace-normalised matrices T (L x L each) as the windows call it,
// from the lag-1 sums (c1r, c1i); block: as block windows do.
template <int L>
void power(const float* T, const float* c1r, const float* c1i, int n, int block, float* v, int* steps, uint8_t* ok) {
    for (int q = 0; q < n; ++q) {
        Sym<L> t;
        for (int i = 0; i < L; ++i)
            for (int j = 0; j < L; ++j) t.a[i][j] = T[((int64_t)q * L + i) * L + j];
        float a[L], nu, hc, hs;
        int s = 0;
        half_angle_of(c1r[q], c1i[q], hc, hs);
        ok[q] = power_top_eigvec<L>(t, hc, hs, kPowerMinSteps, kPowerMaxSteps, block ? kPowerTolBlock : kPowerTol, a,
                                    s, nu);
        steps[q] = s;
        std::memcpy(v + (int64_t)q * L, a, sizeof a);
    }
}

}  // namespace

#define BY_SIZE(call)                      \
    switch (L) {                           \
        case 2: call<2> ARGS; return 0;    \
        case 3: call<3> ARGS; return 0;    \
        case 4: call<4> ARGS; return 0;    \
        case 5: call<5> ARGS; return 0;    \
        case 6: call<6> ARGS; return 0;    \
        case 7: call<7> ARGS; return 0;    \
        case 8: call<8> ARGS; return 0;    \
        case 9: call<9> ARGS; return 0;    \
        case 11: call<11> ARGS; return 0;  \
        case 13: call<13> ARGS; return 0;  \
        case 15: call<15> ARGS; return 0;  \
        case 17: call<17> ARGS; return 0;  \
        default: return -1;                \
    }

extern "C" {
#define ARGS (v, cw, sw, n, omega, ok)
int host_tone(int L, const float* v, const float* cw, const float* sw, int n, float* omega, uint8_t* ok) {
    BY_SIZE(tone)
}
#undef ARGS
#define ARGS (v, wprev, n, omega, steps)
int host_window(int L, const float* v, const float* wprev, int n, float* omega, int* steps) { BY_SIZE(window) }
#undef ARGS
#define ARGS (T, c1r, c1i, n, block, v, steps, ok)
int host_power(int L, const float* T, const float* c1r, const float* c1i, int n, int block, float* v, int* steps,
               uint8_t* ok) {
    BY_SIZE(power)
}
#undef ARGS
}
