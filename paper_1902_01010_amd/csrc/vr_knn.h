// vr_knn.h -- what the two neighbour searches share: the packed key, the
// Gaussian background and the wavefront-wide select of the wave-a-query form.
#pragma once
#include "vr_kd.h"

#include <cmath>

namespace vr {

constexpr int POS_BITS = 22;
constexpr uint64_t POS_MASK = (uint64_t(1) << POS_BITS) - 1;

// ln f_bg (Eq. fvbg): the log density of the trivariate Gaussian of mean
// vbar(x) and covariance sigma(x), particle g, at velocity vq.  The
// quadratic form is u^T adj(S) u / det S with u = vq - vbar; S is positive
// definite iff its leading principal minors S_xx, S_xx S_yy - S_xy^2 and
// det S are positive (Sylvester's criterion), else NaN.
__device__ __forceinline__ double log_fbg(const float* __restrict__ sigma, const float* __restrict__ vbar,
                                          int g, double vqx, double vqy, double vqz) {
    const float* s = sigma + (int64_t)g * 6;  // particle-major
    const double sxx = s[0], syy = s[1], szz = s[2];
    const Sym3Adj A = sym3_adjugate(sxx, syy, szz, s[3], s[4], s[5]);
    if (!(sxx > 0) || !(A.zz > 0) || !(A.det > 0)) return NAN;
    const float* vb = vbar + (int64_t)g * 3;
    const double ux = vqx - (double)vb[0];
    const double uy = vqy - (double)vb[1];
    const double uz = vqz - (double)vb[2];
    const double diag = A.xx * ux * ux + A.yy * uy * uy + A.zz * uz * uz;
    const double offd = A.xy * ux * uy + A.xz * ux * uz + A.yz * uy * uz;
    // 3 ln(2 pi) / 2
    constexpr double HALF3_LN_2PI = 2.7568155996140178;
    return -0.5 * ((diag + 2.0 * offd) / A.det + log(A.det)) - HALF3_LN_2PI;
}

__device__ __forceinline__ bool vless(double a, int pa, double b, int pb) { return a < b || (a == b && pa < pb); }

constexpr int BIG_CAP = 256;              // largest n_se
constexpr int BIG_EXTRA = 192;            // keys appended past n_se before the buffer is cut back
constexpr int BIG_BUF = BIG_CAP + BIG_EXTRA + 64;  // room for one more leaf chunk
constexpr int BIG_J = BIG_BUF / 64;       // buffer slots per lane

// The key of rank r (0-based) among the valid keys of the wavefront, by a
// radix select over byte digits: per digit, a histogram of the keys that
// share the digits chosen so far, and a wave-wide prefix over its 256
// buckets to find the one holding rank r.  Keys are distinct.  hist: 256
// words of LDS.
__device__ __forceinline__ uint64_t wave_select(const uint64_t (&k)[BIG_J], const bool (&v)[BIG_J], int r,
                                                uint32_t* hist) {
    uint64_t lo = ~0ull, hi = 0;
#pragma unroll
    for (int j = 0; j < BIG_J; ++j)
        if (v[j]) {
            lo = min(lo, k[j]);
            hi = max(hi, k[j]);
        }
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (uint64_t)__shfl_xor((unsigned long long)lo, o, 64));
        hi = max(hi, (uint64_t)__shfl_xor((unsigned long long)hi, o, 64));
    }
    if (lo == hi) return lo;
    const int lane = (int)lane_id();
    // digits above the highest differing byte are those of every key
    int shift = ((63 - __clzll(lo ^ hi)) >> 3) << 3;
    uint64_t above = shift + 8 >= 64 ? 0 : ~0ull << (shift + 8);
    uint64_t prefix = lo & above;
    for (;;) {
#pragma unroll
        for (int t = 0; t < 4; ++t) hist[4 * lane + t] = 0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < BIG_J; ++j)
            if (v[j] && (k[j] & above) == prefix) atomicAdd(&hist[(k[j] >> shift) & 255], 1u);
        __builtin_amdgcn_wave_barrier();
        uint32_t c[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) c[t] = hist[4 * lane + t];
        const uint32_t sum = c[0] + c[1] + c[2] + c[3];
        uint32_t incl = sum;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        const uint32_t excl = incl - sum;
        // the lane whose buckets span rank r names the digit
        int digit = -1;
        uint32_t below = excl;
        if ((uint32_t)r >= excl && (uint32_t)r < incl) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (digit < 0 && (uint32_t)r < below + c[t]) digit = 4 * lane + t;
                else if (digit < 0) below += c[t];
            }
        }
        const uint64_t owner = __ballot(digit >= 0);
        const int src = __builtin_ctzll(owner);
        digit = __shfl(digit, src, 64);
        below = __shfl(below, src, 64);
        r -= (int)below;
        prefix |= (uint64_t)digit << shift;
        __builtin_amdgcn_wave_barrier();
        if (shift == 0) break;
        above = ~0ull << shift;
        shift -= 8;
    }
    return prefix;
}

// rank_of[g] = the position of particle g in host_members (-1 beforehand);
// a member outside [0, n) or listed twice raises *bad (vr_knn.hip).
// R where neighbours may be nearer through the box than by their unwrapped
// coordinates (vr_knn_wide.hip); the arguments are those of vr_local_vdensity, already
// checked, off the host offsets on the host, rank_of as above.
int local_vdensity_wide(vr_ctx* ctx, const vr_particles* p, int32_t n_hosts, const int32_t* host_offsets,
                        const int32_t* host_members, const std::vector<int32_t>& off, const int32_t* rank_of,
                        const float* vbar, const float* sigma, int n_se, int n_v, const int32_t* subset,
                        int64_t n_subset, float* R, hipStream_t st);

}  // namespace vr
