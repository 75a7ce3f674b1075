// vr_unbind.hip -- unbinding by directly summed Plummer-softened potentials
// (Sec. 2.2, Eq. binding), all groups batched per pass.
//
// Every pass has two launches.  The potential launch runs over work items
// (group, i-tile, j-range) with the members as float grid-unit coordinates
// (exact small integers) and mass; each lane owns one i and sums 1/sqrt(r^2 + eps^2) terms in FP32 over runs of at most 64 j
// before adding the run into an FP64 accumulator, which is then added
// atomically to the member's FP64 potential.  The per-group launch (one
// workgroup per active group) then finds the potential minimum (candidates
// within the FP32 error band are re-evaluated exactly in FP64, so the chosen
// centre is the FP64 argmin), selects the members nearest to it with an
// 11-bit radix select over (d2, index) keys, takes their mass-weighted mean
// velocity as the frame, evaluates beta_E T + W, and compacts the survivors
// in place (stable, so index order is kept).
//
// The persistent schedule updates the potential incrementally: the group
// kernel keeps each survivor's FP64 sum with it and writes the members it
// removed to a side list; the next pass subtracts those members' terms from
// the survivors' sums (|S| |D| pairs instead of |S|^2).  A group returns to
// a full recompute once the members removed since its last one exceed a
// quarter of its current size, which bounds the error the subtractions add
// to that of a full FP32-tiled sum (a quarter of it).
#include "vr_internal.h"

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstring>

namespace vr {
namespace {

constexpr int UB = 256;                 // threads per workgroup
constexpr int ST_ACTIVE = 0, ST_BOUND = 1, ST_DISSOLVED = 2;
constexpr int MAX_CAND = 64;
constexpr double REFINE_TOL = 4e-5;     // > twice the FP32 error bound of the tiled sums

struct Members {
    float4* p;      // x, y, z in grid units relative to the group's first member (exact integers); mass (1 if uniform)
    float4* v;      // velocity; particle index (bits)
    int uniform;    // every particle has the same mass
};

// Members removed by a group's last pass, at the group's base (stable
// order), and the per-group bookkeeping of the incremental potential:
// nrm = members removed by the last pass; since = removed since the last
// full recompute; mode = 1 when the next pass may subtract them instead of
// recomputing.
struct Removed {
    float* p;  // x, y, z and, unless all masses are equal, mass
    int *nrm, *since, *mode;
};

// Member-parallel set-up: member k of group g (found by bisection of the
// offsets) gets its grid offsets from the group's first member, its
// velocity and mass; its sum, its particle's bound flag and potential are
// reset.
__global__ void k_ub_init(int ng, int64_t M, const int32_t* __restrict__ off, const int32_t* __restrict__ mem,
                          const uint32_t* __restrict__ qx, const uint32_t* __restrict__ qy,
                          const uint32_t* __restrict__ qz, const float* __restrict__ vx, const float* __restrict__ vy,
                          const float* __restrict__ vz, const float* __restrict__ mass, int gb, Members W,
                          double* __restrict__ acc, uint8_t* __restrict__ bound, double* __restrict__ phi) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= M) return;
    int lo = 0, hi = ng - 1;  // last group with off[g] <= k
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= k) lo = mid; else hi = mid - 1;
    }
    const int r = mem[off[lo]];
    const int i = mem[k];
    const int rx = (int)qx[r], ry = (int)qy[r], rz = (int)qz[r];
    W.p[k] = make_float4((float)min_image((int)qx[i] - rx, gb), (float)min_image((int)qy[i] - ry, gb),
                         (float)min_image((int)qz[i] - rz, gb), mass ? mass[i] : 1.f);
    W.v[k] = make_float4(vx[i], vy[i], vz[i], __int_as_float(i));
    acc[k] = 0.0;
    bound[i] = 0;
    phi[i] = NAN;
}

// Per-group state, and nbig = the first group with fewer than wide_min
// members (*nbig holds ng beforehand): the leading groups up to there take
// the wide group kernel.
__global__ void k_ub_state(int ng, const int32_t* __restrict__ off, int n_min, int wide_min, Removed Rm,
                           int* __restrict__ cnt, int* __restrict__ state, int32_t* __restrict__ iters,
                           int* __restrict__ nbig) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= ng) return;
    const int n = off[g + 1] - off[g];
    cnt[g] = n;
    state[g] = n < n_min ? ST_DISSOLVED : ST_ACTIVE;
    iters[g] = 0;
    Rm.nrm[g] = 0;
    Rm.since[g] = 0;
    Rm.mode[g] = 0;
    if (n < wide_min) atomicMin(nbig, g);
}

__global__ void k_ub_zero(int na, const int* __restrict__ active, const int32_t* __restrict__ off,
                          const int* __restrict__ cnt, double* __restrict__ acc) {
    const int g = active[blockIdx.x];
    const int s = off[g], e = s + cnt[g];
    for (int k = s + threadIdx.x; k < e; k += blockDim.x) acc[k] = 0.0;
}

// Sum over staged j of m_j / sqrt(r^2 + eps^2) for one i, in FP32 over at
// most 64 terms (the caller adds it to an FP64 accumulator; 64 same-sign
// FP32 terms stay within 64 * 2^-24 relative).  CHECK = the chunk may hold
// j == i or, with eps = 0, a coincident pair; otherwise every term is
// finite and taken.  r^2 + eps^2 is at least min(eps^2, 1) in grid units
// squared (coordinates are integers), a normal FP32 number (the host refuses
// a smaller nonzero eps^2), so the hardware reciprocal square root needs no
// rescaling for subnormal inputs and gives rsqrtf's result.
template <bool UNIFORM, bool CHECK>
__device__ __forceinline__ float tile_sum(const float4* __restrict__ sj, int t0, int t1, float xi, float yi, float zi,
                                          float eps2, int jbase, int i) {
    float accf = 0.f;
#pragma unroll 4
    for (int t = t0; t < t1; ++t) {
        const float4 q = sj[t];
        const float dx = xi - q.x, dy = yi - q.y, dz = zi - q.z;
        const float s2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2)));
        float rinv;
        if (CHECK) rinv = (jbase + t != i && s2 > 0.f) ? __builtin_amdgcn_rsqf(s2) : 0.f;
        else rinv = __builtin_amdgcn_rsqf(s2);
        accf = UNIFORM ? accf + rinv : fmaf(q.w, rinv, accf);
    }
    return accf;
}

// Potential tiles: item = (group, i0, j0, j1).
template <bool UNIFORM>
__global__ __launch_bounds__(UB) void k_ub_potential(const int4* __restrict__ items, const int32_t* __restrict__ off,
                                                     const int* __restrict__ cnt, Members W, float eps2,
                                                     double* __restrict__ acc, int tile) {
    extern __shared__ float4 sj[];
    const int4 it = items[blockIdx.x];
    const int g = it.x, base = off[g], n = cnt[g];
    const int i = it.y + (int)threadIdx.x;
    const bool valid = i < n;
    const float4 pi = valid ? W.p[base + i] : make_float4(0.f, 0.f, 0.f, 0.f);
    const float xi = pi.x, yi = pi.y, zi = pi.z;
    double accd = 0.0;
    for (int j0 = it.z; j0 < it.w; j0 += tile) {
        const int jn = min(tile, it.w - j0);
        __syncthreads();
        for (int t = threadIdx.x; t < jn; t += blockDim.x) sj[t] = W.p[base + j0 + t];
        __syncthreads();
        // rows of this wavefront: [iw, iw + 64)
        const int iw = it.y + ((int)threadIdx.x & ~63);
        for (int t0 = 0; t0 < jn; t0 += 64) {
            const int t1 = min(t0 + 64, jn);
            const bool check = eps2 == 0.f || (j0 + t0 < iw + 64 && j0 + t1 > iw);
            accd += (double)(check ? tile_sum<UNIFORM, true>(sj, t0, t1, xi, yi, zi, eps2, j0, i)
                                   : tile_sum<UNIFORM, false>(sj, t0, t1, xi, yi, zi, eps2, j0, i));
        }
    }
    if (valid) atomicAdd(&acc[base + i], accd);
}

__device__ __forceinline__ double wsum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

template <int N>
__device__ __forceinline__ void bsum(double (&v)[N], double* sm) {
    const int lane = __lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int k = 0; k < N; ++k) {
        double s = wsum(v[k]);
        if (lane == 0) sm[w * N + k] = s;
    }
    __syncthreads();
    for (int k = 0; k < N; ++k) {
        double s = 0;
        for (int ww = 0; ww < nw; ++ww) s += sm[ww * N + k];
        v[k] = s;
    }
    __syncthreads();
}

__device__ __forceinline__ uint32_t wscan(uint32_t v) {
    const int lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

__device__ __forceinline__ uint32_t bscan(uint32_t v, uint32_t* sm, uint32_t* total) {
    const int lane = __lane_id(), w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint32_t inc = wscan(v);
    if (lane == 63) sm[w] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
    for (int k = 0; k < nw; ++k) {
        if (k < w) pre += sm[k];
        tot += sm[k];
    }
    __syncthreads();
    *total = tot;
    return pre + inc - v;
}

__device__ __forceinline__ uint64_t ref_key(const Members& W, int base, int pos, int px, int py, int pz, int gb) {
    const float4 v = W.p[base + pos];
    const int64_t dx = min_image((int)v.x - px, gb);
    const int64_t dy = min_image((int)v.y - py, gb);
    const int64_t dz = min_image((int)v.z - pz, gb);
    return ((uint64_t)(dx * dx + dy * dy + dz * dz) << 22) | (uint64_t)pos;
}

// Bin of a squared distance for the first step of the frame's select: the
// upper bits of its FP32 value (64 bins an octave over [2^6, 2^38), the rest
// in the end bins), which order as the distances do.
constexpr int SEL_BINS = 2048;
__device__ __forceinline__ int sel_bin(uint64_t d2) {
    const int b = (int)(__float_as_uint((float)d2) >> 17) - ((127 + 6) << 6);
    return min(max(b, 0), SEL_BINS - 1);
}
constexpr int SEL_LIST = 1024;  // keys of the rank's bin that are ranked in LDS

// f(k, v) for every member k of [0, n) with v = load(k), U loads in flight a
// thread, k ascending for each thread.
template <int U, class L, class F>
__device__ __forceinline__ void for_members(int n, L load, F f) {
    const int bs = (int)blockDim.x;
    for (int c0 = (int)threadIdx.x; c0 < n; c0 += U * bs) {
        decltype(load(0)) v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = load(min(c0 + u * bs, n - 1));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c0 + u * bs < n) f(c0 + u * bs, v[u]);
    }
}

// 1 / sqrt(x) of a positive normal x: the hardware estimate (29 bits) and two
// Newton steps, the second with the rounding of its product taken in.  Against
// 64-bit significands, m times this is off by at most 1.93 units of 2^-53
// (mean 0.488; equal masses 1.00 and 0.358), m / sqrt(x) by 1.99 (0.491; 1.49
// and 0.497), at under half the instructions; the plain second step gave 2.17
// (0.517).
__device__ __forceinline__ double rsqrt64(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    const double p = x * y, lost = fma(x, y, -p);
    return fma(0.5 * y, fma(-lost, y, fma(-p, y, 1.0)), y);
}

// One group per workgroup of BS threads.  Bound by the latency of the member
// reads on one CU, so every pass over the members keeps several loads a
// thread in flight, and there are few of them: extreme, candidates, select
// (two: a histogram of distance bins, then the rank's bin), frame, energies
// and compaction.  A single candidate needs no exact sum.  A 120 k-member
// group's first pass 0.60 -> 0.34 ms, all 36 passes of 600 groups 4.65 ->
// 2.0 ms (before: one load in flight, six select passes, a square root and a
// division per exact term, compaction 1,024 members and two scans at a time,
// members in seven arrays).  With split != 0 (no active list)
// BS = UB_WIDE takes the groups before *nbig and BS = UB the others, so the
// largest groups get four times the threads.
constexpr int UB_WIDE = 1024;
template <int BS>
__global__ __launch_bounds__(BS) void k_ub_group(const int* __restrict__ active, const int32_t* __restrict__ off,
                                                 int* __restrict__ cnt, int* __restrict__ state,
                                                 int32_t* __restrict__ iters, Members W, Removed Rm,
                                                 double* __restrict__ acc, double eps2g, double scale,
                                                 double mass_value, double beta_E, double frac_ref, int n_min,
                                                 int n_ref_min, int frame_type, int gb, uint8_t* __restrict__ bound,
                                                 double* __restrict__ phi, int max_iter,
                                                 const int* __restrict__ nbig) {
    constexpr int NW = BS / 64;
    constexpr int BPT = 2048 / BS;  // histogram bins per thread
    static_assert(BS >= 256 && BS <= 2048 && 2048 % BS == 0, "block size");
    __shared__ double smd[4 * NW];
    __shared__ uint32_t smu[NW];
    __shared__ uint32_t hist[2048];
    __shared__ int cand[MAX_CAND];
    __shared__ uint64_t list[SEL_LIST];
    __shared__ int s_p, s_bucket, s_n;
    __shared__ uint32_t s_below;
    __shared__ uint64_t s_key;
    __shared__ uint32_t ckept[64];
    __shared__ double s_min;
    __shared__ int s_minpos;
    // with no active list every group has a block and finished ones leave
    const int g = active ? active[blockIdx.x] : (int)blockIdx.x;
    if (nbig && (BS == UB_WIDE ? g >= *nbig : g < *nbig)) return;
    if (!active && (state[g] != ST_ACTIVE || iters[g] >= max_iter)) return;
    const int base = off[g];
    const int n = cnt[g];
    const int tid = threadIdx.x, lane = __lane_id(), w = tid >> 6, nw = blockDim.x >> 6;
    const bool uniform = W.uniform != 0;

    // 1. largest accumulated 1/r sum = deepest potential (ties: lowest position)
    double best = -1.0;
    int bpos = 0x7FFFFFFF;
    for_members<8>(n, [&](int k) { return acc[base + k]; }, [&](int k, double a) {
        if (a > best || (a == best && k < bpos)) { best = a; bpos = k; }
    });
    for (int o = 32; o > 0; o >>= 1) {
        const double ob = __shfl_xor(best, o, 64);
        const int op = __shfl_xor(bpos, o, 64);
        if (ob > best || (ob == best && op < bpos)) { best = ob; bpos = op; }
    }
    if (lane == 0) { smd[w] = best; smu[w] = (uint32_t)bpos; }
    __syncthreads();
    if (tid == 0) {
        double b = smd[0];
        int bp = (int)smu[0];
        for (int ww = 1; ww < nw; ++ww)
            if (smd[ww] > b || (smd[ww] == b && (int)smu[ww] < bp)) { b = smd[ww]; bp = (int)smu[ww]; }
        s_min = b;
        s_minpos = bp;
        s_n = 0;
    }
    __syncthreads();
    // 2-3. every member within the FP32 error band of the extreme gets an
    // exact FP64 sum; candidates are enumerated in position order, MAX_CAND
    // at a time, so the result does not depend on how many there are.
    const double thr = s_min * (1.0 - REFINE_TOL);
    double cbest = -1.0;
    int cpos = s_minpos;
    for_members<8>(n, [&](int k) { return acc[base + k]; }, [&](int k, double a) {
        if (a >= thr) {
            const int at = atomicAdd(&s_n, 1);
            if (at < MAX_CAND) cand[at] = k;
        }
    });
    __syncthreads();
    const uint32_t total_cand = (uint32_t)s_n;
    for (uint32_t first = 0; total_cand > 1; first += MAX_CAND) {
        if (total_cand > MAX_CAND) {
            uint32_t seen = 0;
            for (int c0 = 0; c0 < n; c0 += blockDim.x) {
                const int k = c0 + tid;
                const bool in = k < n && acc[base + k] >= thr;
                uint32_t tot;
                const uint32_t r = seen + bscan(in ? 1u : 0u, smu, &tot);
                if (in && r >= first && r < first + MAX_CAND) cand[r - first] = k;
                seen += tot;
            }
            __syncthreads();
        }
        const int ncand = (int)min(total_cand - first, (uint32_t)MAX_CAND);
        // NC candidates a pass over the members
        constexpr int NC = 4;
        for (int c = 0; c < ncand; c += NC) {
            int pc[NC];
            double cx[NC], cy[NC], cz[NC], s1[NC];
#pragma unroll
            for (int q = 0; q < NC; ++q) {
                pc[q] = c + q < ncand ? cand[c + q] : -1;
                const float4 v = W.p[base + max(pc[q], 0)];
                cx[q] = (double)v.x;
                cy[q] = (double)v.y;
                cz[q] = (double)v.z;
                s1[q] = 0.0;
            }
            for_members<2>(n, [&](int k) { return W.p[base + k]; }, [&](int k, float4 v) {
                const double x = (double)v.x, y = (double)v.y, z = (double)v.z, m = (double)v.w;
#pragma unroll
                for (int q = 0; q < NC; ++q) {
                    if (pc[q] < 0) continue;  // uniform
                    const double dx = cx[q] - x, dy = cy[q] - y, dz = cz[q] - z;
                    const double r2 = dx * dx + dy * dy + dz * dz;
                    const double t = m * rsqrt64(r2 + eps2g);
                    s1[q] += k == pc[q] || (eps2g == 0.0 && r2 == 0.0) ? 0.0 : t;
                }
            });
            bsum<NC>(s1, smd);
#pragma unroll
            for (int q = 0; q < NC; ++q)
                if (pc[q] >= 0 && (s1[q] > cbest || (s1[q] == cbest && pc[q] < cpos))) { cbest = s1[q]; cpos = pc[q]; }
        }
        if (first + MAX_CAND >= total_cand) break;
    }
    if (tid == 0) s_p = cpos;
    __syncthreads();
    const int p = s_p;
    // 4. velocity frame
    double fr[4] = {0, 0, 0, 0};
    if (frame_type == 1) {
        int64_t nref = (int64_t)ceil(frac_ref * (double)n);
        if (nref < n_ref_min) nref = n_ref_min;
        if (nref > n) nref = n;
        const float4 vp = W.p[base + p];
        const int px = (int)vp.x, py = (int)vp.y, pz = (int)vp.z;
        auto member = [&](int k) { return W.p[base + k]; };
        auto dist2 = [&](float4 v) -> uint64_t {
            const int64_t dx = min_image((int)v.x - px, gb), dy = min_image((int)v.y - py, gb),
                          dz = min_image((int)v.z - pz, gb);
            return (uint64_t)(dx * dx + dy * dy + dz * dz);
        };
        // the key of rank nref - 1: the bin that holds it, then its keys in
        // LDS, each ranked against the others
        uint64_t prefix = 0;
        uint32_t rank = (uint32_t)(nref - 1);
        auto find_bucket = [&]() {
            uint32_t loc = 0;
            for (int k = 0; k < BPT; ++k) loc += hist[tid * BPT + k];
            uint32_t tot;
            const uint32_t ex = bscan(loc, smu, &tot);
            if (rank >= ex && rank < ex + loc) {
                uint32_t c = ex;
                for (int k = 0; k < BPT; ++k) {
                    const uint32_t hh = hist[tid * BPT + k];
                    if (rank < c + hh) { s_bucket = tid * BPT + k; s_below = c; break; }
                    c += hh;
                }
            }
            __syncthreads();
        };
        for (int k = tid; k < SEL_BINS; k += blockDim.x) hist[k] = 0;
        if (tid == 0) s_n = 0;
        __syncthreads();
        for_members<4>(n, member, [&](int k, float4 v) { atomicAdd(&hist[sel_bin(dist2(v))], 1u); });
        __syncthreads();
        find_bucket();
        const int bucket = s_bucket;
        const uint32_t in_bucket = hist[bucket];
        __syncthreads();
        if (in_bucket <= (uint32_t)SEL_LIST) {
            const uint32_t want = rank - s_below;
            for_members<4>(n, member, [&](int k, float4 v) {
                const uint64_t d2 = dist2(v);
                if (sel_bin(d2) == bucket) list[atomicAdd(&s_n, 1)] = (d2 << 22) | (uint64_t)k;
            });
            __syncthreads();
            for (int e = tid; e < (int)in_bucket; e += blockDim.x) {
                const uint64_t key = list[e];
                uint32_t r = 0;
                for (uint32_t j = 0; j < in_bucket; ++j) r += list[j] < key ? 1u : 0u;
                if (r == want) s_key = key;
            }
            __syncthreads();
            prefix = s_key;
        } else {
            // a crowded bin (coincident members): radix select of the whole
            // keys, 11 bits at a time from the top
            for (int shift = 55; shift >= 0; shift -= 11) {
                for (int k = tid; k < 2048; k += blockDim.x) hist[k] = 0;
                __syncthreads();
                const uint64_t hmask = (shift + 11 >= 64) ? 0ull : ~((1ull << (shift + 11)) - 1);
                for (int k = tid; k < n; k += blockDim.x) {
                    const uint64_t key = ref_key(W, base, k, px, py, pz, gb);
                    if (((key ^ prefix) & hmask) == 0) atomicAdd(&hist[(key >> shift) & 2047u], 1u);
                }
                __syncthreads();
                find_bucket();
                prefix |= (uint64_t)s_bucket << shift;
                rank -= s_below;
                __syncthreads();
            }
        }
        for_members<4>(n, member, [&](int k, float4 v) {
            if (((dist2(v) << 22) | (uint64_t)k) > prefix) return;
            const double m = uniform ? mass_value : (double)v.w;
            const float4 u = W.v[base + k];
            fr[0] += m;
            fr[1] += m * (double)u.x;
            fr[2] += m * (double)u.y;
            fr[3] += m * (double)u.z;
        });
    } else {
        for (int k = tid; k < n; k += blockDim.x) {
            const double m = uniform ? mass_value : (double)W.p[base + k].w;
            const float4 u = W.v[base + k];
            fr[0] += m;
            fr[1] += m * (double)u.x;
            fr[2] += m * (double)u.y;
            fr[3] += m * (double)u.z;
        }
    }
    bsum<4>(fr, smd);
    const double vr0 = fr[1] / fr[0], vr1 = fr[2] / fr[0], vr2 = fr[3] / fr[0];
    // 5. energies, removal and stable in-place compaction; survivors
    // keep their sums, removed members go to the side list.  A chunk is CI
    // members a thread, read before any is rewritten; the members before the
    // first removed one stay where they are.
    constexpr int CI = 4;
    const int since0 = Rm.since[g];
    static_assert(CI * NW <= 64, "one wavefront scans the chunk's kept counts");
    uint32_t kept = 0, gone = 0;
    for (int c0 = 0; c0 < n; c0 += CI * BS) {
        float4 P[CI], V[CI];
        double a[CI];
#pragma unroll
        for (int u = 0; u < CI; ++u) {
            const int k = base + min(c0 + u * BS + tid, n - 1);
            P[u] = W.p[k];
            V[u] = W.v[k];
            a[u] = acc[k];
        }
        uint64_t kb[CI];  // kept members of the wavefront
#pragma unroll
        for (int u = 0; u < CI; ++u) {
            bool keep = false;
            if (c0 + u * BS + tid < n) {
                const double m = uniform ? mass_value : (double)P[u].w;
                const double ph = scale * (uniform ? mass_value : 1.0) * a[u];
                const double dx = (double)V[u].x - vr0, dy = (double)V[u].y - vr1, dz = (double)V[u].z - vr2;
                const double T = 0.5 * m * (dx * dx + dy * dy + dz * dz);
                const double Wp = m * ph;
                const double E = beta_E * T + Wp;
                keep = !(E >= 0.0);
                phi[__float_as_int(V[u].w)] = ph;
            }
            kb[u] = __ballot(keep);
            if (lane == 0) ckept[u * NW + w] = (uint32_t)__popcll(kb[u]);
        }
        __syncthreads();
        // kept members before (u, w) in the chunk
        const uint32_t mine = lane < CI * NW ? ckept[lane] : 0u;
        const uint32_t inc = wscan(mine);
        const uint32_t tot = __shfl(inc, CI * NW - 1, 64);
#pragma unroll
        for (int u = 0; u < CI; ++u) {
            const int ci = u * BS + tid;
            const uint32_t kbefore = __shfl(inc - mine, u * NW + w, 64) + (uint32_t)__popcll(kb[u] & lanemask_lt());
            if (c0 + ci >= n) continue;
            if ((kb[u] >> lane) & 1ull) {
                const int dst = base + (int)(kept + kbefore);
                if (dst != base + c0 + ci) {
                    W.p[dst] = P[u];
                    W.v[dst] = V[u];
                    acc[dst] = a[u];
                }
            } else {
                const int64_t k = base + (int)(gone + (uint32_t)ci - kbefore);
                if (uniform) {
                    Rm.p[3 * k] = P[u].x;
                    Rm.p[3 * k + 1] = P[u].y;
                    Rm.p[3 * k + 2] = P[u].z;
                } else {
                    reinterpret_cast<float4*>(Rm.p)[k] = P[u];
                }
            }
        }
        kept += tot;
        gone += (uint32_t)min(CI * BS, n - c0) - tot;
        __syncthreads();
    }
    // the next pass subtracts the removed terms while those removed since
    // the last full recompute stay within a quarter of the survivors; else the
    // sums start from zero
    const int since = since0 + (int)gone;
    const bool incr = 4 * (int64_t)since <= (int64_t)kept;
    if (!incr && kept != (uint32_t)n)
        for (int k = tid; k < (int)kept; k += blockDim.x) acc[base + k] = 0.0;
    if (kept == (uint32_t)n) {
        for (int k = tid; k < n; k += blockDim.x) bound[__float_as_int(W.v[base + k].w)] = 1;
        if (tid == 0) state[g] = ST_BOUND;
    } else if ((int)kept < n_min) {
        if (tid == 0) state[g] = ST_DISSOLVED;
    }
    if (tid == 0) {
        cnt[g] = (int)kept;
        iters[g] += 1;
        Rm.nrm[g] = (int)gone;
        Rm.since[g] = incr ? since : 0;
        Rm.mode[g] = incr ? 1 : 0;
    }
}

// ---- persistent, graph-replayed passes -------------------------------------
// Device-side plan of one pass: the active groups in the given order (the
// group tables come in decreasing size, so the largest work is queued first)
// and the prefix of their work-item counts; item = (i-tile of 64, j-range).
struct UbPlan {
    int n_active;     // groups scheduled in this pass
    int total_items;
    int head;         // work-queue head
    int remaining;    // groups still active after the pass (read by the host)
    int stuck;        // active groups that reached max_iter
    int pad[3];
    double pairs;     // ordered pairs scheduled since the last reset
};

__global__ void k_ub_plan_reset(UbPlan* plan) {
    if (threadIdx.x == 0) plan->pairs = 0.0;
}

// Work items of a full recompute of T tiles of 64 members: every pair of
// tiles once.  Item = (row tile a, chunk c of C column tiles from c C on),
// columns from the diagonal on, so chunk c has rows 0 .. min(T, (c + 1) C) - 1.
__device__ __forceinline__ uint32_t full_items(int T, int C) {
    const int last = (T + C - 1) / C - 1;  // chunks before the last have all their rows
    return (uint32_t)((int64_t)C * last * (last + 1) / 2) + (uint32_t)T;
}
// chunk and row of item l
__device__ __forceinline__ void full_item(int l, int C, int& c, int& a) {
    c = (int)((sqrtf(8.f * (float)l / (float)C + 1.f) - 1.f) * 0.5f);
    while ((int64_t)C * c * (c + 1) / 2 > l) --c;
    while ((int64_t)C * (c + 1) * (c + 2) / 2 <= l) ++c;
    a = l - (int)((int64_t)C * c * (c + 1) / 2);
}

constexpr int PLAN_T = 1024;

__global__ __launch_bounds__(PLAN_T) void k_ub_plan(int ng, const int* __restrict__ cnt, const int* __restrict__ state,
                                                    const int32_t* __restrict__ iters, int max_iter, int jchunk,
                                                    const int* __restrict__ nrm, const int* __restrict__ mode,
                                                    int* __restrict__ act, int* __restrict__ item_off, UbPlan* plan) {
    __shared__ uint32_t sm[32];
    __shared__ double smd[PLAN_T / 64];
    uint32_t carry_g = 0, carry_i = 0;
    double pairs = 0.0;
    for (int base = 0; base < ng; base += PLAN_T) {
        const int g = base + (int)threadIdx.x;
        const bool on = g < ng && state[g] == ST_ACTIVE && iters[g] < max_iter;
        const int n = on ? cnt[g] : 0;
        // j over all members (full) or over the members removed last pass
        const int nj = (on && mode[g]) ? nrm[g] : n;
        pairs += (double)n * (double)(on && mode[g] ? nj : (n > 0 ? n - 1 : 0));
        const uint32_t items = !on ? 0u : mode[g] ? (uint32_t)(((n + 63) / 64) * ((nj + jchunk - 1) / jchunk))
                                                  : full_items((n + 63) / 64, jchunk / 64);
        uint32_t tg, ti;
        const uint32_t pg = bscan(on ? 1u : 0u, sm, &tg);
        const uint32_t pi = bscan(items, sm, &ti);
        if (on) {
            act[carry_g + pg] = g;
            item_off[carry_g + pg] = (int)(carry_i + pi);
        }
        carry_g += tg;
        carry_i += ti;
    }
    pairs = wsum(pairs);
    if (__lane_id() == 0) smd[threadIdx.x >> 6] = pairs;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tp = 0.0;
        for (int k = 0; k < PLAN_T / 64; ++k) tp += smd[k];
        item_off[carry_g] = (int)carry_i;
        plan->n_active = (int)carry_g;
        plan->total_items = (int)carry_i;
        plan->head = 0;
        plan->pairs += tp;
    }
}

// Persistent potential kernel: wavefront w takes item w first, then pops
// items nwaves, nwaves + 1, ... from the queue until it is empty (so a light
// pass costs no burst of atomics on the queue head, and wavefronts beyond the
// item count leave at once); lane = one i of a 64-row tile.
//
// A full recompute takes every pair of tiles once: the lane's own sum runs
// over the columns, the reciprocal distances also go to LDS, and lane j then
// sums its column over the rows -- the same FP32 terms in the same order as
// if its own row had been summed (a pair's squared distance is the same
// either way round).  Bound by VALU issue and, a tenth, by the columns' FP64
// atomics: 10 instruction slots for two ordered pairs against 9 for one (17 KB
// of LDS a wavefront, eight wavefronts a CU; columns in two halves of 32, 16
// wavefronts a CU, were 9% slower).  2.1e10 ordered pairs, largest group
// 120 k: 5.28 -> 3.86 ms; incremental passes lose occupancy (0.83 -> 1.01 ms
// for the first, the only long one).
constexpr int COLS = 68;  // floats a column of 64, padded: eight lanes' 16-byte reads cover all banks
constexpr int STAGE = 512;  // removed members staged at a time
constexpr int UBP = 128;  // threads per workgroup (two slices of LDS below 64 KB)
constexpr int UB_LDS = 64 * COLS * 4 + 64 * 16 + 64 * 4;  // columns, staged j, masses of the rows

// One lane's row of a 64 x 64 tile: the FP32 sum over the members q in
// order, and every reciprocal distance to its column's LDS (stride COLS).
// ZERO: eps = 0, coincident pairs are left out.  q is uniform: for a full
// tile it points to global memory, and the members come through the scalar
// cache (as LDS broadcasts, 8 clocks each on a CU's LDS, they bound the
// kernel: 4.4 ms against 3.9 ms); the last tile of a group is staged in LDS
// and padded.
template <bool UNIFORM, bool ZERO>
__device__ __forceinline__ float tile_rows(const float4* __restrict__ q, float4 pi, float eps2, float* out) {
    // the next block's members are asked for before this block is worked on
    constexpr int U = 8, BLOCKS = UNIFORM ? 4 : 1;
    float4 a[U], b[U];
    float accf = 0.f;
    auto block = [&](const float4 (&v)[U], int t) __attribute__((always_inline)) {
        float r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float dx = pi.x - v[u].x, dy = pi.y - v[u].y, dz = pi.z - v[u].z;
            const float s2 = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, eps2)));
            r[u] = __builtin_amdgcn_rsqf(s2);
            if (ZERO) r[u] = s2 > 0.f ? r[u] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            accf = UNIFORM ? accf + r[u] : fmaf(v[u].w, r[u], accf);
            out[(t + u) * COLS] = r[u];
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = q[u];
    // (with masses the unrolled loop took 270 registers, one wavefront a SIMD)
#pragma unroll BLOCKS
    for (int t = 0; t < 64; t += 2 * U) {
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = q[t + U + u];
        __builtin_amdgcn_sched_barrier(0);
        block(a, t);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 2 * U < 64) {
#pragma unroll
            for (int u = 0; u < U; ++u) a[u] = q[t + 2 * U + u];
        }
        __builtin_amdgcn_sched_barrier(0);
        block(b, t + U);
        __builtin_amdgcn_sched_barrier(0);
    }
    return accf;
}

// The sum of one column over the 64 rows in order.
template <bool UNIFORM>
__device__ __forceinline__ float tile_column(const float* cj, const float* smi) {
    float cs = 0.f;
#pragma unroll
    for (int t0 = 0; t0 < 64; t0 += 32) {
        float4 r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) r[u] = *reinterpret_cast<const float4*>(cj + t0 + 4 * u);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (UNIFORM) {
                cs = (((cs + r[u].x) + r[u].y) + r[u].z) + r[u].w;
            } else {
                const float4 m = *reinterpret_cast<const float4*>(smi + t0 + 4 * u);
                cs = fmaf(m.w, r[u].w, fmaf(m.z, r[u].z, fmaf(m.y, r[u].y, fmaf(m.x, r[u].x, cs))));
            }
        }
    }
    return cs;
}

template <bool UNIFORM>
__global__ __launch_bounds__(UBP, 2) void k_ub_potential_p(UbPlan* plan, const int* __restrict__ act,
                                                       const int* __restrict__ item_off, const int32_t* __restrict__ off,
                                                       const int* __restrict__ cnt, const float4* __restrict__ wp,
                                                       const float* __restrict__ rp, const int* __restrict__ nrm,
                                                       const int* __restrict__ mode, float eps2,
                                                       double* __restrict__ acc, int jchunk) {
    extern __shared__ __align__(16) char ldsall[];
    const int lane = __lane_id(), wv = threadIdx.x >> 6;
    // the wavefront's slice: columns, one tile of members and the rows' masses
    char* slice = ldsall + wv * UB_LDS;
    float* col = reinterpret_cast<float*>(slice);
    float4* sjt = reinterpret_cast<float4*>(slice + 64 * COLS * 4);
    float* smi = reinterpret_cast<float*>(slice + 64 * COLS * 4 + 64 * 16);
    const int na = plan->n_active, total = plan->total_items;
    const int nwaves = (int)(gridDim.x * (blockDim.x >> 6));
    int it = (int)(blockIdx.x * (blockDim.x >> 6)) + wv;
    for (;; ) {
        it = __builtin_amdgcn_readfirstlane(it);
        if (it >= total) break;
        // the group holding item `it`
        int lo = 0, hi = na - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (item_off[mid] <= it) lo = mid; else hi = mid - 1;
        }
        const int g = act[lo];
        const int base = off[g], n = cnt[g];
        const int local = it - item_off[lo];
        double accd = 0.0;
        int i;
        if (mode[g] != 0) {
            // incremental: j over last pass's removed members, staged in LDS
            const int nj = nrm[g];
            const int njc = (nj + jchunk - 1) / jchunk;
            const int i0 = (local / njc) * 64, j0 = (local % njc) * jchunk;
            const int j1 = min(nj, j0 + jchunk);
            i = i0 + lane;
            const float4 pi = i < n ? wp[base + i] : make_float4(0.f, 0.f, 0.f, 0.f);
            float4* sj = reinterpret_cast<float4*>(slice);
            for (int jb = j0; jb < j1; jb += STAGE) {
                const int jn = min(STAGE, j1 - jb);
                __builtin_amdgcn_wave_barrier();
                for (int t = lane; t < jn; t += 64) {
                    const int64_t k = base + jb + t;
                    sj[t] = UNIFORM ? make_float4(rp[3 * k], rp[3 * k + 1], rp[3 * k + 2], 1.f)
                                    : reinterpret_cast<const float4*>(rp)[k];
                }
                __builtin_amdgcn_wave_barrier();
                // a removed member is never i itself; only coincident pairs need care
                for (int t0 = 0; t0 < jn; t0 += 64) {
                    const int t1 = min(t0 + 64, jn);
                    accd -= (double)(eps2 == 0.f ? tile_sum<UNIFORM, true>(sj, t0, t1, pi.x, pi.y, pi.z, eps2, jb, -1)
                                                 : tile_sum<UNIFORM, false>(sj, t0, t1, pi.x, pi.y, pi.z, eps2, jb, -1));
                }
            }
        } else {
            const int T = (n + 63) / 64, C = jchunk / 64;
            int c, a;
            full_item(local, C, c, a);
            i = a * 64 + lane;
            const float4 pi = i < n ? wp[base + i] : make_float4(0.f, 0.f, 0.f, 0.f);
            if (!UNIFORM) smi[lane] = pi.w;
            for (int b = max(a, c * C); b < min(T, (c + 1) * C); ++b) {
                const int jb = b * 64, jn = min(64, n - jb);
                __builtin_amdgcn_wave_barrier();
                if (b == a || jn < 64 || eps2 == 0.f) {
                    // (beyond the last member: infinitely far, 1 / r = 0)
                    sjt[lane] = lane < jn ? wp[base + jb + lane] : make_float4(INFINITY, 0.f, 0.f, 0.f);
                    __builtin_amdgcn_wave_barrier();
                }
                if (b == a) {  // the diagonal tile, row by row
                    accd += (double)tile_sum<UNIFORM, true>(sjt, 0, jn, pi.x, pi.y, pi.z, eps2, jb, i);
                    continue;
                }
                // rows before the last tile are all there
                if (jn < 64 || eps2 == 0.f)
                    accd += (double)(eps2 == 0.f ? tile_rows<UNIFORM, true>(sjt, pi, eps2, col + lane)
                                                 : tile_rows<UNIFORM, false>(sjt, pi, eps2, col + lane));
                else
                    accd += (double)tile_rows<UNIFORM, false>(wp + base + jb, pi, eps2, col + lane);
                __builtin_amdgcn_wave_barrier();
                const float cs = tile_column<UNIFORM>(col + lane * COLS, smi);
                if (lane < jn) atomicAdd(&acc[base + jb + lane], (double)cs);
            }
        }
        if (i < n) atomicAdd(&acc[base + i], accd);
        // (a light pass has no more items than wavefronts: thousands of pops
        // of an empty queue, one address, cost 25 us)
        if (total <= nwaves) break;
        int nx = 0;
        if (lane == 0) nx = atomicAdd(&plan->head, 1);
        it = nwaves + __shfl(nx, 0, 64);
    }
}

__global__ __launch_bounds__(PLAN_T) void k_ub_count(int ng, const int* __restrict__ state,
                                                     const int32_t* __restrict__ iters, int max_iter, UbPlan* plan) {
    __shared__ uint32_t sm[32];
    uint32_t rem = 0, stuck = 0;
    for (int g = threadIdx.x; g < ng; g += PLAN_T) {
        if (state[g] != ST_ACTIVE) continue;
        if (iters[g] < max_iter) ++rem; else ++stuck;
    }
    uint32_t tr, ts;
    bscan(rem, sm, &tr);
    bscan(stuck, sm, &ts);
    if (threadIdx.x == 0) {
        plan->remaining = (int)tr;
        plan->stuck = (int)ts;
    }
}

}  // namespace
}  // namespace vr

using namespace vr;

namespace {

constexpr int PASSES_PER_GRAPH = 4;

// Everything a captured pass depends on; a cached graph is reused only when
// all of it is unchanged.
struct UbGraphKey {
    const void* ptrs[16];
    int ints[12];
    double dbls[6];
};

void ub_graph_release(vr_ctx* ctx) {
    if (ctx->ub_exec) (void)hipGraphExecDestroy((hipGraphExec_t)ctx->ub_exec);
    if (ctx->ub_graph) (void)hipGraphDestroy((hipGraph_t)ctx->ub_graph);
    ctx->ub_exec = nullptr;
    ctx->ub_graph = nullptr;
    ctx->ub_key.clear();
}

// One pass = plan (active list and work items) -> persistent potential over
// the item queue -> one workgroup per active group for frame, energies,
// compaction and, where the next pass recomputes, zeros for its sums.  Passes are
// captured PASSES_PER_GRAPH at a time in a graph that is replayed until no
// group is active; the host reads two counters per replay.
int unbind_persistent(vr_ctx* ctx, const vr_particles* p, int32_t ng, const int32_t* offsets,
                      const vr_unbind_params* up, const Members& W, const Removed& Rm, double* acc, int* cnt, int* state,
                      int32_t* iters, uint8_t* bound, double* phi, int* act, const int* nbig, float eps2f,
                      double eps2g, double scale, hipStream_t st) {
    VR_WS(plan, ctx, UbPlan, WS_D4, 1);
    VR_WS(item_off, ctx, int, WS_D5, (int64_t)ng + 1);
    const bool uniform = W.uniform != 0;
    const int jchunk = ctx->unbind_jchunk;
    const size_t lds = (size_t)(UBP / 64) * UB_LDS;
    int bpc = 0;
    if (uniform)
        VR_HIP(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&bpc, k_ub_potential_p<true>, UBP, lds));
    else
        VR_HIP(ctx, hipOccupancyMaxActiveBlocksPerMultiprocessor(&bpc, k_ub_potential_p<false>, UBP, lds));
    if (ctx->unbind_bpc > 0 && ctx->unbind_bpc < bpc) bpc = ctx->unbind_bpc;
    if (bpc < 1) bpc = 1;
    const unsigned pgrid = (unsigned)(ctx->num_cus * bpc);

    UbGraphKey key;
    std::memset(&key, 0, sizeof key);
    const void* kp[16] = {offsets, W.p, W.v, acc, cnt, state, iters, bound, phi, act, Rm.p, Rm.nrm, Rm.since, Rm.mode,
                          nbig, nullptr};
    std::memcpy(key.ptrs, kp, sizeof kp);
    const int ki[12] = {ng, up->max_iter, jchunk, 0, (int)pgrid, up->n_min, up->n_ref_min, up->frame_type,
                        p->grid_bits, uniform ? 1 : 0, 0, 0};
    std::memcpy(key.ints, ki, sizeof ki);
    const double kd[6] = {(double)eps2f, eps2g, scale, p->mass_value, up->beta_E, up->frac_ref};
    std::memcpy(key.dbls, kd, sizeof kd);
    // plan and item_off are workspace too: their addresses are part of the key
    std::string kbytes((const char*)&key, sizeof key);
    kbytes.append((const char*)&plan, sizeof plan);
    kbytes.append((const char*)&item_off, sizeof item_off);

    if (!ctx->ub_exec || ctx->ub_key != kbytes) {
        ub_graph_release(ctx);
        if (!ctx->cap_stream) VR_HIP(ctx, hipStreamCreateWithFlags((hipStream_t*)&ctx->cap_stream, hipStreamNonBlocking));
        hipStream_t cs = (hipStream_t)ctx->cap_stream;
        VR_HIP(ctx, hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
        for (int k = 0; k < PASSES_PER_GRAPH; ++k) {
            hipLaunchKernelGGL(k_ub_plan, dim3(1), dim3(PLAN_T), 0, cs, ng, cnt, state, iters, up->max_iter, jchunk,
                               Rm.nrm, Rm.mode, act, item_off, plan);
            if (uniform)
                hipLaunchKernelGGL(k_ub_potential_p<true>, dim3(pgrid), dim3(UBP), lds, cs, plan, act, item_off,
                                   offsets, cnt, W.p, Rm.p, Rm.nrm, Rm.mode, eps2f, acc, jchunk);
            else
                hipLaunchKernelGGL(k_ub_potential_p<false>, dim3(pgrid), dim3(UBP), lds, cs, plan, act, item_off,
                                   offsets, cnt, W.p, Rm.p, Rm.nrm, Rm.mode, eps2f, acc, jchunk);
            hipLaunchKernelGGL(k_ub_group<UB_WIDE>, dim3(ng), dim3(UB_WIDE), 0, cs, (const int*)nullptr, offsets, cnt,
                               state, iters, W, Rm, acc, eps2g, scale, p->mass_value, up->beta_E, up->frac_ref,
                               up->n_min, up->n_ref_min, up->frame_type, p->grid_bits, bound, phi, up->max_iter, nbig);
            hipLaunchKernelGGL(k_ub_group<UB>, dim3(ng), dim3(UB), 0, cs, (const int*)nullptr, offsets, cnt, state,
                               iters, W, Rm, acc, eps2g, scale, p->mass_value, up->beta_E, up->frac_ref, up->n_min,
                               up->n_ref_min, up->frame_type, p->grid_bits, bound, phi, up->max_iter, nbig);
        }
        hipLaunchKernelGGL(k_ub_count, dim3(1), dim3(PLAN_T), 0, cs, ng, state, iters, up->max_iter, plan);
        hipGraph_t graph = nullptr;
        const hipError_t le = hipGetLastError();
        const hipError_t ce = hipStreamEndCapture(cs, &graph);
        if (le != hipSuccess || ce != hipSuccess || !graph) {
            if (graph) (void)hipGraphDestroy(graph);
            return set_err(ctx, VR_ERR_HIP, "capturing the unbinding passes failed: %s",
                           hipGetErrorString(le != hipSuccess ? le : ce));
        }
        ctx->ub_graph = graph;
        hipGraphExec_t exec = nullptr;
        const hipError_t ie = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
        if (ie != hipSuccess) {
            ub_graph_release(ctx);
            return set_err(ctx, VR_ERR_HIP, "hipGraphInstantiate: %s", hipGetErrorString(ie));
        }
        ctx->ub_exec = exec;
        ctx->ub_key = kbytes;
    }

    hipLaunchKernelGGL(k_ub_plan_reset, dim3(1), dim3(64), 0, st, plan);
    VR_LAUNCH_CHECK(ctx);
    hipEvent_t e0 = nullptr;
    if (ctx->timing) {
        e0 = timer_event(ctx);
        (void)hipEventRecord(e0, st);
    }
    int* counters = reinterpret_cast<int*>(ctx->pinned);
    for (int launch = 0;; ++launch) {
        VR_HIP(ctx, hipGraphLaunch((hipGraphExec_t)ctx->ub_exec, st));
        VR_HIP(ctx, hipMemcpyAsync(counters, &plan->remaining, 2 * sizeof(int), hipMemcpyDeviceToHost, st));
        VR_HIP(ctx, hipStreamSynchronize(st));
        if (counters[0] == 0) break;
        // every replay advances each remaining group by PASSES_PER_GRAPH
        // passes, so the loop ends after max_iter / PASSES_PER_GRAPH replays
        if ((int64_t)launch * PASSES_PER_GRAPH > (int64_t)up->max_iter + PASSES_PER_GRAPH)
            return set_err(ctx, VR_ERR_HIP, "unbinding replays did not advance");
    }
    const int stuck = counters[1];
    double pairs = 0.0;
    if (ctx->timing) {
        hipEvent_t e1 = timer_event(ctx);
        (void)hipEventRecord(e1, st);
        VR_HIP(ctx, hipMemcpyAsync(ctx->pinned, &plan->pairs, sizeof(double), hipMemcpyDeviceToHost, st));
        VR_HIP(ctx, hipStreamSynchronize(st));
        std::memcpy(&pairs, ctx->pinned, sizeof(double));
        timer_push(ctx, "unbind_persistent", e0, e1, pairs);
    }
    if (stuck > 0)
        return set_err(ctx, VR_ERR_NOT_CONVERGED, "%d groups still lose members after %d passes", stuck, up->max_iter);
    return VR_OK;
}

}  // namespace

namespace vr {
void unbind_release(vr_ctx* ctx) { ub_graph_release(ctx); }
}  // namespace vr

extern "C" int vr_unbind(vr_ctx* ctx, const vr_particles* p, int32_t n_groups, const int32_t* offsets,
                         const int32_t* members, const vr_unbind_params* up, uint8_t* bound, double* phi,
                         int32_t* iters, void* stream) {
    if (!ctx) return VR_ERR_INVALID_ARG;
    int rc = check_particles(ctx, p, true);
    if (rc) return rc;
    if ((rc = check_hosts(ctx, n_groups, offsets, members))) return rc;
    if (!up) return set_err(ctx, VR_ERR_INVALID_ARG, "params is NULL");
    if (!(up->eps >= 0) || !(up->G > 0) || up->n_min < 1 || up->max_iter < 1 || up->n_ref_min < 1 ||
        !(up->frac_ref >= 0) || (up->frame_type != 0 && up->frame_type != 1))
        return set_err(ctx, VR_ERR_INVALID_ARG, "bad unbinding parameters");
    if (up->tile != 0 && (up->tile < 64 || up->tile > 4096 || (up->tile & 63)))
        return set_err(ctx, VR_ERR_INVALID_ARG, "tile must be 0 or a multiple of 64 in [64, 4096]");
    if (n_groups == 0) return VR_OK;
    if (!bound || !phi || !iters) return set_err(ctx, VR_ERR_INVALID_ARG, "NULL output");
    VR_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    std::vector<int32_t> off(n_groups + 1);
    int rc0 = copy_to_host(ctx, off.data(), offsets, (n_groups + 1) * sizeof(int32_t), st);
    if (rc0) return rc0;
    if (off[0] != 0) return set_err(ctx, VR_ERR_INVALID_ARG, "offsets[0] must be 0");
    for (int g = 0; g < n_groups; ++g) {
        if (off[g + 1] < off[g]) return set_err(ctx, VR_ERR_INVALID_ARG, "offsets must be non-decreasing");
        if (off[g + 1] - off[g] > (1 << 22)) return set_err(ctx, VR_ERR_UNSUPPORTED, "group %d exceeds 2^22 members", g);
    }
    const int64_t M = off[n_groups];
    if (M > p->n) return set_err(ctx, VR_ERR_INVALID_ARG, "more members than particles");
    const bool uniform = p->mass == nullptr;
    Members W;
    VR_WS(wp, ctx, float4, WS_C1, M);
    VR_WS(wvel, ctx, float4, WS_C4, M);
    W.p = wp;
    W.v = wvel;
    W.uniform = uniform ? 1 : 0;
    VR_WS(acc, ctx, double, WS_C8, M);
    VR_WS(cnt, ctx, int, WS_D0, n_groups);
    VR_WS(state, ctx, int, WS_D1, n_groups);
    VR_WS(act, ctx, int, WS_D2, n_groups);
    Removed Rm;
    VR_WS(rp, ctx, float, WS_B0, (uniform ? 3 : 4) * M);
    VR_WS(nrm, ctx, int, WS_B4, n_groups); VR_WS(since, ctx, int, WS_B5, n_groups); VR_WS(mode, ctx, int, WS_B6, n_groups);
    Rm.p = rp; Rm.nrm = nrm; Rm.since = since; Rm.mode = mode;
    VR_WS(nbig, ctx, int, WS_D6, 1);
    {
        int rc = fill_i32(ctx, nbig, n_groups, 1, st);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(k_ub_state, dim3(grid_for(n_groups, 256)), dim3(256), 0, st, n_groups, offsets, up->n_min,
                       ctx->unbind_wide, Rm, cnt, state, iters, nbig);
    VR_LAUNCH_CHECK(ctx);
    hipLaunchKernelGGL(k_ub_init, dim3(grid_for(M, 256)), dim3(256), 0, st, n_groups, (int64_t)M, offsets, members,
                       p->qx, p->qy, p->qz, p->vx, p->vy, p->vz, p->mass, p->grid_bits, W, acc, bound, phi);
    VR_LAUNCH_CHECK(ctx);
    const double unit = p->box / ldexp(1.0, p->grid_bits);
    const double epsg = up->eps / unit;
    const double eps2g = epsg * epsg;
    const float eps2f = (float)eps2g;
    if (eps2f > 0.f && eps2f < FLT_MIN)
        return set_err(ctx, VR_ERR_UNSUPPORTED, "softening eps = %g is below the FP32 normal range in grid units",
                       up->eps);
    const double scale = -up->G / unit;  // potential = scale * mass * sum(1/r) in grid units
    int tile = up->tile ? up->tile : (ctx->tuned_tile ? ctx->tuned_tile : 256);
    if (up->persistent)
        return unbind_persistent(ctx, p, n_groups, offsets, up, W, Rm, acc, cnt, state, iters, bound, phi, act, nbig,
                                 eps2f, eps2g, scale, st);
    std::vector<int> hcnt(n_groups), hstate(n_groups), hact;
    std::vector<int4> items;
    for (int pass = 0;; ++pass) {
        if (int rc1 = copy_to_host(ctx, hcnt.data(), cnt, n_groups * sizeof(int), st)) return rc1;
        if (int rc1 = copy_to_host(ctx, hstate.data(), state, n_groups * sizeof(int), st)) return rc1;
        hact.clear();
        items.clear();
        double pairs = 0.0, nmem = 0.0;
        for (int g = 0; g < n_groups; ++g) {
            if (hstate[g] != ST_ACTIVE) continue;
            hact.push_back(g);
            const int n = hcnt[g];
            pairs += (double)n * (double)(n - 1);
            nmem += n;
            const int jchunk = ctx->unbind_jchunk;
            for (int i0 = 0; i0 < n; i0 += UB)
                for (int j0 = 0; j0 < n; j0 += jchunk) items.push_back(make_int4(g, i0, j0, std::min(n, j0 + jchunk)));
        }
        if (hact.empty()) break;
        if (pass >= up->max_iter)
            return set_err(ctx, VR_ERR_NOT_CONVERGED, "%zu groups still lose members after %d passes", hact.size(),
                           up->max_iter);
        const int na = (int)hact.size();
        const int64_t ni = (int64_t)items.size();
        VR_WS(items_d, ctx, int4, WS_D3, ni);
        VR_HIP(ctx, hipMemcpyAsync(act, hact.data(), na * sizeof(int), hipMemcpyHostToDevice, st));
        VR_HIP(ctx, hipMemcpyAsync(items_d, items.data(), ni * sizeof(int4), hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_ub_zero, dim3(na), dim3(256), 0, st, na, act, offsets, cnt, acc);
        VR_LAUNCH_CHECK(ctx);
        const size_t lds = (size_t)tile * sizeof(float4);
        if (uniform)
            VR_TIMED(ctx, "unbind_potential", st, pairs,
                     hipLaunchKernelGGL(k_ub_potential<true>, dim3((unsigned)ni), dim3(UB), lds, st, items_d, offsets,
                                        cnt, W, eps2f, acc, tile));
        else
            VR_TIMED(ctx, "unbind_potential", st, pairs,
                     hipLaunchKernelGGL(k_ub_potential<false>, dim3((unsigned)ni), dim3(UB), lds, st, items_d, offsets,
                                        cnt, W, eps2f, acc, tile));
        VR_LAUNCH_CHECK(ctx);
        VR_TIMED(ctx, "unbind_group", st, nmem,
                 hipLaunchKernelGGL(k_ub_group<UB>, dim3(na), dim3(UB), 0, st, act, offsets, cnt, state, iters, W, Rm,
                                    acc, eps2g, scale, p->mass_value, up->beta_E, up->frac_ref, up->n_min,
                                    up->n_ref_min, up->frame_type, p->grid_bits, bound, phi, up->max_iter,
                                    (const int*)nullptr));
        VR_LAUNCH_CHECK(ctx);
    }
    return VR_OK;
}
