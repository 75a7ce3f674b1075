// vr_knn.hip -- local velocity density ratio R = ln(f_l / f_bg) (Sec. 2.2).
//
// Members are ordered by a KD tree: the device-wide builder splits the hosts
// at medians of the widest dimension down to buckets of a few hundred to
// 2048 members, and one workgroup per bucket (k_buckets) finishes the tree
// in LDS down to leaves of 32, all full but the bucket's last.  A leaf is 32
// consecutive slots; buckets have at most 64 leaves, so one load a lane
// tests a whole bucket's boxes against a wavefront's queries.
//
// LPQ lanes serve one query and a wavefront 64 / LPQ neighbouring ones
// (k_knn).  Every lane takes its own 32 / LPQ members of a leaf and keeps the
// L smallest FP32 squared distances it has met, sorted in registers: an
// insertion is L median-of-three instructions without a branch.  LPQ lanes
// holding KL = n_se / LPQ distances each below B have met n_se members below
// B, so the largest of the lanes' KL-th distances bounds the search.  After
// the walk a bisection over the kept distances finds a threshold X that
// n_se or a few more members meet; a second pass over the visited leaves
// lists them.  Where the list holds more than n_se (ties within FP32
// rounding, or a lane whose list was too short) the largest exact keys leave
// it: a key packs the exact integer squared distance above the member's rank
// in its host's ascending index order, so ties break by particle index
// exactly as the definition says.  Distances are plain differences of the
// unwrapped coordinates; in a host of half the box's width or more they are
// the periodic ones as long as a query's set ends before the members' images
// a box away.  Only the set matters from there on: the
// bandwidth is the n_v-th smallest velocity distance of the set, a member at
// that distance has weight zero, and the sums of the Epanechnikov estimate
// and the Gaussian background follow in FP64.  Queries whose lists overflow
// (many coincident members) or whose sets reach an image go to k_knn_wave, a
// wavefront per query with exact keys of periodic distances throughout.
#include "vr_kd.h"

#include <cmath>
#include <cstring>
#include <type_traits>

namespace vr {
namespace {

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

constexpr int LEAF = 32;           // slots of a leaf
constexpr int BUCKET_MAX = 2048;   // members of a bucket (64 leaves)
constexpr int BUCKET_SMALL = 512;  // and of those that a wavefront finishes, 16 leaves of them at a time
constexpr float PAD = 1e30f;       // coordinate of an empty slot
constexpr float SLACK = 1.000002f; // above the rounding of an FP32 squared distance (3 * 2^-24)

// The neighbour tree over the hosts' members.
struct Slots {
    float *x, *y, *z;   // [n_slots] coordinates (exact integers)
    int *gid, *eid;     // [n_slots] particle (-1: empty), element id (rank = eid - host offset)
    float4* lbox;       // [n_leaves][2] lower and upper corner of a leaf's members
    float4* bbox;       // [n_buckets][2]
    int4* buckets;      // [n_buckets] first list position, members, first leaf, host
    int* leaf_bucket;   // [n_leaves]
    int* host_bucket;   // [n_hosts + 1]
    const float* images;  // [n_hosts][6] ends of the members' images a box away, or null (no host of half the box)
    float box;            // the box's side where there are images, else far off
};

__global__ void k_subset_slot(int64_t ns, int64_t n, const int32_t* __restrict__ subset, const int* __restrict__ slot_of,
                              uint32_t* __restrict__ qpos, uint32_t* __restrict__ qval, int* __restrict__ bad) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= ns) return;
    const int i = subset[s];
    int p = (i >= 0 && i < n) ? slot_of[i] : -1;
    if (p < 0) { atomicOr(bad, 1); p = 0; }
    qpos[s] = (uint32_t)p;
    qval[s] = (uint32_t)s;
}

// cut[i] = the number of sorted ranks below cut[i]
__global__ void k_cuts(int nc, int* __restrict__ cut, int64_t ns, const uint32_t* __restrict__ rank) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nc) return;
    int64_t lo = 0, hi = ns;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (rank[mid] < (uint32_t)cut[i]) lo = mid + 1;
        else hi = mid;
    }
    cut[i] = (int)lo;
}

// the slots of members by rank, in place
__global__ void k_rank_slot(int64_t ns, const int* __restrict__ mem, const int* __restrict__ slot_of,
                            uint32_t* __restrict__ q) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s < ns) q[s] = (uint32_t)slot_of[mem[q[s]]];
}

// slot_of[g] = the position of particle g in host_members (-1 beforehand; the
// bucket build replaces it by the slot); a member outside [0, n) or listed
// twice raises *bad
__global__ void k_rank_of(int64_t M, int64_t n, const int* __restrict__ mem, int* __restrict__ slot_of,
                          int* __restrict__ bad) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= M) return;
    const int g = mem[k];
    if (g < 0 || g >= n || atomicExch(&slot_of[g], (int)k) != -1) atomicOr(bad, 1);
}

// Per host member, at its slot: (vx, vy, vz, mass) as one 16-byte record, so
// a neighbour's velocity and mass are one cache line (and a query's
// neighbours lie in a few leaves), and the member's ln f_bg, so a query
// reads 8 bytes instead of nine floats spread over nine arrays.  The pass
// runs in particle order, where its 12 input arrays are read in full lines;
// a host's members are scattered over the whole particle range, so a pass in
// slot order would fetch a line per value.
__global__ void k_member_records(int64_t n, const int* __restrict__ slot_of, const float* __restrict__ vx,
                                 const float* __restrict__ vy, const float* __restrict__ vz,
                                 const float* __restrict__ mass, const float* __restrict__ vbar,
                                 const float* __restrict__ sigma, float4* __restrict__ V, double* __restrict__ FB) {
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= n) return;
    const int k = slot_of[g];
    if (k < 0) return;
    const float ux = vx[g], uy = vy[g], uz = vz[g];
    V[k] = make_float4(ux, uy, uz, mass ? mass[g] : 0.f);
    FB[k] = log_fbg(sigma, vbar, (int)g, (double)ux, (double)uy, (double)uz);
}

// Slot within a leaf of its i-th member in KD order: lane s of a query's LPQ
// takes members s, s + LPQ, ..., at consecutive slots.  KD neighbours fall to
// different lanes, which keeps the lanes' shares of a ball even.
__device__ __forceinline__ int leaf_slot(int i, int lpq_log2) {
    const int lpq = 1 << lpq_log2;
    return (i & (lpq - 1)) * (LEAF >> lpq_log2) + (i >> lpq_log2);
}

// One workgroup finishes its buckets' trees in LDS (run: the first of them
// and their number).  Each bucket begins at a leaf of the workgroup's
// positions.  The members' three sorted lists (local ids, local id = position
// in list 0) are split by stable partitions, segment by segment: at a multiple of 32 members nearest
// the middle while a segment holds more than a leaf, then in halves down to
// four.  Members, boxes and slots are written in the resulting order.
// Bound by LDS round trips and barriers (three workgroups of 53 KB a CU); on
// the 6.2 M members of a 256^3 box it takes 0.65 ms in place of three to four
// device-wide levels of about 0.25 ms, and leaves of 32 instead of 192 (2,354
// candidate distances a query before, 688 now).
// NT = 64 takes the buckets of up to 512 members, as many as 16 leaves hold.
// (A workgroup of 256 for each of 100,000 hosts of 33 members: 2.92 ms, a
// wavefront for each 0.86, eight of them a wavefront 0.20.)
template <int NT>
__global__ __launch_bounds__(NT) void k_buckets(const int2* __restrict__ runs, const int* __restrict__ l0,
                                                const int* __restrict__ l1, const int* __restrict__ l2,
                                                const int* __restrict__ u0, const int* __restrict__ u1,
                                                const int* __restrict__ u2, const int* __restrict__ g, int* loc,
                                                int lpq_log2, Slots T, int* __restrict__ slot_of) {
    constexpr int PT = 8, MAX = NT * PT;  // consecutive positions a thread, members
    static_assert(MAX == BUCKET_MAX || MAX == BUCKET_SMALL, "bucket sizes");
    __shared__ int cu[3][MAX];
    __shared__ __align__(16) uint16_t ls[3][MAX];
    __shared__ __align__(16) uint16_t pre[3][MAX];
    __shared__ uint8_t side[MAX], sdim[MAX];
    __shared__ unsigned long long wsum[NT / 64];
    // the leaves' buckets, by their numbers in the run
    __shared__ uint8_t lbk[MAX / LEAF];
    __shared__ int4 bks[NT == 64 ? MAX / LEAF : 1];
    int (*lb)[MAX / LEAF] = reinterpret_cast<int (*)[MAX / LEAF]>(&pre[0][0]);  // and, in the end, boxes
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    // (without runs: a workgroup a bucket)
    const int2 run = runs ? runs[blockIdx.x] : make_int2((int)blockIdx.x, 1);
    const int4 head = T.buckets[run.x];
    const int leaf0 = head.z;
    int all = (head.y + LEAF - 1) / LEAF;  // leaves of the run
    if (NT == 64) {
        const int4 last = T.buckets[run.x + run.y - 1];
        all = last.z - leaf0 + (last.y + LEAF - 1) / LEAF;
        if (t < run.y) {
            const int4 bk = T.buckets[run.x + t];
            bks[t] = bk;
            for (int l = bk.z - leaf0; l < bk.z - leaf0 + (bk.y + LEAF - 1) / LEAF; ++l) lbk[l] = (uint8_t)t;
        }
        __syncthreads();
    }
    auto bucket_of = [&](int l) __attribute__((always_inline)) { return NT == 64 ? bks[lbk[l]] : head; };
    // the place of position p in its host's lists, -1: none
    auto place = [&](int p) __attribute__((always_inline)) {
        if (p >= all * LEAF) return -1;
        const int4 bk = bucket_of(p / LEAF);
        const int k = p - (bk.z - leaf0) * LEAF;
        return k < bk.y ? bk.x + k : -1;
    };
    // (a thread's loads of each kind together: 0.30 -> 0.20 ms of those hosts)
    {
        int e[PT], c[3][PT];
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int at = place(t + j * NT);
            e[j] = at >= 0 ? l0[at] : -1;
        }
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            c[0][j] = u0[max(e[j], 0)];
            c[1][j] = u1[max(e[j], 0)];
            c[2][j] = u2[max(e[j], 0)];
        }
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int p = t + j * NT;
            if (e[j] < 0) continue;
#pragma unroll
            for (int d = 0; d < 3; ++d) cu[d][p] = c[d][j];
            ls[0][p] = (uint16_t)p;
            loc[e[j]] = p;
        }
    }
    __syncthreads();
    {
        int e[2][PT];
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int at = place(t + j * NT);
            e[0][j] = at >= 0 ? l1[at] : -1;
            e[1][j] = at >= 0 ? l2[at] : -1;
        }
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int j = 0; j < PT; ++j)
                if (e[d][j] >= 0) e[d][j] = loc[e[d][j]];
#pragma unroll
        for (int j = 0; j < PT; ++j)
            if (e[0][j] >= 0) {
                ls[1][t + j * NT] = (uint16_t)e[0][j];
                ls[2][t + j * NT] = (uint16_t)e[1][j];
            }
    }
    // a thread's positions lie in one leaf
    const int p0 = t * PT;
    const bool have = p0 < all * LEAF;
    const int4 bk = bucket_of(have ? p0 / LEAF : 0);
    const int b = run.x + (NT == 64 && have ? lbk[p0 / LEAF] : 0);
    const int first = (bk.z - leaf0) * LEAF, n = have ? first + bk.y : 0;  // the bucket's positions
    uint32_t se[PT];  // segment of the position: start << 16 | end
#pragma unroll
    for (int j = 0; j < PT; ++j) se[j] = (uint32_t)first << 16 | (uint32_t)n;
    auto middle = [](int s, int e) __attribute__((always_inline)) {
        const int m = e - s;
        return m > LEAF ? s + LEAF * (((m + LEAF - 1) / LEAF) >> 1) : s + (m >> 1);
    };
    int most = have ? (bk.y + LEAF - 1) / LEAF : 1;  // leaves of the largest bucket
    if (NT == 64)
        for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
    else
        most = all;
    const int levels = (most > 1 ? 32 - __clz(most - 1) : 0) + 3;
    __syncthreads();
    for (int lev = 0; lev < levels; ++lev) {
        // the widest dimension of every segment, from the ends of its lists
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int p = p0 + j, s = (int)(se[j] >> 16), e = (int)(se[j] & 0xFFFFu);
            if (p == s && p < n && e - s > 4) {
                int best = 0, ext = -1;
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const int x = cu[d][ls[d][e - 1]] - cu[d][ls[d][s]];
                    if (x > ext) { ext = x; best = d; }
                }
                sdim[s] = (uint8_t)best;
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int p = p0 + j, s = (int)(se[j] >> 16), e = (int)(se[j] & 0xFFFFu);
            if (p < n && e - s > 4) side[ls[sdim[s]][p]] = p < middle(s, e) ? 1 : 0;
        }
        __syncthreads();
        // left flags of the three lists and their block-wide prefix sums
        uint16_t el[3][PT];
        uint32_t fl[3] = {0u, 0u, 0u};
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const uint4 w = *reinterpret_cast<const uint4*>(&ls[d][p0]);
            const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < PT; ++j) {
                el[d][j] = (uint16_t)(ww[j >> 1] >> (16 * (j & 1)));
                const int s = (int)(se[j] >> 16), e = (int)(se[j] & 0xFFFFu);
                if (p0 + j < n && e - s > 4 && side[el[d][j]]) fl[d] |= 1u << j;
            }
        }
        unsigned long long c = (unsigned long long)__popc(fl[0]) | ((unsigned long long)__popc(fl[1]) << 16) |
                               ((unsigned long long)__popc(fl[2]) << 32);
        unsigned long long inc = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(inc, o, 64);
            if (lane >= o) inc += y;
        }
        if (lane == 63) wsum[wv] = inc;
        __syncthreads();
        unsigned long long ex = inc - c;
        for (int w = 0; w < wv; ++w) ex += wsum[w];
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int s = (int)(se[j] >> 16);
            if (p0 + j == s && p0 + j < n) {
#pragma unroll
                for (int d = 0; d < 3; ++d)
                    pre[d][s] = (uint16_t)((uint32_t)(ex >> (16 * d)) + __popc(fl[d] & ((1u << j) - 1u)));
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int p = p0 + j, s = (int)(se[j] >> 16), e = (int)(se[j] & 0xFFFFu);
            if (p >= n || e - s <= 4) continue;
            const int mid = middle(s, e);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int before = (int)(uint16_t)((uint32_t)(ex >> (16 * d)) + __popc(fl[d] & ((1u << j) - 1u)));
                const int r = before - (int)pre[d][s];  // left members of the segment before p
                const int np = (fl[d] >> j) & 1u ? s + r : mid + (p - s - r);
                ls[d][np] = el[d][j];
            }
            se[j] = p < mid ? ((uint32_t)s << 16) | (uint32_t)mid : ((uint32_t)mid << 16) | (uint32_t)e;
        }
        __syncthreads();
    }
    // members into slots, and the boxes of leaves and bucket
    int mn[3] = {INT32_MAX, INT32_MAX, INT32_MAX}, mx[3] = {INT32_MIN, INT32_MIN, INT32_MIN};
    if (have) {
        int a[PT], e[PT], gi[PT];
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            a[j] = p0 + j < n ? ls[0][p0 + j] : first;
            e[j] = l0[bk.x + a[j] - first];
        }
#pragma unroll
        for (int j = 0; j < PT; ++j) gi[j] = g[e[j]];
#pragma unroll
        for (int j = 0; j < PT; ++j) {
            const int p = p0 + j, slot = (leaf0 + (p / LEAF)) * LEAF + leaf_slot(p & (LEAF - 1), lpq_log2);
            const bool in = p < n;
            const int q[3] = {cu[0][a[j]], cu[1][a[j]], cu[2][a[j]]};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                mn[d] = in ? min(mn[d], q[d]) : mn[d];
                mx[d] = in ? max(mx[d], q[d]) : mx[d];
            }
            T.x[slot] = in ? (float)q[0] : PAD;
            T.y[slot] = in ? (float)q[1] : PAD;
            T.z[slot] = in ? (float)q[2] : PAD;
            T.gid[slot] = in ? gi[j] : -1;
            T.eid[slot] = in ? e[j] : 0;
            if (in) slot_of[gi[j]] = slot;
        }
    }
    // a leaf is the 32 positions of four threads
#pragma unroll
    for (int d = 0; d < 3; ++d) {
#pragma unroll
        for (int o = 1; o < 4; o <<= 1) {
            mn[d] = min(mn[d], __shfl_xor(mn[d], o, 64));
            mx[d] = max(mx[d], __shfl_xor(mx[d], o, 64));
        }
    }
    if ((t & 3) == 0 && have) {
        const int l = p0 / LEAF, leaf = leaf0 + l;
        T.lbox[2 * leaf] = make_float4((float)mn[0], (float)mn[1], (float)mn[2], 0.f);
        T.lbox[2 * leaf + 1] = make_float4((float)mx[0], (float)mx[1], (float)mx[2], 0.f);
        T.leaf_bucket[leaf] = b;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            lb[d][l] = mn[d];
            lb[3 + d][l] = -mx[d];
        }
    }
    __syncthreads();
    // the buckets' boxes: a lane per bucket of a run, or all of one bucket
    int m[6];
    if (NT == 64) {
        if (t >= run.y) return;
        const int4 own = T.buckets[run.x + t];
        const int l0 = own.z - leaf0, l1 = l0 + (own.y + LEAF - 1) / LEAF;
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            m[d] = INT32_MAX;
            for (int l = l0; l < l1; ++l) m[d] = min(m[d], lb[d][l]);
        }
    } else {
        if (wv > 0) return;
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            m[d] = lane < all ? lb[d][lane] : INT32_MAX;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) m[d] = min(m[d], __shfl_xor(m[d], o, 64));
        }
        if (lane > 0) return;
    }
    float4* box = T.bbox + 2 * (run.x + (NT == 64 ? t : 0));
    box[0] = make_float4((float)m[0], (float)m[1], (float)m[2], 0.f);
    box[1] = make_float4((float)-m[3], (float)-m[4], (float)-m[5], 0.f);
}

// ---- reductions over a query's lanes and the wavefront ---------------------
// The DPP moves read lanes of the same row of 16, so every lane must be
// active; a query's lanes are aligned to their number.
template <int CTRL>
__device__ __forceinline__ int dpp(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;

// Folds v over groups of N lanes (4 or 16); every lane gets the result.
template <int N, class T, class OP>
__device__ __forceinline__ T fold(T v, OP op) {
    auto mv = [&](auto c, T x) __attribute__((always_inline)) {
        constexpr int C = decltype(c)::value;
        if constexpr (sizeof(T) == 4) {
            return __builtin_bit_cast(T, dpp<C>(__builtin_bit_cast(int, x)));
        } else {
            struct P { int lo, hi; };
            P p = __builtin_bit_cast(P, x);
            p.lo = dpp<C>(p.lo);
            p.hi = dpp<C>(p.hi);
            return __builtin_bit_cast(T, p);
        }
    };
    v = op(v, mv(std::integral_constant<int, DPP_XOR1>{}, v));
    v = op(v, mv(std::integral_constant<int, DPP_XOR2>{}, v));
    if constexpr (N == 16) {
        v = op(v, mv(std::integral_constant<int, DPP_HALF_MIRROR>{}, v));
        v = op(v, mv(std::integral_constant<int, DPP_MIRROR>{}, v));
    }
    return v;
}
struct OpMax { template <class T> __device__ __forceinline__ T operator()(T a, T b) const { return a > b ? a : b; } };
struct OpMin { template <class T> __device__ __forceinline__ T operator()(T a, T b) const { return a < b ? a : b; } };
struct OpAdd { template <class T> __device__ __forceinline__ T operator()(T a, T b) const { return a + b; } };

// Wavefront-wide fold of a 32-bit value, uniform.
template <class T, class OP>
__device__ __forceinline__ T wave_fold(T v, OP op) {
    v = fold<16>(v, op);
    const int b = __builtin_bit_cast(int, v);
    const T r0 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(b, 0));
    const T r1 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(b, 16));
    const T r2 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(b, 32));
    const T r3 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(b, 48));
    const T r = op(op(r0, r1), op(r2, r3));
    return __builtin_bit_cast(T, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, r)));
}

// Squared distance between two boxes.
__device__ __forceinline__ float box_gap2(float4 a0, float4 a1, float4 b0, float4 b1) {
    const float gx = fmaxf(fmaxf(a0.x - b1.x, b0.x - a1.x), 0.f), gy = fmaxf(fmaxf(a0.y - b1.y, b0.y - a1.y), 0.f),
                gz = fmaxf(fmaxf(a0.z - b1.z, b0.z - a1.z), 0.f);
    return fmaf(gx, gx, fmaf(gy, gy, gz * gz));
}

// (no axis adds more than half a box, 2^20: the sum takes at most 42 bits)
__device__ __forceinline__ uint64_t exact_key(int dx, int dy, int dz, int rank) {
    const uint64_t d2 = (uint64_t)((int64_t)dx * dx + (int64_t)dy * dy + (int64_t)dz * dz);
    return (d2 << POS_BITS) | (uint64_t)(uint32_t)rank;
}

constexpr int VMAX = 256;  // leaves one wavefront may visit for one host

// LPQ lanes a query; KL * LPQ >= n_se; L > KL distances kept a lane, so that
// a lane's share of the n_se nearest seldom exceeds its list.
//
// Bound by VALU issue: 8.2 k instructions a wavefront of 16 queries at 32/8,
// half of them the walk (19 leaves of 32, 18 instructions a lane and member),
// a sixth the second pass, against 62 k for 64 queries of the one-lane-a-query
// form with 64-bit keys in LDS that it replaces.  256^3 box, 6.2 M queries,
// 32/8: 11.5 -> 6.0 ms; 48/16, 159 k queries: 4.2 -> 0.24 ms; 256/32, 335 k
// queries (one wavefront a query before): 5.5 -> 1.6 ms.  L = 12 for KL = 8
// (10: 12% slower by the exact removals, 14: 1%).  Four wavefronts a SIMD
// (103 of 128 VGPRs): three were 12% slower, five 8% (spills).  Eight lanes a
// query were 3% slower on the box: a leaf visit's fixed cost falls on half
// the queries.
template <int LPQ, int KL, int L>
__global__ __launch_bounds__(64, 4) void k_knn(const uint32_t* __restrict__ qpos, int64_t q0, int64_t nq, Slots T,
                                            const float4* __restrict__ V, const double* __restrict__ FB,
                                            const int32_t* __restrict__ host_off, int n_se, int n_v, int use_mass,
                                            double mass_value, double mass_sum, float* __restrict__ R,
                                            unsigned xchunk, int* __restrict__ flagged, int* __restrict__ n_flagged,
                                            unsigned long long* __restrict__ ncand) {
    constexpr int W = 64 / LPQ;        // queries of the wavefront
    constexpr int E = LEAF / LPQ;      // members of a leaf a lane takes
    constexpr int CAPL = L + 12;       // listed members a lane
    constexpr int LOG2 = LPQ == 4 ? 2 : 4;
    __shared__ int vis[VMAX];
    __shared__ uint16_t lst[CAPL][64];
    __shared__ int nbr[W][KL * LPQ];
    const int lane = threadIdx.x, sub = lane & (LPQ - 1), q = lane / LPQ;
    const int64_t qi = q0 + (int64_t)xcd_swizzle(blockIdx.x, gridDim.x, xchunk) * W + q;
    int slot = 0;
    bool active = qi < nq;
    if (active) slot = qpos ? (int)qpos[qi] : (int)(qi & ~(int64_t)(LEAF - 1)) + leaf_slot((int)qi & (LEAF - 1), LOG2);
    const int gid = T.gid[slot];
    active = active && gid >= 0;
    if (!__ballot(active)) return;  // the empty half of a small host's leaf
    const int own = slot / LEAF;
    const int obk = T.leaf_bucket[own];
    const int h = active ? T.buckets[obk].w : -1;
    const float qx = T.x[slot], qy = T.y[slot], qz = T.z[slot];
    float d[L];
#pragma unroll
    for (int i = 0; i < L; ++i) d[i] = INFINITY;
    bool over = false;  // the query goes to the exact kernel
    unsigned long long wcand = 0;

    bool pending = active;
    for (uint64_t pm = __ballot(pending); pm; pm = __ballot(pending)) {
        const int hh = __builtin_amdgcn_readlane(h, __builtin_ctzll(pm));
        const bool mine = pending && h == hh;
        // queries of other hosts stand far away and keep nothing
        const float px = mine ? qx : 3.f * PAD, py = mine ? qy : 3.f * PAD, pz = mine ? qz : 3.f * PAD;
        const float4 q4 = make_float4(qx, qy, qz, 0.f);
        const float4 w0 = make_float4(wave_fold(mine ? qx : INFINITY, OpMin{}), wave_fold(mine ? qy : INFINITY, OpMin{}),
                                      wave_fold(mine ? qz : INFINITY, OpMin{}), 0.f);
        const float4 w1 = make_float4(wave_fold(mine ? qx : -INFINITY, OpMax{}),
                                      wave_fold(mine ? qy : -INFINITY, OpMax{}),
                                      wave_fold(mine ? qz : -INFINITY, OpMax{}), 0.f);
        float B = mine ? INFINITY : -1.f;  // squared radius no member of the query's set exceeds
        float Bmax = INFINITY;             // the wavefront's largest (with slack)
        int nvis = 0;
        const int nmine = __popcll(__ballot(mine)) / LPQ;

        // squared distances of the lane's members of a leaf, plus c
        auto distances = [&](int leaf, float c, float (&sd)[E]) __attribute__((always_inline)) {
            const size_t b = (size_t)(uint32_t)leaf * LEAF;  // uniform
            const uint32_t o = (uint32_t)(sub * E);
            float xs[E], ys[E], zs[E];
            __builtin_memcpy(xs, T.x + b + o, sizeof xs);
            __builtin_memcpy(ys, T.y + b + o, sizeof ys);
            __builtin_memcpy(zs, T.z + b + o, sizeof zs);
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const float dx = xs[k] - px, dy = ys[k] - py, dz = zs[k] - pz;
                sd[k] = fmaf(dx, dx, fmaf(dy, dy, fmaf(dz, dz, c)));
            }
        };
        auto scan = [&](int leaf) __attribute__((always_inline)) {
            float sd[E];
            distances(leaf, 0.f, sd);
            wcand += (unsigned long long)(LEAF * nmine);
            // a leaf whose box a ball reaches may still hold no member of it
            float near = sd[0];
#pragma unroll
            for (int k = 1; k < E; ++k) near = fminf(near, sd[k]);
            if (__ballot(near <= B * SLACK) == 0) return;
#pragma unroll
            for (int k = 0; k < E; ++k) {
#pragma unroll
                for (int i = L - 1; i > 0; --i) d[i] = __builtin_amdgcn_fmed3f(sd[k], d[i - 1], d[i]);
                d[0] = fminf(d[0], sd[k]);
            }
            if (nvis < VMAX) vis[nvis] = leaf;  // every lane the same word
            else over = over || mine;
            nvis = min(nvis + 1, VMAX);
            const float b = fold<LPQ>(d[KL - 1], OpMax{});
            B = mine ? b : -1.f;
            // (as integers the radii order as they do as floats, -1 lowest)
            Bmax = __int_as_float(wave_fold(__float_as_int(B), OpMax{})) * SLACK;
        };
        // whether a ball of the wavefront's queries reaches a box
        auto reaches = [&](float4 lo, float4 hi) __attribute__((always_inline)) {
            return __ballot(mine && box_gap2(lo, hi, q4, q4) <= B * SLACK) != 0;
        };
        // visits the lanes' boxes that a ball reaches, those near the queries
        // first (within 0.2 of the largest squared radius: a strict order by
        // distance, a wavefront-wide minimum a box, was 1% slower on the
        // 256^3 box, touching boxes first 6%)
        auto near_first = [&](float4 lo, float4 hi, bool valid, auto visit) __attribute__((always_inline)) {
            const float g2 = box_gap2(lo, hi, w0, w1);
            uint64_t far = __ballot(valid && g2 <= Bmax), near = __ballot(valid && g2 <= 0.2f * Bmax);
            while (far) {
                const int l = __builtin_ctzll(near ? near : far);
                near &= ~(uint64_t(1) << l);
                far &= ~(uint64_t(1) << l);
                auto rl = [&](float f) __attribute__((always_inline)) {
                    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), l));
                };
                if (reaches(make_float4(rl(lo.x), rl(lo.y), rl(lo.z), 0.f), make_float4(rl(hi.x), rl(hi.y), rl(hi.z), 0.f)))
                    visit(l);
            }
        };
        auto bucket = [&](int b) __attribute__((always_inline)) {
            const int4 bk = T.buckets[b];
            const int nl = (bk.y + LEAF - 1) / LEAF;
            const int leaf = bk.z + min(lane, nl - 1);
            near_first(T.lbox[2 * leaf], T.lbox[2 * leaf + 1], lane < nl, [&](int l) __attribute__((always_inline)) {
                // the leaves of the queries themselves were scanned first
                if (__ballot(mine && own == bk.z + l) == 0) scan(bk.z + l);
            });
        };
        // the queries' own leaves first, then the rest of their buckets, then
        // the host's other buckets
        for (uint64_t todo = __ballot(mine); todo;) {
            const int leaf = __builtin_amdgcn_readlane(own, __builtin_ctzll(todo));
            scan(leaf);
            todo &= ~__ballot(own == leaf);
        }
        const int hb0 = T.host_bucket[hh], hb1 = T.host_bucket[hh + 1];
        for (int pass = 0; pass < 2; ++pass) {
            if (pass == 0) {
                for (uint64_t todo = __ballot(mine); todo;) {
                    const int b = __builtin_amdgcn_readlane(obk, __builtin_ctzll(todo));
                    todo &= ~__ballot(obk == b);
                    bucket(b);
                }
                continue;
            }
            for (int g0 = hb0; g0 < hb1; g0 += 64) {
                const int b = min(g0 + lane, hb1 - 1);
                // queries' own buckets are done
                bool done = false;
                for (uint64_t todo = __ballot(mine); todo;) {
                    const int ob = __builtin_amdgcn_readlane(obk, __builtin_ctzll(todo));
                    todo &= ~__ballot(obk == ob);
                    done = done || ob == b;
                }
                near_first(T.bbox[2 * b], T.bbox[2 * b + 1], g0 + lane < hb1 && !done,
                              [&](int l) __attribute__((always_inline)) { bucket(g0 + l); });
            }
        }
        // a threshold X that at least n_se members meet, and hardly more
        auto count_le = [&](float x) __attribute__((always_inline)) {
            int c = 0;
#pragma unroll
            for (int i = 0; i < L; ++i) c += d[i] <= x ? 1 : 0;
            return fold<LPQ>(c, OpAdd{});
        };
        float hi = B;
        if (__ballot(mine && !(B < INFINITY))) {
            // a lane met fewer than KL members (small hosts)
            float m = 0.f;
#pragma unroll
            for (int i = 0; i < L; ++i) m = d[i] < INFINITY ? fmaxf(m, d[i]) : m;
            m = fold<LPQ>(m, OpMax{});
            if (mine && !(B < INFINITY)) hi = m;
        }
        float lo = 0.f;
        int chi = count_le(hi), clo = 0;
        if (mine && chi < n_se) over = true;
        bool found = !mine || chi <= n_se;
        // by the counts' linear interpolation, every third step halving
        for (int it = 0; it < 24 && __ballot(!found); ++it) {
            const float w = it % 3 == 2 ? 0.5f : ((float)(n_se - clo) + 0.5f) * __builtin_amdgcn_rcpf((float)(chi - clo) + 0.5f);
            const float mid = fminf(fmaf(w, hi - lo, lo), hi);
            const int cm = count_le(mid);
            if (!found) {
                if (cm >= n_se) {
                    hi = mid;
                    chi = cm;
                    found = cm == n_se;
                } else {
                    lo = mid;
                    clo = cm;
                }
            }
        }
        const float X = mine ? hi * SLACK : -1.f;
        if (T.images) {
            // how far the query's ball may reach before the nearest image
            const float* im = T.images + 6 * (int64_t)hh;
            const float gap = fminf(fminf(fminf(qx - im[0], im[3] - qx), fminf(qy - im[1], im[4] - qy)),
                                    fminf(qz - im[2], im[5] - qz));
            if (X >= gap * gap * 0.999999f) over = over || mine;
        }
        // the members within X: the sign of d2 - X marks them (SLACK covers its
        // rounding), 32 marks a word, then each lane lists its marks
        int nl = 0;
        __builtin_amdgcn_wave_barrier();
        constexpr int LPW = 32 / E;  // leaves a word
        for (int v0 = 0; v0 < nvis; v0 += LPW) {
            uint32_t mark = 0;
            const int nv = min(LPW, nvis - v0);
            for (int v = 0; v < nv; ++v) {
                float sd[E];
                distances(__builtin_amdgcn_readfirstlane(vis[v0 + v]), -X, sd);
#pragma unroll
                for (int k = 0; k < E; ++k)
                    mark = __builtin_amdgcn_alignbit(mark, __float_as_uint(sd[k]), 31);
            }
            // the first member's mark is the highest of nv * E bits
            mark <<= 32 - nv * E;
            while (mark) {
                const int t = __clz(mark);
                mark &= ~(0x80000000u >> t);
                if (nl < CAPL) lst[nl][lane] = (uint16_t)(v0 * E + t);
                ++nl;
            }
        }
        int total = fold<LPQ>(nl, OpAdd{});
        if (fold<LPQ>(nl, OpMax{}) > CAPL || total < n_se) over = over || mine;
        nl = min(nl, CAPL);
        auto listed = [&](int i) __attribute__((always_inline)) {
            const int code = lst[i][lane];
            return vis[code / E] * LEAF + sub * E + code % E;
        };
        __builtin_amdgcn_wave_barrier();
        // more than n_se: the largest exact keys leave
        bool extra = mine && !over && total > n_se;
        while (__ballot(extra)) {
            uint64_t big = 0;
            int at = 0;
            if (extra)
                for (int i = 0; i < nl; ++i) {
                    const int s = listed(i);
                    const uint64_t key = exact_key((int)(T.x[s] - qx), (int)(T.y[s] - qy), (int)(T.z[s] - qz),
                                                   T.eid[s] - host_off[hh]) + 1;
                    if (key > big) {
                        big = key;
                        at = i;
                    }
                }
            const uint64_t top = fold<LPQ>(big, OpMax{});
            if (extra && big == top) {
                --nl;
                lst[at][lane] = lst[nl][lane];
            }
            __builtin_amdgcn_wave_barrier();
            --total;
            extra = extra && total > n_se;
        }
        int first = nl;  // members listed by the query's lanes before this one
#pragma unroll
        for (int o = 1; o < LPQ; o <<= 1) {
            const int y = __shfl_up(first, o, LPQ);
            if (sub >= o) first += y;
        }
        first -= nl;
        if (mine && !over)
            for (int i = 0; i < nl; ++i) nbr[q][first + i] = listed(i);
        __builtin_amdgcn_wave_barrier();
        pending = pending && !mine;
    }
    if (ncand && lane == 0) atomicAdd(ncand + blockIdx.x % KNN_CAND_SLOTS, wcand);
    // velocity distances of the set, LPQ lanes sharing it
    const bool ok = active && !over;
    const float4 vq = V[ok ? slot : 0];
    const double vqx = (double)vq.x, vqy = (double)vq.y, vqz = (double)vq.z;
    double dv[KL];
    float ms[KL];
    double msum = 0.0;
#pragma unroll
    for (int k = 0; k < KL; ++k) {
        const int a = sub + LPQ * k;
        const bool in = ok && a < n_se;
        const float4 w = V[in ? nbr[q][a] : 0];
        const double ax = vqx - (double)w.x, ay = vqy - (double)w.y, az = vqz - (double)w.z;
        dv[k] = in ? ax * ax + ay * ay + az * az : (double)INFINITY;
        ms[k] = w.w;
        if (in && use_mass) msum += (double)w.w;
    }
    msum = use_mass ? fold<LPQ>(msum, OpAdd{}) : mass_sum;
    // h2, the n_v-th smallest: bisection to a value that n_v of them meet,
    // then the largest of those; equal values are taken off one by one
    auto count_v = [&](double x) __attribute__((always_inline)) {
        int c = 0;
#pragma unroll
        for (int k = 0; k < KL; ++k) c += dv[k] <= x ? 1 : 0;
        return fold<LPQ>(c, OpAdd{});
    };
    auto largest = [&](double x, bool below) __attribute__((always_inline)) {
        double m = -1.0;
#pragma unroll
        for (int k = 0; k < KL; ++k) m = (below ? dv[k] < x : dv[k] <= x) && dv[k] > m ? dv[k] : m;
        return fold<LPQ>(m, OpMax{});
    };
    double vlo = 0.0, vhi = largest(INFINITY, true);
    int clo = 0, chi = n_se;
    bool found = !ok || n_v >= n_se;
    for (int it = 0; it < 48 && __ballot(!found); ++it) {
        const float w = it % 3 == 2 ? 0.5f : ((float)(n_v - clo) + 0.5f) * __builtin_amdgcn_rcpf((float)(chi - clo) + 0.5f);
        const double mid = fmin(vlo + (double)w * (vhi - vlo), vhi);
        const int c = count_v(mid);
        if (!found) {
            if (c >= n_v) {
                vhi = mid;
                chi = c;
                found = c == n_v;
            } else {
                vlo = mid;
                clo = c;
            }
        }
    }
    double h2 = largest(vhi, false);
    for (;;) {
        const double nx = largest(h2, true);
        const bool less = ok && nx >= 0.0 && count_v(nx) >= n_v;
        if (!__ballot(less)) break;
        if (less) h2 = nx;
    }
    // fewer than n_v finite distances: no bandwidth
    if (count_v(h2) < n_v) h2 = (double)NAN;
    double sw = 0.0;
    const double kW = 15.0 / (8.0 * M_PI);
#pragma unroll
    for (int k = 0; k < KL; ++k)
        if (dv[k] < h2) sw += (use_mass ? (double)ms[k] : mass_value) * kW * (1.0 - dv[k] / h2);
    sw = fold<LPQ>(sw, OpAdd{});
    // one logarithm a lane: ln f_l = ln sw - 1.5 ln h2 - ln msum
    const double term = log(sub == 0 ? sw : sub == 1 ? h2 : msum);
    const double t1 = __shfl(term, (lane & ~(LPQ - 1)) + 1, 64), t2 = __shfl(term, (lane & ~(LPQ - 1)) + 2, 64);
    if (sub != 0) return;
    if (ok) {
        const double lfl = h2 == 0.0 ? INFINITY : term - 1.5 * t1 - t2;
        R[gid] = (float)(lfl - FB[slot]);
    } else if (active) {
        flagged[atomicAdd(n_flagged, 1)] = slot;
    }
}

// ---- one wavefront per query, exact keys throughout -------------------------
// For the queries the kernel above could not finish.  Distances are periodic:
// an axis adds the smaller of the difference and what it leaves of the box,
// for a box of members the smaller of the gap to it and those to its images
// (a host's members lie within one box, so nothing else can be nearer).
// Candidates of a visited
// leaf are keyed by the lanes, and those below the current bound are appended
// to an LDS buffer.  When the buffer holds n_se + 192 keys or more, a radix
// select over the wave finds the n_se-th smallest key; the keys up to it are
// kept and it becomes the bound.
__global__ __launch_bounds__(64) void k_knn_wave(const int* __restrict__ flagged, const int* __restrict__ n_flagged,
                                                 Slots T, const float4* __restrict__ V, const double* __restrict__ FB,
                                                 const int32_t* __restrict__ host_off, int n_se, int n_v, int use_mass,
                                                 double mass_value, float* __restrict__ R) {
    __shared__ uint64_t buf[BIG_BUF];
    __shared__ int bslot[BIG_BUF];
    __shared__ uint32_t sel_hist[256];
    __shared__ double sel_d[64];
    __shared__ float sel_m[64];
    const int lane = threadIdx.x;
    const int nf = *n_flagged;
    for (int f = blockIdx.x; f < nf; f += gridDim.x) {
        const int slot = flagged[f];
        const int h = T.buckets[T.leaf_bucket[slot / LEAF]].w;
        const int base = host_off[h];
        const float qx = T.x[slot], qy = T.y[slot], qz = T.z[slot];
        int nb = 0;            // keys in buf (uniform)
        uint64_t W = ~0ull;    // keys below W are taken (uniform)
        auto compact = [&]() __attribute__((always_inline)) {
            uint64_t k[BIG_J];
            int sl[BIG_J];
            bool v[BIG_J];
#pragma unroll
            for (int j = 0; j < BIG_J; ++j) {
                v[j] = lane + 64 * j < nb;
                k[j] = v[j] ? buf[lane + 64 * j] : 0;
                sl[j] = v[j] ? bslot[lane + 64 * j] : 0;
            }
            const uint64_t top = wave_select(k, v, n_se - 1, sel_hist);
            __builtin_amdgcn_wave_barrier();
            int at = 0;
#pragma unroll
            for (int j = 0; j < BIG_J; ++j) {
                const bool keep = v[j] && k[j] <= top;
                const uint64_t m = __ballot(keep);
                if (keep) {
                    const int to = at + __popcll(m & lanemask_lt());
                    buf[to] = k[j];
                    bslot[to] = sl[j];
                }
                at += __popcll(m);
            }
            __builtin_amdgcn_wave_barrier();
            nb = n_se;
            W = top;
        };
        auto axis_gap = [&](float lo, float hi, float q) __attribute__((always_inline)) {
            return fmaxf(fminf(fmaxf(lo - q, q - hi), fminf(lo + T.box - q, q - hi + T.box)), 0.f);
        };
        auto apart = [&](float a, float q) __attribute__((always_inline)) {
            const float d = fabsf(a - q);
            return (int)fminf(d, T.box - d);
        };
        // whether the lane's box may hold a member of the set
        auto near = [&](const float4* box) __attribute__((always_inline)) {
            const float4 lo = box[0], hi = box[1];
            const float gx = axis_gap(lo.x, hi.x, qx), gy = axis_gap(lo.y, hi.y, qy), gz = axis_gap(lo.z, hi.z, qz);
            const float g2 = fmaf(gx, gx, fmaf(gy, gy, gz * gz));
            return nb < n_se || g2 <= (float)(W >> POS_BITS) * SLACK + 1.f;
        };
        // leaves first + i for the bits i of todo, two at a time (a half of
        // the wavefront each), the next two fetched while these are keyed: one
        // leaf after the other, the 64 of a query's own bucket were most of
        // its time (a few flagged queries of 256 neighbours 160 us: 103 us)
        struct Member {
            int slot, gid, eid;
            float x, y, z;
        };
        auto fetch = [&](int first, uint64_t& todo) __attribute__((always_inline)) {
            Member m{0, -1, 0, 0.f, 0.f, 0.f};
            if (!todo) return m;
            const int a = __builtin_ctzll(todo);
            todo &= todo - 1;
            const bool two = todo != 0;
            const int b = two ? __builtin_ctzll(todo) : a;
            todo &= todo - 1;  // (0 stays 0)
            if (lane < LEAF || two) {
                m.slot = (first + (lane < LEAF ? a : b)) * LEAF + (lane & (LEAF - 1));
                m.gid = T.gid[m.slot];
                m.eid = T.eid[m.slot];
                m.x = T.x[m.slot];
                m.y = T.y[m.slot];
                m.z = T.z[m.slot];
            }
            return m;
        };
        auto scan = [&](int first, uint64_t todo) __attribute__((always_inline)) {
            Member next = fetch(first, todo);
            for (bool more = true; more;) {
                const Member c = next;
                more = todo != 0;
                next = fetch(first, todo);
                bool take = false;
                uint64_t key = 0;
                if (c.gid >= 0) {
                    key = exact_key(apart(c.x, qx), apart(c.y, qy), apart(c.z, qz), c.eid - base);
                    take = key < W;
                }
                const uint64_t m = __ballot(take);
                if (take) {
                    const int to = nb + __popcll(m & lanemask_lt());
                    buf[to] = key;
                    bslot[to] = c.slot;
                }
                nb += __popcll(m);
                __builtin_amdgcn_wave_barrier();
                if (nb >= n_se + BIG_EXTRA) compact();
            }
        };
        auto bucket = [&](int b) __attribute__((always_inline)) {
            const int4 bk = T.buckets[b];
            const int nl = (bk.y + LEAF - 1) / LEAF;
            const uint64_t todo = __ballot(lane < nl && near(T.lbox + 2 * (bk.z + min(lane, nl - 1))));
            if (todo) scan(bk.z, todo);
        };
        // the query's own bucket first, then the host's others, 64 at a time
        const int ob = T.leaf_bucket[slot / LEAF], b1 = T.host_bucket[h + 1];
        bucket(ob);
        for (int b0 = T.host_bucket[h]; b0 < b1; b0 += 64) {
            const int b = min(b0 + lane, b1 - 1);
            for (uint64_t todo = __ballot(b0 + lane < b1 && b != ob && near(T.bbox + 2 * b)); todo; todo &= todo - 1)
                bucket(b0 + __builtin_ctzll(todo));
        }
        if (nb > n_se) compact();
        // the n_se spatial neighbours: velocity distances and the mass of the set
        const float4 vq = V[slot];
        const double vqx = (double)vq.x, vqy = (double)vq.y, vqz = (double)vq.z;
        double dv[BIG_CAP / 64];
        int ps[BIG_CAP / 64];
        float mm[BIG_CAP / 64];
        double msum = 0.0;
#pragma unroll
        for (int j = 0; j < BIG_CAP / 64; ++j) {
            const int a = lane + 64 * j;
            dv[j] = INFINITY;
            ps[j] = 0x7FFFFFFF;
            mm[j] = 0.f;
            if (a < n_se) {
                const float4 w = V[bslot[a]];
                msum += use_mass ? (double)w.w : mass_value;
                const double ax = vqx - (double)w.x, ay = vqy - (double)w.y, az = vqz - (double)w.z;
                dv[j] = ax * ax + ay * ay + az * az;
                ps[j] = (int)(buf[a] & POS_MASK);
                mm[j] = w.w;
            }
        }
        for (int o = 32; o > 0; o >>= 1) msum += __shfl_xor(msum, o, 64);
        // the n_v nearest in velocity, smallest first, by (dv2, rank)
        for (int i = 0; i < n_v; ++i) {
            double bd = INFINITY;
            int bp = 0x7FFFFFFF;
            float bm = 0.f;
#pragma unroll
            for (int j = 0; j < BIG_CAP / 64; ++j)
                if (vless(dv[j], ps[j], bd, bp)) {
                    bd = dv[j];
                    bp = ps[j];
                    bm = mm[j];
                }
            for (int o = 32; o > 0; o >>= 1) {
                const double od = __shfl_xor(bd, o, 64);
                const int op = __shfl_xor(bp, o, 64);
                const float om = __shfl_xor(bm, o, 64);
                if (vless(od, op, bd, bp)) {
                    bd = od;
                    bp = op;
                    bm = om;
                }
            }
#pragma unroll
            for (int j = 0; j < BIG_CAP / 64; ++j)
                if (ps[j] == bp) {
                    dv[j] = INFINITY;
                    ps[j] = 0x7FFFFFFF;
                }
            if (lane == 0) {
                sel_d[i] = bd;
                sel_m[i] = bm;
            }
        }
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) {
            const double kW = 15.0 / (8.0 * M_PI);
            const double h2 = sel_d[n_v - 1];
            double sw = 0.0;
            if (h2 != 0.0)
                for (int a = 0; a < n_v; ++a) {
                    const double m = use_mass ? (double)sel_m[a] : mass_value;
                    sw += m * kW * (1.0 - sel_d[a] / h2);
                }
            const double lfl = h2 == 0.0 ? INFINITY : log(sw) - 1.5 * log(h2) - log(msum);
            R[T.gid[slot]] = (float)(lfl - FB[slot]);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <int LPQ, int KL, int L>
int launch_knn(vr_ctx* ctx, const uint32_t* qpos, int64_t nq, int64_t n_queries, const Slots& T, const float4* V,
               const double* FB, const int32_t* host_off, const vr_particles* p, int n_se, int n_v, float* R,
               int* flagged, int* n_flagged, hipStream_t st) {
    const int use_mass = p->mass ? 1 : 0;
    double mass_sum = 0.0;  // of n_se equal masses, added one by one
    for (int k = 0; k < n_se; ++k) mass_sum += p->mass_value;
    // a launch holds fewer than 2^32 threads, LPQ of them a query
    constexpr int64_t QMAX = int64_t(1) << 26;
    VR_TIMED(ctx, "knn", st, n_queries,
             for (int64_t q0 = 0; q0 < nq; q0 += QMAX)
                 hipLaunchKernelGGL((k_knn<LPQ, KL, L>), dim3(grid_for(std::min(nq - q0, QMAX), 64 / LPQ)), dim3(64), 0,
                                    st, qpos, q0, nq, T, V, FB, host_off, n_se, n_v, use_mass, p->mass_value, mass_sum,
                                    R, (unsigned)ctx->xcd_chunk, flagged, n_flagged,
                                    ctx->timing ? ctx->knn_cand : nullptr));
    VR_LAUNCH_CHECK(ctx);
    // almost always without work: a few wavefronts that stride over the flagged
    // queries; as many as the CUs hold where a host's faces flag them by the
    // thousand
    const unsigned nw = (unsigned)std::min<int64_t>(n_queries, (T.images ? 20 : 4) * ctx->num_cus);
    hipLaunchKernelGGL(k_knn_wave, dim3(std::max(nw, 1u)), dim3(64), 0, st, flagged, n_flagged, T, V, FB, host_off, n_se,
                       n_v, use_mass, p->mass_value, R);
    VR_LAUNCH_CHECK(ctx);
    return VR_OK;
}

}  // namespace
}  // namespace vr

using namespace vr;

extern "C" int vr_local_vdensity(vr_ctx* ctx, const vr_particles* p, int32_t n_hosts, const int32_t* host_offsets,
                                 const int32_t* host_members, const float* vbar, const float* sigma, int32_t n_se,
                                 int32_t n_v, const int32_t* subset, int64_t n_subset, float* R, void* stream) {
    if (!ctx) return VR_ERR_INVALID_ARG;
    int rc = check_particles(ctx, p, true);
    if (rc) return rc;
    if ((rc = check_hosts(ctx, n_hosts, host_offsets, host_members))) return rc;
    if (n_v < 2 || n_v > n_se || n_se > 256 || (n_se > 64 && n_v > 32))
        return set_err(ctx, VR_ERR_INVALID_ARG,
                       "need 2 <= n_v <= n_se <= 256, and n_v <= 32 when n_se > 64 (got n_se=%d, n_v=%d)", n_se, n_v);
    if (subset && n_subset < 0) return set_err(ctx, VR_ERR_INVALID_ARG, "n_subset < 0");
    if (n_hosts == 0 || (subset && n_subset == 0)) return VR_OK;
    if (!vbar || !sigma || !R) return set_err(ctx, VR_ERR_INVALID_ARG, "NULL array");
    VR_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t st = (hipStream_t)stream;
    std::vector<int32_t> off;
    rc = read_host_offsets(ctx, n_hosts, host_offsets, p->n, n_se, off, st);
    if (rc) return rc;
    for (int h = 0; h < n_hosts; ++h)
        if ((int64_t)off[h + 1] - off[h] > (int64_t(1) << POS_BITS))
            return set_err(ctx, VR_ERR_UNSUPPORTED, "host %d has more than 2^%d members", h, POS_BITS);
    const int64_t M = off[n_hosts];
    VR_WS(slot_of, ctx, int32_t, WS_C2, p->n);
    VR_WS(dup, ctx, int, WS_FLAG, 4);
    rc = fill_i32(ctx, slot_of, -1, p->n, st);
    if (rc) return rc;
    rc = fill_i32(ctx, dup, 0, 2, st);
    if (rc) return rc;
    hipLaunchKernelGGL(k_rank_of, dim3(grid_for(M, 256)), dim3(256), 0, st, M, p->n, host_members, slot_of, dup);
    VR_LAUNCH_CHECK(ctx);
    int duph = 0;
    rc = read_back(ctx, dup, &duph, sizeof duph, st);
    if (rc) return rc;
    if (duph) return set_err(ctx, VR_ERR_INVALID_ARG, "host_members lists a particle twice or outside [0, n)");
    // Device-wide levels down to buckets of at most `cap` members.
    const int cap = std::min(BUCKET_MAX, 16 * ctx->knn_leaf);
    std::vector<int> nc(n_hosts, cap);
    KdTree tree;
    rc = kd_build(ctx, p, n_hosts, host_offsets, host_members, off, nc, KD_BUCKETS, 2, tree, st);
    if (rc) return rc;
    // The buckets follow from the sizes: every node above `cap` is halved.
    auto each_bucket = [&](int s, int n, auto&& put) {
        if (n <= cap) return put(s, n);
        // (a host of 2^22 members is halved 14 times)
        std::pair<int, int> todo[32] = {{s, n}};
        for (int left = 1; left > 0;) {
            const auto [at, m] = todo[--left];
            if (m > cap) {
                todo[left++] = {at + m / 2, m - m / 2};
                todo[left++] = {at, m / 2};
            } else {
                put(at, m);
            }
        }
    };
    // A host's leaves are its own, so small hosts pad theirs: two members take
    // 32 slots.  The hosts are searched in ranges whose slots stay within 5/4
    // of the members (or 2^24 where nothing caps the workspace), at least one
    // host each: one range where the hosts have 128 members or more.
    struct Range {
        int h0, h1;
        int64_t nb, leaves, fit;  // buckets, their leaves, buckets a wavefront finishes
    };
    std::vector<Range> ranges;
    Range most{0, 0, 0, 0, 0};  // of each the largest
    {
        const int64_t room = std::max(M + M / 4, ctx->max_ws ? int64_t(0) : int64_t(1) << 24) / LEAF;
        Range r{0, 0, 0, 0, 0};
        auto close = [&](int h) {
            r.h1 = h;
            ranges.push_back(r);
            most.h1 = std::max(most.h1, r.h1 - r.h0);
            most.nb = std::max(most.nb, r.nb);
            most.leaves = std::max(most.leaves, r.leaves);
            r = Range{h, h, 0, 0, 0};
        };
        for (int h = 0; h < n_hosts; ++h) {
            int64_t nb = 0, leaves = 0, fit = 0;
            each_bucket(off[h], off[h + 1] - off[h], [&](int, int n) {
                ++nb;
                leaves += (n + LEAF - 1) / LEAF;
                fit += n <= BUCKET_SMALL;
            });
            if (r.leaves > 0 && r.leaves + leaves > std::min<int64_t>(room, INT32_MAX / LEAF)) close(h);
            r.nb += nb;
            r.leaves += leaves;
            r.fit += fit;
        }
        close(n_hosts);
    }
    const int nr = (int)ranges.size();
    Slots T{};
    Carve cv;
    auto layout = [&]() {
        const int64_t n_slots = most.leaves * LEAF;
        T.x = cv.add<float>(n_slots);
        T.y = cv.add<float>(n_slots);
        T.z = cv.add<float>(n_slots);
        T.gid = cv.add<int>(n_slots);
        T.eid = cv.add<int>(n_slots);
        T.lbox = cv.add<float4>(2 * most.leaves);
        T.bbox = cv.add<float4>(2 * most.nb);
        T.leaf_bucket = cv.add<int>(most.leaves);
        // one upload: buckets, the hosts' first ones, the workgroups' runs of them
        T.buckets = cv.add<int4>(most.nb + (2 * most.nb + most.h1 + 5) / 4);
    };
    layout();
    const size_t total = cv.bytes;
    cv.bytes = 0;
    cv.base = static_cast<char*>(ws(ctx, WS_C3, total));
    if (!cv.base) return VR_ERR_OUT_OF_MEMORY;
    layout();
    VR_WS(V, ctx, float4, WS_C0, most.leaves * LEAF);
    VR_WS(FB, ctx, double, WS_C1, most.leaves * LEAF);
    VR_WS(flagged, ctx, int, WS_C4, subset ? n_subset : M);
    const int lpq_log2 = n_se > 64 ? 4 : 2;
    uint32_t *qp = nullptr, *qv = nullptr;
    std::vector<int> cut;  // the ranges' queries, by rank
    auto subset_places = [&](int64_t places) -> int {
        VR_WS(bad, ctx, int, WS_FLAG2, 4);
        if ((rc = fill_i32(ctx, bad, 0, 1, st))) return rc;
        hipLaunchKernelGGL(k_subset_slot, dim3(grid_for(n_subset, 256)), dim3(256), 0, st, n_subset, p->n, subset,
                           slot_of, qp, qv, bad);
        VR_LAUNCH_CHECK(ctx);
        int badh = 0;
        if ((rc = read_back(ctx, bad, &badh, sizeof badh, st))) return rc;
        if (badh) return set_err(ctx, VR_ERR_INVALID_ARG, "subset lists a particle that is in no host");
        int bits = 1;
        while ((int64_t(1) << bits) < places) ++bits;
        return sort_pairs_u32(ctx, qp, qv, n_subset, bits, st);
    };
    if (subset) {
        VR_WS(qp_w, ctx, uint32_t, WS_C5, n_subset);
        VR_WS(qv_w, ctx, uint32_t, WS_C6, n_subset);
        qp = qp_w;
        qv = qv_w;
        if (nr > 1) {
            if ((rc = subset_places(M))) return rc;  // slot_of still holds the ranks
            cut.resize(nr + 1);
            VR_WS(cut_d, ctx, int, WS_C7, nr + 1);
            int* up = static_cast<int*>(upload_begin(ctx, (nr + 1) * sizeof(int)));
            if (!up) return VR_ERR_HIP;
            for (int i = 0; i <= nr; ++i) up[i] = i < nr ? off[ranges[i].h0] : (int)M;
            VR_HIP(ctx, hipMemcpyAsync(cut_d, up, (nr + 1) * sizeof(int), hipMemcpyHostToDevice, st));
            if ((rc = upload_end(ctx, st))) return rc;
            hipLaunchKernelGGL(k_cuts, dim3(grid_for(nr + 1, 64)), dim3(64), 0, st, nr + 1, cut_d, n_subset, qp);
            VR_LAUNCH_CHECK(ctx);
            if ((rc = read_back(ctx, cut_d, cut.data(), (nr + 1) * sizeof(int), st))) return rc;
        }
    }
    int* nfl = dup + 1;  // zero since the fill above
    T.images = nullptr;
    T.box = tree.images ? (float)(1 << p->grid_bits) : 1e30f;
    for (int ri = 0; ri < nr; ++ri) {
        const Range& r = ranges[ri];
        if (nr > 1 && subset && cut[ri] == cut[ri + 1]) continue;
        if (nr > 1 && ((rc = fill_i32(ctx, slot_of, -1, p->n, st)) || (rc = fill_i32(ctx, nfl, 0, 1, st)))) return rc;
        const int64_t nb = r.nb, n_slots = r.leaves * LEAF;
        const int nh = r.h1 - r.h0;
        // The small buckets get their own launch where the chip could not hold
        // them all beside the others anyway: the launches follow each other, 59
        // and 45 us where a workgroup each took 59 in all (300 buckets).
        const bool split = r.fit > 3 * ctx->num_cus;
        // runs of one large bucket, then those of small ones
        const int64_t n_large = nb - (split ? r.fit : 0);
        int64_t n_runs = n_large;
        const int2* runs = nullptr;
        {
            const size_t room = nb * (sizeof(int4) + sizeof(int2)) + ((size_t)nh + 2) * sizeof(int);
            int4* up = static_cast<int4*>(upload_begin(ctx, room));
            if (!up) return VR_ERR_HIP;
            int* uh = reinterpret_cast<int*>(up + nb);
            int2* ur = reinterpret_cast<int2*>(uh + ((nh + 2) & ~1));
            int2 run = make_int2(0, 0);  // the run of small buckets being filled
            int k = 0, leaf = 0, filled = 0;
            int64_t at = 0;
            auto close = [&]() {
                if (run.y > 0) ur[n_runs++] = run;
                run.y = filled = 0;
            };
            for (int h = r.h0; h < r.h1; ++h) {
                uh[h - r.h0] = k;
                each_bucket(off[h], off[h + 1] - off[h], [&](int s, int n) {
                    const int nl = (n + LEAF - 1) / LEAF;
                    up[k] = make_int4(s, n, leaf, h - r.h0);
                    if (split && n <= BUCKET_SMALL) {
                        if (filled + nl > BUCKET_SMALL / LEAF) close();
                        if (run.y++ == 0) run.x = k;
                        filled += nl;
                    } else if (split) {
                        close();
                        ur[at++] = make_int2(k, 1);
                    }
                    ++k;
                    leaf += nl;
                });
            }
            uh[nh] = k;
            close();
            T.host_bucket = reinterpret_cast<int*>(T.buckets + nb);
            if (split) runs = reinterpret_cast<int2*>(T.host_bucket + ((nh + 2) & ~1));
            const size_t used = (char*)(ur + (split ? n_runs : 0)) - (char*)up;
            VR_HIP(ctx, hipMemcpyAsync(T.buckets, up, used, hipMemcpyHostToDevice, st));
            if ((rc = upload_end(ctx, st))) return rc;
        }
        if (tree.images) T.images = tree.images + 6 * (int64_t)r.h0;
        auto build = [&](auto kernel, int64_t n, const int2* run, int threads) {
            if (n > 0)
                hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(threads), 0, st, run, tree.list[0], tree.list[1],
                                   tree.list[2], tree.elem_u[0], tree.elem_u[1], tree.elem_u[2], tree.elem_g,
                                   tree.scratch, lpq_log2, T, slot_of);
        };
        build(k_buckets<256>, n_large, runs, 256);
        build(k_buckets<64>, n_runs - n_large, runs + n_large, 64);
        VR_LAUNCH_CHECK(ctx);
        hipLaunchKernelGGL(k_member_records, dim3(grid_for(p->n, 256)), dim3(256), 0, st, p->n, slot_of, p->vx, p->vy,
                           p->vz, p->mass, vbar, sigma, V, FB);
        VR_LAUNCH_CHECK(ctx);
        const uint32_t* qpos = nullptr;
        int64_t nq = n_slots, n_queries = off[r.h1] - off[r.h0];
        if (subset && nr == 1) {
            if ((rc = subset_places(n_slots))) return rc;
            qpos = qp;
            nq = n_queries = n_subset;
        } else if (subset) {
            uint32_t* q = qp + cut[ri];
            nq = n_queries = cut[ri + 1] - cut[ri];
            hipLaunchKernelGGL(k_rank_slot, dim3(grid_for(nq, 256)), dim3(256), 0, st, nq, host_members, slot_of, q);
            VR_LAUNCH_CHECK(ctx);
            int bits = 1;
            while ((int64_t(1) << bits) < n_slots) ++bits;
            if ((rc = sort_pairs_u32(ctx, q, qv, nq, bits, st))) return rc;
            qpos = q;
        }
        const int32_t* ho = host_offsets + r.h0;
        if (n_se <= 32)
            rc = launch_knn<4, 8, 12>(ctx, qpos, nq, n_queries, T, V, FB, ho, p, n_se, n_v, R, flagged, nfl, st);
        else if (n_se <= 64)
            rc = launch_knn<4, 16, 22>(ctx, qpos, nq, n_queries, T, V, FB, ho, p, n_se, n_v, R, flagged, nfl, st);
        else if (n_se <= 128)
            rc = launch_knn<16, 8, 14>(ctx, qpos, nq, n_queries, T, V, FB, ho, p, n_se, n_v, R, flagged, nfl, st);
        else  // up to the paper's defaults (n_se 256, n_v 32)
            rc = launch_knn<16, 16, 24>(ctx, qpos, nq, n_queries, T, V, FB, ho, p, n_se, n_v, R, flagged, nfl, st);
        if (rc) return rc;
    }
    return VR_OK;
}
