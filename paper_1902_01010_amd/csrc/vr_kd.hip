// vr_kd.hip -- level-synchronous KD trees over the members of many hosts,
// built from presorted lists.
//
// For each dimension d the members are sorted once by (host, u_d, index)
// with the device radix sort.  Every node then owns the same position range
// in the three lists, and the list of dimension d holds its members in
// (u_d, index) order, so the member of rank floor(n/2) -- the split point --
// and the bounding box are read off directly.  One level costs a handful of
// element-parallel passes for all nodes of all hosts at once: entropy
// histograms (cells tree), the split decision per node, a left/right flag
// per member with counts per tile of positions, and a stable partition of
// each list from the tiles' prefixes: five launches, three without histograms
// (eleven and eight before: 12 k members in ten levels 1.0 -> 0.5 ms).  No
// node is ever handled by a single workgroup, so the few huge top-level
// nodes cost no more per member than the many small ones.  The levels and
// the active-node counts that size their launches follow from the host
// sizes alone, so the whole build is queued without waiting on the device;
// the kernels read the true counts, which only nodes of coincident members
// (kept as leaves) make smaller.
#include "vr_kd.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <type_traits>

namespace vr {
namespace {

constexpr int KB = 256;
constexpr int HCH = 2048;  // positions per histogram block
// Up to this many members a block takes 256 positions (a 12 k host's level
// would keep 6 of 256 CUs busy with 2,048: histograms 16 -> 4 us), beyond it
// BIG_TILE in the flags and the partition, whose blocks add up to M / tile
// counts each, and HCH in the histograms.
constexpr int64_t SMALL_M = 1 << 20;
constexpr int BIG_TILE = 1024;
// A level whose largest node spans more tiles than this scans their counts
// first; below, every block of the partition adds up those it needs.
// (One host, seven levels, all levels scanned and none: 2^22 members 1.62 and
// 1.61 ms, 2^23 3.56 and 3.64, 2^25 14.7 and 15.9, 2^28 113 and 160.)
constexpr int64_t SCAN_TILES = 4096;
// Counters of a build: leaves, nodes, and from CN_ACTIVE on the active nodes
// of every level.
constexpr int MAX_LEVELS = 64;
enum { CN_LEAVES = 0, CN_NODES = 1, CN_ACTIVE = 2, CN_COUNT = CN_ACTIVE + MAX_LEVELS + 1 };
constexpr int HASH_SLOTS = 256;  // partial sums of the content hash

// One element's share of the content hash of a build's inputs: a 64-bit
// mix of its position, member, unwrapped coordinates and host.  The shares
// are summed, so the hash covers every element whatever the order of the
// additions.
__device__ __forceinline__ unsigned long long elem_hash(int64_t e, int i, int a, int b, int c, int h) {
    uint64_t x = (uint64_t)e * 0x9E3779B97F4A7C15ull;
    x ^= (uint64_t)(uint32_t)i * 0xC2B2AE3D27D4EB4Full;
    x ^= (((uint64_t)(uint32_t)a << 32) | (uint32_t)b) * 0x165667B19E3779F9ull;
    x ^= (((uint64_t)(uint32_t)c << 32) | (uint32_t)h) * 0x27D4EB2F165667C5ull;
    x ^= x >> 31;
    x *= 0xBF58476D1CE4E5B9ull;
    x ^= x >> 29;
    x *= 0x94D049BB133111EBull;
    x ^= x >> 32;
    return (unsigned long long)x;
}

// Element arrays by element id, and the sort keys of the presort; the
// HASH_SLOTS words of hash (zeroed beforehand) receive partial sums of the
// content hash of (member, coordinates, host) over all elements, one slot
// per wavefront in turn, so no single address takes every wavefront's add.
__global__ void k_elems(int64_t M, int n_hosts, const int32_t* __restrict__ off, const int32_t* __restrict__ mem,
                        const uint32_t* __restrict__ qx, const uint32_t* __restrict__ qy,
                        const uint32_t* __restrict__ qz, const float* __restrict__ mass, int gb, int* __restrict__ u0,
                        int* __restrict__ u1, int* __restrict__ u2, int* __restrict__ g, float* __restrict__ m,
                        int* __restrict__ host, unsigned long long* __restrict__ hash, int* __restrict__ hbox) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long hv = 0;
    int hm = -1, um[3] = {0, 0, 0};
    // host with off[h] <= e < off[h+1]: the block's first and last elements
    // search among all hosts, the others between those two
    __shared__ int hrange[2];
    auto host_at = [&](int64_t at, int lo, int hi) {
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (off[mid] <= at) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    if (threadIdx.x < 2)
        hrange[threadIdx.x] = host_at(min(((int64_t)blockIdx.x + threadIdx.x) * blockDim.x, M) - threadIdx.x, 0, n_hosts - 1);
    __syncthreads();
    if (e < M) {
        const int lo = host_at(e, hrange[0], hrange[1]);
        const int h = lo;
        const int r = mem[off[h]];
        const int i = mem[e];
        const int rx = (int)qx[r], ry = (int)qy[r], rz = (int)qz[r];
        const int a = rx + min_image((int)qx[i] - rx, gb), b = ry + min_image((int)qy[i] - ry, gb),
                  c = rz + min_image((int)qz[i] - rz, gb);
        u0[e] = a;
        u1[e] = b;
        u2[e] = c;
        g[e] = i;
        host[e] = h;
        if (mass) m[e] = mass[i];
        hv = elem_hash(e, i, a, b, c, h);
        hm = h;
        um[0] = a;
        um[1] = b;
        um[2] = c;
    }
    if (hbox) {
        // the host's extent: minima of u and of -u.  A block inside one host
        // (its members are consecutive) reduces; one with several collects them
        // in LDS, and only the hosts that reach beyond it need atomics (every
        // run of lanes by itself, 100,000 hosts of 33 members: 262 us, now
        // 96).  Values only decrease, so a plain read that is already
        // no larger makes the atomic unnecessary.
        __shared__ int hb[256][6];
        const int h0 = hrange[0], nh = hrange[1] - h0 + 1;
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        if (nh == 1) {
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                int v = e < M ? (k < 3 ? um[k] : -um[k - 3]) : INT_MAX;
                for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
                if (lane == 0) hb[w][k] = v;
            }
            __syncthreads();
            if (threadIdx.x < 6) {
                const int k = threadIdx.x;
                const int v = min(min(hb[0][k], hb[1][k]), min(hb[2][k], hb[3][k]));
                int* at = hbox + 6 * (int64_t)h0 + k;
                if (v < *at) atomicMin(at, v);
            }
        } else {
            for (int k = threadIdx.x; k < 6 * nh; k += blockDim.x) (&hb[0][0])[k] = INT_MAX;
            __syncthreads();
            if (hm >= 0)
#pragma unroll
                for (int k = 0; k < 6; ++k) atomicMin(&hb[hm - h0][k], k < 3 ? um[k] : -um[k - 3]);
            __syncthreads();
            const int64_t b0 = (int64_t)blockIdx.x * blockDim.x;
            for (int k = threadIdx.x; k < 6 * nh; k += blockDim.x) {
                const int h = h0 + k / 6, v = (&hb[0][0])[k];
                int* at = hbox + 6 * (int64_t)h0 + k;
                if (off[h] >= b0 && off[h + 1] <= b0 + blockDim.x) *at = v;
                else if (v < *at) atomicMin(at, v);
            }
        }
    }
    // every lane of the wavefront reaches the sum
    for (int o = 32; o > 0; o >>= 1) hv += (unsigned long long)__shfl_xor((long long)hv, o, 64);
    if ((threadIdx.x & 63) == 0 && hv)
        atomicAdd(&hash[((uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) % HASH_SLOTS], hv);
}

// The hosts' extents: the largest of them in words[1], and words[0] raised when
// a host spans half the box or more on some axis.  There the periodic distance
// of two members can be below their coordinates' difference, where one of them
// comes near the other's image a box away (images: the near ends of all
// members' images, whole numbers below 2^23).
__global__ void k_host_box(int n_hosts, int half, const int* __restrict__ hbox, float* __restrict__ images,
                           unsigned long long* __restrict__ words) {
    int most = 0;
    for (int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; h < n_hosts; h += (int64_t)gridDim.x * blockDim.x) {
        const int* b = hbox + 6 * h;
        for (int d = 0; d < 3; ++d) {
            const int lo = b[d], hi = -b[3 + d];
            most = max(most, hi - lo);
            const bool wide = hi - lo >= half;
            images[6 * h + d] = wide ? (float)(hi - 2 * half) : -1e30f;
            images[6 * h + 3 + d] = wide ? (float)(lo + 2 * half) : 1e30f;
            if (wide) words[0] = 1;
        }
    }
    for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
    if (__lane_id() == 0) atomicMax(&words[1], (unsigned long long)most);
}

// Sort keys (host, coordinate); blockIdx.y: the dimension d0 + y of u (a batch
// of sorts, one after the other).  cb bits hold a coordinate relative to its
// host's smallest (hbox), or, without hbox, shifted into 22 bits (unwrapped
// ones lie in [-2^20, 3 * 2^20)).
template <class K>
__global__ void k_presort_keys(int64_t M, int d0, const int* __restrict__ u0, const int* __restrict__ u1,
                               const int* __restrict__ u2, const int* __restrict__ host, const int* __restrict__ hbox,
                               int cb, K* __restrict__ key, uint32_t* __restrict__ val) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= M) return;
    const int d = d0 + (int)blockIdx.y;
    const int* u = d == 0 ? u0 : (d == 1 ? u1 : u2);
    key += blockIdx.y * M;
    val += blockIdx.y * M;
    const int h = host[e], base = hbox ? hbox[6 * (int64_t)h + d] : -(1 << 20);
    key[e] = (K)h << cb | (K)(uint32_t)(u[e] - base);
    val[e] = (uint32_t)e;
}

// Positions and roots of the first level: every position's node is its host's
// root (hosts keep their ranges in every list), the coordinates in list-0
// order (c0 null: none) and zeros for the first histograms; a root's bounding
// box, which is its region, is read off its sorted lists.
__global__ void k_start(int64_t M, int n_hosts, const int32_t* __restrict__ off, const int* __restrict__ ncell,
                        const int* __restrict__ host, const int* __restrict__ l0, const int* __restrict__ l1,
                        const int* __restrict__ l2, const int* __restrict__ u0, const int* __restrict__ u1,
                        const int* __restrict__ u2, KdNode* __restrict__ nodes, int* __restrict__ active,
                        int* __restrict__ counters, int* __restrict__ leaves, int* __restrict__ leaf_min,
                        int* __restrict__ seg_node, int* __restrict__ c0, int* __restrict__ c1, int* __restrict__ c2,
                        uint32_t* __restrict__ hist, int64_t hist_words) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t k = p; k < hist_words; k += (int64_t)gridDim.x * blockDim.x) hist[k] = 0;
    if (p >= M) return;
    seg_node[p] = host[p];
    if (c0) {
        const int e = l0[p];
        c0[p] = u0[e];
        c1[p] = u1[e];
        c2[p] = u2[e];
    }
    if (p >= n_hosts) return;
    const int h = (int)p;
    KdNode nd;
    nd.host = h;
    nd.start = off[h];
    nd.end = off[h + 1];
    nd.slot = -1;
    nd.dim = -1;
    nd.t = 0;
    nd.left = nd.right = -1;
    const int s = nd.start, e = nd.end - 1;
    nd.lo[0] = nd.bmin[0] = u0[l0[s]]; nd.hi[0] = nd.bmax[0] = u0[l0[e]];
    nd.lo[1] = nd.bmin[1] = u1[l1[s]]; nd.hi[1] = nd.bmax[1] = u1[l1[e]];
    nd.lo[2] = nd.bmin[2] = u2[l2[s]]; nd.hi[2] = nd.bmax[2] = u2[l2[e]];
    if (nd.end - nd.start > ncell[h]) {
        nd.slot = atomicAdd(&counters[CN_ACTIVE], 1);
        active[nd.slot] = h;
    } else {
        leaves[atomicAdd(&counters[CN_LEAVES], 1)] = h;
    }
    nodes[h] = nd;
    leaf_min[h] = 0x7FFFFFFF;
}

// Mass histograms (counts for uniform mass) of the active nodes, nb bins per
// dimension spanning the members' extent.  A block whose positions all
// belong to one node accumulates in LDS first.  The bin of a coordinate is
// taken in 32 bits: a node spans less than 2^22 of them and nb <= 64.
// The three coordinates carried in list-0 order (null when no histogram
// needs them), permuted with list 0 at every level.
struct CoordsL0 {
    const int* in[3];
    int* out[3];
};

// Nodes of one chunk that get LDS histograms: slots [base, base + HK), base
// the slot of the chunk's first active end. Deep levels put several small
// nodes in a chunk; a node outside the window adds to global memory.
constexpr int HK = 8;

template <bool COUNTS>
__global__ __launch_bounds__(KB) void k_hist(int64_t M, const int* __restrict__ seg_node, const KdNode* __restrict__ nodes,
                                             const int* __restrict__ l0, const int* __restrict__ c0,
                                             const int* __restrict__ c1, const int* __restrict__ c2,
                                             const float* __restrict__ mass, int nb, int hch,
                                             uint32_t* __restrict__ hc, double* __restrict__ hm) {
    __shared__ uint32_t lc[COUNTS ? HK * 3 * 64 : 1];
    __shared__ double lm[COUNTS ? 1 : HK * 3 * 64];
    const int64_t p0 = (int64_t)blockIdx.x * hch;
    const int64_t p1 = min(p0 + hch, M);
    const KdNode& nf = nodes[seg_node[p0]];
    const KdNode& nl = nodes[seg_node[p1 - 1]];
    const bool af = nf.slot >= 0 && nf.dim < 0, al = nl.slot >= 0 && nl.dim < 0;
    if (&nf == &nl && !af) return;  // one node, not active this level
    const int base = af ? nf.slot : (al ? max(0, nl.slot - (HK - 1)) : -1);
    const int nb3 = 3 * nb;
    for (int k = threadIdx.x; k < HK * nb3; k += blockDim.x) {
        if (COUNTS) lc[k] = 0;
        else lm[k] = 0.0;
    }
    __syncthreads();
    for (int64_t p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
        const KdNode& nd = nodes[seg_node[p]];
        if (nd.slot < 0 || nd.dim >= 0) continue;
        const int li = base >= 0 ? nd.slot - base : -1;
        const bool local = li >= 0 && li < HK;
        const int u[3] = {c0[p], c1[p], c2[p]};  // coordinates in list-0 order
        const double w = COUNTS ? 1.0 : (double)mass[l0[p]];
        for (int d = 0; d < 3; ++d) {
            if (nd.bmax[d] == nd.bmin[d]) continue;
            const int bin = (int)((uint32_t)(u[d] - nd.bmin[d]) * (uint32_t)nb / (uint32_t)(nd.bmax[d] - nd.bmin[d] + 1));
            if (local) {
                if (COUNTS) atomicAdd(&lc[li * nb3 + d * nb + bin], 1u);
                else atomicAdd(&lm[li * nb3 + d * nb + bin], w);
            } else {
                const int64_t at = ((int64_t)nd.slot * 3 + d) * nb + bin;
                if (COUNTS) atomicAdd(&hc[at], 1u);
                else atomicAdd(&hm[at], w);
            }
        }
    }
    if (base < 0) return;
    __syncthreads();
    // a nonzero entry belongs to an active node seen above, so its slot
    // base + k / nb3 is in range
    for (int k = threadIdx.x; k < HK * nb3; k += blockDim.x) {
        const int64_t at = (int64_t)base * nb3 + k;
        if (COUNTS) {
            if (lc[k]) atomicAdd(&hc[at], lc[k]);
        } else if (lm[k] != 0.0) {
            atomicAdd(&hm[at], lm[k]);
        }
    }
}

// Normalised Shannon entropy of each dimension's histogram (the entropy
// equation of Sec. 2.2) for every active node: one wavefront per node, one
// lane per bin, so the logarithms of a node are taken in parallel.
__global__ __launch_bounds__(256) void k_entropy(const int* __restrict__ nact, const int* __restrict__ active,
                                                 const KdNode* __restrict__ nodes, int nb, int counts,
                                                 const uint32_t* __restrict__ hc, const double* __restrict__ hm,
                                                 double* __restrict__ S) {
    const int i = (int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    const int lane = __lane_id();
    if (i >= *nact) return;
    const KdNode& nd = nodes[active[i]];
    __shared__ double sh[4][3][65];
    const int w = threadIdx.x >> 6;
    // totals and entropy sums run over the bins in order, as a serial loop
    // would, one lane a dimension; the logarithms are spread over the lanes
    double h[3];
    for (int d = 0; d < 3; ++d) {
        const int64_t at = ((int64_t)i * 3 + d) * nb + lane;
        h[d] = lane < nb ? (counts ? (double)hc[at] : hm[at]) : 0.0;
        sh[w][d][lane] = h[d];
    }
    __builtin_amdgcn_wave_barrier();
    double tot = 0.0;
    if (lane < 3)
        for (int k = 0; k < nb; ++k) tot += sh[w][lane][k];
    __builtin_amdgcn_wave_barrier();
    for (int d = 0; d < 3; ++d) {
        const double td = __shfl(tot, d, 64);
        double term = 0.0;
        if (h[d] > 0) {
            const double pk = h[d] / td;
            term = -pk * log(pk);
        }
        sh[w][d][lane] = term;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < 3) {
        double sacc = 0.0;
        for (int k = 0; k < nb; ++k) sacc += sh[w][lane][k];
        S[3 * (int64_t)i + lane] = nd.bmax[lane] == nd.bmin[lane] ? 0.0 : sacc / log((double)nb);
    }
}

// Reserves n[k] slots of each of three global counters for every lane; one
// atomic per wavefront and counter, all three in flight.  Every lane of the
// wavefront must call it.
__device__ __forceinline__ void wave_reserve3(int* const (&counter)[3], const int (&n)[3], int (&first)[3]) {
    const int lane = __lane_id();
    int x[3], base[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        x[k] = n[k];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(x[k], o, 64);
            if (lane >= o) x[k] += t;
        }
        base[k] = 0;
    }
    if (lane == 63) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (x[k] > 0) base[k] = atomicAdd(counter[k], x[k]);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) first[k] = __shfl(base[k], 63, 64) + x[k] - n[k];
}

// Split decision of every active node and creation of its children (their
// bounding boxes follow from the partition).  All lanes reserve (the counters
// are reserved per wavefront).
__global__ __launch_bounds__(256) void k_split(const int* nact, const int* __restrict__ active, KdNode* nodes,
                                               const int* __restrict__ l0, const int* __restrict__ l1,
                                               const int* __restrict__ l2, const int* __restrict__ u0,
                                               const int* __restrict__ u1, const int* __restrict__ u2, int mode,
                                               const double* __restrict__ Sdim, const int* __restrict__ ncell,
                                               int* next_active, int* leaves, int* __restrict__ leaf_min,
                                               int* counters, int* nnext) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < *nact;
    const int id = valid ? active[i] : 0;
    KdNode nd;
    int best = -1;
    if (valid) {
        nd = nodes[id];
        if (mode == KD_BUCKETS) {
            int widest = 0;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int ext = nd.bmax[d] - nd.bmin[d];
                if (best < 0 || ext > widest) {
                    best = d;
                    widest = ext;
                }
            }
        } else {
            const double S[3] = {Sdim[3 * (int64_t)i], Sdim[3 * (int64_t)i + 1], Sdim[3 * (int64_t)i + 2]};
            double Sb = 0.0;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if (nd.bmax[d] == nd.bmin[d]) continue;
                if (best < 0 || (mode == KD_MIN_ENTROPY ? S[d] < Sb - 1e-12 : S[d] > Sb + 1e-12)) {
                    best = d;
                    Sb = S[d];
                }
            }
        }
    }
    const bool split = valid && best >= 0;
    // every member coincides: the node stays a leaf
    const bool stays = valid && best < 0;
    const int n = split ? nd.end - nd.start : 0, nl = n / 2;
    const int nc = split ? ncell[nd.host] : 0;
    const bool lact = split && nl > nc, ract = split && n - nl > nc;
    // the split value is fetched while the slots are reserved
    const int* lb = best == 0 ? l0 : (best == 1 ? l1 : l2);
    const int* ub = best == 0 ? u0 : (best == 1 ? u1 : u2);
    const int t = split ? ub[lb[nd.start + nl]] : 0;
    int slot[3];
    wave_reserve3({&counters[CN_NODES], nnext, &counters[CN_LEAVES]},
                  {split ? 2 : 0, (int)lact + (int)ract, (int)stays + (split ? (int)!lact + (int)!ract : 0)}, slot);
    const int c0 = slot[0], na0 = slot[1], nl0 = slot[2];
    if (stays) {
        nodes[id].slot = -1;
        leaves[nl0] = id;
    }
    if (!split) return;
    KdNode L = nd, R = nd;
    L.end = nd.start + nl;
    R.start = nd.start + nl;
#pragma unroll
    for (int d = 0; d < 3; ++d)
        if (d == best) {
            L.hi[d] = t - 1;
            R.lo[d] = t;
        }
    int ka = na0, kl = nl0;
    L.slot = lact ? ka++ : -1;
    R.slot = ract ? ka : -1;
    L.dim = R.dim = -1;
    L.left = L.right = R.left = R.right = -1;
    nodes[c0] = L;
    nodes[c0 + 1] = R;
    nodes[id].dim = best;
    nodes[id].t = t;
    nodes[id].left = c0;
    nodes[id].right = c0 + 1;
    leaf_min[c0] = leaf_min[c0 + 1] = 0x7FFFFFFF;
    if (lact) next_active[L.slot] = c0; else leaves[kl++] = c0;
    if (ract) next_active[R.slot] = c0 + 1; else leaves[kl] = c0 + 1;
}

// The left flags of the three lists at once (list j at lf[j * M + p]).  A
// node splits at rank nl = n / 2 of its list along the split dimension d,
// which is ordered by (u_d, element): the list along d takes its flag from
// the position, and an element of the other two lists goes left when its
// (u_d, element) is below the median's (t, em), em = that list's entry at
// rank nl.  tail[j * tiles + tile]: the tile's left members of the node that
// its last position is in.
template <int NT>
__global__ __launch_bounds__(NT) void k_lflag3(int64_t M, const int* __restrict__ seg_node,
                                               const KdNode* __restrict__ nodes, const int* __restrict__ l0,
                                               const int* __restrict__ l1, const int* __restrict__ l2,
                                               const int* __restrict__ u0, const int* __restrict__ u1,
                                               const int* __restrict__ u2, uint8_t* __restrict__ lf,
                                               uint32_t* __restrict__ tail) {
    __shared__ uint32_t cnt[NT / 64][3];
    const int64_t p0 = (int64_t)blockIdx.x * NT, p = p0 + threadIdx.x;
    const int last = seg_node[min(p0 + NT, M) - 1];
    uint32_t f = 0;
    int id = -1;
    if (p < M) {
        id = seg_node[p];
        const KdNode& nd = nodes[id];
        const int dim = nd.dim;
        if (dim >= 0) {
            const int nl = (nd.end - nd.start) / 2;
            const uint32_t own = (p - nd.start) < nl ? 1 : 0;
            const int* ld = dim == 0 ? l0 : (dim == 1 ? l1 : l2);
            const int* ud = dim == 0 ? u0 : (dim == 1 ? u1 : u2);
            // the two other lists, in order
            const int ea = (dim == 0 ? l1 : l0)[p], eb = (dim == 2 ? l1 : l2)[p];
            const int em = ld[nd.start + nl], t = nd.t;
            const int ua = ud[ea], ub = ud[eb];
            const uint32_t a = ua < t || (ua == t && ea < em) ? 1 : 0;
            const uint32_t b = ub < t || (ub == t && eb < em) ? 1 : 0;
            f = dim == 0 ? own | a << 1 | b << 2 : dim == 1 ? a | own << 1 | b << 2 : a | b << 1 | own << 2;
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const uint32_t bit = (f >> j) & 1u;
        if (p < M) lf[j * M + p] = (uint8_t)bit;
        const uint64_t m = __ballot(bit && id == last);
        if (__lane_id() == 0) cnt[threadIdx.x >> 6][j] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint32_t s = 0;
        for (int w = 0; w < NT / 64; ++w) s += cnt[w][threadIdx.x];
        tail[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = s;
    }
}

// Stable partition of the three lists inside every split node; the
// position's node moves to its child, the entries that come to lie at a
// child's ends give its bounding box, and the next level's histograms are
// cleared.  A member's rank among its node's left members is the tile's own
// prefix of flags, from the node's start where the node begins in the tile;
// a node that began in an earlier tile is the last of every tile from there
// on, so the tails of those tiles add up to what is missing.  (Scanned flags
// took three more launches and 24 bytes a member and level: 1.42 ms against
// 1.18 ms for the 15 levels of a 256^3 box.)
// (SCANNED: the tails' prefix sums, whose difference of two is that sum.)
template <int IT, bool SCANNED>
__global__ __launch_bounds__(KB) void k_part3(int64_t M, int* __restrict__ seg_node, KdNode* __restrict__ nodes,
                                              const int* __restrict__ l0, const int* __restrict__ l1,
                                              const int* __restrict__ l2, const int* __restrict__ u0,
                                              const int* __restrict__ u1, const int* __restrict__ u2,
                                              const uint8_t* __restrict__ lf, const uint32_t* __restrict__ tail,
                                              int* __restrict__ o0, int* __restrict__ o1, int* __restrict__ o2,
                                              CoordsL0 c, uint32_t* __restrict__ hist, int64_t hist_words) {
    constexpr int NW = KB / 64, CH = NW * IT;  // chunks of 64 positions
    __shared__ uint16_t pre[3][KB * IT];
    __shared__ uint32_t cc[3][CH];
    __shared__ uint32_t before[NW][3];
    const int tid = threadIdx.x, lane = __lane_id(), w = tid >> 6;
    const int64_t tile = blockIdx.x, tiles = gridDim.x, p0 = tile * (KB * IT);
    for (int64_t k = tile * KB + tid; k < hist_words; k += tiles * KB) hist[k] = 0;
    const int* lists[3] = {l0, l1, l2};
    const int* us[3] = {u0, u1, u2};
    int* outs[3] = {o0, o1, o2};
    // left members before the tile of the node that reaches into it
    uint32_t b[3] = {0, 0, 0};
    {
        const KdNode& nd = nodes[seg_node[p0]];
        if (nd.dim >= 0 && nd.start < p0) {
            const int64_t k0 = nd.start / (KB * IT);
            if (SCANNED) {
                if (tid == 0)
                    for (int j = 0; j < 3; ++j) b[j] = tail[j * tiles + tile] - tail[j * tiles + k0];
            } else {
                for (int64_t k = k0 + tid; k < tile; k += KB)
                    for (int j = 0; j < 3; ++j) b[j] += tail[j * tiles + k];
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        for (int o = 32; o > 0; o >>= 1) b[j] += __shfl_xor(b[j], o, 64);
        if (lane == 0) before[w][j] = b[j];
    }
    int node[IT], e[3][IT];
    uint32_t f[IT];
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int64_t p = p0 + k * KB + tid;
        const bool valid = p < M;
        node[k] = valid ? seg_node[p] : -1;
        f[k] = 0;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            e[j][k] = valid ? lists[j][p] : 0;
            f[k] |= valid && lf[j * M + p] ? 1u << j : 0u;
        }
    }
#pragma unroll
    for (int k = 0; k < IT; ++k)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const uint64_t m = __ballot((f[k] >> j) & 1u);
            pre[j][k * KB + tid] = (uint16_t)__popcll(m & lanemask_lt());
            if (lane == 0) cc[j][k * NW + w] = (uint32_t)__popcll(m);
        }
    __syncthreads();
    if (w < 3) {
        const uint32_t v = lane < CH ? cc[w][lane] : 0u;
        uint32_t x = v;
#pragma unroll
        for (int o = 1; o < CH; o <<= 1) {
            const uint32_t t = __shfl_up(x, o, 64);
            if (lane >= o) x += t;
        }
        if (lane < CH) cc[w][lane] = x - v;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        b[j] = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) b[j] += before[k][j];
    }
    // flags before position q of the tile
    auto prefix = [&](int j, int q) { return cc[j][q >> 6] + (uint32_t)pre[j][q]; };
#pragma unroll
    for (int k = 0; k < IT; ++k) {
        const int64_t p = p0 + k * KB + tid;
        if (p >= M) continue;
        const KdNode& nd = nodes[node[k]];
        if (nd.dim < 0) {
#pragma unroll
            for (int j = 0; j < 3; ++j) outs[j][p] = e[j][k];
            if (c.in[0])
                for (int d = 0; d < 3; ++d) c.out[d][p] = c.in[d][p];
            continue;
        }
        const int s = nd.start, end = nd.end, nl = (end - s) / 2, left = nd.left, right = nd.right;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const uint32_t at = prefix(j, k * KB + tid);
            const int rl = (int)(s >= p0 ? at - prefix(j, (int)(s - p0)) : at + b[j]);
            const int np = (f[k] >> j) & 1u ? s + rl : s + nl + ((int)p - s - rl);
            outs[j][np] = e[j][k];
            if (j == 0 && c.in[0])
                for (int d = 0; d < 3; ++d) c.out[d][np] = c.in[d][p];
            if (np == s) nodes[left].bmin[j] = us[j][e[j][k]];
            if (np == s + nl - 1) nodes[left].bmax[j] = us[j][e[j][k]];
            if (np == s + nl) nodes[right].bmin[j] = us[j][e[j][k]];
            if (np == end - 1) nodes[right].bmax[j] = us[j][e[j][k]];
        }
        seg_node[p] = p < s + nl ? left : right;
    }
}

// Members by position in list-0 order, and the smallest index of each leaf.
// c0..c2: the coordinates in list-0 order.
__global__ void k_final(int64_t M, const int* __restrict__ l0, const int* __restrict__ seg_node,
                        const int* __restrict__ c0, const int* __restrict__ c1, const int* __restrict__ c2,
                        const int* __restrict__ g, const float* __restrict__ m, Elems F, int* __restrict__ leaf_min) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = p < M;
    const int e = valid ? l0[p] : 0;
    const int gi = valid ? g[e] : 0x7FFFFFFF;
    if (valid) {
        F.u[0][p] = c0[p];
        F.u[1][p] = c1[p];
        F.u[2][p] = c2[p];
        F.gidx[p] = gi;
        if (m) F.mass[p] = m[e];
    }
    // smallest particle index per leaf: leaves are runs of positions, so a
    // minimum over each run of the wavefront, then one atomic a run
    const int lane = __lane_id(), key = valid ? seg_node[p] : -1;
    int v = gi;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(v, o, 64), k = __shfl_up(key, o, 64);
        if (lane >= o && k == key) v = min(v, t);
    }
    const int next = __shfl_down(key, 1, 64);
    if (valid && (lane == 63 || next != key)) atomicMin(&leaf_min[key], v);
}

}  // namespace

int read_host_offsets(vr_ctx* ctx, int32_t n_hosts, const int32_t* host_offsets, int64_t n, int64_t min_size,
                      std::vector<int32_t>& off, hipStream_t st) {
    off.assign(n_hosts + 1, 0);
    if (n_hosts == 0) return VR_OK;
    int rc0 = copy_to_host(ctx, off.data(), host_offsets, (n_hosts + 1) * sizeof(int32_t), st);
    if (rc0) return rc0;
    if (off[0] != 0) return set_err(ctx, VR_ERR_INVALID_ARG, "host_offsets[0] must be 0");
    for (int h = 0; h < n_hosts; ++h) {
        const int64_t NH = (int64_t)off[h + 1] - off[h];
        if (NH < min_size)
            return set_err(ctx, VR_ERR_INVALID_ARG, "host %d has %lld members (need >= %lld)", h, (long long)NH,
                           (long long)min_size);
    }
    if (off[n_hosts] > n) return set_err(ctx, VR_ERR_INVALID_ARG, "more host members than particles");
    return VR_OK;
}

int kd_build(vr_ctx* ctx, const vr_particles* p, int32_t n_hosts, const int32_t* host_offsets,
             const int32_t* host_members, const std::vector<int32_t>& off, const std::vector<int>& ncell, int mode,
             int nbins, KdTree& tree, hipStream_t st) {
    int64_t node_cap = 0;
    for (int h = 0; h < n_hosts; ++h) {
        const int64_t NH = (int64_t)off[h + 1] - off[h];
        const int64_t minleaf = std::max<int64_t>(1, (ncell[h] + 1) / 2);
        node_cap += NH <= ncell[h] ? 1 : 2 * ((NH + minleaf - 1) / minleaf) + 1;
    }
    const int64_t M = off[n_hosts];
    const int use_mass = p->mass ? 1 : 0;
    const int counts = use_mass ? 0 : 1;
    int hb = 0;  // bits of a host
    while ((1 << hb) < n_hosts) ++hb;
    // Sorts that do not fill the device run the three dimensions together
    // (a third of the launches); with a workspace cap one after the other,
    // in a third of the room.
    const bool batch = M <= SORT_BATCH_MAX && ctx->max_ws == 0;
    const bool small = M <= SMALL_M;
    const int64_t tile = small ? KB : BIG_TILE, tiles = (M + tile - 1) / tile;
    // one workspace region holds every array of the build
    Carve cv;
    int *U[3], *G, *H, *L[3], *Lalt[3], *seg, *leaf_min, *act0, *act1, *leaves, *ncell_d, *counters, *hbox;
    int *C0[3], *C0alt[3];
    const int64_t MF = mode != KD_BUCKETS ? M : 1;  // coordinates in list-0 order, members by position
    // Bucket trees know their hosts' extents: keys relative to a host's box
    // save a sort pass or two of four to five and mostly fit 32 bits (48/16
    // neighbours of 200 k members, the whole search: 541 -> 518 us).
    // For the other trees the extents cost k_elems what the passes gain
    // (1.6 M members, cells and search: 3958 -> 4014 us).
    const bool extents = mode == KD_BUCKETS;
    const int64_t HB = extents ? 6 * (int64_t)n_hosts : 1;
    float *Ms, *images;
    uint8_t* lf8;
    uint32_t* tail;
    uint64_t* pkey;
    unsigned long long* hsh;
    KdNode* nodes;
    Elems F;
    auto layout = [&]() {
        for (int d = 0; d < 3; ++d) U[d] = cv.add<int>(M);
        G = cv.add<int>(M);
        H = cv.add<int>(M);
        Ms = cv.add<float>(use_mass ? M : 1);
        for (int d = 0; d < 3; ++d) L[d] = cv.add<int>(M);
        for (int d = 0; d < 3; ++d) Lalt[d] = cv.add<int>(M);
        for (int d = 0; d < 3; ++d) C0[d] = cv.add<int>(MF);
        for (int d = 0; d < 3; ++d) C0alt[d] = cv.add<int>(MF);
        seg = cv.add<int>(M);
        lf8 = cv.add<uint8_t>(3 * M);
        tail = cv.add<uint32_t>(3 * tiles);
        pkey = cv.add<uint64_t>(batch ? 3 * M : M);
        nodes = cv.add<KdNode>(node_cap);
        act0 = cv.add<int>(node_cap);
        act1 = cv.add<int>(node_cap);
        leaves = cv.add<int>(node_cap);
        leaf_min = cv.add<int>(node_cap);
        for (int d = 0; d < 3; ++d) F.u[d] = cv.add<int>(MF);
        F.gidx = cv.add<int>(MF);
        F.mass = cv.add<float>(use_mass ? MF : 1);
        hbox = cv.add<int>(HB);
        images = cv.add<float>(HB);
        // one upload: content hash, wide-host flag and largest extent, counters,
        // cell sizes
        hsh = cv.add<unsigned long long>(HASH_SLOTS + 2 + (CN_COUNT + n_hosts + 1) / 2);
    };
    layout();
    const size_t total = cv.bytes;
    cv.bytes = 0;
    cv.base = static_cast<char*>(ws(ctx, WS_KD, total));
    if (!cv.base) return VR_ERR_OUT_OF_MEMORY;
    layout();
    if (!use_mass) F.mass = nullptr;
    counters = reinterpret_cast<int*>(hsh + HASH_SLOTS + 2);
    ncell_d = counters + CN_COUNT;
    {
        const size_t nb = (HASH_SLOTS + 2) * sizeof(*hsh) + (CN_COUNT + (size_t)n_hosts) * sizeof(int);
        char* up = static_cast<char*>(upload_begin(ctx, nb));
        if (!up) return VR_ERR_HIP;
        std::memset(up, 0, (HASH_SLOTS + 2) * sizeof(*hsh) + CN_COUNT * sizeof(int));
        int* cn = reinterpret_cast<int*>(up + (HASH_SLOTS + 2) * sizeof(*hsh));
        cn[CN_NODES] = n_hosts;
        std::memcpy(cn + CN_COUNT, ncell.data(), (size_t)n_hosts * sizeof(int));
        VR_HIP(ctx, hipMemcpyAsync(hsh, up, nb, hipMemcpyHostToDevice, st));
        int rc = upload_end(ctx, st);
        if (rc) return rc;
        if (extents && (rc = fill_i32(ctx, hbox, INT_MAX, HB, st))) return rc;
    }
    hipLaunchKernelGGL(k_elems, dim3(grid_for(M, 256)), dim3(256), 0, st, M, n_hosts, host_offsets, host_members,
                       p->qx, p->qy, p->qz, p->mass, p->grid_bits, U[0], U[1], U[2], G, Ms, H, hsh,
                       extents ? hbox : nullptr);
    VR_LAUNCH_CHECK(ctx);
    if (extents) {
        // (few workgroups: their atomics meet on one word, a million hosts' 160 us)
        hipLaunchKernelGGL(k_host_box, dim3(std::min(grid_for(n_hosts, 256), 256u)), dim3(256), 0, st, n_hosts, 1 << (p->grid_bits - 1),
                           hbox, images, hsh + HASH_SLOTS);
        VR_LAUNCH_CHECK(ctx);
    }
    // The lists a level reads: first the sorted ones, where they are kept (read
    // only), then Lalt and L in turn.
    int* Lin[3] = {L[0], L[1], L[2]};
    int* Lout[3] = {Lalt[0], Lalt[1], Lalt[2]};
    int* Lnext[3] = {L[0], L[1], L[2]};
    // The three lists sorted by (host, u_d, element) depend only on the
    // elements' members, unwrapped coordinates and hosts.  The context keeps
    // the last build's lists and reuses them when this build's content hash and
    // size match (the entropy cells and the neighbour tree of
    // one search are built over the same members); without room for them
    // under the workspace cap it simply sorts.
    {
        unsigned long long parts[HASH_SLOTS + 2];
        int rc = read_back(ctx, hsh, parts, sizeof parts, st);
        if (rc) return rc;
        tree.images = parts[HASH_SLOTS] != 0 ? images : nullptr;
        unsigned long long h64 = 0;
        for (int k = 0; k < HASH_SLOTS; ++k) h64 += parts[k];
        int cb = 22;  // bits of a coordinate
        if (extents)
            for (cb = 1; (1ull << cb) <= parts[HASH_SLOTS + 1];) ++cb;
        const int bits = cb + hb;
        const std::string err_before = ctx->err;
        int* pre = static_cast<int*>(ws(ctx, WS_KD_PRE, 3 * (size_t)M * sizeof(int)));
        if (!pre) ctx->err = err_before;  // no room for the kept lists: not an error
        const bool hit = pre && ctx->kd_pre_ptr == pre && ctx->kd_pre_m == M && ctx->kd_pre_hash == h64;
        if (hit) {
            for (int d = 0; d < 3; ++d) Lin[d] = pre + d * M;
        } else {
            ctx->kd_pre_m = -1;
            if (pre)
                for (int d = 0; d < 3; ++d) Lin[d] = pre + d * M;
            const int step = batch && pre ? 3 : 1;  // dimensions a sort
            auto presort = [&](auto* keys) {
                using K = std::remove_pointer_t<decltype(keys)>;
                for (int d = 0; d < 3; d += step) {
                    uint32_t* ld = reinterpret_cast<uint32_t*>(Lin[d]);
                    K* kin;
                    uint32_t* vin;
                    int e;
                    if constexpr (sizeof(K) == 4) e = sort_input_u32(ctx, keys, ld, step * M, bits, &kin, &vin);
                    else e = sort_input_u64(ctx, keys, ld, step * M, bits, &kin, &vin);
                    if (e) return e;
                    hipLaunchKernelGGL(k_presort_keys<K>, dim3(grid_for(M, 256), step), dim3(256), 0, st, M, d, U[0], U[1],
                                       U[2], H, extents ? hbox : nullptr, cb, kin, vin);
                    VR_LAUNCH_CHECK(ctx);
                    if (step == 3) e = sort_batch(ctx, kin, vin, keys, ld, M, 3, bits, st);
                    else if constexpr (sizeof(K) == 4) e = sort_pairs_u32_from(ctx, kin, vin, keys, ld, M, bits, st);
                    else e = sort_pairs_u64_from(ctx, kin, vin, keys, ld, M, bits, st);
                    if (e) return e;
                }
                return (int)VR_OK;
            };
            if ((rc = bits <= 32 ? presort(reinterpret_cast<uint32_t*>(pkey)) : presort(pkey))) return rc;
            if (pre) {
                ctx->kd_pre_ptr = pre;
                ctx->kd_pre_m = M;
                ctx->kd_pre_hash = h64;
            }
        }
    }
    int* cur = act0;
    int* nxt = act1;
    const unsigned gM = grid_for(M, 256);
    // Active nodes and their members per level as the sizes alone give them
    // (a node splits at rank floor(n/2) while it holds more than ncell; the
    // sizes of one host's nodes on a level are two consecutive integers).
    // A node of coincident members that stays a leaf only lowers the true
    // counts, which the kernels read from the device; these bound the grids
    // and the number of levels, so no level waits for the host.
    std::vector<int64_t> plan_na, plan_members, plan_largest;
    {
        struct Sz { int64_t s0, c0, c1; };  // c0 nodes of size s0, c1 of size s0 + 1
        std::vector<std::pair<Sz, int>> sz;  // of the hosts that split, with their cells' size
        for (int h = 0; h < n_hosts; ++h)
            if (off[h + 1] - off[h] > ncell[h]) sz.push_back({Sz{(int64_t)off[h + 1] - off[h], 1, 0}, ncell[h]});
        for (;;) {
            int64_t na = 0, mem = 0, largest = 0;
            for (auto& [z, nc] : sz) {
                int64_t a0 = z.s0 > nc ? z.c0 : 0, a1 = z.s0 + 1 > nc ? z.c1 : 0;
                na += a0 + a1;
                mem += a0 * z.s0 + a1 * (z.s0 + 1);
                if (a0 + a1 > 0) largest = std::max(largest, z.s0 + 1);
                // children of the active ones: floor and ceil halves
                int64_t lo = INT64_MAX, cnt[3] = {0, 0, 0};
                const int64_t sizes[2] = {z.s0, z.s0 + 1}, counts[2] = {a0, a1};
                for (int k = 0; k < 2; ++k)
                    if (counts[k] > 0) lo = std::min(lo, sizes[k] / 2);
                if (lo == INT64_MAX) {
                    z = Sz{0, 0, 0};
                    continue;
                }
                for (int k = 0; k < 2; ++k) {
                    if (counts[k] == 0) continue;
                    const int64_t f = sizes[k] / 2, c = sizes[k] - f;
                    cnt[f - lo] += counts[k];
                    cnt[c - lo] += counts[k];
                }
                // the halves of two consecutive sizes span at most lo .. lo + 1
                z = Sz{lo, cnt[0], cnt[1] + cnt[2]};
            }
            if (na == 0) break;
            plan_na.push_back(na);
            plan_members.push_back(mem);
            plan_largest.push_back(largest);
            if (plan_na.size() > MAX_LEVELS) return set_err(ctx, VR_ERR_NOT_CONVERGED, "KD build exceeded 64 levels");
        }
    }
    // histograms and entropies of the widest level
    uint32_t* hc = nullptr;
    double *hm = nullptr, *Sdim = nullptr;
    int64_t hwords = 0;  // 32-bit words a node
    if (mode != KD_BUCKETS && !plan_na.empty()) {
        const int64_t na = *std::max_element(plan_na.begin(), plan_na.end());
        hwords = 3 * nbins * (counts ? 1 : 2);
        hc = static_cast<uint32_t*>(ws(ctx, WS_KD_HIST, na * hwords * sizeof(uint32_t)));
        Sdim = static_cast<double*>(ws(ctx, WS_KD_S, (size_t)na * 3 * sizeof(double)));
        if (!hc || !Sdim) return VR_ERR_OUT_OF_MEMORY;
        hm = reinterpret_cast<double*>(hc);
    }
    const bool have_c0 = mode != KD_BUCKETS;
    // (buckets that are whole hosts need no nodes)
    if (have_c0 || !plan_na.empty())
        hipLaunchKernelGGL(k_start, dim3(gM), dim3(256), 0, st, M, n_hosts, host_offsets, ncell_d, H, Lin[0], Lin[1], Lin[2],
                       U[0], U[1], U[2], nodes, act0, counters, leaves, leaf_min, seg, have_c0 ? C0[0] : nullptr, C0[1],
                       C0[2], hc, plan_na.empty() ? 0 : plan_na[0] * hwords);
    VR_LAUNCH_CHECK(ctx);
    const int hch = small ? KB : HCH;
    for (int level = 0; level < (int)plan_na.size(); ++level) {
        const int na = (int)plan_na[level];
        const int* nact = counters + CN_ACTIVE + level;
        hipEvent_t e0 = nullptr;
        if (ctx->timing) {
            e0 = timer_event(ctx);
            (void)hipEventRecord(e0, st);
        }
        if (mode != KD_BUCKETS) {
            if (counts)
                hipLaunchKernelGGL(k_hist<true>, dim3(grid_for(M, hch)), dim3(KB), 0, st, M, seg, nodes, Lin[0], C0[0],
                                   C0[1], C0[2], Ms, nbins, hch, hc, hm);
            else
                hipLaunchKernelGGL(k_hist<false>, dim3(grid_for(M, hch)), dim3(KB), 0, st, M, seg, nodes, Lin[0], C0[0],
                                   C0[1], C0[2], Ms, nbins, hch, hc, hm);
            VR_LAUNCH_CHECK(ctx);
            hipLaunchKernelGGL(k_entropy, dim3(grid_for((int64_t)na * 64, 256)), dim3(256), 0, st, nact, cur, nodes,
                               nbins, counts, hc, hm, Sdim);
            VR_LAUNCH_CHECK(ctx);
        }
        hipLaunchKernelGGL(k_split, dim3(grid_for(na, 256)), dim3(256), 0, st, nact, cur, nodes, Lin[0], Lin[1], Lin[2],
                           U[0], U[1], U[2], mode, Sdim, ncell_d, nxt, leaves, leaf_min, counters,
                           counters + CN_ACTIVE + level + 1);
        VR_LAUNCH_CHECK(ctx);
        CoordsL0 cl0{};
        if (have_c0) cl0 = CoordsL0{{C0[0], C0[1], C0[2]}, {C0alt[0], C0alt[1], C0alt[2]}};
        const int64_t hz = level + 1 < (int)plan_na.size() ? plan_na[level + 1] * hwords : 0;
        // (flags: one position a thread; the partition, which has the tile's
        // prefix to pass round: four.  Box of 256^3, 15 levels: 0.87 + 1.18 ms,
        // the other way round 1.28 + 1.99 ms)
        auto partition = [&](auto tile_t) {
            constexpr int TILE = decltype(tile_t)::value;
            hipLaunchKernelGGL(k_lflag3<TILE>, dim3((unsigned)tiles), dim3(TILE), 0, st, M, seg, nodes, Lin[0], Lin[1],
                               Lin[2], U[0], U[1], U[2], lf8, tail);
            VR_LAUNCH_CHECK(ctx);
            const bool scanned = plan_largest[level] > SCAN_TILES * TILE;
            if (scanned) {
                const int e = scan_u32(ctx, tail, tail, 3 * tiles, nullptr, st);
                if (e) return e;
            }
            hipLaunchKernelGGL((scanned ? k_part3<TILE / KB, true> : k_part3<TILE / KB, false>), dim3((unsigned)tiles),
                               dim3(KB), 0, st, M, seg, nodes, Lin[0], Lin[1], Lin[2], U[0], U[1], U[2], lf8, tail, Lout[0],
                               Lout[1], Lout[2], cl0, hc, hz);
            VR_LAUNCH_CHECK(ctx);
            return (int)VR_OK;
        };
        int rc = small ? partition(std::integral_constant<int, KB>{}) : partition(std::integral_constant<int, BIG_TILE>{});
        if (rc) return rc;
        for (int j = 0; j < 3; ++j) {
            Lin[j] = Lout[j];
            std::swap(Lout[j], Lnext[j]);
            std::swap(C0[j], C0alt[j]);
        }
        if (ctx->timing) {
            hipEvent_t e1 = timer_event(ctx);
            (void)hipEventRecord(e1, st);
            timer_push(ctx, "kd_level", e0, e1, (double)plan_members[level]);
        }
        std::swap(cur, nxt);
    }
    for (int d = 0; d < 3; ++d) tree.elem_u[d] = U[d];
    tree.use_mass = use_mass;
    if (mode == KD_BUCKETS) {
        for (int d = 0; d < 3; ++d) tree.list[d] = Lin[d];
        tree.elem_g = G;
        tree.scratch = Lout[0];
        return VR_OK;
    }
    int nleaf = 0;
    int rc = read_back(ctx, counters + CN_LEAVES, &nleaf, sizeof nleaf, st);
    if (rc) return rc;
    hipLaunchKernelGGL(k_final, dim3(gM), dim3(256), 0, st, M, Lin[0], seg, C0[0], C0[1], C0[2], G,
                       use_mass ? Ms : nullptr, F, leaf_min);
    VR_LAUNCH_CHECK(ctx);
    tree.nodes = nodes;
    tree.leaves = leaves;
    tree.n_leaves = nleaf;
    tree.seg_node = seg;
    tree.leaf_min = leaf_min;
    tree.F = F;
    return VR_OK;
}

}  // namespace vr
