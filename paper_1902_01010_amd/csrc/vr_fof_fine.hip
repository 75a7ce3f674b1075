// vr_fof_fine.hip -- 3D friends-of-friends with a two-level grid (Sec. 2.1,
// Eq. fof3d).
//
// Coarse cells have side S = 2^s >= ellx, so every link joins a cell to
// itself or to one of its 26 neighbours; each coarse cell is cut into r^3 <=
// 64 fine cells of side f = 2^k with 3 (f-1)^2 < ellx^2, so all members of a
// fine cell are linked to each other: the union-find runs over fine cells.
// Particles are sorted by (coarse cell in row-major order, fine cell).  A
// coarse cell's occupied fine cells are one 64-bit mask; for a fine cell A
// and a neighbour offset, two tables of exact integer bounds give the fine
// cells whose box lies wholly within ellx of A's (certain links) and those
// that may hold a link (possible), so one AND finds the candidates of a
// whole coarse cell without touching them.
//
// 1. Every fine cell hooks onto its smallest certain neighbour of smaller
//    index (no finds, no atomics), and the trees are flattened: that merges
//    the halos but for their seams and outskirts.
// 2. The remaining certain pairs unite, and the trees are flattened again.
// 3. The possible pairs with different roots test their particles.
// A coarse cell whose fine cells share one root carries it, so an equal root
// settles a whole neighbour cell with one load.
//
// Bound by the latency and the cache lines of scattered reads.  A thread that
// walks every candidate fine cell of 14 coarse cells (45 on average, 600 in a
// halo's outskirts, a cache line each) took 4.05 ms on a 256^3 box, half of it
// for records that the box bound then rejects, and 0.31 ms on 14 k particles
// for the longest walk; a wavefront a dense coarse cell 0.86 and 0.31 ms, and
// 5.6 ms where stellar discs put thousands of particles into a fine cell
// (the particle tests of one pair ran on one lane).  Now: 3.7 ms in all on
// the box, 0.17 ms on the 14 k, 1.2 ms in place of 8.4 ms with the discs.
//
// Every decision compares an exact integer squared distance d2 with l2c =
// ceil(ell2): for an integer d2, d2 < ell2 exactly when d2 < l2c, so the
// integer test decides as the plain definition's FP64 test does.
#include "vr_grid.h"

namespace vr {
namespace {

struct FineGrid {
    int gb, s, k, b, lr, r;
    int nc;   // coarse cells per side
};

// Sort key of particle i: its fine-cell key (coarse cell in row-major order,
// then the fine cell inside it) above the particle's offsets inside its fine
// cell (3 k bits), which the sort carries along without ordering by them.
// With grid_bits <= 21 the whole key takes at most 63 bits.
__global__ void k_finekey(int64_t n, const uint32_t* __restrict__ qx, const uint32_t* __restrict__ qy,
                          const uint32_t* __restrict__ qz, FineGrid G, uint64_t* __restrict__ key,
                          uint32_t* __restrict__ idx) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t x = qx[i], y = qy[i], z = qz[i];
    const uint64_t ck = ((uint64_t)(z >> G.s) << (2 * G.b)) | ((uint64_t)(y >> G.s) << G.b) | (uint64_t)(x >> G.s);
    const uint32_t m = (uint32_t)G.r - 1;
    const uint64_t sub = ((uint64_t)((z >> G.k) & m) << (2 * G.lr)) | ((uint64_t)((y >> G.k) & m) << G.lr) |
                         (uint64_t)((x >> G.k) & m);
    const uint32_t om = (1u << G.k) - 1u;
    const uint64_t off = ((uint64_t)(z & om) << (2 * G.k)) | ((uint64_t)(y & om) << G.k) | (uint64_t)(x & om);
    key[i] = (((ck << (3 * G.lr)) | sub) << (3 * G.k)) | off;
    idx[i] = (uint32_t)i;
}

// In place after the sort: the fine-cell key, and the coordinates rebuilt
// from it and the carried offsets (sequential, where a gather through the
// sorted order would fetch a cache line per coordinate).
__global__ void k_decode_q(int64_t n, FineGrid G, uint64_t* __restrict__ key, uint32_t* __restrict__ sx,
                           uint32_t* __restrict__ sy, uint32_t* __restrict__ sz) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const uint64_t e = key[p];
    const uint64_t kf = e >> (3 * G.k);
    const uint32_t om = (1u << G.k) - 1u;
    const uint32_t ox = (uint32_t)e & om, oy = (uint32_t)(e >> G.k) & om, oz = (uint32_t)(e >> (2 * G.k)) & om;
    const int lr3 = 3 * G.lr;
    const uint64_t ck = kf >> lr3;
    const uint32_t sub = (uint32_t)(kf & ((1ull << lr3) - 1));
    const uint32_t ncm = (uint32_t)G.nc - 1u, rm = (uint32_t)G.r - 1u;
    const uint32_t fx = (uint32_t)(ck & ncm) * (uint32_t)G.r + (sub & rm);
    const uint32_t fy = (uint32_t)((ck >> G.b) & ncm) * (uint32_t)G.r + ((sub >> G.lr) & rm);
    const uint32_t fz = (uint32_t)(ck >> (2 * G.b)) * (uint32_t)G.r + (sub >> (2 * G.lr));
    key[p] = kf;
    sx[p] = (fx << G.k) | ox;
    sy[p] = (fy << G.k) | oy;
    sz[p] = (fz << G.k) | oz;
}

__global__ void k_key_flags(int64_t n, const uint64_t* __restrict__ key, uint32_t* __restrict__ flag) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) flag[p] = (p == 0 || key[p] != key[p - 1]) ? 1u : 0u;
}

__global__ void k_fine_starts(int64_t n, const uint64_t* __restrict__ key, const uint32_t* __restrict__ scan,
                              uint32_t* __restrict__ fine_start, uint32_t* __restrict__ fid) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const bool start = (p == 0 || key[p] != key[p - 1]);
    const uint32_t f = start ? scan[p] : scan[p] - 1;
    fid[p] = f;
    if (start) fine_start[f] = (uint32_t)p;
    if (p == n - 1) fine_start[f + 1] = (uint32_t)n;
}

// Pairs of fine cells with more than HEAVY particle pairs to test are listed
// for k_link_heavy, which tests 64 at a time.
constexpr uint32_t HEAVY = 32;
struct HeavyList {
    uint2* pair;
    int* count;
    uint32_t cap;
};
__device__ __forceinline__ bool defer_pair(HeavyList H, uint32_t A, uint32_t B) {
    const uint32_t at = (uint32_t)atomicAdd(H.count, 1);
    if (at >= H.cap) return false;
    H.pair[at] = make_uint2(A, B);
    return true;
}

// Whether some particle of [a0, a1) lies within the linking length of one of
// [b0, b1).
__device__ __forceinline__ bool test_particles(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1,
                                               const uint32_t* __restrict__ sx, const uint32_t* __restrict__ sy,
                                               const uint32_t* __restrict__ sz, int gb, int64_t l2c) {
    for (uint32_t pp = a0; pp < a1; ++pp) {
        const int px = (int)sx[pp], py = (int)sy[pp], pz = (int)sz[pp];
        for (uint32_t q = b0; q < b1; ++q) {
            const int dx = min_image((int)sx[q] - px, gb);
            const int dy = min_image((int)sy[q] - py, gb);
            const int dz = min_image((int)sz[q] - pz, gb);
            if ((int64_t)dx * dx + (int64_t)dy * dy + (int64_t)dz * dz < l2c) return true;
        }
    }
    return false;
}

// Number of occupied coarse cells before coarse cell `cell` (row-major
// index): the prefix count of its 64-cell word plus the occupancy bits
// below `cell` in that word (two independent loads).  Occupied cells are
// numbered in sorted order, so this is also the coarse index of `cell`
// when it is occupied.
__device__ __forceinline__ uint32_t coarse_rank(const uint64_t* __restrict__ occ, const uint32_t* __restrict__ pre,
                                                uint64_t cell) {
    const uint64_t w = cell >> 6;
    return pre[w] + (uint32_t)__popcll(occ[w] & ((1ull << (cell & 63)) - 1ull));
}

// Neighbour offsets (dx, dy, dz) in ascending cell order, o = 9 (dz + 1) +
// 3 (dy + 1) + dx + 1; OWN is the cell itself, larger ones are the forward
// half of the neighbourhood.
constexpr int NOFF = 27, OWN = 13;

// What the link passes read.
struct Links {
    FineGrid G;
    int64_t l2c;
    const uint2* frec;      // [nfine] coarse cell, fine cell inside it
    uint4* crec;            // [ncoarse] mask of fine cells (two words), first fine cell, common root or -1
    const uint32_t* nbits;  // [ncoarse] occupied neighbours, bit o
    const uint64_t* key;    // fine-cell key by sorted position
    const uint32_t* fine_start;
    const uint64_t* occ;    // occupancy bits of the coarse cells, and
    const uint32_t* pre;    // the count of occupied ones before each 64
    const uint64_t* cert;   // [64][NOFF] certain and possible partners
    const uint64_t* poss;
    const uint32_t *sx, *sy, *sz;
    int* uf;                // [nfine] union-find parents
};

// cert, poss: block o, lane a
__global__ __launch_bounds__(64) void k_pair_tables(FineGrid G, int64_t l2c, uint64_t* __restrict__ cert,
                                                    uint64_t* __restrict__ poss) {
    const int o = (int)blockIdx.x, a = (int)threadIdx.x, rm = G.r - 1;
    const int ox = o % 3 - 1, oy = (o / 3) % 3 - 1, oz = o / 9 - 1;
    const int64_t f = int64_t(1) << G.k;
    uint64_t mc = 0, mp = 0;
    for (int b = 0; b < G.r * G.r * G.r; ++b) {
        const int gx = abs(ox * G.r + (b & rm) - (a & rm));
        const int gy = abs(oy * G.r + ((b >> G.lr) & rm) - ((a >> G.lr) & rm));
        const int gz = abs(oz * G.r + (b >> (2 * G.lr)) - (a >> (2 * G.lr)));
        // exact bounds of the squared distance between members of the boxes
        const int64_t ux = (gx + 1) * f - 1, uy = (gy + 1) * f - 1, uz = (gz + 1) * f - 1;
        const int64_t lx = gx ? (gx - 1) * f + 1 : 0, ly = gy ? (gy - 1) * f + 1 : 0, lz = gz ? (gz - 1) * f + 1 : 0;
        if (ux * ux + uy * uy + uz * uz < l2c) mc |= 1ull << b;
        if (lx * lx + ly * ly + lz * lz < l2c) mp |= 1ull << b;
    }
    cert[a * NOFF + o] = mc;
    poss[a * NOFF + o] = mp;
}

// Per coarse cell: the mask of its fine cells and its occupied neighbours.
// Two cells in three of a cosmological box have none, and cost the later
// passes one coalesced word.
__global__ void k_coarse_rec(const uint32_t* __restrict__ ncoarse, const uint32_t* __restrict__ cfs, const uint2* __restrict__ frec,
                             const uint64_t* __restrict__ key, const uint32_t* __restrict__ fine_start, FineGrid G,
                             const uint64_t* __restrict__ occ, uint4* __restrict__ crec, uint32_t* __restrict__ nbits) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= *ncoarse) return;
    const uint32_t f0 = cfs[c], f1 = cfs[c + 1];
    const uint64_t ck = key[fine_start[f0]] >> (3 * G.lr);
    const int ncm = G.nc - 1;
    const int cx = (int)(ck & ncm), cy = (int)((ck >> G.b) & ncm), cz = (int)(ck >> (2 * G.b));
    uint64_t row[9];
#pragma unroll
    for (int r = 0; r < 9; ++r)
        row[r] = ((uint64_t)((cz + r / 3 - 1) & ncm) * (uint64_t)G.nc + (uint64_t)((cy + r % 3 - 1) & ncm)) *
                 (uint64_t)G.nc;
    uint32_t nb = 0;
    if (cx > 0 && cx < ncm) {
        uint64_t v[9];
#pragma unroll
        for (int r = 0; r < 9; ++r) {
            const uint64_t i0 = row[r] + (uint64_t)(cx - 1);
            const int o = (int)(i0 & 63);
            v[r] = occ[i0 >> 6] >> o;
            if (o > 61) v[r] |= occ[(i0 >> 6) + 1] << (64 - o);
        }
#pragma unroll
        for (int r = 0; r < 9; ++r) nb |= (uint32_t)(v[r] & 7ull) << (3 * r);
    } else {
        for (int r = 0; r < 9; ++r)
            for (int d = 0; d < 3; ++d) {
                const uint64_t i = row[r] + (uint64_t)((cx + d - 1) & ncm);
                nb |= (uint32_t)((occ[i >> 6] >> (i & 63)) & 1ull) << (3 * r + d);
            }
    }
    nbits[c] = nb & ~(1u << OWN);
    uint64_t m = 0;
    for (uint32_t F = f0; F < f1; ++F) m |= 1ull << frec[F].y;
    crec[c] = make_uint4((uint32_t)m, (uint32_t)(m >> 32), f0, ~0u);
}

__device__ __forceinline__ uint64_t mask_of(uint4 r) { return ((uint64_t)r.y << 32) | r.x; }

// The coarse indices of a cell's neighbours, one row of three at a time.
struct NeighbourRow {
    uint32_t first;  // coarse index of the row's first occupied neighbour
    bool wrap;       // the row wraps round the box: indices by lookup
    uint64_t base;
    int cx;
};
__device__ __forceinline__ NeighbourRow neighbour_row(const Links& K, uint64_t ck, int r) {
    const FineGrid& G = K.G;
    const int ncm = G.nc - 1;
    const int cx = (int)(ck & ncm), cy = (int)((ck >> G.b) & ncm), cz = (int)(ck >> (2 * G.b));
    NeighbourRow n;
    n.cx = cx;
    n.base = ((uint64_t)((cz + r / 3 - 1) & ncm) * (uint64_t)G.nc + (uint64_t)((cy + r % 3 - 1) & ncm)) *
             (uint64_t)G.nc;
    n.wrap = cx == 0 || cx == ncm;
    n.first = n.wrap ? 0u : coarse_rank(K.occ, K.pre, n.base + (uint64_t)(cx - 1));
    return n;
}
// coarse index of neighbour d (0..2) of the row whose occupied ones are bits
// (own: the cell itself also lies in the row)
__device__ __forceinline__ uint32_t neighbour(const Links& K, const NeighbourRow& n, uint32_t bits, int d) {
    if (!n.wrap) return n.first + (uint32_t)__popc(bits & ((1u << d) - 1u));
    return coarse_rank(K.occ, K.pre, n.base + (uint64_t)((n.cx + d - 1) & (K.G.nc - 1)));
}

// Hooks every fine cell F onto the first certain neighbour of smaller index
// found in ascending cell order (itself if none): parents are smaller than
// their children, so there are no cycles, and nothing waits for another
// thread.
__global__ __launch_bounds__(256) void k_hook(const uint32_t* __restrict__ nfine, Links K) {
    const int64_t F = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (F >= *nfine) return;
    const uint2 fr = K.frec[F];
    const uint32_t c = fr.x, a = fr.y;
    const uint4 own = K.crec[c];
    const uint32_t nb = K.nbits[c];
    const uint32_t back = nb & ((1u << OWN) - 1u);
    int par = (int)F;
    if (back) {
        const uint64_t ck = K.key[K.fine_start[own.z]] >> (3 * K.G.lr);
        for (int r = 0; r < 5 && par == (int)F; ++r) {
            uint32_t bits = (nb >> (3 * r)) & 7u;
            if (r == 4) bits = (bits & 1u) | 2u;  // up to the own cell
            if (!(r == 4 ? bits & 1u : bits)) continue;
            const NeighbourRow n = neighbour_row(K, ck, r);
            for (int d = 0; d < (r == 4 ? 1 : 3); ++d) {
                if (!((bits >> d) & 1u)) continue;
                const uint32_t c2 = neighbour(K, n, bits, d);
                if (c2 >= c) continue;  // across the box edge
                const uint4 cr = K.crec[c2];
                const uint64_t m = mask_of(cr) & K.cert[a * NOFF + 3 * r + d];
                if (m) {
                    par = (int)(cr.z + (uint32_t)__popcll(mask_of(cr) & ((m & (0 - m)) - 1ull)));
                    break;
                }
            }
        }
    }
    if (par == (int)F) {
        const uint64_t m = mask_of(own) & K.cert[a * NOFF + OWN] & ((1ull << a) - 1ull);
        if (m) par = (int)(own.z + (uint32_t)__popcll(mask_of(own) & ((m & (0 - m)) - 1ull)));
    }
    K.uf[F] = par;
}

__global__ void k_flatten(const uint32_t* __restrict__ nfine, int* uf) {
    const int64_t F = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (F >= *nfine) return;
    int p = uf[F];
    if (p == (int)F) return;
    for (int g = uf[p]; g != p; g = uf[p]) p = g;
    uf[F] = p;
}

// The root that all fine cells of a coarse cell share, or -1.
__global__ void k_coarse_root(const uint32_t* __restrict__ ncoarse, const int* __restrict__ uf, uint4* __restrict__ crec) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= *ncoarse) return;
    const uint4 r = crec[c];
    const uint32_t n = (uint32_t)__popcll(mask_of(r));
    const int root = uf[r.z];
    bool same = true;
    for (uint32_t j = 1; j < n && same; ++j) same = uf[r.z + j] == root;
    crec[c].w = same ? (uint32_t)root : ~0u;
}

// Unites fine cell A with its partners among the own cell's later fine cells
// and the forward neighbours: the certain ones (TEST false), or the possible
// ones that are not certain, by testing their particles.  The roots are
// flattened when the pass starts; a partner whose parent is A's root is done.
// LPC = 16: a lane per neighbour.
template <bool TEST, int LPC>
__global__ __launch_bounds__(256) void k_link_cells(const uint32_t* __restrict__ nfine, Links K, unsigned xchunk, HeavyList H) {
    const int64_t t = (int64_t)xcd_swizzle(blockIdx.x, gridDim.x, xchunk) * blockDim.x + threadIdx.x;
    const int64_t A = t / LPC;
    if (A >= *nfine) return;
    const uint2 fr = K.frec[A];
    const uint32_t c = fr.x, a = fr.y;
    const uint32_t fwd = K.nbits[c] >> (OWN + 1);
    const uint4 own = K.crec[c];
    const int r0 = K.uf[A];
    int ra = r0;
    auto partners = [&](uint4 cr, uint64_t m) __attribute__((always_inline)) {
        // four partners' parents a round trip
        while (m) {
            uint32_t B[4];
            int pb[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                B[j] = ~0u;
                if (m) {
                    B[j] = cr.z + (uint32_t)__popcll(mask_of(cr) & ((m & (0 - m)) - 1ull));
                    m &= m - 1;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) pb[j] = B[j] != ~0u ? K.uf[B[j]] : 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // ra may be stale, but roots once equal stay equal
                if (B[j] == ~0u || pb[j] == ra || pb[j] == r0) continue;
                const int rb = uf_find(K.uf, pb[j]);
                if (rb == ra) continue;
                ra = uf_find(K.uf, ra);
                if (ra == rb) continue;
                if (TEST) {
                    const uint32_t a0 = K.fine_start[A], a1 = K.fine_start[A + 1];
                    const uint32_t b0 = K.fine_start[B[j]], b1 = K.fine_start[B[j] + 1];
                    // a listed pair unites nothing yet, and every pair that its
                    // union would have settled is listed too: four tests first
                    // (1 M particles in halos: both kernels 1.05 -> 0.29 ms)
                    if ((uint64_t)(a1 - a0) * (b1 - b0) > HEAVY &&
                        !test_particles(a0, a0 + 1, b0, min(b1, b0 + 4), K.sx, K.sy, K.sz, K.G.gb, K.l2c) &&
                        defer_pair(H, (uint32_t)A, B[j]))
                        continue;
                    if (!test_particles(a0, a1, b0, b1, K.sx, K.sy, K.sz, K.G.gb, K.l2c)) continue;
                }
                uf_union(K.uf, ra, rb);
            }
        }
    };
    auto candidates = [&](int o) __attribute__((always_inline)) {
        const uint64_t mc = K.cert[a * NOFF + o];
        return TEST ? K.poss[a * NOFF + o] & ~mc : mc;
    };
    if constexpr (LPC == 16) {
        // a lane a neighbour, the first one for the own cell
        const int part = (int)(t % LPC), o = OWN + part;
        if (part > 0) {
            if (part > 13 || !((fwd >> (part - 1)) & 1u)) return;
            const uint64_t ck = K.key[K.fine_start[own.z]] >> (3 * K.G.lr);
            const int r = o / 3, d = o % 3;
            uint32_t c2 = c + 1;  // the own row's last neighbour follows the own cell
            NeighbourRow n;
            if (r > 4 || ((int)(ck & (K.G.nc - 1)) == K.G.nc - 1)) {
                n = neighbour_row(K, ck, r);
                c2 = neighbour(K, n, r == 4 ? 4u : (fwd >> (3 * r - OWN - 1)) & 7u, d);
            }
            const uint4 cr = K.crec[c2];
            if ((int)cr.w != r0) partners(cr, mask_of(cr) & candidates(o));
            return;
        }
    }
    if ((int)own.w != r0) {
        const uint64_t later = a == 63 ? 0ull : ~0ull << (a + 1);
        const uint64_t m = mask_of(own) & later;
        if (m) partners(own, m & candidates(OWN));
    }
    if (LPC > 1 || !fwd) return;
    const uint64_t ck = K.key[K.fine_start[own.z]] >> (3 * K.G.lr);
    // rows 4 (behind the own cell) to 8
    for (int r = 4; r < 9; ++r) {
        uint32_t bits = (fwd >> (r == 4 ? 0 : 3 * r - OWN - 1)) & (r == 4 ? 1u : 7u);
        if (!bits) continue;
        NeighbourRow n = neighbour_row(K, ck, r);
        if (r == 4) {
            // the own row's last neighbour follows the own cell
            bits = 4u;
            n.first = c + 1;
        }
        for (int d = 0; d < 3; ++d) {
            if (!((bits >> d) & 1u)) continue;
            const uint4 cr = K.crec[neighbour(K, n, bits, d)];
            if ((int)cr.w == r0) continue;  // one component with A
            partners(cr, mask_of(cr) & candidates(3 * r + d));
        }
    }
}

// occupancy bits per 64-cell word (the scan turns them into the prefix
// counts of coarse_rank); the extra last word counts nothing
__global__ void k_occ_count(int64_t words, const uint64_t* __restrict__ occ, uint32_t* __restrict__ cnt) {
    const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w <= words) cnt[w] = w < words ? (uint32_t)__popcll(occ[w]) : 0u;
}

// fine-cell records: coarse cell, fine cell inside it
__global__ void k_frec(const uint32_t* __restrict__ nfine, const uint32_t* __restrict__ fine_start, const uint64_t* __restrict__ key,
                       const uint32_t* __restrict__ cid, int lr3, uint2* __restrict__ frec) {
    const int64_t F = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (F >= *nfine) return;
    frec[F] = make_uint2(cid[F], (uint32_t)key[fine_start[F]] & ((1u << lr3) - 1u));
}

// coarse-cell starts among the fine cells: flag[F] = 1 where F < bound opens a
// coarse cell
__global__ void k_coarse_flags(int64_t bound, const uint32_t* __restrict__ nfine, const uint32_t* __restrict__ fine_start,
                               const uint64_t* __restrict__ key, int lr3, uint32_t* __restrict__ flag) {
    const int64_t F = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (F >= bound) return;
    flag[F] = F < *nfine && (F == 0 || (key[fine_start[F]] >> lr3) != (key[fine_start[F - 1]] >> lr3)) ? 1u : 0u;
}

// after an exclusive scan of the flags in place: cid[F] = coarse index of F,
// cfs[c] = first fine cell of coarse cell c, cfs[ncoarse] = nfine
__global__ void k_coarse_starts(const uint32_t* __restrict__ nfine, const uint32_t* __restrict__ fine_start,
                                const uint64_t* __restrict__ key, int lr3, uint32_t* __restrict__ cid,
                                uint32_t* __restrict__ cfs, unsigned long long* __restrict__ occ) {
    const int64_t F = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (F >= *nfine) return;
    const uint64_t ck = key[fine_start[F]] >> lr3;
    const bool start = F == 0 || ck != (key[fine_start[F - 1]] >> lr3);
    const uint32_t c = start ? cid[F] : cid[F] - 1;
    cid[F] = c;
    if (start) {
        cfs[c] = (uint32_t)F;
        atomicOr(&occ[ck >> 6], 1ull << (ck & 63));
    }
    if (F == *nfine - 1) cfs[c + 1] = *nfine;
}

__device__ __forceinline__ int uf_root(const int* uf, int a) {
    int p = uf[a];
    while (p != a) {
        a = p;
        p = uf[a];
    }
    return a;
}

// The listed pairs of fine cells, a wavefront each: the smaller cell's
// particles one after another (those beyond ellx of the other's box are
// passed over), 64 of the larger's at a time.
__global__ __launch_bounds__(64) void k_link_heavy(HeavyList H, Links K) {
    const uint32_t n = min((uint32_t)*H.count, H.cap);
    const FineGrid G = K.G;
    const int64_t f = int64_t(1) << G.k, l2c = K.l2c;
    const uint32_t *sx = K.sx, *sy = K.sy, *sz = K.sz;
    for (uint32_t it = blockIdx.x; it < n; it += gridDim.x) {
        const uint2 pr = H.pair[it];
        const int ra = uf_root(K.uf, (int)pr.x), rb = uf_root(K.uf, (int)pr.y);
        if (ra == rb) continue;
        uint2 s = make_uint2(K.fine_start[pr.x], K.fine_start[pr.x + 1]);  // fewer particles
        uint2 l = make_uint2(K.fine_start[pr.y], K.fine_start[pr.y + 1]);  // more
        if (s.y - s.x > l.y - l.x) {
            const uint2 t = s;
            s = l;
            l = t;
        }
        // the larger cell's box: its first particle rounded down to the fine grid
        const int bx = (int)(sx[l.x] >> G.k << G.k), by = (int)(sy[l.x] >> G.k << G.k), bz = (int)(sz[l.x] >> G.k << G.k);
        bool hit = false;
        for (uint32_t p = s.x; p < s.y && !hit; ++p) {
            const int px = (int)sx[p], py = (int)sy[p], pz = (int)sz[p];
            auto gap = [&](int b, int x) __attribute__((always_inline)) {
                const int64_t d = min_image(b - x, G.gb);  // the box starts d above x
                return d > 0 ? d : d + f - 1 < 0 ? -(d + f - 1) : int64_t(0);
            };
            const int64_t gx = gap(bx, px), gy = gap(by, py), gz = gap(bz, pz);
            if (gx * gx + gy * gy + gz * gz >= l2c) continue;
            for (uint32_t q0 = l.x; q0 < l.y && !hit; q0 += 64) {
                const uint32_t q = q0 + threadIdx.x;
                bool in = false;
                if (q < l.y) {
                    const int dx = min_image((int)sx[q] - px, G.gb);
                    const int dy = min_image((int)sy[q] - py, G.gb);
                    const int dz = min_image((int)sz[q] - pz, G.gb);
                    in = (int64_t)dx * dx + (int64_t)dy * dy + (int64_t)dz * dz < l2c;
                }
                hit = __ballot(in) != 0;
            }
        }
        if (hit && threadIdx.x == 0) uf_union(K.uf, ra, rb);
    }
}

// Smallest original index per component.  Members of a fine cell are in
// index order (the sort is stable), so its first member's is its smallest:
// every root first stores its own (no atomics for the many singletons), then
// the other fine cells lower it.
__global__ void k_root_idx_f(const uint32_t* __restrict__ nfine, const int* __restrict__ uf, const uint32_t* __restrict__ fine_start,
                             const uint32_t* __restrict__ idx, int* __restrict__ mn) {
    const int64_t F = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (F < *nfine && uf[F] == (int)F) mn[F] = (int)idx[fine_start[F]];
}

__global__ void k_min_orig_f(const uint32_t* __restrict__ nfine, const int* __restrict__ uf, const uint32_t* __restrict__ fine_start,
                             const uint32_t* __restrict__ idx, int* __restrict__ mn, int stride) {
    const int64_t F = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * stride;
    const bool valid = F < *nfine && uf[F] != (int)F;
    wave_atomic_min(mn, valid ? uf[F] : 0, valid ? (int)idx[fine_start[F]] : 0x7FFFFFFF, valid);
}

__global__ void k_label_f(int64_t n, const int* __restrict__ uf, const uint32_t* __restrict__ fid,
                          const uint32_t* __restrict__ idx, const int* __restrict__ mn, int32_t* __restrict__ label) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) label[idx[p]] = mn[uf[fid[p]]];
}

}  // namespace

bool fof3d_fine_applicable(int gb, int s) {
    const int b = gb - s;
    return b >= 2 && b <= 12;  // 4 .. 4096 coarse cells a side
}

// Up to this many particles the link passes take a lane per fine cell and
// neighbour: their time is the longest chain of one cell's partners, beyond it
// the pairs that threads test before others have joined them.  The call without
// and with it: a halo 247 -> 230 us at 14 k particles, 261 -> 233 at 28 k, from
// -6 to 9% (three halos) at 35 k, 270 -> 286 at 48 k, 300 -> 330 at 117 k; a box,
// whose pairs are spread wider, 251 -> 183 at 14 k, 328 -> 311 at 111 k, 355 -> 371
// at 262 k, 904 -> 1330 at 2.1 M.
constexpr int64_t LANE_PER_NEIGHBOUR = 32768;

int fof3d_fine(vr_ctx* ctx, const vr_particles* p, double ell2, int s, int32_t* label, hipStream_t st) {
    const int64_t n = p->n;
    FineGrid G;
    G.gb = p->grid_bits;
    G.s = s;
    int k = 0;
    while (k + 1 <= s && 3.0 * (double)((int64_t(2) << k) - 1) * (double)((int64_t(2) << k) - 1) < ell2) ++k;
    G.k = k;
    G.b = G.gb - s;
    G.lr = s - k;
    G.r = 1 << G.lr;
    G.nc = 1 << G.b;
    const int key_bits = 3 * (G.gb - k);
    VR_WS(key, ctx, uint64_t, WS_A0, n);
    VR_WS(idx, ctx, uint32_t, WS_A1, n);
    VR_WS(sx, ctx, uint32_t, WS_A2, n);
    VR_WS(sy, ctx, uint32_t, WS_A3, n);
    VR_WS(sz, ctx, uint32_t, WS_A4, n);
    VR_WS(scan, ctx, uint32_t, WS_A5, n);
    VR_WS(fine_start, ctx, uint32_t, WS_A6, n + 1);
    VR_WS(fid, ctx, uint32_t, WS_A7, n);
    VR_WS(tot, ctx, uint32_t, WS_FLAG, 4);
    const unsigned gn = grid_for(n, 256);
    uint64_t* kin;
    uint32_t* iin;
    const int off_bits = 3 * k;
    int rc = sort_input_u64(ctx, key, idx, n, off_bits + key_bits, &kin, &iin, off_bits);
    if (rc) return rc;
    hipLaunchKernelGGL(k_finekey, dim3(gn), dim3(256), 0, st, n, p->qx, p->qy, p->qz, G, kin, iin);
    VR_LAUNCH_CHECK(ctx);
    if ((rc = sort_pairs_u64_from(ctx, kin, iin, key, idx, n, off_bits + key_bits, st, off_bits))) return rc;
    hipLaunchKernelGGL(k_decode_q, dim3(gn), dim3(256), 0, st, n, G, key, sx, sy, sz);
    VR_LAUNCH_CHECK(ctx);
    hipLaunchKernelGGL(k_key_flags, dim3(gn), dim3(256), 0, st, n, key, scan);
    VR_LAUNCH_CHECK(ctx);
    if ((rc = scan_u32(ctx, scan, scan, n, tot, st))) return rc;
    hipLaunchKernelGGL(k_fine_starts, dim3(gn), dim3(256), 0, st, n, key, scan, fine_start, fid);
    VR_LAUNCH_CHECK(ctx);
    // The kernels read the counts of cells from the device (tot); the host
    // waits for them only where they save more than the wait.
    const bool bound = n <= FEW_POINTS && ctx->max_ws == 0;
    uint32_t nfine = (uint32_t)n;
    if (!bound && (rc = read_back(ctx, tot, &nfine, sizeof nfine, st))) return rc;
    // coarse index per fine cell, first fine cell per coarse cell, the
    // occupancy bit of every coarse cell with prefix counts per 64 cells
    // (nc^3 / 8 + nc^3 / 16 bytes), and the records of both levels
    const uint64_t ncell3 = (uint64_t)G.nc * (uint64_t)G.nc * (uint64_t)G.nc;
    const int64_t owords = (int64_t)(ncell3 >> 6) + 1;  // nc >= 4: ncell3 is a multiple of 64
    uint32_t* cid = scan;  // the fine-start flags are no longer needed
    VR_WS(cfs, ctx, uint32_t, WS_B2, (int64_t)nfine + 1);
    VR_WS(occ, ctx, unsigned long long, WS_B4, owords);
    VR_WS(pre, ctx, uint32_t, WS_B5, owords + 1);
    VR_WS(frec, ctx, uint2, WS_B6, (int64_t)nfine);
    // (the union-find and what the passes read beside the records lie in the
    // sort's other buffers: particles in cells of their own, the most there can
    // be, then need no more room than one tree over the particles did)
    VR_WS(uf, ctx, int, WS_SORT_VALS_B, (int64_t)nfine);
    if ((rc = fill_u32(ctx, reinterpret_cast<uint32_t*>(occ), 0u, 2 * owords, st))) return rc;
    const unsigned gf = grid_for(nfine, 256);
    hipLaunchKernelGGL(k_coarse_flags, dim3(gf), dim3(256), 0, st, (int64_t)nfine, tot, fine_start, key, 3 * G.lr, cid);
    VR_LAUNCH_CHECK(ctx);
    if ((rc = scan_u32(ctx, cid, cid, nfine, tot + 1, st))) return rc;
    uint32_t ncoarse = nfine;
    if (!bound && (rc = read_back(ctx, tot + 1, &ncoarse, sizeof ncoarse, st))) return rc;
    hipLaunchKernelGGL(k_coarse_starts, dim3(gf), dim3(256), 0, st, tot, fine_start, key, 3 * G.lr, cid, cfs, occ);
    VR_LAUNCH_CHECK(ctx);
    hipLaunchKernelGGL(k_occ_count, dim3(grid_for(owords, 256)), dim3(256), 0, st, owords - 1,
                       reinterpret_cast<const uint64_t*>(occ), pre);
    VR_LAUNCH_CHECK(ctx);
    if ((rc = scan_u32(ctx, pre, pre, owords, nullptr, st))) return rc;
    VR_WS(crec, ctx, uint4, WS_B3, (int64_t)ncoarse);
    uint64_t* tables = nullptr;
    uint32_t* nbits = nullptr;
    int* mn = nullptr;
    Carve cv;
    auto layout = [&]() {
        tables = cv.add<uint64_t>(2 * 64 * NOFF);
        nbits = cv.add<uint32_t>(ncoarse);
        mn = cv.add<int>(nfine);
    };
    layout();
    const size_t rest = cv.bytes;
    cv.bytes = 0;
    cv.base = static_cast<char*>(ws(ctx, WS_SORT_KEYS_B, rest));
    if (!cv.base) return VR_ERR_OUT_OF_MEMORY;
    layout();
    const int64_t l2c = (int64_t)std::ceil(ell2);  // ell2 < 2^40: exact
    const uint64_t* occ_c = reinterpret_cast<const uint64_t*>(occ);
    const unsigned gc = grid_for(ncoarse, 256);
    hipLaunchKernelGGL(k_pair_tables, dim3(NOFF), dim3(64), 0, st, G, l2c, tables, tables + 64 * NOFF);
    VR_LAUNCH_CHECK(ctx);
    hipLaunchKernelGGL(k_frec, dim3(gf), dim3(256), 0, st, tot, fine_start, key, cid, 3 * G.lr, frec);
    VR_LAUNCH_CHECK(ctx);
    hipLaunchKernelGGL(k_coarse_rec, dim3(gc), dim3(256), 0, st, tot + 1, cfs, frec, key, fine_start, G, occ_c,
                       crec, nbits);
    VR_LAUNCH_CHECK(ctx);
    VR_WS(cnt, ctx, int, WS_FLAG2, 4);
    if ((rc = fill_i32(ctx, cnt, 0, 1, st))) return rc;
    // the fine cells' coarse indices now sit in their records: their array
    // takes the listed pairs
    const HeavyList H{reinterpret_cast<uint2*>(cid), cnt, (uint32_t)(n / 2)};
    const Links K{G, l2c, frec, crec, nbits, key, fine_start, occ_c, pre, tables, tables + 64 * NOFF, sx, sy, sz, uf};
    const unsigned xc = (unsigned)ctx->xcd_chunk;
    const bool lanes = n <= LANE_PER_NEIGHBOUR;
    VR_TIMED(ctx, "fof_link3d", st, 0,
             hipLaunchKernelGGL(k_hook, dim3(gf), dim3(256), 0, st, tot, K);
             hipLaunchKernelGGL(k_flatten, dim3(gf), dim3(256), 0, st, tot, uf);
             hipLaunchKernelGGL(k_coarse_root, dim3(gc), dim3(256), 0, st, tot + 1, uf, crec));
    VR_LAUNCH_CHECK(ctx);
    VR_TIMED(ctx, "fof_link3d", st, 0,
             if (lanes) hipLaunchKernelGGL((k_link_cells<false, 16>), dim3(16 * gf), dim3(256), 0, st, tot, K, xc, H);
             else hipLaunchKernelGGL((k_link_cells<false, 1>), dim3(gf), dim3(256), 0, st, tot, K, xc, H);
             hipLaunchKernelGGL(k_flatten, dim3(gf), dim3(256), 0, st, tot, uf);
             hipLaunchKernelGGL(k_coarse_root, dim3(gc), dim3(256), 0, st, tot + 1, uf, crec));
    VR_LAUNCH_CHECK(ctx);
    VR_TIMED(ctx, "fof_link3d", st, n,
             if (lanes) hipLaunchKernelGGL((k_link_cells<true, 16>), dim3(16 * gf), dim3(256), 0, st, tot, K, xc, H);
             else hipLaunchKernelGGL((k_link_cells<true, 1>), dim3(gf), dim3(256), 0, st, tot, K, xc, H);
             hipLaunchKernelGGL(k_link_heavy, dim3((unsigned)(8 * ctx->num_cus)), dim3(64), 0, st, H, K);
             hipLaunchKernelGGL(k_flatten, dim3(gf), dim3(256), 0, st, tot, uf));
    VR_LAUNCH_CHECK(ctx);
    hipLaunchKernelGGL(k_root_idx_f, dim3(gf), dim3(256), 0, st, tot, uf, fine_start, idx, mn);
    VR_LAUNCH_CHECK(ctx);
    if (nfine > 65536)
        hipLaunchKernelGGL(k_min_orig_f, dim3(grid_for(nfine, 64 * 256)), dim3(256), 0, st, tot, uf, fine_start, idx, mn,
                           64);
    hipLaunchKernelGGL(k_min_orig_f, dim3(gf), dim3(256), 0, st, tot, uf, fine_start, idx, mn, 1);
    VR_LAUNCH_CHECK(ctx);
    hipLaunchKernelGGL(k_label_f, dim3(gn), dim3(256), 0, st, n, uf, fid, idx, mn, label);
    VR_LAUNCH_CHECK(ctx);
    return VR_OK;
}

}  // namespace vr
