// vr_prims.hip -- device-wide primitives: exclusive scan, stable LSD radix
// sort of (key, index) pairs, fills.  Written for wave64: ranks inside a
// wavefront come from 64-bit ballots, tiles are staged through LDS so that the
// scatter writes contiguous runs per digit.
#include "vr_internal.h"

namespace vr {
namespace {

constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;
constexpr int SCAN_ONE = 1024;          // threads of the one-workgroup scan
// Up to here one workgroup of two rounds, one launch, is faster than tile sums
// and their application (4 us each with the gap): 14 k items 13 -> 7 us.
constexpr int64_t SCAN_ONE_MAX = 2 * SCAN_ONE * 8;
// Up to here every block of the application adds up the tile sums before its
// own (at most eight a thread): a launch of its own for their scan cost 5-9 us.
constexpr int64_t SCAN_RAW_TILES = 2048;

__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    const int lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        uint32_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// Block-wide exclusive scan of one value per thread (smem: a word per wavefront).
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* smem, uint32_t* total) {
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    uint32_t inc = wave_incl_scan(v);
    if (lane == 63) smem[w] = inc;
    __syncthreads();
    uint32_t wpre = 0, tot = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
        if (i < w) wpre += smem[i];
        tot += smem[i];
    }
    __syncthreads();
    if (total) *total = tot;
    return wpre + inc - v;
}

// Eight consecutive items of a lane; a full tile of aligned input moves as
// 16-byte words (uint32) or one 8-byte word (flags), since a lane's eight
// 4-byte accesses 32 bytes apart ran at half the rate.
__device__ __forceinline__ void load8(const uint32_t* in, int64_t base, int64_t n, uint32_t (&v)[8]) {
    if ((((uintptr_t)in) & 15) == 0 && base + 8 <= n) {
        const uint4 a = reinterpret_cast<const uint4*>(in + base)[0];
        const uint4 b = reinterpret_cast<const uint4*>(in + base)[1];
        v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = base + j < n ? in[base + j] : 0u;
    }
}

__device__ __forceinline__ void load8(const uint8_t* in, int64_t base, int64_t n, uint32_t (&v)[8]) {
    if ((((uintptr_t)in) & 7) == 0 && base + 8 <= n) {
        const uint2 w = *reinterpret_cast<const uint2*>(in + base);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[j] = (w.x >> (8 * j)) & 255u;
            v[4 + j] = (w.y >> (8 * j)) & 255u;
        }
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = base + j < n ? (uint32_t)in[base + j] : 0u;
    }
}

// The exclusive sums of a lane's eight items, the first of them off.
__device__ __forceinline__ void store8(uint32_t* out, int64_t base, int64_t n, const uint32_t (&v)[8], uint32_t off) {
    uint32_t o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        o[j] = off;
        off += v[j];
    }
    if ((((uintptr_t)out) & 15) == 0 && base + 8 <= n) {
        reinterpret_cast<uint4*>(out + base)[0] = make_uint4(o[0], o[1], o[2], o[3]);
        reinterpret_cast<uint4*>(out + base)[1] = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (base + j < n) out[base + j] = o[j];
    }
}

template <class In>
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_reduce(const In* in, int64_t n, uint32_t* part) {
    static_assert(SCAN_ITEMS == 8, "a lane's items");
    __shared__ uint32_t sm[8];
    uint32_t v[8], s = 0;
    load8(in, (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS, n, v);
#pragma unroll
    for (int j = 0; j < 8; ++j) s += v[j];
    uint32_t tot;
    block_excl_scan(s, sm, &tot);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// part: the tiles' sums, scanned already or (raw) not: then the block adds up
// those of the tiles before its own.
template <class In>
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_apply(const In* in, uint32_t* out, int64_t n, const uint32_t* part,
                                                           int raw, uint32_t* total_dev) {
    __shared__ uint32_t sm[8], smp[8];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t v[8], s = 0, before = 0;
    load8(in, base, n, v);
    if (raw) {
        for (unsigned k = threadIdx.x; k < blockIdx.x; k += SCAN_BLOCK) before += part[k];
        uint32_t tot;
        block_excl_scan(before, smp, &tot);
        before = tot;
    } else {
        before = part[blockIdx.x];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) s += v[j];
    const uint32_t off = before + block_excl_scan(s, sm, nullptr);
    store8(out, base, n, v, off);
    if (total_dev && blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_BLOCK - 1) *total_dev = off + s;
}

// A short scan in one workgroup.
template <class In>
__global__ __launch_bounds__(SCAN_ONE) void k_scan_one(const In* in, uint32_t* out, int64_t n, uint32_t* total_dev) {
    __shared__ uint32_t sm[SCAN_ONE / 64];
    uint32_t carry = 0;
    for (int64_t t0 = 0; t0 < n; t0 += SCAN_ONE * 8) {
        const int64_t base = t0 + (int64_t)threadIdx.x * 8;
        uint32_t v[8], s = 0, tot;
        load8(in, base, n, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) s += v[j];
        const uint32_t off = carry + block_excl_scan(s, sm, &tot);
        store8(out, base, n, v, off);
        carry += tot;
    }
    if (total_dev && threadIdx.x == 0) *total_dev = carry;
}

template <class T>
__global__ void k_fill(T* p, T v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_iota(uint32_t* p, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = (uint32_t)i;
}

// ---- radix sort ------------------------------------------------------------
constexpr int RS_BLOCK = 256;
constexpr int RS_WAVES = RS_BLOCK / 64;
constexpr int RS_ITEMS = 16;                   // keys per thread and tile of a large sort
constexpr int RS_ITEMS_SMALL = 4;              // of a small one
constexpr int RS_RADIX = 256;
// Up to this many tiles a scatter block adds up the tiles' digit counts
// itself (a row of 256 counts each, 128 KB from the L2) instead of reading
// their scan, which takes two launches of 4-5 us: a pass of 64 k keys
// 31 -> 14 us.
constexpr int RS_FUSED_TILES = 128;
// Tiles of 1,024 keys as long as RS_FUSED_TILES of them hold the sort: with
// 4,096 keys a tile 64 k keys kept 16 of 256 CUs busy.
constexpr int64_t RS_SMALL_MAX = (int64_t)RS_FUSED_TILES * RS_BLOCK * RS_ITEMS_SMALL;
// One workgroup sorts all digits in LDS, one launch: 2 us a digit against 14.
constexpr int RS_ONE = 1024;
constexpr int RS_ONE_ITEMS = 4;
constexpr int64_t RS_ONE_MAX = RS_ONE * RS_ONE_ITEMS;

static_assert(SORT_BATCH_MAX <= (int64_t)RS_FUSED_TILES * RS_BLOCK * RS_ITEMS, "batches need the fused passes");

// Digit counts of a tile: digit-major (hist[d * num_tiles + tile]) for the
// scan, or a row per tile (ROWS).  blockIdx.y: the sort of a batch, whose
// arrays follow each other.
template <class K, int ITEMS, bool ROWS>
__global__ __launch_bounds__(RS_BLOCK) void k_radix_count(const K* __restrict__ keys, int64_t n, int shift,
                                                          uint32_t* __restrict__ hist, int num_tiles) {
    __shared__ uint32_t h[RS_RADIX];
    keys += (int64_t)blockIdx.y * n;
    hist += (int64_t)blockIdx.y * RS_RADIX * num_tiles;
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (RS_BLOCK * ITEMS);
#pragma unroll 4
    for (int j = 0; j < ITEMS; ++j) {
        int64_t i = base + j * RS_BLOCK + threadIdx.x;
        if (i < n) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[ROWS ? (int64_t)blockIdx.x * RS_RADIX + threadIdx.x : (int64_t)threadIdx.x * num_tiles + blockIdx.x] =
        h[threadIdx.x];
}

// Ranks of a wavefront's ITEMS x 64 keys (item j of lane l is its key
// 64 j + l) among its own keys with the same digit, by ballots; wcnt counts
// the wavefront's keys per digit.
template <class K, class C, int ITEMS>
__device__ __forceinline__ void wave_ranks(const K (&key)[ITEMS], int64_t base, int64_t n, int shift, C* wcnt,
                                           uint32_t (&rank)[ITEMS]) {
    const int lane = __lane_id();
    const uint64_t lt = lanemask_lt();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const bool valid = base + j * 64 + lane < n;
        const uint32_t d = (uint32_t)(key[j] >> shift) & 255u;
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        uint32_t before = 0;
        if (valid) before = wcnt[d];
        rank[j] = before + (uint32_t)__popcll(m & lt);
        // the highest peer lane publishes the new running count of the digit
        if (valid && lane == 63 - __clzll(m)) wcnt[d] = (C)(before + (uint32_t)__popcll(m));
        __builtin_amdgcn_wave_barrier();
    }
}

// Stable scatter of one 8-bit digit: every wavefront ranks its ITEMS x 64
// keys by ballots, the block turns the per-wave digit counts into tile
// offsets, and the tile moves out through LDS in digit order -- the keys
// first, then the values through the same buffer, so the block needs LDS for
// one array of keys only (four blocks of 64-bit keys per CU).  All loads are
// issued before the first rank (taken one by one between the ranks, they
// made a 12 k sort's pass 16 us).  FUSED: offs holds the tiles' rows of
// counts, not their scan.
template <class K, int ITEMS, bool FUSED>
__global__ __launch_bounds__(RS_BLOCK) void k_radix_scatter(const K* __restrict__ kin, const uint32_t* __restrict__ vin,
                                                             K* __restrict__ kout, uint32_t* __restrict__ vout,
                                                             int64_t n, int shift,
                                                             const uint32_t* __restrict__ offs, int num_tiles) {
    constexpr int TILE = RS_BLOCK * ITEMS;
    constexpr int LK = FUSED && sizeof(K) * TILE < 8 * RS_RADIX * 4 ? (int)(8 * RS_RADIX * 4 / sizeof(K)) : TILE;
    __shared__ uint32_t wcnt[RS_WAVES][RS_RADIX];
    __shared__ uint32_t toff[RS_RADIX];
    __shared__ uint32_t goff[RS_RADIX];
    __shared__ uint32_t sm[8];
    __shared__ __align__(16) K lk[LK];
    uint32_t* lv = reinterpret_cast<uint32_t*>(lk);
    kin += (int64_t)blockIdx.y * n;
    vin += (int64_t)blockIdx.y * n;
    kout += (int64_t)blockIdx.y * n;
    vout += (int64_t)blockIdx.y * n;
    offs += (int64_t)blockIdx.y * RS_RADIX * num_tiles;
    const int tid = threadIdx.x, lane = __lane_id(), w = tid >> 6;
    const int64_t tbase = (int64_t)blockIdx.x * TILE;
    const int64_t base = tbase + (int64_t)w * (ITEMS * 64);
    K key[ITEMS];
    uint32_t val[ITEMS], rank[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t i = base + j * 64 + lane;
        key[j] = i < n ? kin[i] : K(0);
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t i = base + j * 64 + lane;
        val[j] = i < n ? vin[i] : 0u;
    }
    for (int i = tid; i < RS_WAVES * RS_RADIX; i += RS_BLOCK) (&wcnt[0][0])[i] = 0;
    if (FUSED) {
        // rows w, w + 4, ...; four digits a lane: counts of all tiles and of
        // those before this one
        uint4* sums = reinterpret_cast<uint4*>(lk);
        uint4 a = make_uint4(0, 0, 0, 0), b = a;
#pragma unroll 8
        for (int t = w; t < num_tiles; t += RS_WAVES) {
            const uint4 c = reinterpret_cast<const uint4*>(offs + (int64_t)t * RS_RADIX)[lane];
            const uint32_t k = t < (int)blockIdx.x ? ~0u : 0u;
            a.x += c.x, a.y += c.y, a.z += c.z, a.w += c.w;
            b.x += c.x & k, b.y += c.y & k, b.z += c.z & k, b.w += c.w & k;
        }
        sums[w * 64 + lane] = a;
        sums[(RS_WAVES + w) * 64 + lane] = b;
        __syncthreads();
        const uint32_t* s32 = reinterpret_cast<const uint32_t*>(lk);
        uint32_t all = 0, before = 0;
#pragma unroll
        for (int k = 0; k < RS_WAVES; ++k) {
            all += s32[k * RS_RADIX + tid];
            before += s32[(RS_WAVES + k) * RS_RADIX + tid];
        }
        goff[tid] = before + block_excl_scan(all, sm, nullptr);
    } else {
        goff[tid] = offs[(int64_t)tid * num_tiles + blockIdx.x];
        __syncthreads();
    }
    wave_ranks(key, base, n, shift, wcnt[w], rank);
    __syncthreads();
    // digit totals, per-wave prefixes and the tile-level exclusive offsets
    {
        const int d = tid;
        uint32_t run = 0;
#pragma unroll
        for (int ww = 0; ww < RS_WAVES; ++ww) {
            uint32_t c = wcnt[ww][d];
            wcnt[ww][d] = run;
            run += c;
        }
        toff[d] = block_excl_scan(run, sm, nullptr);
    }
    __syncthreads();
    // a key's place in the tile, in digit order
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t i = base + j * 64 + lane;
        if (i < n) {
            const uint32_t d = (uint32_t)(key[j] >> shift) & 255u;
            rank[j] += toff[d] + wcnt[w][d];
            lk[rank[j]] = key[j];
        }
    }
    __syncthreads();
    const int cnt = (int)((n - tbase) < TILE ? (n - tbase) : TILE);
    uint32_t dst[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int i = tid + j * RS_BLOCK;
        if (i < cnt) {
            const K k = lk[i];
            const uint32_t d = (uint32_t)(k >> shift) & 255u;
            dst[j] = goff[d] + (uint32_t)i - toff[d];
            kout[dst[j]] = k;
        }
    }
    __syncthreads();
    // the values through the same buffer, to the places their keys went
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t i = base + j * 64 + lane;
        if (i < n) lv[rank[j]] = val[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int i = tid + j * RS_BLOCK;
        if (i < cnt) vout[dst[j]] = lv[i];
    }
}

// A sort of up to RS_ONE x ITEMS pairs: one workgroup takes every digit with
// the pairs in registers and LDS; in and out may be the same arrays.
template <class K, int ITEMS>
__global__ __launch_bounds__(RS_ONE) void k_radix_one(const K* kin, const uint32_t* vin, K* kout, uint32_t* vout, int n,
                                                      int first_bit, int bits) {
    constexpr int WAVES = RS_ONE / 64;
    __shared__ K lk[RS_ONE * ITEMS];
    __shared__ uint32_t lv[RS_ONE * ITEMS];
    __shared__ uint16_t wcnt[WAVES][RS_RADIX];
    __shared__ uint32_t toff[RS_RADIX];
    __shared__ uint32_t sm[WAVES];
    kin += (int64_t)blockIdx.x * n;
    vin += (int64_t)blockIdx.x * n;
    kout += (int64_t)blockIdx.x * n;
    vout += (int64_t)blockIdx.x * n;
    const int tid = threadIdx.x, lane = __lane_id(), w = tid >> 6;
    const int base = w * (ITEMS * 64);
    K key[ITEMS];
    uint32_t val[ITEMS], rank[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int i = base + j * 64 + lane;
        key[j] = i < n ? kin[i] : K(0);
        val[j] = i < n ? vin[i] : 0u;
    }
    for (int shift = first_bit; shift < bits; shift += 8) {
        for (int i = tid; i < WAVES * RS_RADIX / 2; i += RS_ONE) reinterpret_cast<uint32_t*>(&wcnt[0][0])[i] = 0;
        __syncthreads();
        wave_ranks(key, base, n, shift, wcnt[w], rank);
        __syncthreads();
        uint32_t run = 0;
        if (tid < RS_RADIX) {
#pragma unroll
            for (int ww = 0; ww < WAVES; ++ww) {
                const uint32_t c = wcnt[ww][tid];
                wcnt[ww][tid] = (uint16_t)run;
                run += c;
            }
        }
        const uint32_t ex = block_excl_scan(run, sm, nullptr);
        if (tid < RS_RADIX) toff[tid] = ex;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (base + j * 64 + lane < n) {
                const uint32_t d = (uint32_t)(key[j] >> shift) & 255u;
                const uint32_t at = rank[j] + toff[d] + wcnt[w][d];
                lk[at] = key[j];
                lv[at] = val[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const int i = base + j * 64 + lane;
            if (i < n) {
                key[j] = lk[i];
                val[j] = lv[i];
            }
        }
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int i = base + j * 64 + lane;
        if (i < n) {
            kout[i] = key[j];
            vout[i] = val[j];
        }
    }
}

template <class K>
int sort_input_impl(vr_ctx* ctx, K* keys, uint32_t* vals, int64_t n, int bits, K** kin, uint32_t** vin,
                    int first_bit = 0) {
    *kin = keys;
    *vin = vals;
    if (n <= 1 || bits <= first_bit || ((bits - first_bit + 7) / 8) % 2 == 0) return VR_OK;
    VR_WS(kalt, ctx, K, WS_SORT_KEYS_B, n);
    VR_WS(valt, ctx, uint32_t, WS_SORT_VALS_B, n);
    *kin = kalt;
    *vin = valt;
    return VR_OK;
}

// One pass over `batch` sorts of n pairs each.
template <class K, int ITEMS, bool FUSED>
int radix_pass(vr_ctx* ctx, const K* k0, const uint32_t* v0, K* k1, uint32_t* v1, int64_t n, int batch, int shift,
               uint32_t* hist, int num_tiles, hipStream_t s) {
    hipLaunchKernelGGL((k_radix_count<K, ITEMS, FUSED>), dim3(num_tiles, batch), dim3(RS_BLOCK), 0, s, k0, n, shift,
                       hist, num_tiles);
    VR_LAUNCH_CHECK(ctx);
    if (!FUSED) {
        int rc = scan_u32(ctx, hist, hist, (int64_t)RS_RADIX * num_tiles, nullptr, s);
        if (rc) return rc;
    }
    VR_TIMED(ctx, "radix_scatter", s, n * batch,
             hipLaunchKernelGGL((k_radix_scatter<K, ITEMS, FUSED>), dim3(num_tiles, batch), dim3(RS_BLOCK), 0, s, k0,
                                v0, k1, v1, n, shift, hist, num_tiles));
    VR_LAUNCH_CHECK(ctx);
    return VR_OK;
}

// Input pairs in (kin, vin), which is either (keys, vals) or the alternate
// buffers; passes ping-pong between the two pairs, and the result is copied
// into (keys, vals) only where it ends in the other one.  batch > 1: that
// many sorts whose arrays follow each other (n pairs each, within
// SORT_BATCH_MAX).
template <class K>
int sort_pairs_impl(vr_ctx* ctx, K* kin, uint32_t* vin, K* keys, uint32_t* vals, int64_t n, int bits,
                    hipStream_t s, int first_bit = 0, int batch = 1) {
    const int64_t m = n * batch;
    if (n <= 1 || bits <= first_bit) {
        if (n == 1 && kin != keys) {
            VR_HIP(ctx, hipMemcpyAsync(keys, kin, m * sizeof(K), hipMemcpyDeviceToDevice, s));
            VR_HIP(ctx, hipMemcpyAsync(vals, vin, m * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
        }
        return VR_OK;
    }
    // (a cap on the workspace leaves the counts the room of the larger tiles)
    const bool one = n <= RS_ONE_MAX, small = n <= RS_SMALL_MAX && ctx->max_ws == 0;
    const int tile = RS_BLOCK * (small ? RS_ITEMS_SMALL : RS_ITEMS);
    const int num_tiles = (int)((n + tile - 1) / tile);
    const bool fused = num_tiles <= RS_FUSED_TILES;
    K* kalt = keys;
    uint32_t* valt = vals;
    if (!one || kin != keys) {
        kalt = wsT<K>(ctx, WS_SORT_KEYS_B, m);
        valt = wsT<uint32_t>(ctx, WS_SORT_VALS_B, m);
        if (!kalt || !valt) return VR_ERR_OUT_OF_MEMORY;
    }
    if (kin != keys && (kin != kalt || vin != valt))
        return set_err(ctx, VR_ERR_INVALID_ARG, "sort input is neither the output nor the alternate buffers");
    if (one) {
        VR_TIMED(ctx, "radix_scatter", s, m,
                 if (n <= RS_ONE) hipLaunchKernelGGL((k_radix_one<K, 1>), dim3(batch), dim3(RS_ONE), 0, s, kin, vin,
                                                     keys, vals, (int)n, first_bit, bits);
                 else hipLaunchKernelGGL((k_radix_one<K, RS_ONE_ITEMS>), dim3(batch), dim3(RS_ONE), 0, s, kin, vin,
                                         keys, vals, (int)n, first_bit, bits));
        VR_LAUNCH_CHECK(ctx);
        return VR_OK;
    }
    VR_WS(hist, ctx, uint32_t, WS_SORT_HIST, (int64_t)RS_RADIX * num_tiles * batch);
    K* k0 = kin; K* k1 = kin == keys ? kalt : keys;
    uint32_t* v0 = vin; uint32_t* v1 = vin == vals ? valt : vals;
    const int passes = (bits - first_bit + 7) / 8;
    for (int p = 0; p < passes; ++p) {
        const int shift = first_bit + p * 8;
        int rc;
        if (small) rc = radix_pass<K, RS_ITEMS_SMALL, true>(ctx, k0, v0, k1, v1, n, batch, shift, hist, num_tiles, s);
        else if (fused) rc = radix_pass<K, RS_ITEMS, true>(ctx, k0, v0, k1, v1, n, batch, shift, hist, num_tiles, s);
        else rc = radix_pass<K, RS_ITEMS, false>(ctx, k0, v0, k1, v1, n, 1, shift, hist, num_tiles, s);
        if (rc) return rc;
        std::swap(k0, k1);
        std::swap(v0, v1);
    }
    if (k0 != keys) {
        VR_HIP(ctx, hipMemcpyAsync(keys, k0, m * sizeof(K), hipMemcpyDeviceToDevice, s));
        VR_HIP(ctx, hipMemcpyAsync(vals, v0, m * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
    }
    return VR_OK;
}

}  // namespace

namespace {

template <class In>
int scan_impl(vr_ctx* ctx, const In* in, uint32_t* out, int64_t n, uint32_t* total_dev, int depth, hipStream_t s) {
    if (n <= SCAN_ONE_MAX) {
        hipLaunchKernelGGL(k_scan_one<In>, dim3(1), dim3(SCAN_ONE), 0, s, in, out, n, total_dev);
        VR_LAUNCH_CHECK(ctx);
        return VR_OK;
    }
    const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    // partial sums live in a fresh region per recursion level; two levels
    // cover 2048^3 items
    static const int slots[2] = {WS_SCAN_TMP2, WS_SCAN_TMP};
    if (depth >= 2) return set_err(ctx, VR_ERR_UNSUPPORTED, "scan of %lld elements too deep", (long long)n);
    uint32_t* part = wsT<uint32_t>(ctx, slots[depth], nb);
    if (!part) return VR_ERR_OUT_OF_MEMORY;
    hipLaunchKernelGGL(k_scan_reduce<In>, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, part);
    VR_LAUNCH_CHECK(ctx);
    const bool raw = nb <= SCAN_RAW_TILES;
    if (!raw) {
        int rc = scan_impl<uint32_t>(ctx, part, part, nb, nullptr, depth + 1, s);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(k_scan_apply<In>, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, out, n, part, raw ? 1 : 0,
                       total_dev);
    VR_LAUNCH_CHECK(ctx);
    return VR_OK;
}

}  // namespace

int scan_u32(vr_ctx* ctx, const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total_dev, hipStream_t s) {
    if (n <= 0) {
        if (total_dev) return fill_u32(ctx, total_dev, 0u, 1, s);
        return VR_OK;
    }
    return scan_impl<uint32_t>(ctx, in, out, n, total_dev, 0, s);
}

int scan_u8(vr_ctx* ctx, const uint8_t* in, uint32_t* out, int64_t n, hipStream_t s) {
    if (n <= 0) return VR_OK;
    return scan_impl<uint8_t>(ctx, in, out, n, nullptr, 0, s);
}

int sort_pairs_u32(vr_ctx* ctx, uint32_t* keys, uint32_t* vals, int64_t n, int bits, hipStream_t s) {
    return sort_pairs_impl<uint32_t>(ctx, keys, vals, keys, vals, n, bits, s);
}

int sort_pairs_u64(vr_ctx* ctx, uint64_t* keys, uint32_t* vals, int64_t n, int bits, hipStream_t s) {
    return sort_pairs_impl<uint64_t>(ctx, keys, vals, keys, vals, n, bits, s);
}

int sort_input_u64(vr_ctx* ctx, uint64_t* keys, uint32_t* vals, int64_t n, int bits, uint64_t** kin,
                   uint32_t** vin, int first_bit) {
    return sort_input_impl<uint64_t>(ctx, keys, vals, n, bits, kin, vin, first_bit);
}

int sort_pairs_u64_from(vr_ctx* ctx, uint64_t* kin, uint32_t* vin, uint64_t* keys, uint32_t* vals, int64_t n,
                        int bits, hipStream_t s, int first_bit) {
    return sort_pairs_impl<uint64_t>(ctx, kin, vin, keys, vals, n, bits, s, first_bit);
}

int sort_batch(vr_ctx* ctx, uint64_t* kin, uint32_t* vin, uint64_t* keys, uint32_t* vals, int64_t n, int batch,
               int bits, hipStream_t s) {
    if (n > SORT_BATCH_MAX) return set_err(ctx, VR_ERR_UNSUPPORTED, "batched sort of %lld pairs each", (long long)n);
    return sort_pairs_impl<uint64_t>(ctx, kin, vin, keys, vals, n, bits, s, 0, batch);
}

int sort_batch(vr_ctx* ctx, uint32_t* kin, uint32_t* vin, uint32_t* keys, uint32_t* vals, int64_t n, int batch,
               int bits, hipStream_t s) {
    if (n > SORT_BATCH_MAX) return set_err(ctx, VR_ERR_UNSUPPORTED, "batched sort of %lld pairs each", (long long)n);
    return sort_pairs_impl<uint32_t>(ctx, kin, vin, keys, vals, n, bits, s, 0, batch);
}

int sort_input_u32(vr_ctx* ctx, uint32_t* keys, uint32_t* vals, int64_t n, int bits, uint32_t** kin,
                   uint32_t** vin) {
    return sort_input_impl<uint32_t>(ctx, keys, vals, n, bits, kin, vin);
}

int sort_pairs_u32_from(vr_ctx* ctx, uint32_t* kin, uint32_t* vin, uint32_t* keys, uint32_t* vals, int64_t n,
                        int bits, hipStream_t s) {
    return sort_pairs_impl<uint32_t>(ctx, kin, vin, keys, vals, n, bits, s);
}

int fill_i32(vr_ctx* ctx, int32_t* p, int32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return VR_OK;
    hipLaunchKernelGGL(k_fill<int32_t>, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
    VR_LAUNCH_CHECK(ctx);
    return VR_OK;
}

int fill_u32(vr_ctx* ctx, uint32_t* p, uint32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return VR_OK;
    hipLaunchKernelGGL(k_fill<uint32_t>, dim3(grid_for(n, 256)), dim3(256), 0, s, p, v, n);
    VR_LAUNCH_CHECK(ctx);
    return VR_OK;
}

int iota_u32(vr_ctx* ctx, uint32_t* p, int64_t n, hipStream_t s) {
    if (n <= 0) return VR_OK;
    hipLaunchKernelGGL(k_iota, dim3(grid_for(n, 256)), dim3(256), 0, s, p, n);
    VR_LAUNCH_CHECK(ctx);
    return VR_OK;
}

}  // namespace vr
