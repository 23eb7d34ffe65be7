// Device radix sort (stable LSD, up to 8-bit digits) with 32-bit values, used for
// the (tile, depth) order of the tile lists, and below it the two passes of the depth
// order, whose digits (up to 11 bits) follow the depth range.
//
// Keys are 64-bit (tile << 32) | depth_bits or 32-bit (tile id, or a point's slot). The
// digits come from a view of the key that keeps only its significant bits:
//   KV_TILE_DEPTH (64-bit): (tile << dbits) | (depth_bits - zmin)
//   KV_SUB        (32-bit): key - zmin
// Both views preserve the key order among the keys of one render.
//
// Each pass is reduce-then-scan, with no waiting between workgroups:
//   up:      per chunk of 1,024 to 4,096 keys, the digit counts -> matrix [digit][chunk]
//   rowscan: one workgroup per digit scans its row in place and writes the row total
//   down:    per chunk, the digits' global bases come from an exclusive scan of the
//            row totals (256 words, done by every workgroup); keys are ranked stably
//            per digit with wave ballots (a 64-lane match mask built from one ballot
//            per digit bit, rank = popcount of the lower lanes), staged through LDS in
//            digit order and written as contiguous runs at the offsets of the matrix.
// A single-pass "decoupled look-back" form was measured slower here: its prefix
// frontier advances only a window of chunks per cross-XCD round trip.
#include "recogs_internal.hpp"

#include <algorithm>

namespace recogs {

enum : int { KV_TILE_DEPTH = 0, KV_SUB = 1 };

template <typename KT, int VIEW>
__device__ __forceinline__ uint32_t digit_of(KT key, uint32_t zmin, int dbits, int shift, uint32_t dmask) {
    if constexpr (VIEW == KV_TILE_DEPTH) return (uint32_t)(sort_view((uint64_t)key, zmin, dbits) >> shift) & dmask;
    else return ((uint32_t)key - zmin) >> shift & dmask;
}

// exclusive scan of one value per thread over a 256-thread workgroup
__device__ __forceinline__ uint32_t block_excl_scan256(uint32_t v, uint32_t *s_w, uint32_t &total) {
    const uint32_t lane = lane_id(), w = threadIdx.x >> 6;
    const uint32_t inc = wave_incl_scan(v);
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t pre = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t x = s_w[k];
        if (k < (int)w) pre += x;
        total += x;
    }
    __syncthreads();
    return pre + inc - v;
}

// The count may live in device memory (dyn_count non-null: the graph-capturable renders,
// whose host code never reads it back); grids are then sized for the capacity and
// workgroups past the live count return at once.

// per-chunk digit counts -> cnt[digit * chunks + chunk]; a chunk is 256 x ITEMS keys.
template <typename KT, int VIEW, int ITEMS>
__global__ __launch_bounds__(256) void k_radix_up(const KT *__restrict__ kin, uint32_t K, uint32_t zmin, int dbits,
                                                  int shift, int nbits, uint32_t *__restrict__ cnt, uint32_t chunks,
                                                  const uint32_t *dyn_count) {
    constexpr uint32_t CHUNK = 256 * ITEMS;
    const uint32_t t = threadIdx.x;
    const uint32_t base = blockIdx.x * CHUNK;
    if (dyn_count) K = *dyn_count;
    if (base >= K) return;
    __shared__ uint32_t h[256];
    h[t] = 0;
    __syncthreads();
    const uint32_t dmask = (1u << nbits) - 1u;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = base + r * 256 + t;
        if (idx < K) atomicAdd(&h[digit_of<KT, VIEW>(kin[idx], zmin, dbits, shift, dmask)], 1u);
    }
    __syncthreads();
    if (t <= dmask) cnt[(size_t)t * chunks + blockIdx.x] = h[t];
}

// workgroup d: cnt[d][c] <- sum_{c' < c} cnt[d][c'];  tot[d] <- sum_c cnt[d][c].
// Four counts per thread, so a row of up to 1,024 chunks is one round of loads.
__global__ __launch_bounds__(256) void k_radix_rowscan(uint32_t *__restrict__ cnt, uint32_t chunks, uint32_t chunk_keys,
                                                       uint32_t *__restrict__ tot, uint32_t K,
                                                       const uint32_t *dyn_count) {
    __shared__ uint32_t s_w[4];
    const uint32_t d = blockIdx.x, t = threadIdx.x;
    uint32_t *row = cnt + (size_t)d * chunks;
    // the row's first 1,024 entries are loaded before the device count arrives (it would
    // cost a memory round trip of its own); entries past the live chunks are not summed
    uint32_t v0[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v0[i] = 4 * t + i < chunks ? row[4 * t + i] : 0u;
    if (dyn_count) K = *dyn_count;
    const uint32_t live = (K + chunk_keys - 1) / chunk_keys;   // chunks holding keys; row stride stays `chunks`
    uint32_t run = 0, total;
    for (uint32_t c0 = 0; c0 < live; c0 += 1024) {
        const uint32_t c = c0 + 4 * t;
        uint32_t v[4], sum = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = c + i < live ? (c0 == 0 ? v0[i] : row[c + i]) : 0u;
            sum += v[i];
        }
        uint32_t e = run + block_excl_scan256(sum, s_w, total);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (c + i < live) row[c + i] = e;
            e += v[i];
        }
        run += total;
    }
    if (t == 0) tot[d] = run;
}

template <typename KT, int VIEW, int ITEMS>
__global__ __launch_bounds__(256) void k_radix_down(const KT *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                    KT *__restrict__ kout, uint32_t *__restrict__ vout, uint32_t K,
                                                    uint32_t zmin, int dbits, int shift, int nbits,
                                                    const uint32_t *__restrict__ off, const uint32_t *__restrict__ dtot,
                                                    uint32_t chunks, const uint32_t *dyn_count) {
    constexpr uint32_t CHUNK = 256 * ITEMS;
    const uint32_t t = threadIdx.x, lane = lane_id(), w = t >> 6;
    const uint32_t chunk = xcd_chunk<0, 3>(blockIdx.x, gridDim.x);
    const uint32_t cbase = chunk * (uint32_t)CHUNK;
    // every global load of the workgroup goes out first (the chunk's keys and values, the
    // digit totals, this chunk's digit offsets): one memory round trip, not three
    KT key[ITEMS];
    uint32_t val[ITEMS], rank[ITEMS];
    if (dyn_count) K = *dyn_count;
    if (cbase >= K) return;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = cbase + w * (64 * ITEMS) + r * 64 + lane;
        const bool valid = idx < K;
        key[r] = valid ? kin[idx] : (KT)0;
        val[r] = valid ? vin[idx] : 0u;
    }
    __shared__ uint32_t s_whist[4][256];   // per-wave digit counts, then per-wave digit prefix
    __shared__ uint32_t s_gbase[256];      // global position of this chunk's first key of each digit
    __shared__ uint32_t s_lstart[256];     // position in the LDS stage of each digit
    __shared__ uint32_t s_w[4];
    __shared__ KT s_keys[CHUNK];
    __shared__ uint32_t s_vals[CHUNK];

    const uint32_t dmask = (1u << nbits) - 1u;
    const uint32_t tot_t = t <= dmask ? dtot[t] : 0u;
    const uint32_t off_t = t <= dmask ? off[(size_t)t * chunks + chunk] : 0u;
    for (int i = t; i < 4 * 256; i += 256) (&s_whist[0][0])[i] = 0;
    {
        uint32_t all;
        const uint32_t dbase = block_excl_scan256(tot_t, s_w, all);
        if (t <= dmask) s_gbase[t] = dbase + off_t;
    }
    __syncthreads();
    // stable rank within the wave, round by round (wave w holds a contiguous quarter)
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = cbase + w * (64 * ITEMS) + r * 64 + lane;
        const bool valid = idx < K;
        const uint32_t d = digit_of<KT, VIEW>(key[r], zmin, dbits, shift, dmask);
        const uint64_t m = wave_match(valid, d, nbits);
        const uint32_t below = rank_below(m);
        uint32_t prior = 0;
        if (valid) prior = s_whist[w][d];
        rank[r] = prior + below;
        if (valid && below == 0) s_whist[w][d] = prior + (uint32_t)__popcll(m);
    }
    __syncthreads();
    // per digit (thread t = digit t): prefix over waves and chunk total
    uint32_t tot = 0;
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) {
        const uint32_t c = s_whist[ww][t];
        s_whist[ww][t] = tot;
        tot += c;
    }
    uint32_t total;
    s_lstart[t] = block_excl_scan256(tot, s_w, total);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = cbase + w * (64 * ITEMS) + r * 64 + lane;
        if (idx < K) {
            const uint32_t d = digit_of<KT, VIEW>(key[r], zmin, dbits, shift, dmask);
            const uint32_t pos = s_lstart[d] + s_whist[w][d] + rank[r];
            s_keys[pos] = key[r];
            s_vals[pos] = val[r];
        }
    }
    __syncthreads();
    const uint32_t nvalid = min((uint32_t)CHUNK, K - cbase);
    for (uint32_t j = t; j < nvalid; j += 256) {
        const KT k = s_keys[j];
        const uint32_t d = digit_of<KT, VIEW>(k, zmin, dbits, shift, dmask);
        const uint32_t dst = s_gbase[d] + (j - s_lstart[d]);
        kout[dst] = k;
        vout[dst] = s_vals[j];
    }
}

// ---------------------------------------------------------------------------
// Host side: sort K (key, value) pairs across the two buffers over `total_bits`
// significant bits (passes of equal width, <= 8 bits each). Returns 1 if the result
// is in the alternate buffers (kb/vb), 0 if in ka/va. `ghist` holds 8 x 256 words
// (each pass's digit totals); `cnt` 256 x ceil(K / 4096) words of scratch.
// ---------------------------------------------------------------------------
int sort_passes(int total_bits) { return (total_bits + 7) / 8; }

// keys per thread of a pass over K keys: long chunks (long contiguous output runs) when
// there are enough keys to fill the GPU with them, shorter ones otherwise
static int sort_items(uint32_t K) { return K >= (1u << 22) ? 16 : (K >= (1u << 20) ? 8 : 4); }

// Words of the digit-count matrix any sort of at most K_max keys needs: chunks of the
// shortest length (1,024 keys), whatever length a sort takes or is given.
size_t sort_count_words(uint64_t K_max) {
    const uint64_t chunks = (K_max + 1023) / 1024;
    return 256 * (size_t)(chunks > 0 ? chunks : 1);
}

// The first pass of a sort whose digit counts the key emission writes (KeyCount): the
// sort then runs with chunks of 2,048 keys (kKeyCountItems per thread).
constexpr int kKeyCountItems = 8;
static_assert(256u * kKeyCountItems == kEmitKeys, "a counted chunk is one emission block");
KeyCount key_sort_first_count(uint32_t *cnt, uint32_t K_max, int total_bits) {
    if (total_bits <= 0) return KeyCount{nullptr, 0u, 0};   // one tile: no pass to count for
    const int passes = sort_passes(total_bits);
    const int per = (total_bits + passes - 1) / passes;
    const uint32_t chunk = 256u * (uint32_t)kKeyCountItems;
    return KeyCount{cnt, (K_max + chunk - 1) / chunk, per < total_bits ? per : total_bits};
}

template <typename KT, int VIEW>
static int radix_sort(KT *ka, uint32_t *va, KT *kb, uint32_t *vb, uint32_t K, uint32_t zmin, int dbits, int total_bits,
                      uint32_t *ghist, uint32_t *cnt, hipStream_t st, const uint32_t *dyn_count = nullptr,
                      bool first_counted = false) {
    if (K == 0 || total_bits == 0) return 0;   // K is the count, or its upper bound with dyn_count
    const int passes = sort_passes(total_bits);
    const int per = (total_bits + passes - 1) / passes;
    uint32_t bits = 0;
    int rem = total_bits;
    for (int p = 0; p < passes; ++p) {
        const int nb = rem < per ? rem : per;
        bits |= (uint32_t)nb << (4 * p);
        rem -= nb;
    }
    // first_counted: the first pass's counts are in cnt already (KeyCount), in its chunks
    const int items = first_counted ? kKeyCountItems : sort_items(K);
    const uint32_t chunk_keys = 256u * (uint32_t)items;
    const uint32_t chunks = (K + chunk_keys - 1) / chunk_keys;
    int alt = 0, shift = 0;
    for (int p = 0; p < passes; ++p) {
        const int nb = (bits >> (4 * p)) & 15;
        const KT *kin = alt ? kb : ka;
        const uint32_t *vin = alt ? vb : va;
        KT *kout = alt ? ka : kb;
        uint32_t *vout = alt ? va : vb;
        uint32_t *tot = ghist + 256 * p;
#define RECOGS_PASS(IT)                                                                                                    \
    if (p > 0 || !first_counted)                                                                                           \
        hipLaunchKernelGGL((k_radix_up<KT, VIEW, IT>), dim3(chunks), dim3(256), 0, st, kin, K, zmin, dbits, shift, nb,     \
                           cnt, chunks, dyn_count);                                                                        \
    hipLaunchKernelGGL(k_radix_rowscan, dim3(1u << nb), dim3(256), 0, st, cnt, chunks, chunk_keys, tot, K, dyn_count);     \
    hipLaunchKernelGGL((k_radix_down<KT, VIEW, IT>), dim3(chunks), dim3(256), 0, st, kin, vin, kout, vout, K, zmin, dbits, \
                       shift, nb, cnt, tot, chunks, dyn_count);
        if (items == 16) { RECOGS_PASS(16) }
        else if (items == 8) { RECOGS_PASS(8) }
        else { RECOGS_PASS(4) }
#undef RECOGS_PASS
        alt ^= 1;
        shift += nb;
    }
    return alt;
}

// ---------------------------------------------------------------------------
// The two passes of the depth order behind the scan's (which orders the pairs by their low
// kScanBits depth bits): digits as depth_digits takes them from the header's depth range, up to
// 2^kDepthBitsMax of them, known on the device only. The same three kernels as above, with
// the per-wave digit counts in 16 bits and a thread holding the digits nd / 256 t .. of
// nd > 256. Three passes of 8-bit digits over the raw upper 24 bits before, the last of them with
// the emission's gather and sums (whose atomics want few digits a chunk): scan to offsets
// 105 -> 92 us at 1M Gaussians, 69 -> 59 us at 200k.
// ---------------------------------------------------------------------------
constexpr uint32_t kDepthDigitsMax = 1u << kDepthBitsMax;

struct DepthPass {
    const uint32_t *hdr;   // H_V, H_ZMIN_RAW, H_ZMAX
    uint32_t bound;        // V or a bound of it
    int second;            // which of the two passes
};
// the pass's count of pairs, shift, base and bits (uniform; one read of the header)
struct DepthArgs {
    uint32_t V, base;
    int shift, nb;
};
__device__ __forceinline__ DepthArgs depth_args(const DepthPass &p) {
    const DepthDigits d = depth_digits(p.hdr[H_ZMIN_RAW], p.hdr[H_ZMAX]);
    return DepthArgs{p.hdr[H_V], d.base, p.second ? d.nb1 : 0, p.second ? d.nb2 : d.nb1};
}
__device__ __forceinline__ uint32_t depth_digit(uint32_t z, const DepthArgs &a, uint32_t dmask) {
    return ((z >> kScanBits) - a.base) >> a.shift & dmask;
}

template <int ITEMS>
__global__ __launch_bounds__(256) void k_depth_up(const uint32_t *__restrict__ kin, DepthPass p, uint32_t *__restrict__ cnt,
                                                  uint32_t chunks) {
    __shared__ uint32_t h[kDepthDigitsMax];
    const uint32_t t = threadIdx.x, base = blockIdx.x * (256u * ITEMS);
    uint32_t kk[ITEMS];   // loaded below the bound, before the header is in
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) kk[r] = base + r * 256 + t < p.bound ? kin[base + r * 256 + t] : 0u;
    const DepthArgs a = depth_args(p);
    if (base >= a.V) return;
    const uint32_t nd = 1u << a.nb;
    for (uint32_t d = t; d < nd; d += 256) h[d] = 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
        if (base + r * 256 + t < a.V) atomicAdd(&h[depth_digit(kk[r], a, nd - 1u)], 1u);
    __syncthreads();
    for (uint32_t d = t; d < nd; d += 256) cnt[(size_t)d * chunks + blockIdx.x] = h[d];
}

// k_radix_rowscan over the rows blockIdx.x, + gridDim.x, .. of the pass's digits
__global__ __launch_bounds__(256) void k_depth_rowscan(uint32_t *__restrict__ cnt, uint32_t chunks, uint32_t chunk_keys,
                                                       uint32_t *__restrict__ tot, DepthPass p) {
    __shared__ uint32_t s_w[4];
    const uint32_t t = threadIdx.x;
    uint32_t v0[4];   // the first row's first entries, before the header is in
#pragma unroll
    for (int i = 0; i < 4; ++i) v0[i] = 4 * t + i < chunks ? cnt[(size_t)blockIdx.x * chunks + 4 * t + i] : 0u;
    const DepthArgs a = depth_args(p);
    const uint32_t live = (a.V + chunk_keys - 1) / chunk_keys, nd = 1u << a.nb;
    for (uint32_t d = blockIdx.x; d < nd; d += gridDim.x) {
        uint32_t *row = cnt + (size_t)d * chunks;
        uint32_t run = 0, total;
        for (uint32_t c0 = 0; c0 < live; c0 += 1024) {
            const uint32_t c = c0 + 4 * t;
            uint32_t v[4], sum = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[i] = c + i < live ? (c0 == 0 && d == blockIdx.x ? v0[i] : row[c + i]) : 0u;
                sum += v[i];
            }
            uint32_t e = run + block_excl_scan256(sum, s_w, total);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (c + i < live) row[c + i] = e;
                e += v[i];
            }
            run += total;
        }
        if (t == 0) tot[d] = run;
    }
}

template <int ITEMS>
__global__ __launch_bounds__(256) void k_depth_down(const uint32_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                                    uint32_t *__restrict__ kout, uint32_t *__restrict__ vout, DepthPass p,
                                                    const uint32_t *__restrict__ off, const uint32_t *__restrict__ dtot,
                                                    uint32_t chunks) {
    constexpr uint32_t CHUNK = 256 * ITEMS;
    __shared__ uint16_t s_whist[4][kDepthDigitsMax];   // per-wave digit counts, then per-wave digit prefix
    __shared__ uint32_t s_gbase[kDepthDigitsMax];      // global position of this chunk's first key of each digit
    __shared__ uint16_t s_lstart[kDepthDigitsMax];     // position in the LDS stage of each digit
    __shared__ uint32_t s_w[4];
    __shared__ uint32_t s_keys[CHUNK], s_vals[CHUNK];
    const uint32_t t = threadIdx.x, lane = lane_id(), w = t >> 6;
    const uint32_t chunk = xcd_chunk<2, 4>(blockIdx.x, gridDim.x), cbase = chunk * CHUNK;
    uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];   // loaded below the bound, before the header is in
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = cbase + w * (64 * ITEMS) + r * 64 + lane;
        key[r] = idx < p.bound ? kin[idx] : 0u;
        val[r] = idx < p.bound ? vin[idx] : 0u;
    }
    const DepthArgs a = depth_args(p);
    if (cbase >= a.V) return;
    const uint32_t nd = 1u << a.nb, dmask = nd - 1u;
    const uint32_t dpt = nd > 256u ? nd / 256u : 1u, d0 = dpt * t;   // this thread's digits: d0 .. d0 + dpt, below nd
    {
        uint32_t tot[kDepthDigitsMax / 256], ofs[kDepthDigitsMax / 256], sum = 0, all;
#pragma unroll
        for (uint32_t i = 0; i < kDepthDigitsMax / 256; ++i) {
            const bool in = i < dpt && d0 + i < nd;
            tot[i] = in ? dtot[d0 + i] : 0u;
            ofs[i] = in ? off[(size_t)(d0 + i) * chunks + chunk] : 0u;
        }
        for (uint32_t ww = 0; ww < 4; ++ww)
            for (uint32_t d = t; d < nd; d += 256) s_whist[ww][d] = 0;
#pragma unroll
        for (uint32_t i = 0; i < kDepthDigitsMax / 256; ++i) sum += tot[i];
        uint32_t dbase = block_excl_scan256(sum, s_w, all);
#pragma unroll
        for (uint32_t i = 0; i < kDepthDigitsMax / 256; ++i) {
            if (i < dpt && d0 + i < nd) s_gbase[d0 + i] = dbase + ofs[i];
            dbase += tot[i];
        }
    }
    __syncthreads();
    // stable rank within the wave, round by round (wave w holds a contiguous quarter)
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = cbase + w * (64 * ITEMS) + r * 64 + lane;
        const bool valid = idx < a.V;
        const uint32_t d = depth_digit(key[r], a, dmask);
        const uint64_t m = wave_match(valid, d, a.nb);
        const uint32_t below = rank_below(m);
        uint32_t prior = 0;
        if (valid) prior = s_whist[w][d];
        rank[r] = prior + below;
        if (valid && below == 0) s_whist[w][d] = (uint16_t)(prior + (uint32_t)__popcll(m));
    }
    __syncthreads();
    {
        uint32_t dt[kDepthDigitsMax / 256], sum = 0, all;   // per digit: prefix over waves and chunk total
#pragma unroll
        for (uint32_t i = 0; i < kDepthDigitsMax / 256; ++i) {
            dt[i] = 0;
            if (i < dpt && d0 + i < nd) {
#pragma unroll
                for (int ww = 0; ww < 4; ++ww) {
                    const uint32_t c = s_whist[ww][d0 + i];
                    s_whist[ww][d0 + i] = (uint16_t)dt[i];
                    dt[i] += c;
                }
            }
            sum += dt[i];
        }
        uint32_t ls = block_excl_scan256(sum, s_w, all);
#pragma unroll
        for (uint32_t i = 0; i < kDepthDigitsMax / 256; ++i) {
            if (i < dpt && d0 + i < nd) s_lstart[d0 + i] = (uint16_t)ls;
            ls += dt[i];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint32_t idx = cbase + w * (64 * ITEMS) + r * 64 + lane;
        if (idx < a.V) {
            const uint32_t d = depth_digit(key[r], a, dmask);
            const uint32_t pos = (uint32_t)s_lstart[d] + s_whist[w][d] + rank[r];
            s_keys[pos] = key[r];
            s_vals[pos] = val[r];
        }
    }
    __syncthreads();
    const uint32_t nvalid = min(CHUNK, a.V - cbase);
    for (uint32_t j = t; j < nvalid; j += 256) {
        const uint32_t k = s_keys[j], d = depth_digit(k, a, dmask);
        const uint32_t dst = s_gbase[d] + (j - s_lstart[d]);
        kout[dst] = k;
        vout[dst] = s_vals[j];
    }
}

// One of the two passes from (ka, va) to (kb, vb), for at most K_max pairs (sizes the grids
// and the count matrix); tot: kDepthDigitsMax words.
void launch_depth_pass(const uint32_t *ka, const uint32_t *va, uint32_t *kb, uint32_t *vb, uint32_t K_max, bool second,
                       const uint32_t *hdr, uint32_t *tot, uint32_t *cnt, hipStream_t st) {
    if (K_max == 0) return;
    const int items = sort_items(K_max);
    const uint32_t chunk_keys = 256u * (uint32_t)items, chunks = (K_max + chunk_keys - 1) / chunk_keys;
    const DepthPass p{hdr, K_max, second ? 1 : 0};
#define RECOGS_PASS(IT)                                                                                                    \
    hipLaunchKernelGGL(k_depth_up<IT>, dim3(chunks), dim3(256), 0, st, ka, p, cnt, chunks);                                \
    hipLaunchKernelGGL(k_depth_rowscan, dim3(256), dim3(256), 0, st, cnt, chunks, chunk_keys, tot, p);                     \
    hipLaunchKernelGGL(k_depth_down<IT>, dim3(chunks), dim3(256), 0, st, ka, va, kb, vb, p, cnt, tot, chunks);
    if (items == 16) { RECOGS_PASS(16) }
    else if (items == 8) { RECOGS_PASS(8) }
    else { RECOGS_PASS(4) }
#undef RECOGS_PASS
}

// words of the count matrix that passes over at most n pairs need (sort_items' chunks)
size_t depth_count_words(uint64_t n) {
    const uint64_t chunks = std::max({(std::min<uint64_t>(n, 1u << 20) + 1023) / 1024,
                                      (std::min<uint64_t>(n, 1u << 22) + 2047) / 2048, (n + 4095) / 4096, (uint64_t)1});
    return kDepthDigitsMax * (size_t)chunks;
}

// One row scan of a digit-count matrix [2^nbits][chunks] (K keys, chunk_keys per chunk).
void launch_rowscan(uint32_t *cnt, uint32_t chunks, uint32_t chunk_keys, uint32_t *tot, uint32_t K, int nbits,
                    hipStream_t st) {
    hipLaunchKernelGGL(k_radix_rowscan, dim3(1u << nbits), dim3(256), 0, st, cnt, chunks, chunk_keys, tot, K, nullptr);
}

int radix_sort_tile_depth64(uint64_t *ka, uint32_t *va, uint64_t *kb, uint32_t *vb, uint32_t K, uint32_t zmin, int dbits,
                            int total_bits, uint32_t *ghist, uint32_t *cnt, hipStream_t st) {
    return radix_sort<uint64_t, KV_TILE_DEPTH>(ka, va, kb, vb, K, zmin, dbits, total_bits, ghist, cnt, st);
}

// first_counted: the key emission wrote the first pass's counts (key_sort_first_count).
int radix_sort_u32(uint32_t *ka, uint32_t *va, uint32_t *kb, uint32_t *vb, uint32_t K, uint32_t sub, int total_bits,
                   uint32_t *ghist, uint32_t *cnt, hipStream_t st, bool first_counted) {
    return radix_sort<uint32_t, KV_SUB>(ka, va, kb, vb, K, sub, 0, total_bits, ghist, cnt, st, nullptr, first_counted);
}

// The same with the count read from device memory; K_max bounds it (sizes the grids and the
// count matrix).
int radix_sort_u32_dyn(uint32_t *ka, uint32_t *va, uint32_t *kb, uint32_t *vb, uint32_t K_max, const uint32_t *dyn_count,
                       int total_bits, uint32_t *ghist, uint32_t *cnt, hipStream_t st, bool first_counted) {
    return radix_sort<uint32_t, KV_SUB>(ka, va, kb, vb, K_max, 0u, 0, total_bits, ghist, cnt, st, dyn_count, first_counted);
}

}  // namespace recogs
