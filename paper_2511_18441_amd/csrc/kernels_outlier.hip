// Statistical outlier removal of a point cloud (Sec. 3.2, Fig. 2 caption: mean distance
// to 16 neighbours, standard-deviation scale 0.007):
//   D_i = mean distance from point i to its k nearest other points (all others when
//         there are fewer), mu / sigma = mean and population standard deviation of D,
//   keep i  iff  D_i <= mu + std_ratio sigma.
//
// Exact k-nearest neighbours through a hashed uniform grid:
//   1. bounding box (reduction), then per-axis 1024-bin histograms over it; the cell
//      size h is the largest 1%-99% quantile extent divided by ceil(2 n^(1/3)) (at most
//      128), so far-away stray points do not coarsen the grid for the rest;
//   2. each point's cell (floor((x - min) / h) per axis) goes to the slot made of its
//      coordinates modulo powers of two (2^b slots, b = log2 of about 2n, at least 4 bits
//      per axis); a radix sort by slot orders the points, and a binary search gives each
//      slot's first point, so the points of consecutive slots are one run (slot order is
//      also the query order: queries of one wave start in nearby cells);
//   3. per query, the cubes of cells of Chebyshev radius 1, then 2, then 5 are searched (no
//      two cells of one cube share a slot; points of far cells that do are scanned too),
//      a row of cells along x being one run of points; the search ends once the k-th
//      distance is within (r - 1/16) h, the distance below which no unscanned cell lies
//      (the 1/16 absorbs float32 rounding of the cell coordinates). A query has 2, 16 and
//      64 lanes in the three searches (4 and 16 of the last two where many queries are
//      left, and then the largest cube in shells), which merge their lists of the k
//      smallest. Queries that even the largest cube leaves open (far stray points) go to a
//      search of the whole cloud by the bounding boxes of its runs of 64 points.
//      314k points (a brush selection): 285 us for the four, against 980 with one thread
//      per query over the 27 cells one by one, one wave per query with a cell per lane for
//      the rest, and a scan of the whole cloud for each stray point.
//   4. mu and sigma from compensated float32 sums (float-float, TwoSum) in a fixed order:
//      a pass for the sum of D, a pass for the sum of (D - mu)^2; the threshold, the keep
//      mask (float32 comparison) and the compaction of the kept points (input order)
//      follow. No double precision on the GPU.
#include "recogs_internal.hpp"

namespace recogs {

int radix_sort_u32(uint32_t *, uint32_t *, uint32_t *, uint32_t *, uint32_t, uint32_t, int, uint32_t *, uint32_t *,
                   hipStream_t, bool = false);
void launch_excl_scan_u32(uint32_t *, uint32_t, uint32_t *, hipStream_t);

constexpr int kOlBins = 1024;
constexpr int kOlMaxDim = 128;
constexpr int kOlRing1 = 1, kOlRing2 = 2, kOlRing3 = 5;   // cube radii of the three searches
constexpr int kOlShell0 = 3;                   // first cube of the third in shells
constexpr int kOlR1 = 1, kOlC1 = 2, kOlR2 = 4, kOlC2 = 4, kOlR3 = 16, kOlC3 = 4;   // their lanes per query: rows x candidates
constexpr int kOlR2Many = 2, kOlC2Many = 2, kOlR3Many = 8, kOlC3Many = 2;          // with long lists
// which lists are long: `total` queries of n points
template <int K> __device__ __forceinline__ bool ol_many2(uint32_t total, uint32_t n) {
    return total >= (K < 16 ? 8192u : K < 32 ? 16384u : 49152u) && total > n - n / 16u;
}
template <int K> __device__ __forceinline__ bool ol_many3(uint32_t total, uint32_t n) {
    return total >= 32768u || (K < 16 && total >= 8192u + 512u * (K - 4) && total > n - n / 16u);
}
constexpr int kOlListBlocks = 2048;            // grid of the second and third (grid-stride over their lists)
static_assert(2 * kOlRing3 + 1 <= 16, "one search's cells must fit in 16 slot residues per axis");
constexpr int kOlLeaf = 64;                    // points per bounding box of the whole-cloud search
constexpr int kOlFarBlocks = 1024;             // grid of the whole-cloud searches (grid-stride over the queries)
constexpr int kOlFarThreads = 512;
constexpr int kOlRedBlocks = 512;              // grid of the reductions (grid-stride)
constexpr int64_t kOlSample = 32768;           // points of the histograms' sample, about
constexpr uint32_t kOlScanFold = 2048;         // most workgroup counts that the compaction sums by itself
constexpr int kOlItems = 4;                    // points per thread of the keep/compaction passes
constexpr int kOlBlock = 256 * kOlItems;
constexpr float kOlClamp = 1048576.f;          // cell coordinates are clamped to +-2^20
// Ring-search guard: a float32 cell coordinate f = (v - min) / h is within 3 2^-24 |f|
// of its exact value, so for |f| <= 2^16 two coordinates are within 0.024 cells of the
// exact difference; the stop bound keeps kOlMargin = 1/16 cell of slack for it. Queries
// beyond 2^16 cells from the box corner scan the whole cloud.
constexpr float kOlQueryLimit = 65536.f;
constexpr float kOlMargin = 1.f / 16.f;

// Workspace header (device, written by the setup kernels).
struct OlHdr {
    float mn[3], mx[3];   // bounding box
    float h, inv_h;       // cell size and its reciprocal
    uint32_t bx, by, bz;  // slot bits per axis
    uint32_t ndefer;      // queries left to the whole-cloud search
    uint32_t nslow[2];    // queries left to the second and to the third cube search
    float thr;            // mu + std_ratio sigma
    float mu, sigma;
};

__device__ __forceinline__ void ol_load(const float *__restrict__ pts, int64_t stride, int64_t i, float &x, float &y,
                                        float &z) {
    x = pts[i];
    y = pts[stride + i];
    z = pts[2 * stride + i];
}

__device__ __forceinline__ int ol_coord(float v, float mn, float inv_h) {
    const float f = fminf(fmaxf(floorf((v - mn) * inv_h), -kOlClamp), kOlClamp);
    return (int)f;
}

// Slot of a cell: its coordinates modulo 2^bx, 2^by, 2^bz, packed (bx + by + bz = the
// slot bits, each at least 4). Cells that differ by less than 16 along every axis get
// different slots, so the cells of one search (at most 11 x 11 x 11) never share a slot
// and a slot's run can be scanned without checking each point's cell: the points of
// far cells that share it are real points of the cloud, and only add candidates.
__device__ __forceinline__ uint32_t ol_slot(int cx, int cy, int cz, uint32_t bx, uint32_t by, uint32_t bz) {
    return ((uint32_t)cx & ((1u << bx) - 1u)) | (((uint32_t)cy & ((1u << by) - 1u)) << bx) |
           (((uint32_t)cz & ((1u << bz) - 1u)) << (bx + by));
}

__device__ __forceinline__ float wave_min(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// 1a. per-workgroup bounding boxes -> part[blk][6]; also zeroes the histograms
__global__ __launch_bounds__(256) void k_ol_bbox(const float *__restrict__ pts, int64_t n, int64_t stride,
                                                 float *__restrict__ part, uint32_t *__restrict__ hist) {
    __shared__ float s[4][6];
    for (int k = (int)(blockIdx.x * 256 + threadIdx.x); k < 3 * kOlBins; k += (int)gridDim.x * 256) hist[k] = 0u;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        float p[3];
        ol_load(pts, stride, i, p[0], p[1], p[2]);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], p[a]);
            hi[a] = fmaxf(hi[a], p[a]);
        }
    }
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = wave_min(lo[a]);
        hi[a] = wave_max(hi[a]);
    }
    if (lane_id() == 0)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            s[w][a] = lo[a];
            s[w][3 + a] = hi[a];
        }
    __syncthreads();
    if (threadIdx.x < 6) {
        float v = s[0][threadIdx.x];
        for (int k = 1; k < 4; ++k) v = threadIdx.x < 3 ? fminf(v, s[k][threadIdx.x]) : fmaxf(v, s[k][threadIdx.x]);
        part[blockIdx.x * 6 + threadIdx.x] = v;
    }
}

// 1b. per-axis histograms over the box (LDS counts, then one atomic per bin and
// workgroup; integer counts, so the result is independent of the order), of one point in
// every step: they only place the cell size, which no result depends on, and neighbouring
// points fall into the same bins, whose LDS atomics then wait for each other (15 us over
// all points of a 314k cloud). The point within the step follows the golden ratio's
// multiples, so that an order with a period (interleaved scans, points dealt in turn) does
// not show only one of its phases: with always the first, a cloud of 131,072 points dealt
// in turn to one small and three large clusters took cells a hundred times too small.
// Every workgroup reduces the partial boxes for itself (wave w the bounds w and w + 4);
// workgroup 0 stores the box and clears the queues' counts.
__global__ __launch_bounds__(256) void k_ol_hist(const float *__restrict__ pts, int64_t n, int64_t stride,
                                                 int64_t ns, uint32_t step, const float *__restrict__ part, int nblk,
                                                 OlHdr *__restrict__ hdr, uint32_t *__restrict__ hist) {
    __shared__ uint32_t s_h[3 * kOlBins];
    __shared__ float s_box[6];
    for (int k = threadIdx.x; k < 3 * kOlBins; k += 256) s_h[k] = 0;
    for (int a = (int)(threadIdx.x >> 6); a < 6; a += 4) {
        const bool lo = a < 3;
        float v = lo ? INFINITY : -INFINITY;
        for (int b = (int)lane_id(); b < nblk; b += 64) v = lo ? fminf(v, part[b * 6 + a]) : fmaxf(v, part[b * 6 + a]);
        v = lo ? wave_min(v) : wave_max(v);
        if (lane_id() == 0) {
            s_box[a] = v;
            if (blockIdx.x == 0) {
                if (lo) hdr->mn[a] = v;
                else hdr->mx[a - 3] = v;
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) hdr->ndefer = hdr->nslow[0] = hdr->nslow[1] = 0;
    __syncthreads();
    float mn[3], sc[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        mn[a] = s_box[a];
        const float e = s_box[3 + a] - mn[a];
        sc[a] = e > 0.f ? (float)kOlBins / e : 0.f;
    }
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < ns; q += (int64_t)gridDim.x * 256) {
        const uint32_t phase = __umulhi((uint32_t)q * 0x9e3779b9u, step);   // 0 .. step - 1
        float p[3];
        ol_load(pts, stride, min(q * step + phase, n - 1), p[0], p[1], p[2]);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            int b = (int)((p[a] - mn[a]) * sc[a]);
            b = b < 0 ? 0 : (b >= kOlBins ? kOlBins - 1 : b);
            atomicAdd(&s_h[a * kOlBins + b], 1u);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < 3 * kOlBins; k += 256)
        if (s_h[k]) atomicAdd(&hist[k], s_h[k]);
}

// 1c. cell size from the 1%-99% quantile extents: wave a scans axis a's 1024 bins (16
// per lane, then a wave scan) and finds the first bins whose cumulative count passes 1%
// and 99% of the points; then thread 0 sets h.
// (ns: the histograms' points)
__global__ __launch_bounds__(192) void k_ol_setup(const uint32_t *__restrict__ hist, int64_t ns, int64_t n, uint32_t slot_bits,
                                                  OlHdr *__restrict__ hdr) {
    __shared__ float s_ext[3];
    constexpr int PER = kOlBins / 64;
    const int a = threadIdx.x >> 6, l = (int)lane_id();
    const uint64_t lo_need = (uint64_t)ns / 100u, hi_need = (uint64_t)ns * 99u / 100u;
    uint32_t c[PER];
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        c[q] = hist[a * kOlBins + l * PER + q];
        mine += c[q];
    }
    const uint32_t incl = wave_incl_scan(mine);
    // first bin (in lane-major order) where the running count exceeds `need`
    auto first_over = [&](uint64_t need) -> int {
        int bin = kOlBins;
        uint64_t cum = incl - mine;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            cum += c[q];
            if (bin == kOlBins && cum > need) bin = l * PER + q;
        }
        int best = bin;
        for (int o = 32; o > 0; o >>= 1) best = min(best, __shfl_xor(best, o));
        return best;
    };
    int blo = first_over(lo_need);
    int bhi = first_over(hi_need < (uint64_t)ns ? hi_need : (uint64_t)ns - 1);
    blo = blo >= kOlBins ? 0 : blo;
    bhi = bhi >= kOlBins ? kOlBins - 1 : bhi;
    if (l == 0) {
        const float e = hdr->mx[a] - hdr->mn[a];
        s_ext[a] = (float)(bhi - blo + 1) * (e / (float)kOlBins);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const float L = fmaxf(s_ext[0], fmaxf(s_ext[1], s_ext[2]));
        // D = ceil(2 n^(1/3)), the least D with D^3 >= 8 n, capped at kOlMaxDim
        int D = 1;
        while (D < kOlMaxDim && (uint64_t)D * D * D < 8u * (uint64_t)n) ++D;
        float h = L / (float)D;
        if (!(h > 0.f) || !isfinite(h)) h = 1.f;   // all points coincide (or a degenerate box)
        hdr->h = h;
        hdr->inv_h = 1.f / h;
        hdr->bz = slot_bits / 3;
        hdr->by = (slot_bits - slot_bits / 3) / 2;
        hdr->bx = slot_bits - hdr->bz - hdr->by;
    }
}

// 2. slot keys
__global__ __launch_bounds__(256) void k_ol_key(const float *__restrict__ pts, int64_t n, int64_t stride,
                                                const OlHdr *__restrict__ hdr, uint32_t *__restrict__ keys,
                                                uint32_t *__restrict__ vals) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    float x, y, z;
    ol_load(pts, stride, i, x, y, z);
    const float ih = hdr->inv_h;
    keys[i] = ol_slot(ol_coord(x, hdr->mn[0], ih), ol_coord(y, hdr->mn[1], ih), ol_coord(z, hdr->mn[2], ih), hdr->bx,
                      hdr->by, hdr->bz);
    vals[i] = (uint32_t)i;
}

// number of keys below `key` among the sorted keys[0, n), by the whole wave: 64 probes a
// round, so n is cut by 65 per memory round trip
__device__ __forceinline__ uint32_t wave_lower_bound(const uint32_t *__restrict__ keys, uint32_t n, uint32_t key) {
    uint32_t lo = 0, len = n;
    while (len > 0) {
        const uint32_t step = (len + 64u) / 65u, p = step * (lane_id() + 1u) - 1u;   // probe within [0, len)
        const bool below = p < len && keys[lo + p] < key;
        const uint32_t c = (uint32_t)__builtin_popcountll(wave_ballot(below));
        lo += c * step;
        const uint32_t rest = len - c * step;   // up to the probe that was not below, if any
        len = c < 64u ? min(step - 1u, rest) : rest;
    }
    return lo;
}

// 2b. workgroups [0, sblk): each slot's first point in slot order, start[s] = the number of
// keys below s, for the slots and one past the last (a run of slots [s, t) holds the points
// [start[s], start[t])): a wave finds where its 64 slots begin and end (14 us with a
// binary search over all keys per slot, now 6 with the gather), each lane its own slot
// between them.
// The others: the points in slot order as float4 (x, y, z, input index bits): one 16-byte
// load per candidate in the searches below; and the bounding box of each run of kOlLeaf
// (one wave's) as two float4.
__global__ __launch_bounds__(256) void k_ol_gather(const float *__restrict__ pts, int64_t n, int64_t stride,
                                                   const uint32_t *__restrict__ keys, const uint32_t *__restrict__ svals,
                                                   uint32_t slots, uint32_t sblk, uint32_t *__restrict__ start,
                                                   float4 *__restrict__ spts, float4 *__restrict__ boxes) {
    if (blockIdx.x < sblk) {
        const uint32_t s0 = blockIdx.x * 256u + (threadIdx.x & ~63u), s = s0 + lane_id();
        if (s0 > slots) return;
        uint32_t lo = wave_lower_bound(keys, (uint32_t)n, s0);
        uint32_t hi = lo + wave_lower_bound(keys + lo, (uint32_t)n - lo, s0 + 64u);
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (keys[mid] < s) lo = mid + 1;
            else hi = mid;
        }
        if (s <= slots) start[s] = lo;
        return;
    }
    static_assert(kOlLeaf == 64, "a leaf is a wave's points");
    const int64_t j = (int64_t)(blockIdx.x - sblk) * 256 + threadIdx.x;
    float p[3] = {0.f, 0.f, 0.f};
    if (j < n) {
        const uint32_t i = svals[j];
        ol_load(pts, stride, i, p[0], p[1], p[2]);
        spts[j] = make_float4(p[0], p[1], p[2], __uint_as_float(i));
    }
    float lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = wave_min(j < n ? p[a] : INFINITY);
        hi[a] = wave_max(j < n ? p[a] : -INFINITY);
    }
    if (lane_id() == 0 && j < n) {
        boxes[2 * (j / kOlLeaf)] = make_float4(lo[0], lo[1], lo[2], 0.f);
        boxes[2 * (j / kOlLeaf) + 1] = make_float4(hi[0], hi[1], hi[2], 0.f);
    }
}

// The K smallest squared distances, ascending (+inf: none yet). One more is put in its
// place by one median of three per entry: entry q becomes the median of d2 and the old
// entries q - 1 and q.
template <int K> __device__ __forceinline__ void ol_insert(float (&best)[K], float d2) {
    if (d2 < best[K - 1]) {
#pragma unroll
        for (int q = K - 1; q > 0; --q) best[q] = __builtin_amdgcn_fmed3f(d2, best[q - 1], best[q]);
        best[0] = fminf(best[0], d2);
    }
}
__device__ __forceinline__ void ol_ce(float &a, float &b) {   // compare and exchange (as bits: no value is negative or NaN)
    const uint32_t u = __float_as_uint(a), v = __float_as_uint(b);
    a = __uint_as_float(min(u, v));
    b = __uint_as_float(max(u, v));
}
// every lane of an aligned group of G lanes <- the K smallest of the group's lists: the
// element-wise minima of a list and its partner's reversed hold the K smallest of both as
// a bitonic sequence, which log2 K rounds of exchanges sort
template <int K, int G> __device__ __forceinline__ void ol_merge_lanes(float (&best)[K]) {
#pragma unroll
    for (int o = 1; o < G; o <<= 1) {
        float t[K];
#pragma unroll
        for (int a = 0; a < K; ++a) t[a] = __shfl_xor(best[a], o, 64);
#pragma unroll
        for (int a = 0; a < K; ++a) best[K - 1 - a] = fminf(best[K - 1 - a], t[a]);
#pragma unroll
        for (int s = K / 2; s > 0; s >>= 1)
#pragma unroll
            for (int a = 0; a < K; ++a)
                if (!(a & s)) ol_ce(best[a], best[a + s]);
    }
}
// N candidates, loaded together, against query i at (x, y, z); the first `count` count
template <int K, int N>
__device__ __forceinline__ void ol_take(float (&best)[K], const float4 (&c)[N], uint32_t count, uint32_t i, float x, float y,
                                        float z) {
#pragma unroll
    for (uint32_t u = 0; u < (uint32_t)N; ++u) {
        if (u < count) {   // (skipped by the wave once none of its lanes has more)
            const float ex = c[u].x - x, ey = c[u].y - y, ez = c[u].z - z;
            const float d2 = __builtin_fmaf(ex, ex, __builtin_fmaf(ey, ey, ez * ez));
            if (__float_as_uint(c[u].w) != i) ol_insert<K>(best, d2);   // (i: the query itself)
        }
    }
}
template <int K> __device__ __forceinline__ float ol_mean(const float (&best)[K], int want) {
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < K; ++q) sum += q < want ? sqrtf(best[q]) : 0.f;
    return want > 0 ? sum / (float)want : 0.f;
}

// 3. k nearest neighbours within the cube of cells of radius RING, G = GR GC consecutive
// lanes per query: its (2 RING + 1)^2 rows of cells are dealt to GR groups, and GC lanes
// take neighbouring candidates of a row (one line of memory then serves several lanes).
// More lanes per query fill the GPU and balance the rows, fewer leave less to merge:
// measured at 314k points, (GR, GC) of the radius-1 search (1, 1) 135, (1, 2) 119, (1, 4) 137,
// (1, 8) 193 us; of the radius-2 search (4, 2) 91, (8, 2) 76, (4, 4) 68; of the radius-5
// search (16, 2) 75, (8, 8) 49, (16, 4) 42. The queries are all points in slot order (list
// null) or the listed slot positions, `total` of them, grid-stride. A query not settled
// goes to the list `slow` (or, with slow null, to the whole-cloud search, as does any
// beyond the coordinate guard).
struct OlSearch {
    const float4 *__restrict__ spts;
    int64_t n;
    OlHdr *hdr;
    const uint32_t *__restrict__ start;
    uint32_t *__restrict__ defer;
    float *__restrict__ dmean;
};
// hd: the header, read by the caller in one go with the list's length
template <int K, int RING, int GR, int GC>
__device__ __forceinline__ void ol_search(const OlSearch &sr, const OlHdr &hd, const uint32_t *__restrict__ list, uint32_t total,
                                          uint32_t *__restrict__ slow, uint32_t *nslow) {
    const float4 *__restrict__ spts = sr.spts;
    const uint32_t *__restrict__ start = sr.start;
    const int64_t n = sr.n;
    OlHdr *hdr = sr.hdr;
    constexpr int SIDE = 2 * RING + 1, ROWS = SIDE * SIDE, G = GR * GC;
    const float mnx = hd.mn[0], mny = hd.mn[1], mnz = hd.mn[2], ih = hd.inv_h, h = hd.h;
    const uint32_t bx = hd.bx, by = hd.by, bz = hd.bz;
    const uint32_t mx = (1u << bx) - 1u, my = (1u << by) - 1u, mz = (1u << bz) - 1u;
    const int want = n - 1 < (int64_t)K ? (int)(n - 1) : K;
    const int g = (int)(threadIdx.x % G), gr = g / GC;
    const uint32_t gc = (uint32_t)(g % GC);
    const uint32_t last = (uint32_t)n - 1u;
    for (uint32_t q = (blockIdx.x * 256u + threadIdx.x) / G; q < total; q += gridDim.x * (256u / G)) {
        const uint32_t s = list ? list[q] : q;
        const float4 me = spts[s];
        const uint32_t i = __float_as_uint(me.w);
        const float x = me.x, y = me.y, z = me.z;
        float best[K];
#pragma unroll
        for (int a = 0; a < K; ++a) best[a] = INFINITY;
        const bool clamped = fabsf((x - mnx) * ih) > kOlQueryLimit || fabsf((y - mny) * ih) > kOlQueryLimit ||
                             fabsf((z - mnz) * ih) > kOlQueryLimit;
        bool done = want == 0;
        if (!done && !clamped) {
            const uint32_t cx = (uint32_t)ol_coord(x, mnx, ih), cy = (uint32_t)ol_coord(y, mny, ih),
                           cz = (uint32_t)ol_coord(z, mnz, ih);
            // a row of cells is one run of slots, or two where it wraps around the residues
            const uint32_t x0 = (cx - RING) & mx, x1 = (cx + RING) & mx;
            const bool wrap = x0 > x1;
            auto row = [&](int r) {   // the row's first slot (x residue 0)
                return (((cy + (uint32_t)(r % SIDE) - RING) & my) << bx) |
                       (((cz + (uint32_t)(r / SIDE) - RING) & mz) << (bx + by));
            };
            constexpr uint32_t NB = 8;   // candidates in flight per lane
            auto run = [&](uint32_t a, uint32_t b) {
                for (uint32_t j = a + gc; j < b; j += NB * GC) {
                    float4 c[NB];
                    const uint32_t left = (b - j + GC - 1) / GC;   // this lane's candidates
#pragma unroll
                    for (uint32_t u = 0; u < NB; ++u) c[u] = spts[min(j + u * GC, last)];
                    ol_take<K, NB>(best, c, left, i, x, y, z);
                }
            };
            uint32_t base = row(gr < ROWS ? gr : 0);
            uint32_t a = start[base + x0], b = start[base + (wrap ? mx : x1) + 1u];
            for (int r = gr; r < ROWS; r += GR) {
                // the next row's run is looked up while this one is scanned
                const int rn = r + GR;
                const uint32_t nbase = row(rn < ROWS ? rn : r);
                const uint32_t na = start[nbase + x0], nb = start[nbase + (wrap ? mx : x1) + 1u];
                run(a, b);
                if (wrap) run(start[base], start[base + x1 + 1u]);
                base = nbase;
                a = na;
                b = nb;
            }
            ol_merge_lanes<K, G>(best);
            float kth = best[0];
#pragma unroll
            for (int a2 = 1; a2 < K; ++a2) kth = a2 == want - 1 ? best[a2] : kth;
            const float bound = ((float)RING - kOlMargin) * h;
            done = kth <= bound * bound;
        }
        if (g == 0) {
            if (done) sr.dmean[i] = ol_mean<K>(best, want);
            else if (clamped || !slow) sr.defer[atomicAdd(&hdr->ndefer, 1u)] = i;
            else slow[atomicAdd(nslow, 1u)] = s;
        }
    }
}

// The third search for a long list: the cube of radius kOlShell0, then shell by shell up to
// kOlRing3, with the stop test between (the k-th distance is within a bound iff the lanes'
// lists hold k entries within it). Points that fill a volume settle at radius 3 or 4, whose
// cubes have a quarter and half of radius 5's cells.
template <int K, int GR, int GCI>
__device__ __forceinline__ void ol_search_shells(const OlSearch &sr, const OlHdr &hd, const uint32_t *__restrict__ list,
                                                 uint32_t total) {
    constexpr int G = GR * GCI;
    constexpr uint32_t GC = GCI, NB = 8;   // candidates in flight per lane
    const float4 *__restrict__ spts = sr.spts;
    const uint32_t *__restrict__ start = sr.start;
    const int64_t n = sr.n;
    OlHdr *hdr = sr.hdr;
    const float mnx = hd.mn[0], mny = hd.mn[1], mnz = hd.mn[2], ih = hd.inv_h, h = hd.h;
    const uint32_t bx = hd.bx, by = hd.by, bz = hd.bz;
    const uint32_t mx = (1u << bx) - 1u, my = (1u << by) - 1u, mz = (1u << bz) - 1u;
    const int want = n - 1 < (int64_t)K ? (int)(n - 1) : K;
    const uint32_t last = (uint32_t)n - 1u;
    const int l = (int)(threadIdx.x % G), gr = l / (int)GC;
    const uint32_t gc = (uint32_t)l % GC;
    for (uint32_t q = (blockIdx.x * 256u + threadIdx.x) / G; q < total; q += gridDim.x * (256u / G)) {
        const float4 me = spts[list[q]];
        const uint32_t i = __float_as_uint(me.w);
        const float x = me.x, y = me.y, z = me.z;
        const uint32_t cx = (uint32_t)ol_coord(x, mnx, ih), cy = (uint32_t)ol_coord(y, mny, ih),
                       cz = (uint32_t)ol_coord(z, mnz, ih);
        float best[K];
#pragma unroll
        for (int a = 0; a < K; ++a) best[a] = INFINITY;
        auto run = [&](uint32_t a, uint32_t b) {
            for (uint32_t j = a + gc; j < b; j += NB * GC) {
                float4 c[NB];
                const uint32_t left = (b - j + GC - 1) / GC;   // this lane's candidates
#pragma unroll
                for (uint32_t u = 0; u < NB; ++u) c[u] = spts[min(j + u * GC, last)];
                ol_take<K, NB>(best, c, left, i, x, y, z);
            }
        };
        bool done = false;
        for (int r = kOlShell0; r <= kOlRing3 && !done; ++r) {
            // pieces t of the shell: the side^2 rows of the cube, whole on its faces and, for
            // the others, their first cell; then the others' last cells. The first cube: its rows.
            const bool cube = r == kOlShell0;
            const int side = 2 * r + 1, rows = side * side, inner = cube ? 0 : side - 2, pieces = rows + inner * inner;
            const int rcp = 65536 / side + 1, rcp_in = inner ? 65536 / inner + 1 : 0;   // exact quotients below 256
            struct Piece { uint32_t a, b, a2, b2; };   // one run of points, or two where it wraps
            auto piece = [&](int t) {
                int dy, dz, x0 = -r, x1 = r;
                if (t < rows) {
                    dz = (t * rcp) >> 16;
                    dy = t - dz * side - r;
                    dz -= r;
                    if (!cube && max(abs(dy), abs(dz)) < r) x1 = -r;
                } else {
                    dz = ((t - rows) * rcp_in) >> 16;
                    dy = t - rows - dz * inner - (r - 1);
                    dz -= r - 1;
                    x0 = r;
                }
                const uint32_t base = (((cy + (uint32_t)dy) & my) << bx) | (((cz + (uint32_t)dz) & mz) << (bx + by));
                const uint32_t u0 = (cx + (uint32_t)x0) & mx, u1 = (cx + (uint32_t)x1) & mx;
                const bool wrap = u0 > u1;
                Piece p{start[base + u0], start[base + (wrap ? mx : u1) + 1u], 0u, 0u};
                if (wrap) {
                    p.a2 = start[base];
                    p.b2 = start[base + u1 + 1u];
                }
                return p;
            };
            Piece p = piece(gr);
            for (int t = gr; t < pieces; t += GR) {
                const Piece nx = piece(t + GR < pieces ? t + GR : t);   // looked up while this one is scanned
                run(p.a, p.b);
                if (p.b2 > p.a2) run(p.a2, p.b2);
                p = nx;
            }
            const float bound = ((float)r - kOlMargin) * h, b2 = bound * bound;
            uint32_t c = 0;
#pragma unroll
            for (int a = 0; a < K; ++a) c += best[a] <= b2 ? 1u : 0u;
#pragma unroll
            for (int o = 1; o < G; o <<= 1) c += __shfl_xor(c, o);
            done = c >= (uint32_t)want;
        }
        ol_merge_lanes<K, G>(best);
        if (l == 0) {
            if (done) sr.dmean[i] = ol_mean<K>(best, want);
            else sr.defer[atomicAdd(&hdr->ndefer, 1u)] = i;
        }
    }
}

// The three searches. Many lanes per query are for lists that would leave the GPU idle, or
// for rows of many points; where nearly all of the cloud is left (a volume's points, about
// 1/8 per cell: a row holds none or one), few lanes waste less, and the lists are long enough.
// The whole filter over uniform points in a cube, k = 4 / 8 / 16 / 32, us, the wide forms alone
// (radius 5 at once) and by this rule: 20,000 points 189 / 220 / 253 / 394 and 155 / 182 / 223 /
// 394; 100,000 638 / 823 / 955 / 1685 and 334 / 456 / 725 / 1538; 400,000 1684 / 3686 / 4377 /
// 4737 and 772 / 1074 / 1823 / 2851; over a regular grid of 14,000, k = 4 and 8, 183 / 186 and
// 123 / 149. Below the lines the wide forms win (5,000 points, k = 4 / 8 / 16, 118 / 136 / 148
// against 121 / 173 / 151; a plane's regular grid of 14,000 with k = 16 119 against 139; a sheet's
// 20,000 with k = 32 162 against 176), and where a sixteenth or more of the cloud has
// settled its rows hold many points (a brush's 47,000 points with k = 32, three quarters left:
// 261 against 295; 400,000 in clusters, k = 16, 480 against 509).
template <int K> __global__ __launch_bounds__(256) void k_ol_knn1(OlSearch sr, uint32_t *slow) {
    const OlHdr hd = *sr.hdr;
    ol_search<K, kOlRing1, kOlR1, kOlC1>(sr, hd, nullptr, (uint32_t)sr.n, slow, sr.hdr->nslow);
}
template <int K>
__global__ __launch_bounds__(256) void k_ol_knn2(OlSearch sr, const uint32_t *list, uint32_t *slow) {
    const OlHdr hd = *sr.hdr;
    const uint32_t total = hd.nslow[0];
    if (ol_many2<K>(total, (uint32_t)sr.n))
        ol_search<K, kOlRing2, kOlR2Many, kOlC2Many>(sr, hd, list, total, slow, sr.hdr->nslow + 1);
    else
        ol_search<K, kOlRing2, kOlR2, kOlC2>(sr, hd, list, total, slow, sr.hdr->nslow + 1);
}
template <int K> __global__ __launch_bounds__(256) void k_ol_knn3(OlSearch sr, const uint32_t *list) {
    const OlHdr hd = *sr.hdr;
    const uint32_t total = hd.nslow[1];
    if (ol_many3<K>(total, (uint32_t)sr.n)) ol_search_shells<K, kOlR3Many, kOlC3Many>(sr, hd, list, total);
    else ol_search<K, kOlRing3, kOlR3, kOlC3>(sr, hd, list, total, nullptr, nullptr);
}

// 3b. the deferred queries, one workgroup each (grid-stride over the list): each thread
// tests the boxes of the cloud's runs of kOlLeaf points. A full run holds more than K other
// points, so the smallest of the boxes' largest distances bounds the k-th distance; only
// runs whose box reaches within that bound (with a margin far above float32 rounding) are
// scanned, eight at a time per wave, a point per lane. (A scan of the whole cloud per query
// is bound by the caches: 237 us for the 538 stray points of a 314k cloud.)
template <int K>
__global__ __launch_bounds__(kOlFarThreads) void k_ol_knn_far(const float4 *__restrict__ spts, const float4 *__restrict__ boxes,
                                                    const float *__restrict__ pts,
                                                    int64_t n, int64_t stride, const OlHdr *__restrict__ hdr,
                                                    const uint32_t *__restrict__ defer, float *__restrict__ dmean) {
    constexpr int NW = kOlFarThreads / 64;
    __shared__ float s_tau[NW];
    __shared__ float s_l[NW][K];
    const uint32_t nd = hdr->ndefer;
    const int want = n - 1 < (int64_t)K ? (int)(n - 1) : K;
    const uint32_t w = threadIdx.x >> 6, l = lane_id();
    const int64_t leaves = (n + kOlLeaf - 1) / kOlLeaf, full = n / kOlLeaf;
    const uint32_t last = (uint32_t)n - 1u;
    for (uint32_t q = blockIdx.x; q < nd; q += gridDim.x) {
        const uint32_t i = defer[q];
        float p[3];
        ol_load(pts, stride, i, p[0], p[1], p[2]);
        // squared distances to a box: the least and the largest
        auto reach = [&](int64_t f, float &hi2) {
            const float4 a = boxes[2 * f], b = boxes[2 * f + 1];
            const float lo[3] = {a.x, a.y, a.z}, hi[3] = {b.x, b.y, b.z};
            float l2 = 0.f;
            hi2 = 0.f;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float u = lo[k] - p[k], v = p[k] - hi[k];   // both <= 0 inside
                const float o = fmaxf(fmaxf(u, v), 0.f), e = fmaxf(fabsf(u), fabsf(v));
                l2 = __builtin_fmaf(o, o, l2);
                hi2 = __builtin_fmaf(e, e, hi2);
            }
            return l2;
        };
        float tau = INFINITY;
        for (int64_t f = threadIdx.x; f < full; f += kOlFarThreads) {
            float hi2;
            (void)reach(f, hi2);
            tau = fminf(tau, hi2);
        }
        tau = wave_min(tau);
        if (l == 0) s_tau[w] = tau;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NW; ++k) tau = fminf(tau, s_tau[k]);
        tau = tau * (1.f + 2e-5f);   // (inf stays inf)
        float best[K];
#pragma unroll
        for (int a = 0; a < K; ++a) best[a] = INFINITY;
        // neighbouring boxes go to different waves
        for (int64_t f0 = 0; f0 < leaves; f0 += kOlFarThreads) {
            const int64_t f = f0 + (int64_t)l * NW + w;
            float hi2;
            const bool near = f < leaves && reach(f, hi2) <= tau;
            uint64_t mm = wave_ballot(near);
            while (mm) {
                float4 c[8];
                uint32_t count = 0;   // (a lane's candidates are in the order of the runs: the last may be short)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const uint32_t j = (uint32_t)(f0 + (mm ? (int64_t)__builtin_ctzll(mm) * NW + w : 0)) * kOlLeaf + l;
                    count += mm && j <= last ? 1u : 0u;
                    mm &= mm - 1;
                    c[u] = spts[min(j, last)];
                }
                ol_take<K, 8>(best, c, count, i, p[0], p[1], p[2]);
            }
        }
        ol_merge_lanes<K, 64>(best);
        if (l == 0)
#pragma unroll
            for (int a = 0; a < K; ++a) s_l[w][a] = best[a];
        __syncthreads();
        if (w == 0) {
#pragma unroll
            for (int a = 0; a < K; ++a) best[a] = s_l[l % NW][a];
            ol_merge_lanes<K, NW>(best);
            if (l == 0) dmean[i] = ol_mean<K>(best, want);
        }
        __syncthreads();   // s_l and s_tau are reused by the next query
    }
}

// Compensated float32 sums: a value held as hi + lo, each addition through Knuth's
// TwoSum (the rounding error of hi + b is exact and goes to lo).
struct FF { float hi, lo; };
__device__ __forceinline__ FF ff_add(FF a, float b) {
    const float s = a.hi + b, bb = s - a.hi;
    return FF{s, a.lo + ((a.hi - (s - bb)) + (b - bb))};
}
__device__ __forceinline__ FF ff_merge(FF a, FF b) {
    const float s = a.hi + b.hi, bb = s - a.hi;
    return FF{s, (a.lo + b.lo) + ((a.hi - (s - bb)) + (b.hi - bb))};
}
__device__ __forceinline__ FF ff_wave(FF a) {   // butterfly over the wave, the same order every run
    for (int o = 32; o > 0; o >>= 1) a = ff_merge(a, FF{__shfl_xor(a.hi, o), __shfl_xor(a.lo, o)});
    return a;
}
// the workgroup's 256-thread sum (every wave reaches it), fixed order; valid in thread 0
__device__ __forceinline__ FF ff_block(FF a, FF (*s)[1]) {
    a = ff_wave(a);
    if (lane_id() == 0) s[threadIdx.x >> 6][0] = a;
    __syncthreads();
    return ff_merge(ff_merge(s[0][0], s[1][0]), ff_merge(s[2][0], s[3][0]));
}
// sum of the nblk partials part[0..nblk) by one wave (lanes stride, then the butterfly)
__device__ __forceinline__ FF ff_parts(const float2 *__restrict__ part, int nblk) {
    FF a{0.f, 0.f};
    for (int k = (int)lane_id(); k < nblk; k += 64) a = ff_merge(a, FF{part[k].x, part[k].y});
    return ff_wave(a);
}

// 4a. per workgroup: compensated sum of D -> part[blk]
__global__ __launch_bounds__(256) void k_ol_sum(const float *__restrict__ dmean, int64_t n, float2 *__restrict__ part) {
    __shared__ FF s[4][1];
    FF a{0.f, 0.f};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) a = ff_add(a, dmean[i]);
    a = ff_block(a, s);
    if (threadIdx.x == 0) part[blockIdx.x] = make_float2(a.hi, a.lo);
}

// 4b. per workgroup: mu from the partial sums (every workgroup the same bits), then the
// compensated sum of (D - mu)^2 -> part2[blk]; workgroup 0 stores mu
__global__ __launch_bounds__(256) void k_ol_var(const float *__restrict__ dmean, int64_t n, const float2 *__restrict__ part,
                                                int nblk, float2 *__restrict__ part2, OlHdr *__restrict__ hdr) {
    __shared__ FF s[4][1];
    __shared__ float s_mu;
    if (threadIdx.x < 64) {
        const FF t = ff_parts(part, nblk);
        if (threadIdx.x == 0) s_mu = (t.hi + t.lo) / (float)n;
    }
    __syncthreads();
    const float mu = s_mu;
    FF a{0.f, 0.f};
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const float d = dmean[i] - mu;
        a = ff_add(a, d * d);
    }
    a = ff_block(a, s);
    if (threadIdx.x == 0) {
        part2[blockIdx.x] = make_float2(a.hi, a.lo);
        if (blockIdx.x == 0) hdr->mu = mu;
    }
}

// 4c. threshold from the summed squares (every workgroup the same bits: one wave, a fixed
// order; workgroup 0 stores it), keep mask and kept count per workgroup of kOlBlock points
__global__ __launch_bounds__(256) void k_ol_keep(const float *__restrict__ dmean, int64_t n, const float2 *__restrict__ part2,
                                                 int nblk, float std_ratio, OlHdr *__restrict__ hdr,
                                                 uint8_t *__restrict__ keep, uint32_t *__restrict__ part) {
    __shared__ uint32_t s_w[4];
    __shared__ float s_thr;
    const int64_t base = (int64_t)blockIdx.x * kOlBlock;
    float d[kOlItems];
#pragma unroll
    for (int k = 0; k < kOlItems; ++k) {
        const int64_t i = base + k * 256 + threadIdx.x;
        d[k] = i < n ? dmean[i] : 0.f;
    }
    if (threadIdx.x < 64) {
        const FF t = ff_parts(part2, nblk);
        if (threadIdx.x == 0) {
            const float sigma = sqrtf(fmaxf((t.hi + t.lo) / (float)n, 0.f));
            s_thr = hdr->mu + std_ratio * sigma;
            if (blockIdx.x == 0) {
                hdr->sigma = sigma;
                hdr->thr = s_thr;
            }
        }
    }
    __syncthreads();
    const float thr = s_thr;
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kOlItems; ++k) {
        const int64_t i = base + k * 256 + threadIdx.x;
        if (i < n) {
            const bool kp = d[k] <= thr;
            keep[i] = kp ? 1 : 0;
            c += kp ? 1u : 0u;
        }
    }
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane_id() == 0) s_w[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

// 4d. compaction of the kept points in input order: from the scanned counts, or (fold, few
// workgroups) each workgroup sums the counts before its own, and the last one stores the
// total: one launch fewer
__global__ __launch_bounds__(256) void k_ol_write(const float *__restrict__ pts, int64_t n, int64_t stride,
                                                 const uint8_t *__restrict__ keep, const uint32_t *__restrict__ part,
                                                 float *__restrict__ out, int64_t out_stride, int fold,
                                                 uint32_t *__restrict__ count) {
    __shared__ uint32_t s_w[4];
    const int64_t base = (int64_t)blockIdx.x * kOlBlock;
    const int l = (int)lane_id(), w = (int)(threadIdx.x >> 6);
    uint32_t run;
    if (fold) {
        uint32_t a = 0;
        for (uint32_t c = threadIdx.x; c < blockIdx.x; c += 256) a += part[c];
        for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
        if (l == 0) s_w[w] = a;
        __syncthreads();
        run = s_w[0] + s_w[1] + s_w[2] + s_w[3];
        __syncthreads();
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *count = run + part[blockIdx.x];
    } else {
        run = part[blockIdx.x];
    }
#pragma unroll
    for (int k = 0; k < kOlItems; ++k) {
        const int64_t i = base + k * 256 + threadIdx.x;
        const bool take = i < n && keep[i] != 0;
        const uint64_t bal = __ballot(take);
        const uint32_t below = (uint32_t)__popcll(bal & ((1ull << l) - 1ull));
        if (l == 0) s_w[w] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t before = run;
        for (int q = 0; q < w; ++q) before += s_w[q];
        const uint32_t total = s_w[0] + s_w[1] + s_w[2] + s_w[3];
        __syncthreads();
        if (take) {
            const int64_t o = (int64_t)before + below;
            out[o] = pts[i];
            out[out_stride + o] = pts[stride + i];
            out[2 * out_stride + o] = pts[2 * stride + i];
        }
        run += total;
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
int outlier_slot_bits(int64_t n) {
    int b = 12;   // at least 4 bits per axis
    while (b < 22 && ((int64_t)1 << b) < 2 * n) ++b;
    return b;
}

static size_t al(size_t x) { return (x + 255) / 256 * 256; }

// Workspace pieces for n points (offsets in bytes, in this order).
struct OlLayout {
    size_t hdr, keys0, vals0, keys1, vals1, hist, shist, scount, ranges, bpart, spart, kpart, defer, slow, spts, boxes, total;
};

size_t sort_count_words(uint64_t);

static OlLayout ol_layout(int64_t n) {
    OlLayout L;
    const size_t nn = (size_t)(n > 0 ? n : 1);
    const size_t slots = (size_t)1 << outlier_slot_bits(n);
    size_t o = 0;
    auto take = [&](size_t b) { const size_t at = o; o += al(b); return at; };
    L.hdr = take(sizeof(OlHdr));
    L.keys0 = take(4 * nn);
    L.vals0 = take(4 * nn);
    L.keys1 = take(4 * nn);
    L.vals1 = take(4 * nn);
    L.hist = take(4 * 256 * kMaxPasses);   // the sort's digit totals
    L.shist = take(4 * 3 * kOlBins);
    L.scount = take(4 * sort_count_words((uint64_t)nn));
    L.ranges = take(4 * (slots + 1));
    L.bpart = take(4 * 6 * kOlRedBlocks);
    L.spart = take(8 * 2 * kOlRedBlocks);   // two float2 partials per reduction workgroup
    L.kpart = take(4 * ((nn + kOlBlock - 1) / kOlBlock + 1));
    L.defer = take(4 * nn);
    L.slow = take(4 * nn);
    L.spts = take(16 * nn);
    L.boxes = take(32 * ((nn + kOlLeaf - 1) / kOlLeaf));
    L.total = o;
    return L;
}

size_t outlier_workspace_bytes(int64_t n) { return ol_layout(n).total; }

// slow1, slow2: the lists of the second and third search (nn words each)
template <int K>
static void knn_launch(const float *pts, int64_t n, int64_t stride, OlHdr *hdr, const float4 *spts, const float4 *boxes,
                       const uint32_t *start, uint32_t *slow1, uint32_t *slow2, uint32_t *defer, float *dmean, hipStream_t st) {
    const auto grid = [&](int lanes, int64_t most) {
        const int64_t b = (n * lanes + 255) / 256;
        return dim3((unsigned)(b < most ? b : most));
    };
    const OlSearch sr{spts, n, hdr, start, defer, dmean};
    hipLaunchKernelGGL((k_ol_knn1<K>), grid(kOlR1 * kOlC1, (int64_t)1 << 31), dim3(256), 0, st, sr, slow1);
    hipLaunchKernelGGL((k_ol_knn2<K>), grid(kOlR2 * kOlC2, kOlListBlocks), dim3(256), 0, st, sr, slow1, slow2);
    hipLaunchKernelGGL((k_ol_knn3<K>), grid(kOlR3 * kOlC3, kOlListBlocks), dim3(256), 0, st, sr, slow2);
    const unsigned far = (unsigned)(n < kOlFarBlocks ? n : kOlFarBlocks);
    hipLaunchKernelGGL((k_ol_knn_far<K>), dim3(far), dim3(kOlFarThreads), 0, st, spts, boxes, pts, n, stride, hdr, defer, dmean);
}

// k in {4, 8, 16, 32}: false (nothing launched) otherwise. out may be null (no compaction).
bool launch_outliers(const float *pts, int64_t n, int64_t stride, int k, float std_ratio, float *dmean, uint8_t *keep,
                     float *out, int64_t out_stride, uint32_t *count, void *ws, hipStream_t st) {
    if (k != 4 && k != 8 && k != 16 && k != 32) return false;
    const OlLayout L = ol_layout(n);
    char *b = (char *)ws;
    OlHdr *hdr = (OlHdr *)(b + L.hdr);
    uint32_t *k0 = (uint32_t *)(b + L.keys0), *v0 = (uint32_t *)(b + L.vals0);
    uint32_t *k1 = (uint32_t *)(b + L.keys1), *v1 = (uint32_t *)(b + L.vals1);
    uint32_t *kpart = (uint32_t *)(b + L.kpart);
    if (n == 0) {
        launch_excl_scan_u32(kpart, 0u, count, st);   // writes the count 0
        return true;
    }
    const int bits = outlier_slot_bits(n);
    const uint32_t slots = 1u << bits;
    const int rb = (int)((n + 255) / 256 < kOlRedBlocks ? (n + 255) / 256 : kOlRedBlocks);
    uint32_t *shist = (uint32_t *)(b + L.shist);
    float *bpart = (float *)(b + L.bpart);
    hipLaunchKernelGGL(k_ol_bbox, dim3(rb), dim3(256), 0, st, pts, n, stride, bpart, shist);
    const int64_t step = (n + kOlSample - 1) / kOlSample, ns = (n + step - 1) / step;
    hipLaunchKernelGGL(k_ol_hist, dim3((unsigned)((ns + 255) / 256)), dim3(256), 0, st, pts, n, stride, ns, (uint32_t)step,
                       bpart, rb, hdr, shist);
    hipLaunchKernelGGL(k_ol_setup, dim3(1), dim3(192), 0, st, shist, ns, n, (uint32_t)bits, hdr);
    hipLaunchKernelGGL(k_ol_key, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, pts, n, stride, hdr, k0, v0);
    const int alt = radix_sort_u32(k0, v0, k1, v1, (uint32_t)n, 0u, bits, (uint32_t *)(b + L.hist),
                                   (uint32_t *)(b + L.scount), st);
    const uint32_t *sk = alt ? k1 : k0, *sv = alt ? v1 : v0;
    uint32_t *start = (uint32_t *)(b + L.ranges);
    uint32_t *defer = (uint32_t *)(b + L.defer), *slow1 = (uint32_t *)(b + L.slow);
    uint32_t *slow2 = alt ? v0 : v1;   // the sort's other value buffer
    float4 *spts = (float4 *)(b + L.spts), *boxes = (float4 *)(b + L.boxes);
    const uint32_t sblk = (slots + 256u) / 256u;
    hipLaunchKernelGGL(k_ol_gather, dim3(sblk + (unsigned)((n + 255) / 256)), dim3(256), 0, st, pts, n, stride, sk, sv, slots,
                       sblk, start, spts, boxes);
    if (k == 4) knn_launch<4>(pts, n, stride, hdr, spts, boxes, start, slow1, slow2, defer, dmean, st);
    else if (k == 8) knn_launch<8>(pts, n, stride, hdr, spts, boxes, start, slow1, slow2, defer, dmean, st);
    else if (k == 16) knn_launch<16>(pts, n, stride, hdr, spts, boxes, start, slow1, slow2, defer, dmean, st);
    else knn_launch<32>(pts, n, stride, hdr, spts, boxes, start, slow1, slow2, defer, dmean, st);
    float2 *sp1 = (float2 *)(b + L.spart), *sp2 = sp1 + kOlRedBlocks;
    hipLaunchKernelGGL(k_ol_sum, dim3(rb), dim3(256), 0, st, dmean, n, sp1);
    hipLaunchKernelGGL(k_ol_var, dim3(rb), dim3(256), 0, st, dmean, n, sp1, rb, sp2, hdr);
    const uint32_t nblk = (uint32_t)((n + kOlBlock - 1) / kOlBlock);
    hipLaunchKernelGGL(k_ol_keep, dim3(nblk), dim3(256), 0, st, dmean, n, sp2, rb, std_ratio, hdr, keep, kpart);
    const int fold = out && nblk <= kOlScanFold;
    if (!fold) launch_excl_scan_u32(kpart, nblk, count, st);
    if (out)
        hipLaunchKernelGGL(k_ol_write, dim3(nblk), dim3(256), 0, st, pts, n, stride, keep, kpart, out, out_stride, fold, count);
    return true;
}

}  // namespace recogs
