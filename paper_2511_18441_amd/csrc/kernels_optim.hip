// Pieces of the background optimiser (Sec. 3.3 / 4.1): the L1 and SSIM terms of the
// loss of eq. 4 with their gradients (eq. 7), and the Adam step that moves the SH coefficients.
#include <cmath>
#include <cstring>

#include "optim_device.hpp"

namespace recogs {

void launch_fill_u32(uint32_t *p, uint32_t v, int64_t count, hipStream_t st);

// loss = scale sum |y - t| (overwritten by the caller's fill), dL/dy = scale sign(y - t)
// with sign(0) = 0. With vec (all three arrays 16-byte aligned) 4 elements per step.
__device__ __forceinline__ float sgn(float d) { return d > 0.f ? 1.f : (d < 0.f ? -1.f : 0.f); }

__global__ __launch_bounds__(1024) void k_loss_l1(const float *__restrict__ y, const float *__restrict__ tg, int64_t count,
                                                 float scale, float *__restrict__ dldy, float *__restrict__ loss, int vec) {
    __shared__ float s_w[16];
    float sum = 0.f;
    const int64_t n4 = vec ? count / 4 : 0;
    const float4 *y4 = reinterpret_cast<const float4 *>(y), *t4 = reinterpret_cast<const float4 *>(tg);
    float4 *d4 = reinterpret_cast<float4 *>(dldy);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    auto one = [&](const float4 a, const float4 b, int64_t i) {
        const float4 d = make_float4(a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w);
        d4[i] = make_float4(scale * sgn(d.x), scale * sgn(d.y), scale * sgn(d.z), scale * sgn(d.w));
        sum += fabsf(d.x) + fabsf(d.y) + fabsf(d.z) + fabsf(d.w);
    };
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + 3 * stride < n4; i += 4 * stride) {   // four groups' loads in flight
        float4 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) { a[u] = y4[i + u * stride]; b[u] = t4[i + u * stride]; }
#pragma unroll
        for (int u = 0; u < 4; ++u) one(a[u], b[u], i + u * stride);
    }
    for (; i < n4; i += stride) one(y4[i], t4[i], i);
    for (int64_t i = 4 * n4 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        const float d = y[i] - tg[i];
        dldy[i] = scale * sgn(d);
        sum += fabsf(d);
    }
    sum = wave_sum(sum);
    if (lane_id() == 0) s_w[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        float w = 0.f;
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) w += s_w[k];   // the waves' sums in order
        atomicAdd(loss, scale * w);
    }
}

void launch_loss_l1(const float *y, const float *tg, int64_t count, float scale, float *dldy, float *loss, hipStream_t st) {
    if (count <= 0) return;
    // few workgroups (of 16 waves): each adds its partial sum with one same-address atomic
    int64_t blocks = (count + 1023) / 1024;
    if (blocks > 128) blocks = 128;
    const int vec = ((reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(tg) | reinterpret_cast<uintptr_t>(dldy)) &
                     15u) == 0;
    hipLaunchKernelGGL(k_loss_l1, dim3((unsigned)blocks), dim3(1024), 0, st, y, tg, count, scale, dldy, loss, vec);
}

// Adam, element-wise: m <- b1 m + (1 - b1) g, v <- b2 v + (1 - b2) g^2,
// p <- p - lr (m / c1) / (sqrt(v / c2) + eps) with the bias corrections c1 = 1 - b1^step,
// c2 = 1 - b2^step (their reciprocals computed by the host in double precision).
__global__ __launch_bounds__(256) void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                                              float *__restrict__ v, int64_t count, AdamArgs a) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) {
        float pi = ld_stream(p + i), mi = ld_stream(m + i), vi = ld_stream(v + i);
        adam_update(pi, ld_stream(g + i), mi, vi, a);
        st_stream(m + i, mi);
        st_stream(v + i, vi);
        st_stream(p + i, pi);
    }
}

// The same update on four consecutive values per thread (16-byte loads and stores: the
// step moves 28 bytes per coefficient and is bound by HBM).
__global__ __launch_bounds__(256) void k_adam4(float4 *__restrict__ p, const float4 *__restrict__ g,
                                               float4 *__restrict__ m, float4 *__restrict__ v, int64_t count4,
                                               AdamArgs a) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count4; i += stride) {
        const float4 gi = ld_stream(g + i);
        float4 mi = ld_stream(m + i), vi = ld_stream(v + i), pi = ld_stream(p + i);
        adam_update(pi.x, gi.x, mi.x, vi.x, a);
        adam_update(pi.y, gi.y, mi.y, vi.y, a);
        adam_update(pi.z, gi.z, mi.z, vi.z, a);
        adam_update(pi.w, gi.w, mi.w, vi.w, a);
        st_stream(m + i, mi);
        st_stream(v + i, vi);
        st_stream(p + i, pi);
    }
}

void launch_adam(float *p, const float *g, float *m, float *v, int64_t count, float lr, float b1, float b2, float eps,
                 float ic1, float ic2, hipStream_t st) {
    if (count <= 0) return;
    const AdamArgs a{lr, b1, b2, eps, ic1, ic2};
    const bool vec = ((reinterpret_cast<uintptr_t>(p) | reinterpret_cast<uintptr_t>(g) | reinterpret_cast<uintptr_t>(m) |
                       reinterpret_cast<uintptr_t>(v)) & 15u) == 0;
    int64_t done = 0;
    if (vec && count >= 4) {
        const int64_t c4 = count / 4;
        int64_t blocks = (c4 + 255) / 256;
        if (blocks > 8192) blocks = 8192;
        hipLaunchKernelGGL(k_adam4, dim3((unsigned)blocks), dim3(256), 0, st, (float4 *)p, (const float4 *)g, (float4 *)m,
                           (float4 *)v, c4, a);
        done = 4 * c4;
    }
    const int64_t rest = count - done;
    if (rest <= 0) return;
    int64_t blocks = (rest + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(k_adam, dim3((unsigned)blocks), dim3(256), 0, st, p + done, g + done, m + done, v + done, rest, a);
}

// ---------------------------------------------------------------------------
// SSIM term of eq. 4 over HWC float images, per channel, with the 11 x 11 Gaussian
// window (sigma 1.5, zero outside the image): local means, variances and covariance
// are separable blurs; S = (2 mu_y mu_t + C1)(2 s_yt + C2) / ((mu_y^2 + mu_t^2 + C1)
// (s_y^2 + s_t^2 + C2)). Its gradient: S depends on y through mu_y = G*y, E_yy = G*(y^2)
// and E_yt = G*(y t), so dS/dy = G*a + 2 y (G*b) + t (G*c) with a, b, c the partial
// derivatives of S in those maps. Two passes:
//   k_ssim_fwd: the three maps a, b, c per value and each workgroup's sum of S;
//   k_ssim_bwd: the blurs of a, b, c and the gradient; its first workgroup first adds
//               the workgroups' sums in a fixed order (the loss).
// Bound by the vector units (about 140 operations per value in the forward, 80 in the
// backward) and by LDS reads beside them. The three channels are one image of 3 W floats
// per row whose x taps are 3 apart, so every access is a run of consecutive floats (the
// maps are stored the same way). A workgroup takes 64 pixels x 8 rows: each thread first
// blurs one column (of 222: the tile's 192 floats and 15 on either side) down the rows
// from registers, straight from memory (18 rows for 8: the halo costs loads only), then
// the blurred rows go through LDS, one 16-byte read per tap for all the blurred
// quantities, for the blur along x. S needs s_y^2 + s_t^2 only as a sum, so four
// quantities are blurred (y, t, (y - t)^2, y t): with l1 and c1 the two factors of S's
// numerator and m = mu_y - mu_t, the denominator's are l1 + m^2 and c1 + G*(y - t)^2 - m^2.
// Where the images agree the additions are zero and S is 1 to the rounding of three
// products, as with five blurred quantities; from y^2 + t^2, whose blur is rounded apart
// from that of 2 y t, the loss of equal flat images was off by up to 1.3e-5, and the
// gradient's error against 64 bits at 1920x1080 was 4.1e-6 for 3.4e-6, in the same time.
// Tiles are numbered so that one XCD's
// workgroups take a band of rows, whose halos then meet in its L2. Both passes at
// 1920x1080: 150 -> 69 us against a workgroup per 16 x 16 tile and channel, blurred
// along x first with one output and 77 LDS reads per thread (at 1280x720: 78 -> 42 us).
// ---------------------------------------------------------------------------
namespace {
constexpr int kSsimR = 5;                     // window radius (11 taps)
constexpr int kSsimTaps = 2 * kSsimR + 1;
constexpr int kSsimPx = 64;                   // pixels of a workgroup's tile along x
constexpr int kSsimCols = 3 * kSsimPx;        // its floats along x
constexpr int kSsimExt = kSsimCols + 6 * kSsimR;   // with the halo (222 <= 256 threads)
constexpr int kSsimRows = 8;                  // its rows
constexpr int kSsimIn = kSsimRows + 2 * kSsimR;    // rows read
constexpr int kSsimRounds = kSsimCols * kSsimRows / 256;   // values per thread of the blur along x
static_assert(kSsimExt <= 256 && kSsimCols * kSsimRows % 256 == 0, "one thread per column, whole rounds along x");
constexpr float kSsimC1 = 0.01f * 0.01f, kSsimC2 = 0.03f * 0.03f;
}  // namespace

struct SsimWindow { float g[kSsimTaps]; };
// the order of a blur's taps: the outer, small weights first, so that the running sum (and
// its rounding) stays small until the last few
__device__ constexpr int ssim_tap(int i) { return i & 1 ? kSsimTaps - 1 - i / 2 : i / 2; }

// tile (tx, ty) of workgroup b of a grid of 8 * per workgroups (workgroup b runs on XCD
// b mod 8, which takes tiles [per x, per x + per) in row order); false past the last tile
__device__ __forceinline__ bool ssim_tile(uint32_t b, uint32_t per, uint32_t gx, uint32_t tiles, uint32_t &tile, int &px0,
                                          int &row0) {
    tile = (b & 7u) * per + (b >> 3);
    if (tile >= tiles) return false;
    px0 = (int)(tile % gx) * kSsimPx;
    row0 = (int)(tile / gx) * kSsimRows;
    return true;
}

// part_l1 (optional): also the tile's sum of |y - t| (the L1 term)
__global__ __launch_bounds__(256) void k_ssim_fwd(const float *__restrict__ y, const float *__restrict__ t, int W, int H,
                                                  SsimWindow win, float *__restrict__ maps, float *__restrict__ part,
                                                  float *__restrict__ part_l1, uint32_t gx, uint32_t tiles, uint32_t per) {
    __shared__ float4 s_v[kSsimRows][kSsimExt];   // blurred along y: y, t, (y - t)^2, y t
    __shared__ float s_w[4], s_w1[4];
    uint32_t tile;
    int px0, row0;
    if (!ssim_tile(blockIdx.x, per, gx, tiles, tile, px0, row0)) return;
    const int tid = (int)threadIdx.x;
    const int64_t RW = 3 * (int64_t)W, HW3 = RW * H;
    float asum = 0.f, ssum = 0.f;
    if (tid < kSsimExt) {
        const int64_t e = 3 * (int64_t)px0 - 3 * kSsimR + tid;
        const bool col = e >= 0 && e < RW;
        float u[kSsimIn], v[kSsimIn];
#pragma unroll
        for (int r = 0; r < kSsimIn; ++r) {   // (every load unconditional: value 0 stands in outside)
            const int yy = row0 + r - kSsimR;
            const int64_t q = col && yy >= 0 && yy < H ? yy * RW + e : 0;
            u[r] = y[q];
            v[r] = t[q];
        }
#pragma unroll
        for (int r = 0; r < kSsimIn; ++r) {   // zero outside the image
            const int yy = row0 + r - kSsimR;
            const bool in = col && yy >= 0 && yy < H;
            u[r] = in ? u[r] : 0.f;
            v[r] = in ? v[r] : 0.f;
        }
        if (part_l1 && tid >= 3 * kSsimR && tid < 3 * kSsimR + kSsimCols) {
#pragma unroll
            for (int o = 0; o < kSsimRows; ++o) asum += fabsf(u[o + kSsimR] - v[o + kSsimR]);   // 0 outside
        }
        float d2[kSsimIn], p[kSsimIn];
#pragma unroll
        for (int r = 0; r < kSsimIn; ++r) {
            d2[r] = (u[r] - v[r]) * (u[r] - v[r]);
            p[r] = u[r] * v[r];
        }
#pragma unroll
        for (int o = 0; o < kSsimRows; ++o) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < kSsimTaps; ++i) {
                const int j = ssim_tap(i);
                const float g = win.g[j];
                a.x += g * u[o + j]; a.y += g * v[o + j]; a.z += g * d2[o + j]; a.w += g * p[o + j];
            }
            s_v[o][tid] = a;
        }
    }
    __syncthreads();
#pragma unroll 2
    for (int i = 0; i < kSsimRounds; ++i) {
        const int k = tid + 256 * i, o = k / kSsimCols, x = k % kSsimCols;
        const int64_t e = 3 * (int64_t)px0 + x;
        const int yy = row0 + o;
        float my = 0.f, mt = 0.f, ed = 0.f, eyt = 0.f;
#pragma unroll
        for (int n = 0; n < kSsimTaps; ++n) {
            const int j = ssim_tap(n);
            const float4 a = s_v[o][x + 3 * j];
            const float g = win.g[j];
            my += g * a.x; mt += g * a.y; ed += g * a.z; eyt += g * a.w;
        }
        if (e < RW && yy < H) {
            const float syt = __builtin_fmaf(-my, mt, eyt), m = my - mt;
            const float l1 = 2.f * my * mt + kSsimC1, l2 = __builtin_fmaf(m, m, l1);
            const float c1 = 2.f * syt + kSsimC2, c2 = c1 + __builtin_fmaf(-m, m, ed);
            // 1 / (l2 c2): the hardware reciprocal and one Newton step (kept out where it
            // is not finite: den zero or infinite)
            const float den = l2 * c2, rc = __builtin_amdgcn_rcpf(den);
            const float nr = __builtin_fmaf(__builtin_fmaf(-den, rc, 1.f), rc, rc);
            const float inv = __builtin_isfinite(nr) ? nr : rc;
            const float S = l1 * c1 * inv;
            const float dS_dsyt = 2.f * l1 * inv;
            const float dS_dsyy = -S * (l2 * inv);
            const float dS_dmy = 2.f * mt * c1 * inv - S * 2.f * my * (c2 * inv);
            const int64_t q = yy * RW + e;
            maps[q] = dS_dmy - 2.f * my * dS_dsyy - mt * dS_dsyt;   // a
            maps[HW3 + q] = dS_dsyy;                                // b
            maps[2 * HW3 + q] = dS_dsyt;                            // c
            ssum += S;
        }
    }
    ssum = wave_sum(ssum);
    if (lane_id() == 0) s_w[tid >> 6] = ssum;
    if (part_l1) {
        asum = wave_sum(asum);
        if (lane_id() == 0) s_w1[tid >> 6] = asum;
    }
    __syncthreads();
    // the workgroup's sums, added to the others in a fixed order by the backward
    if (tid == 0) part[tile] = ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
    if (part_l1 && tid == 0) part_l1[tile] = ((s_w1[0] + s_w1[1]) + s_w1[2]) + s_w1[3];
}

// The n partial sums added in a fixed order by one workgroup (thread t: entries t,
// t + 256, ... in turn, then the waves' sums in order): the same bits on every run.
// Eight loads in flight per thread. The total is returned to thread 0.
__device__ __forceinline__ float fixed_order_sum(const float *__restrict__ part, uint32_t n, float *s_w /* [4] */) {
    float acc = 0.f;
    for (uint32_t k0 = threadIdx.x; k0 < n; k0 += 256u * 8u) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = k0 + 256u * i < n ? part[k0 + 256u * i] : 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (k0 + 256u * i < n) acc += v[i];
    }
    acc = wave_sum(acc);
    if (lane_id() == 0) s_w[threadIdx.x >> 6] = acc;
    __syncthreads();
    return ((s_w[0] + s_w[1]) + s_w[2]) + s_w[3];
}

// One gradient value from its SSIM term d: after the L1 term (l1_scale sign(diff)), or the
// stored value with accumulate, in this order and with no fused multiply-add, so that both
// terms in one call have the bits of the two calls.
__device__ __forceinline__ float ssim_grad(float d, bool with_l1, float l1_scale, float diff, int accumulate, const float *prev) {
#pragma clang fp contract(off)
    if (with_l1) d = l1_scale * sgn(diff) + d;
    return accumulate ? *prev + d : d;
}

// part / nparts / weight / loss: the loss weight + gscale (sum of S), plus l1_scale (sum
// of |y - t|) with part_l1, summed by workgroup 0 before its tile. With part_l1 the
// gradient also takes l1_scale sign(y - t), added before the SSIM term is (the bits of
// the L1 gradient written first and the SSIM gradient added to it).
__global__ __launch_bounds__(256) void k_ssim_bwd(const float *__restrict__ y, const float *__restrict__ t, int W, int H,
                                                  SsimWindow win, const float *__restrict__ maps, float gscale,
                                                  int accumulate, float *__restrict__ dldy, const float *__restrict__ part,
                                                  uint32_t nparts, float weight, float *__restrict__ loss,
                                                  const float *__restrict__ part_l1, float l1_scale, uint32_t gx,
                                                  uint32_t tiles, uint32_t per) {
    __shared__ float2 s_ab[kSsimRows][kSsimExt];   // a, b blurred along y
    __shared__ float s_c[kSsimRows][kSsimExt];     // c
    __shared__ float s_lw[4], s_lw1[4];
    const int tid = (int)threadIdx.x;
    if (blockIdx.x == 0) {
        const float ss = fixed_order_sum(part, nparts, s_lw);
        if (part_l1) {
            const float sa = fixed_order_sum(part_l1, nparts, s_lw1);
            if (tid == 0) *loss = (weight + gscale * ss) + l1_scale * sa;
        } else if (tid == 0) {
            *loss = weight + gscale * ss;
        }
    }
    uint32_t tile;
    int px0, row0;
    if (!ssim_tile(blockIdx.x, per, gx, tiles, tile, px0, row0)) return;
    const int64_t RW = 3 * (int64_t)W, HW3 = RW * H;
    if (tid < kSsimExt) {
        const int64_t e = 3 * (int64_t)px0 - 3 * kSsimR + tid;
        const bool col = e >= 0 && e < RW;
        float m[3][kSsimIn];
#pragma unroll
        for (int r = 0; r < kSsimIn; ++r) {
            const int yy = row0 + r - kSsimR;
            const int64_t q = col && yy >= 0 && yy < H ? yy * RW + e : 0;
#pragma unroll
            for (int k = 0; k < 3; ++k) m[k][r] = maps[k * HW3 + q];
        }
#pragma unroll
        for (int r = 0; r < kSsimIn; ++r) {
            const int yy = row0 + r - kSsimR;
            const bool in = col && yy >= 0 && yy < H;
#pragma unroll
            for (int k = 0; k < 3; ++k) m[k][r] = in ? m[k][r] : 0.f;
        }
#pragma unroll
        for (int o = 0; o < kSsimRows; ++o) {
            float a = 0.f, b = 0.f, c = 0.f;
#pragma unroll
            for (int i = 0; i < kSsimTaps; ++i) {
                const int j = ssim_tap(i);
                const float g = win.g[j];
                a += g * m[0][o + j]; b += g * m[1][o + j]; c += g * m[2][o + j];
            }
            s_ab[o][tid] = make_float2(a, b);
            s_c[o][tid] = c;
        }
    }
    __syncthreads();
#pragma unroll 2
    for (int i = 0; i < kSsimRounds; ++i) {
        const int k = tid + 256 * i, o = k / kSsimCols, x = k % kSsimCols;
        const int64_t e = 3 * (int64_t)px0 + x;
        const int yy = row0 + o;
        const bool in = e < RW && yy < H;
        const int64_t q = in ? yy * RW + e : 0;
        const float yp = in ? y[q] : 0.f, tp = in ? t[q] : 0.f;
        float ga = 0.f, gb = 0.f, gc = 0.f;
#pragma unroll
        for (int n = 0; n < kSsimTaps; ++n) {
            const int j = ssim_tap(n);
            const float2 ab = s_ab[o][x + 3 * j];
            const float g = win.g[j];
            ga += g * ab.x; gb += g * ab.y; gc += g * s_c[o][x + 3 * j];
        }
        if (in) dldy[q] = ssim_grad(gscale * (ga + 2.f * yp * gb + tp * gc), part_l1 != nullptr, l1_scale, yp - tp, accumulate,
                                    dldy + q);
    }
}

// Scratch floats of the SSIM term: 9 per pixel (the maps), then 6 per 16 x 16 tile of the
// image, which hold the workgroups' partial sums of S and of |y - t|: two per 64 x 8 tile
// (at most two such tiles per 16 x 16 one, where the image is narrow).
size_t dssim_scratch_floats(int W, int H) {
    if (W <= 0 || H <= 0) return 0;
    const size_t tiles = (size_t)((W + 15) / 16) * (size_t)((H + 15) / 16);
    return (size_t)9 * (size_t)W * (size_t)H + 6 * tiles;
}

// maps: dssim_scratch_floats(W, H) floats of scratch. loss <- weight (1 - mean S); dL/dy
// (=, or += with accumulate) -weight dS/dy averaged over 3 H W values.
// with_l1: also the L1 term, l1_scale sum |y - t| and its gradient (eq. 4 and eq. 7 in one pass)
void launch_dssim(const float *y, const float *t, int W, int H, float weight, float *dldy, int accumulate, float *loss,
                  float *maps, hipStream_t st, int with_l1, float l1_scale) {
    SsimWindow win;
    double g[2 * kSsimR + 1], sum = 0.0;
    for (int j = 0; j <= 2 * kSsimR; ++j) {
        const double r = j - kSsimR;
        g[j] = std::exp(-(r * r) / (2.0 * 1.5 * 1.5));
        sum += g[j];
    }
    for (int j = 0; j <= 2 * kSsimR; ++j) win.g[j] = (float)(g[j] / sum);
    if (W <= 0 || H <= 0) {   // no pixels: weight (1 - SSIM) with SSIM taken as 0
        uint32_t wbits;
        std::memcpy(&wbits, &weight, 4);
        launch_fill_u32(reinterpret_cast<uint32_t *>(loss), wbits, 1, st);
        return;
    }
    const double N = 3.0 * (double)W * (double)H;
    const uint32_t gx = (uint32_t)((W + kSsimPx - 1) / kSsimPx), gy = (uint32_t)((H + kSsimRows - 1) / kSsimRows);
    const uint32_t tiles = gx * gy, per = (tiles + 7u) / 8u;
    float *part = maps + (size_t)9 * (size_t)W * (size_t)H;
    float *part_l1 = with_l1 ? part + tiles : nullptr;
    hipLaunchKernelGGL(k_ssim_fwd, dim3(8u * per), dim3(256), 0, st, y, t, W, H, win, maps, part, part_l1, gx, tiles, per);
    hipLaunchKernelGGL(k_ssim_bwd, dim3(8u * per), dim3(256), 0, st, y, t, W, H, win, maps, (float)(-weight / N), accumulate,
                       dldy, part, tiles, weight, loss, part_l1, l1_scale, gx, tiles, per);
}

}  // namespace recogs
