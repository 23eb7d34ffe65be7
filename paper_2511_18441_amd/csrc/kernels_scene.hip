// Per-Gaussian streaming kernels: covariance (eq. 1), selection, recolour (eq. 6).
// One thread per Gaussian, planar (SoA) loads: consecutive lanes read consecutive
// elements of each plane.
#include "recogs_internal.hpp"

namespace recogs {

void launch_fill_u32(uint32_t *p, uint32_t v, int64_t count, hipStream_t st);

// eq. (1): Sigma = R S S^T R^T, S = diag(exp(log_scale)), R from the normalised
// quaternion (w, x, y, z).
__global__ __launch_bounds__(256) void k_covariance(const float *__restrict__ ls, const float *__restrict__ q,
                                                    float *__restrict__ cov, int64_t n, int64_t stride) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float w = q[i], x = q[stride + i], y = q[2 * stride + i], z = q[3 * stride + i];
    const float inv = 1.0f / sqrtf(w * w + x * x + y * y + z * z);
    w *= inv; x *= inv; y *= inv; z *= inv;
    const float R00 = 1.f - 2.f * (y * y + z * z), R01 = 2.f * (x * y - w * z), R02 = 2.f * (x * z + w * y);
    const float R10 = 2.f * (x * y + w * z), R11 = 1.f - 2.f * (x * x + z * z), R12 = 2.f * (y * z - w * x);
    const float R20 = 2.f * (x * z - w * y), R21 = 2.f * (y * z + w * x), R22 = 1.f - 2.f * (x * x + y * y);
    const float s0 = expf(ls[i]), s1 = expf(ls[stride + i]), s2 = expf(ls[2 * stride + i]);
    const float M00 = R00 * s0, M01 = R01 * s1, M02 = R02 * s2;
    const float M10 = R10 * s0, M11 = R11 * s1, M12 = R12 * s2;
    const float M20 = R20 * s0, M21 = R21 * s1, M22 = R22 * s2;
    cov[i] = M00 * M00 + M01 * M01 + M02 * M02;
    cov[stride + i] = M00 * M10 + M01 * M11 + M02 * M12;
    cov[2 * stride + i] = M00 * M20 + M01 * M21 + M02 * M22;
    cov[3 * stride + i] = M10 * M10 + M11 * M11 + M12 * M12;
    cov[4 * stride + i] = M10 * M20 + M11 * M21 + M12 * M22;
    cov[5 * stride + i] = M20 * M20 + M21 * M21 + M22 * M22;
}

// Selection: depth > znear, projected centre in the closed disk, DC colour in the
// closed ball. Bound by HBM (12 bytes of position, three coefficients and a mask byte per
// Gaussian); a thread takes VEC consecutive Gaussians (4 where every plane is 16-byte
// aligned: 16-byte position loads and one 4-byte mask store; 1 otherwise), and its
// coefficient loads go out with the position loads, not behind the near-plane test: 31 ->
// 21 us at 3M Gaussians in f16 (57 MB). The count is reduced per workgroup (wave ballots,
// then LDS) and added with one atomic per workgroup: same-address device atomics are
// serialised far from the CU, so a grid-stride loop over at most kSelectBlocks workgroups
// bounds them. SOLO (one workgroup, up to kSelectSolo Gaussians): the workgroup stores
// the count itself, so no launch has to zero it first (one of the two launches is the
// larger part of such a call). Where the lines lie, us per call and, of calls in a graph, on
// the GPU: one workgroup against several, 2,048 Gaussians 7.4 and 4.0 against 9.9 and 5.1,
// 4,096 7.2 and 5.1 against 10.1 and 5.2, 8,192 8.1 and 8.2 against 10.1 and 5.2 (it makes
// several rounds), 16,384 14.1 against 10.2; VEC 4 against 1 on the GPU, several workgroups,
// 8,192 Gaussians 5.2 against 4.5 (too few waves), 32,768 5.4 both, 65,536 5.7 against 6.8.
constexpr unsigned kSelectBlocks = 1024;
constexpr int64_t kSelectSolo = 4096, kSelectVec = 32768;

template <typename T, int VEC> struct Pack { T v[VEC]; };
template <typename T, int VEC> __device__ __forceinline__ Pack<T, VEC> ld_pack(const T *p) {
    typedef T vec_t __attribute__((ext_vector_type(VEC)));
    Pack<T, VEC> r;
    if constexpr (VEC == 1) {
        r.v[0] = *p;
    } else {
        const vec_t x = *reinterpret_cast<const vec_t *>(p);
#pragma unroll
        for (int k = 0; k < VEC; ++k) r.v[k] = x[k];
    }
    return r;
}
template <int DT> struct Raw { typedef uint16_t T; };
template <> struct Raw<RECOGS_F32> { typedef float T; };

template <int DT, int VEC, int NT, bool SOLO>
__global__ __launch_bounds__(NT) void k_select(SceneDev sc, CamDev cam, float scx, float scy, float r2,
                                               float ref0, float ref1, float ref2, float rho2,
                                               uint8_t *__restrict__ mask, int32_t *__restrict__ count) {
    __shared__ uint32_t s_cnt[NT / 64];
    typedef typename Raw<DT>::T raw;
    uint32_t wave_cnt = 0;
    for (int64_t g0 = (int64_t)blockIdx.x * NT * VEC; g0 < sc.n; g0 += (int64_t)gridDim.x * NT * VEC) {
        const int64_t i = g0 + (int64_t)threadIdx.x * VEC;
        uint32_t sel = 0;   // bit k: Gaussian i + k selected
        auto test = [&](float mx, float my, float mz, float d0, float d1, float d2c) {
            const float z = dot3c(cam.R[6], mx, cam.R[7], my, cam.R[8], mz, cam.t[2]);
            const float x = dot3c(cam.R[0], mx, cam.R[1], my, cam.R[2], mz, cam.t[0]);
            const float y = dot3c(cam.R[3], mx, cam.R[4], my, cam.R[5], mz, cam.t[1]);
            const float u = cam.fx * (x / z) + cam.cx, v = cam.fy * (y / z) + cam.cy;
            const float du = u - scx, dv = v - scy;
            const float d2 = du * du + dv * dv;
            const float c0 = kSH0 * d0 + 0.5f - ref0;
            const float c1 = kSH0 * d1 + 0.5f - ref1;
            const float c2 = kSH0 * d2c + 0.5f - ref2;
            return (z > cam.znear) && (d2 <= r2) && (c0 * c0 + c1 * c1 + c2 * c2 <= rho2);
        };
        if (i + VEC <= sc.n) {
            Pack<float, VEC> m[3];
            Pack<raw, VEC> c[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) m[a] = ld_pack<float, VEC>(sc.means + a * sc.stride + i);
#pragma unroll
            for (int a = 0; a < 3; ++a) c[a] = ld_pack<raw, VEC>((const raw *)sc.sh + a * sc.stride + i);
            uint32_t bytes = 0;
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                const bool t = test(m[0].v[k], m[1].v[k], m[2].v[k], Store<DT>::ldc(&c[0].v[k], 0),
                                    Store<DT>::ldc(&c[1].v[k], 0), Store<DT>::ldc(&c[2].v[k], 0));
                sel |= (t ? 1u : 0u) << k;
                bytes |= (t ? 1u : 0u) << (8 * k);
            }
            if constexpr (VEC == 4) *reinterpret_cast<uint32_t *>(mask + i) = bytes;
            else mask[i] = (uint8_t)bytes;
        } else {
            for (int k = 0; k < VEC && i + k < sc.n; ++k) {
                const int64_t j = i + k;
                const bool t = test(sc.means[j], sc.means[sc.stride + j], sc.means[2 * sc.stride + j], Store<DT>::ldc(sc.sh, j),
                                    Store<DT>::ldc(sc.sh, sc.stride + j), Store<DT>::ldc(sc.sh, 2 * sc.stride + j));
                sel |= (t ? 1u : 0u) << k;
                mask[j] = t ? 1 : 0;
            }
        }
#pragma unroll
        for (int k = 0; k < VEC; ++k) wave_cnt += (uint32_t)__popcll(wave_ballot((sel >> k) & 1u));
    }
    if (lane_id() == 0) s_cnt[threadIdx.x >> 6] = wave_cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) c += s_cnt[w];
        if constexpr (SOLO) *count = (int32_t)c;
        else if (c) atomicAdd(count, (int32_t)c);
    }
}

// Recolour on coefficients: C'_k = M C_k (k >= 1), C'_0 = M C_0 + ((M - I) 1/2 + b)/Y00.
// A thread reads the mask bytes of four consecutive Gaussians with one load.
constexpr int kRecolorPer = 4;
// One recoloured value, held in a float32 register before it is stored: the compiler may
// otherwise fold the conversion to f16 into the last multiply-add (one rounding instead
// of two) in one of the kernels that share this and not in the other.
__device__ __forceinline__ float recolor_value(const float *M, int r, float c0, float c1, float c2, bool dc, float off) {
    float v = M[r * 3] * c0 + M[r * 3 + 1] * c1 + M[r * 3 + 2] * c2;
    if (dc) v += off;
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ float recolor_offset(const float *M, const float *bb, int r) {
    return ((M[r * 3] + M[r * 3 + 1] + M[r * 3 + 2] - 1.0f) * 0.5f + bb[r]) / kSH0;
}
template <int DT>
__global__ __launch_bounds__(256) void k_recolor(SceneDev sc, int ncoef, void *__restrict__ dst,
                                                 const uint8_t *__restrict__ mask, const float *__restrict__ Mp,
                                                 const float *__restrict__ bp) {
    const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * kRecolorPer;
    // the matrix and offset (uniform) are loaded with the mask, not after it
    float M[9], bb[3];
#pragma unroll
    for (int k = 0; k < 9; ++k) M[k] = Mp[k];
#pragma unroll
    for (int r = 0; r < 3; ++r) bb[r] = bp[r];
    uint32_t sel = 0;   // byte k: Gaussian i0 + k selected
    if (i0 + kRecolorPer <= sc.n && ((uintptr_t)mask & 3u) == 0) {
        sel = *reinterpret_cast<const uint32_t *>(mask + i0);
    } else {
        for (int k = 0; k < kRecolorPer; ++k)
            if (i0 + k < sc.n && mask[i0 + k]) sel |= 1u << (8 * k);
    }
    // The selected Gaussians of the wave (a sparse selection leaves one or two per wave)
    // are listed in index order in LDS; then each group of 16 lanes recolours one of them,
    // four at a time: lane k of a group takes coefficient k's three planes, so a Gaussian
    // costs three loads and three stores of up to 16 lanes each, and a wave's Gaussians
    // cost one memory round trip per four instead of one each. A lane loads its planes
    // before it stores them, so the destination may alias the source.
    __shared__ uint16_t s_list[4][64 * kRecolorPer];
    const uint64_t m = wave_ballot(sel != 0u);
    if (!m) return;
    const int l = (int)lane_id(), w = (int)(threadIdx.x >> 6);
    const uint32_t nsel_l = ((sel & 0xffu) ? 1u : 0u) + ((sel >> 8 & 0xffu) ? 1u : 0u) +
                            ((sel >> 16 & 0xffu) ? 1u : 0u) + ((sel >> 24) ? 1u : 0u);   // selected of the lane
    const uint32_t incl = wave_incl_scan(nsel_l);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    {
        uint32_t pos = incl - nsel_l;
#pragma unroll
        for (int k = 0; k < kRecolorPer; ++k)
            if ((sel >> (8 * k)) & 0xffu) s_list[w][pos++] = (uint16_t)(l * kRecolorPer + k);
    }
    wave_sync();   // the list written before any lane reads it
    float off[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) off[r] = recolor_offset(M, bb, r);
    const int64_t wbase = i0 - (int64_t)l * kRecolorPer;   // the first Gaussian of lane 0
    const int grp = l >> 4, co = l & 15;
    for (uint32_t j0 = 0; j0 < total; j0 += 4) {
        const uint32_t j = j0 + (uint32_t)grp;
        if (j < total && co < ncoef) {
            const int64_t g = wbase + (int64_t)s_list[w][j];
            const float c0 = Store<DT>::ldc(sc.sh, (int64_t)(3 * co) * sc.stride + g);
            const float c1 = Store<DT>::ldc(sc.sh, (int64_t)(3 * co + 1) * sc.stride + g);
            const float c2 = Store<DT>::ldc(sc.sh, (int64_t)(3 * co + 2) * sc.stride + g);
#pragma unroll
            for (int r = 0; r < 3; ++r)
                Store<DT>::st(dst, (int64_t)(3 * co + r) * sc.stride + g, recolor_value(M, r, c0, c1, c2, co == 0, off[r]));
        }
    }
}

// Recolour into a whole copy (copy_unselected with a destination of its own): every
// coefficient is read and written once, so the pass is bound by HBM. A thread streams VEC
// consecutive Gaussians (16 bytes of a plane where every plane is 16-byte aligned, one
// element otherwise) of kCopyCoefs coefficients' three planes each, unselected ones as
// their stored bits; the coefficient groups are the grid's y, so small scenes fill the GPU
// too. 3M Gaussians of degree 3 in f16 (576 MB): 622 -> 100 us (5.8 TB/s) against four
// Gaussians per lane, element by element.
constexpr int kCopyCoefs = 4;
template <int DT, int VEC>
__global__ __launch_bounds__(256) void k_recolor_copy(SceneDev sc, int ncoef, void *__restrict__ dst,
                                                      const uint8_t *__restrict__ mask, const float *__restrict__ Mp,
                                                      const float *__restrict__ bp) {
    typedef typename Raw<DT>::T raw;
    typedef raw vec_t __attribute__((ext_vector_type(VEC)));
    const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * VEC;
    if (i0 >= sc.n) return;
    float M[9], bb[3];
#pragma unroll
    for (int k = 0; k < 9; ++k) M[k] = Mp[k];
#pragma unroll
    for (int r = 0; r < 3; ++r) bb[r] = bp[r];
    const raw *src = (const raw *)sc.sh;
    raw *out = (raw *)dst;
    const int k0 = (int)blockIdx.y * kCopyCoefs, k1 = min(ncoef, k0 + kCopyCoefs);
    float off[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) off[r] = recolor_offset(M, bb, r);
    auto one = [&](int co, raw (&c)[3]) {   // a selected Gaussian's three values, as k_recolor
        const float c0 = Store<DT>::ldc(&c[0], 0), c1 = Store<DT>::ldc(&c[1], 0), c2 = Store<DT>::ldc(&c[2], 0);
#pragma unroll
        for (int r = 0; r < 3; ++r) Store<DT>::st(&c[r], 0, recolor_value(M, r, c0, c1, c2, co == 0, off[r]));
    };
    if (i0 + VEC <= sc.n) {
        uint32_t sel = 0;   // bit j: Gaussian i0 + j selected
#pragma unroll
        for (int j = 0; j < VEC; ++j) sel |= (mask[i0 + j] ? 1u : 0u) << j;
        vec_t x[kCopyCoefs][3];
#pragma unroll
        for (int q = 0; q < kCopyCoefs; ++q)
            if (k0 + q < k1)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    x[q][c] = __builtin_nontemporal_load(
                        reinterpret_cast<const vec_t *>(src + (int64_t)(3 * (k0 + q) + c) * sc.stride + i0));
#pragma unroll
        for (int q = 0; q < kCopyCoefs; ++q)
            if (k0 + q < k1) {
                if (sel) {
#pragma unroll
                    for (int j = 0; j < VEC; ++j)
                        if ((sel >> j) & 1u) {
                            raw c[3] = {x[q][0][j], x[q][1][j], x[q][2][j]};
                            one(k0 + q, c);
                            x[q][0][j] = c[0]; x[q][1][j] = c[1]; x[q][2][j] = c[2];
                        }
                }
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    __builtin_nontemporal_store(
                        x[q][c], reinterpret_cast<vec_t *>(out + (int64_t)(3 * (k0 + q) + c) * sc.stride + i0));
            }
    } else {
        for (int64_t i = i0; i < sc.n; ++i)
            for (int k = k0; k < k1; ++k) {
                raw c[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) c[a] = src[(int64_t)(3 * k + a) * sc.stride + i];
                if (mask[i]) one(k, c);
#pragma unroll
                for (int a = 0; a < 3; ++a) out[(int64_t)(3 * k + a) * sc.stride + i] = c[a];
            }
    }
}

// ---------------------------------------------------------------------------
// host launchers
// ---------------------------------------------------------------------------
void launch_covariance(const float *ls, const float *q, float *cov, int64_t n, int64_t stride, hipStream_t st) {
    if (n <= 0) return;
    hipLaunchKernelGGL(k_covariance, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, ls, q, cov, n, stride);
}

// whether planes of `bytes`-byte elements at p with this stride start on 16-byte lines of
// VEC-element groups
static bool planes_aligned(const void *p, int64_t stride, int bytes, int align) {
    return (reinterpret_cast<uintptr_t>(p) % (uintptr_t)align) == 0 && (stride * bytes) % align == 0;
}

template <int DT, int VEC>
static void select_dt(const SceneDev &sc, const CamDev &cam, const recogs_select_params &p, uint8_t *mask, int32_t *count,
                      hipStream_t st) {
    const float r2 = p.radius * p.radius, rho2 = p.color_radius * p.color_radius;
    if (sc.n <= kSelectSolo) {
        hipLaunchKernelGGL((k_select<DT, VEC, 1024, true>), dim3(1), dim3(1024), 0, st, sc, cam, p.cx, p.cy, r2, p.ref[0],
                           p.ref[1], p.ref[2], rho2, mask, count);
        return;
    }
    launch_fill_u32((uint32_t *)count, 0u, 1, st);
    const int64_t need = (sc.n + 256 * VEC - 1) / (256 * VEC);
    hipLaunchKernelGGL((k_select<DT, VEC, 256, false>), dim3((unsigned)(need < kSelectBlocks ? need : kSelectBlocks)), dim3(256),
                       0, st, sc, cam, p.cx, p.cy, r2, p.ref[0], p.ref[1], p.ref[2], rho2, mask, count);
}

// mask [n] and *count are written (the count 0 for an empty scene)
void launch_select(int dt, const SceneDev &sc, const CamDev &cam, const recogs_select_params &p, uint8_t *mask,
                   int32_t *count, hipStream_t st) {
    if (sc.n <= 0) {
        launch_fill_u32((uint32_t *)count, 0u, 1, st);
        return;
    }
    const int eb = dt == RECOGS_F32 ? 4 : 2;
    const bool vec = (sc.n <= kSelectSolo || sc.n >= kSelectVec) && planes_aligned(sc.means, sc.stride, 4, 16) &&
                     planes_aligned(sc.sh, sc.stride, eb, 4 * eb) && planes_aligned(mask, 0, 1, 4);
#define RECOGS_SELECT(DT)                                                     \
    if (vec) select_dt<DT, 4>(sc, cam, p, mask, count, st);                   \
    else select_dt<DT, 1>(sc, cam, p, mask, count, st)
    if (dt == RECOGS_F32) { RECOGS_SELECT(RECOGS_F32); }
    else if (dt == RECOGS_F16) { RECOGS_SELECT(RECOGS_F16); }
    else { RECOGS_SELECT(RECOGS_BF16); }
#undef RECOGS_SELECT
}

template <int DT>
static void recolor_dt(const SceneDev &sc, int ncoef, void *dst, const uint8_t *mask, const float *M, const float *b, int copy,
                       hipStream_t st) {
    constexpr int VEC = 16 / Store<DT>::bytes;
    const dim3 bl(256);
    // (a destination that is the source already holds the unselected coefficients)
    if (copy && dst != sc.sh) {
        const unsigned gy = (unsigned)((ncoef + kCopyCoefs - 1) / kCopyCoefs);
        if (planes_aligned(sc.sh, sc.stride, Store<DT>::bytes, 16) && planes_aligned(dst, sc.stride, Store<DT>::bytes, 16))
            hipLaunchKernelGGL((k_recolor_copy<DT, VEC>), dim3((unsigned)((sc.n + 256 * VEC - 1) / (256 * VEC)), gy), bl, 0, st,
                               sc, ncoef, dst, mask, M, b);
        else
            hipLaunchKernelGGL((k_recolor_copy<DT, 1>), dim3((unsigned)((sc.n + 255) / 256), gy), bl, 0, st, sc, ncoef, dst, mask,
                               M, b);
        return;
    }
    const int64_t threads = (sc.n + kRecolorPer - 1) / kRecolorPer;
    hipLaunchKernelGGL(k_recolor<DT>, dim3((unsigned)((threads + 255) / 256)), bl, 0, st, sc, ncoef, dst, mask, M, b);
}

void launch_recolor(int dt, const SceneDev &sc, int ncoef, void *dst, const uint8_t *mask, const float *M,
                    const float *b, int copy_unselected, hipStream_t st) {
    if (sc.n <= 0) return;
    if (dt == RECOGS_F32) recolor_dt<RECOGS_F32>(sc, ncoef, dst, mask, M, b, copy_unselected, st);
    else if (dt == RECOGS_F16) recolor_dt<RECOGS_F16>(sc, ncoef, dst, mask, M, b, copy_unselected, st);
    else recolor_dt<RECOGS_BF16>(sc, ncoef, dst, mask, M, b, copy_unselected, st);
}

}  // namespace recogs
