// HIP kernels of the forward 3DGS rasterizer for CDNA4 (gfx950, wave64).
//
//   k_preprocess   per Gaussian (x views): activation, 3D covariance, camera
//                  transform, projection, EWA 2D covariance + conic (FP64
//                  fallback when near-singular), SH colour, screen footprint
//   k_bucket_*     the visible Gaussians of each view in depth order: counted
//                  into buckets of depth ranges, scattered, every bucket
//                  sorted in LDS; the FP64 conics of the near-singular ones
//   k_chunk_totals, k_scan_*
//                  exclusive scans of per-block counts (chunk totals, then
//                  each chunk; wave64 DPP scans)
//   k_compact      visible Gaussians as (depth key, record, packed tile
//                  rectangle) triples; the FP64 conics of the near-singular
//                  Gaussians
//   k_sort_*       LSD radix sort passes, 8-bit digits, reduce-then-scan,
//                  LDS-atomic digit counts, ballot/mbcnt ranking inside a
//                  wave, DPP scans; the tile digits of the (tile | depth)
//                  keys on the duplicates, and the depth digits on the visible
//                  Gaussians of the views that the buckets do not take
//   k_sorted_sums  tile counts per 256 depth-ordered Gaussians
//   k_duplicate    one (tile | depth) key per (Gaussian, overlapped tile)
//   k_duplicate_culled
//                  the same, keeping only the tiles where the Gaussian can
//                  reach the skip threshold at some pixel (count, then emit)
//   k_ranges       [start, end) of every tile in the sorted list
//   k_tile_*       the tile digit placed by counting instead (per-unit tile
//                  counts from 2D difference grids, their prefixes, then
//                  every (Gaussian, tile) entry written straight to its sorted
//                  position; the ranges are the tile starts)
//   k_blend        front-to-back compositing, one wave64 per 8x8 pixel block,
//                  Gaussians staged per wave in LDS, per-wave early exit
//
// Numerics: all kernels are compiled with -ffp-contract=off; every fused
// multiply-add is written explicitly so the FP32 operation sequence is fixed.
#include "tigas_internal.h"

namespace tigas {

// ------------------------------------------------------------ wave helpers

__device__ __forceinline__ uint32_t lane_id() {
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ uint32_t bits_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
__device__ __forceinline__ uint32_t readlane(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}

// Inclusive prefix sum over the 64 lanes of a wave with DPP row shifts and
// row broadcasts (all 64 lanes must be active).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return readlane(wave_incl_scan(v), 63); }

// Inclusive prefix maximum over the 64 lanes of a wave (same lane pattern as
// wave_incl_scan; lanes without a source see 0, the identity for unsigned
// maxima).
__device__ __forceinline__ uint32_t wave_incl_max(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));  // row_shr:2
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));  // row_shr:4
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));  // row_shr:8
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));  // row_bcast:15
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return v;
}

// x, from which nothing is formed ahead of this point: addresses and constants
// that the compiler keeps over a loop for a rare step in it take registers.
__device__ __forceinline__ uint32_t fresh(uint32_t x) {
    asm volatile("" : "+v"(x));
    return x;
}

// Exclusive scan over a workgroup of NT threads; *total receives the sum.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* lds, uint32_t* total) {
    const uint32_t incl = wave_incl_scan(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 63) lds[w] = incl;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) {
        const uint32_t s = lds[i];
        off += (i < w) ? s : 0u;
        tot += s;
    }
    *total = tot;
    __syncthreads();
    return off + incl - v;
}

template <int NT>
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t* lds) {
    uint32_t tot;
    block_excl_scan<NT>(v, lds, &tot);
    return tot;
}

// ------------------------------------------------------ double-float helpers
// Error-free transformations (Knuth two-sum, fma two-product) so that the
// pixel position of a Gaussian is carried as an unevaluated FP32 sum hi + lo.

struct df {
    float hi, lo;
};
__device__ __forceinline__ df two_sum(float a, float b) {
    const float s = a + b;
    const float bb = s - a;
    const float e = (a - (s - bb)) + (b - bb);
    return {s, e};
}
__device__ __forceinline__ df quick_two_sum(float a, float b) {
    const float s = a + b;
    return {s, b - (s - a)};
}
__device__ __forceinline__ df df_add(df a, df b) {
    df s = two_sum(a.hi, b.hi);
    s.lo = s.lo + (a.lo + b.lo);
    return quick_two_sum(s.hi, s.lo);
}
__device__ __forceinline__ df df_mulf(df a, float b) {
    const float p = a.hi * b;
    float e = __builtin_fmaf(a.hi, b, -p);
    e = __builtin_fmaf(a.lo, b, e);
    return quick_two_sum(p, e);
}
__device__ __forceinline__ df df_div(df a, df b) {
    const float q1 = a.hi / b.hi;
    const df p = df_mulf(b, q1);
    const df r = df_add(a, df{-p.hi, -p.lo});
    const float q2 = r.hi / b.hi;
    return quick_two_sum(q1, q2);
}

// --------------------------------------------------------- attribute decode

__device__ __forceinline__ float h2f(uint32_t bits16, int storage) {
    if (storage == 2) return __uint_as_float(bits16 << 16);  // bfloat16
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits16);
}
__device__ __forceinline__ void unpack8(const uint4 u, float* f, int storage) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        f[2 * i] = h2f(w[i] & 0xffffu, storage);
        f[2 * i + 1] = h2f(w[i] >> 16, storage);
    }
}

// Real spherical harmonics with the Condon-Shortley phase, degree <= 3
// (textbook normalisations), colour = 0.5 + sum Y_i k_i, clamped below at 0.
constexpr float SH_C0 = 0.28209479177387814f;
constexpr float SH_C1 = 0.48860251190291992f;
constexpr float SH_C2A = 1.0925484305920792f;
constexpr float SH_C2B = 0.31539156525252005f;
constexpr float SH_C2C = 0.54627421529603959f;
constexpr float SH_C3A = 0.59004358992664352f;
constexpr float SH_C3B = 2.8906114426405538f;
constexpr float SH_C3C = 0.45704579946446577f;
constexpr float SH_C3D = 0.3731763325901154f;
constexpr float SH_C3E = 1.4453057213202769f;

template <int DEG>
__device__ __forceinline__ void sh_colour(const float* k, float x, float y, float z, int deg, float* rgb) {
    float Y[16];
    Y[0] = SH_C0;
    if (DEG >= 1) {
        Y[1] = -SH_C1 * y;
        Y[2] = SH_C1 * z;
        Y[3] = -SH_C1 * x;
    }
    if (DEG >= 2) {
        const float xx = x * x, yy = y * y, zz = z * z;
        Y[4] = SH_C2A * (x * y);
        Y[5] = -SH_C2A * (y * z);
        Y[6] = SH_C2B * (3.0f * zz - 1.0f);
        Y[7] = -SH_C2A * (x * z);
        Y[8] = SH_C2C * (xx - yy);
        if (DEG >= 3) {
            Y[9] = -SH_C3A * (y * (3.0f * xx - yy));
            Y[10] = SH_C3B * (x * y * z);
            Y[11] = -SH_C3C * (y * (5.0f * zz - 1.0f));
            Y[12] = SH_C3D * (z * (5.0f * zz - 3.0f));
            Y[13] = -SH_C3C * (x * (5.0f * zz - 1.0f));
            Y[14] = SH_C3E * (z * (xx - yy));
            Y[15] = -SH_C3A * (x * (xx - 3.0f * yy));
        }
    }
    float s[3] = {0.5f, 0.5f, 0.5f};
    auto add = [&](int i) {
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) s[ch] = __builtin_fmaf(Y[i], k[i * 3 + ch], s[ch]);
    };
    // a uniform branch per degree: a select per coefficient takes 48 more
    // instructions a view (32 views of 3M records 1.95 ms, with the branches 1.90)
    add(0);
    if (DEG >= 1 && deg >= 1) {
#pragma unroll
        for (int i = 1; i < 4; ++i) add(i);
        if (DEG >= 2 && deg >= 2) {
#pragma unroll
            for (int i = 4; i < 9; ++i) add(i);
            if (DEG >= 3 && deg >= 3) {
#pragma unroll
                for (int i = 9; i < 16; ++i) add(i);
            }
        }
    }
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) rgb[ch] = fmaxf(s[ch], 0.0f);
}

// ------------------------------------------------------------- preprocess

constexpr float NEAR_Z = 0.2f;
constexpr float DILATION = 0.3f;
constexpr float ALPHA_MIN = 1.0f / 255.0f;
// log2(1/255): below it, 2^e < 1/255 and a Gaussian is skipped at the pixel.
constexpr float LOG2_ALPHA_MIN = -7.99435343685886f;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN255 = 5.5412635451584258f;
constexpr float KAPPA_INV = 1.0f / 64.0f;  // FP64 fallback when a*c > 64 det

// FP64 recomputation of the 2D covariance from the FP32 inputs.
__device__ __forceinline__ void cov2d_fp64(const float* q32, const float* ls32, float mx, float my, float mz,
                                        const ViewParams& v, double* abc) {
    double qw = q32[0], qx = q32[1], qy = q32[2], qz = q32[3];
    const double inv = 1.0 / sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
    qw *= inv; qx *= inv; qy *= inv; qz *= inv;
    const double R[9] = {1 - 2 * (qy * qy + qz * qz), 2 * (qx * qy - qw * qz), 2 * (qx * qz + qw * qy),
                         2 * (qx * qy + qw * qz), 1 - 2 * (qx * qx + qz * qz), 2 * (qy * qz - qw * qx),
                         2 * (qx * qz - qw * qy), 2 * (qy * qz + qw * qx), 1 - 2 * (qx * qx + qy * qy)};
    const double s[3] = {exp((double)ls32[0]), exp((double)ls32[1]), exp((double)ls32[2])};
    double M[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) M[i * 3 + j] = R[i * 3 + j] * s[j];
    const double d[3] = {(double)mx - (double)v.cam[0], (double)my - (double)v.cam[1], (double)mz - (double)v.cam[2]};
    double p[3];
    for (int i = 0; i < 3; ++i)
        p[i] = (double)v.V[i * 3] * d[0] + (double)v.V[i * 3 + 1] * d[1] + (double)v.V[i * 3 + 2] * d[2];
    double rx = p[0] / p[2], ry = p[1] / p[2];
    rx = fmin(fmax(rx, -(double)v.lim_x), (double)v.lim_x);
    ry = fmin(fmax(ry, -(double)v.lim_y), (double)v.lim_y);
    const double fxz = (double)v.fx / p[2], fyz = (double)v.fy / p[2];
    double T0[3], T1[3];
    for (int j = 0; j < 3; ++j) {
        T0[j] = fxz * ((double)v.V[j] - rx * (double)v.V[6 + j]);
        T1[j] = fyz * ((double)v.V[3 + j] - ry * (double)v.V[6 + j]);
    }
    double m0[3], m1[3];
    for (int k = 0; k < 3; ++k) {
        m0[k] = T0[0] * M[k] + T0[1] * M[3 + k] + T0[2] * M[6 + k];
        m1[k] = T1[0] * M[k] + T1[1] * M[3 + k] + T1[2] * M[6 + k];
    }
    abc[0] = m0[0] * m0[0] + m0[1] * m0[1] + m0[2] * m0[2] + (double)DILATION;
    abc[1] = m0[0] * m1[0] + m0[1] * m1[1] + m0[2] * m1[2];
    abc[2] = m1[0] * m1[0] + m1[1] * m1[1] + m1[2] * m1[2] + (double)DILATION;
}

// SH coefficients of Gaussian g (the words of degree <= DEG) decoded to FP32.
template <int ST, int DEG>
__device__ __forceinline__ void load_sh(const SceneView& s, int64_t n, int64_t g, float* k) {
    if (ST == 0) {
        const float4* sh = reinterpret_cast<const float4*>(s.sh);
        constexpr int NP = ((DEG + 1) * (DEG + 1) * 3 + 3) / 4;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const float4 t = sh[g * s.sh_stride + p];
            k[4 * p] = t.x;
            k[4 * p + 1] = t.y;
            k[4 * p + 2] = t.z;
            k[4 * p + 3] = t.w;
        }
    } else {
        const uint4* sh = reinterpret_cast<const uint4*>(s.sh);
        constexpr int NP = ((DEG + 1) * (DEG + 1) * 3 + 7) / 8;
#pragma unroll
        for (int p = 0; p < NP; ++p) unpack8(sh[g * s.sh_stride + p], &k[8 * p], ST);
    }
}

// Bit d set when the SH coefficients of degrees 0..d are all finite.
__host__ __device__ constexpr int sh_degree_of(int i) {  // float i of the [16][3] coefficient block
    return i < 3 ? 0 : i < 12 ? 1 : i < 27 ? 2 : 3;
}
template <int DEG>
__device__ __forceinline__ uint32_t sh_finite(const float* k) {
    uint32_t bad = 0;  // bit d: a coefficient of degree d is not finite
#pragma unroll
    for (int i = 0; i < 3 * (DEG + 1) * (DEG + 1); ++i)
        bad |= __builtin_isfinite(k[i]) ? 0u : (1u << sh_degree_of(i));
    // lowest bad degree b: degrees below b are fine
    return (bad & (0u - bad)) - 1u;
}

// The lane whose record is the sample of a wave's visible ones (mask m, not
// empty): the first at or after one that varies from wave to wave.
__device__ __forceinline__ uint32_t sample_lane(uint64_t m, uint32_t wid) {
    const uint32_t r = (wid * 0x9E3779B1u) >> 26;
    const uint64_t rot = (m >> r) | (m << ((64u - r) & 63u));
    return ((uint32_t)__builtin_ctzll(rot) + r) & 63u;
}

template <int ST, int DEG>
__global__ __launch_bounds__(K1_THREADS) void k_preprocess(SceneView s, const ViewParams* __restrict__ views,
                                                           int nviews, uint32_t rec_base, uint32_t n_pad,
                                                           uint32_t view_base, PreOut o) {
    __shared__ uint32_t red[2][K1_THREADS / 64][3];
    const int64_t g = (int64_t)blockIdx.x * K1_THREADS + threadIdx.x;
    const bool in = g < s.n;
    const int64_t n = s.n;

    // ---- view-independent attributes
    float mx = 0.f, my = 0.f, mz = 0.f;
    float q[4] = {1.f, 0.f, 0.f, 0.f}, ls[3] = {0.f, 0.f, 0.f}, logit = 0.f;
    if (in) {
        mx = s.mean[g];
        my = s.mean[n + g];
        mz = s.mean[2 * n + g];
        if (ST == 0) {
            const float4* a = reinterpret_cast<const float4*>(s.attr);
            const float4 r = a[g], m = a[n + g];
            q[0] = r.x; q[1] = r.y; q[2] = r.z; q[3] = r.w;
            ls[0] = m.x; ls[1] = m.y; ls[2] = m.z; logit = m.w;
        } else {
            float f[8];
            unpack8(reinterpret_cast<const uint4*>(s.attr)[g], f, ST);
            q[0] = f[0]; q[1] = f[1]; q[2] = f[2]; q[3] = f[3];
            ls[0] = f[4]; ls[1] = f[5]; ls[2] = f[6]; logit = f[7];
        }
    }
    const float qn2 = q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3];
    bool ok = in && qn2 > 0.0f && __builtin_isfinite(qn2) && __builtin_isfinite(mx) && __builtin_isfinite(my) &&
              __builtin_isfinite(mz) && __builtin_isfinite(ls[0]) && __builtin_isfinite(ls[1]) &&
              __builtin_isfinite(ls[2]) && __builtin_isfinite(logit);
    // opacity and its log2 (folded into the blend exponent)
    const float op = 1.0f / (1.0f + expf(-logit));
    ok = ok && op >= ALPHA_MIN;
    const float L = log2f(op);
    // alpha >= 1/255 support: Q <= 2 ln(255 o); widened by 2^-9 relative and
    // 2^-12 absolute so FP32 evaluation error cannot push a contributing
    // pixel outside the footprint
    const float k2 = 2.0f * __builtin_fmaf(L, 0.69314718055994531f, LN255);
    const float k2m = __builtin_fmaf(k2, 1.0f + 1.0f / 512.0f, 1.0f / 4096.0f);
    // M = Rq diag(exp(ls)), Sigma = M M^T
    float M[9];
    float smax = 0.0f;  // largest scale: bounds the screen footprint before the EWA step
    {
        const float inv = 1.0f / sqrtf(qn2);
        const float w = q[0] * inv, x = q[1] * inv, y = q[2] * inv, z = q[3] * inv;
        const float R[9] = {1.f - 2.f * (y * y + z * z), 2.f * (x * y - w * z), 2.f * (x * z + w * y),
                            2.f * (x * y + w * z), 1.f - 2.f * (x * x + z * z), 2.f * (y * z - w * x),
                            2.f * (x * z - w * y), 2.f * (y * z + w * x), 1.f - 2.f * (x * x + y * y)};
        const float sc[3] = {expf(ls[0]), expf(ls[1]), expf(ls[2])};
        smax = fmaxf(sc[0], fmaxf(sc[1], sc[2]));
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) M[i * 3 + j] = R[i * 3 + j] * sc[j];
    }

    float k[48];
    bool sh_loaded = false;
    uint32_t sh_fin = 0;  // bit d: the coefficients of degrees 0..d are all finite
    bool sh_checked = false;

    for (int vi = 0; vi < nviews; ++vi) {
        const ViewParams& v = views[vi];
        const uint32_t rec = rec_base + (uint32_t)vi * n_pad + (uint32_t)g;
        // FP32 order key (also the near-plane test)
        const float z32 = __builtin_fmaf(v.V[6], mx, __builtin_fmaf(v.V[7], my, __builtin_fmaf(v.V[8], mz, v.tz_key)));
        bool vis = ok && z32 > NEAR_Z;
        uint32_t touched = 0, tiles = 0, fb = 0;  // lists and tiles met, FP64 fallback
        float4 r0, r1, r2;  // of touched records only
        uint2 bb, tr = {0u, 0u};
        if (vis) {
            // camera-space centre, double-float: d = mu - t exactly, p = V d
            const df dX = two_sum(mx, -v.cam[0]), dY = two_sum(my, -v.cam[1]), dZ = two_sum(mz, -v.cam[2]);
            const df px = df_add(df_add(df_mulf(dX, v.V[0]), df_mulf(dY, v.V[1])), df_mulf(dZ, v.V[2]));
            const df py = df_add(df_add(df_mulf(dX, v.V[3]), df_mulf(dY, v.V[4])), df_mulf(dZ, v.V[5]));
            const df pz = df_add(df_add(df_mulf(dX, v.V[6]), df_mulf(dY, v.V[7])), df_mulf(dZ, v.V[8]));
            const float zc = pz.hi;
            // pixel centre of the Gaussian: u = fx x/z + cx, v = fy y/z + cy
            const df u = df_add(df_mulf(df_div(px, pz), v.fx), df{v.cx, 0.0f});
            const df w = df_add(df_mulf(df_div(py, pz), v.fy), df{v.cy, 0.0f});
            // start the SH loads now when the footprint can reach the image, so
            // they arrive during the EWA step: the footprint half-width is at
            // most 3.34 (f/z (1 + lim) max scale + 0.55) pixels
            {
                const float rb = 3.4f * (fmaxf(v.fx, v.fy) / zc * (1.0f + fmaxf(v.lim_x, v.lim_y)) * smax + 0.6f) + 1.0f;
                const bool maybe = u.hi > -rb && u.hi < (float)v.width + rb && w.hi > -rb && w.hi < (float)v.height + rb;
                if (maybe && !sh_loaded) {
                    load_sh<ST, DEG>(s, n, g, k);
                    sh_loaded = true;
                }
            }
            // EWA: T = J V with the Jacobian at the clamped direction; Sigma2D = (T M)(T M)^T + 0.3 I
            const float iz = 1.0f / zc;
            const float rx = fminf(fmaxf(px.hi * iz, -v.lim_x), v.lim_x);
            const float ry = fminf(fmaxf(py.hi * iz, -v.lim_y), v.lim_y);
            const float fxz = v.fx * iz, fyz = v.fy * iz;
            float T0[3], T1[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                T0[j] = fxz * __builtin_fmaf(-rx, v.V[6 + j], v.V[j]);
                T1[j] = fyz * __builtin_fmaf(-ry, v.V[6 + j], v.V[3 + j]);
            }
            float m0[3], m1[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                m0[c] = __builtin_fmaf(T0[0], M[c], __builtin_fmaf(T0[1], M[3 + c], T0[2] * M[6 + c]));
                m1[c] = __builtin_fmaf(T1[0], M[c], __builtin_fmaf(T1[1], M[3 + c], T1[2] * M[6 + c]));
            }
            float a = __builtin_fmaf(m0[0], m0[0], __builtin_fmaf(m0[1], m0[1], m0[2] * m0[2])) + DILATION;
            float b = __builtin_fmaf(m0[0], m1[0], __builtin_fmaf(m0[1], m1[1], m0[2] * m1[2]));
            float c = __builtin_fmaf(m1[0], m1[0], __builtin_fmaf(m1[1], m1[1], m1[2] * m1[2])) + DILATION;
            const float ac = a * c;
            const float det = ac - b * b;
            float ca, cb, cc;
            if (!(det > ac * KAPPA_INV)) {
                // near-singular 2D covariance: its conic is recomputed in FP64
                // by conic_fp64 (listed below); a and c are sums of squares
                // and exact enough for the footprint
                ca = cb = cc = 0.0f;
                fb = 1;
            } else {
                const float id = 1.0f / det;
                ca = c * id;
                cb = -b * id;
                cc = a * id;
            }
            // conservative footprint: bounding box of the widened support ellipse
            const float ex = sqrtf(k2m * a), ey = sqrtf(k2m * c);
            vis = vis && __builtin_isfinite(u.hi) && __builtin_isfinite(w.hi) && __builtin_isfinite(ex) &&
                  __builtin_isfinite(ey) && __builtin_isfinite(ca) && __builtin_isfinite(cb) && __builtin_isfinite(cc);
            if (vis) {
                const float mg = 1.0f / 256.0f;
                // pixel i is inside when |i + 0.5 - u| <= ex
                const float fw = (float)v.width, fh = (float)v.height;
                const float xl = fminf(fmaxf(u.hi - ex - 0.5f - mg, -1.0f), fw);
                const float xr = fminf(fmaxf(u.hi + ex - 0.5f + mg, -1.0f), fw);
                const float yl = fminf(fmaxf(w.hi - ey - 0.5f - mg, -1.0f), fh);
                const float yr = fminf(fmaxf(w.hi + ey - 0.5f + mg, -1.0f), fh);
                const int x0 = max((int)ceilf(xl), 0), x1 = min((int)floorf(xr), v.width - 1);
                const int y0 = max((int)ceilf(yl), 0), y1 = min((int)floorf(yr), v.height - 1);
                if (x0 <= x1 && y0 <= y1) {
                    int tx0 = x0 >> v.tw_log, tx1 = x1 >> v.tw_log;
                    int ty0 = y0 >> v.th_log, ty1 = y1 >> v.th_log;
                    tiles = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
                    // the lists' rectangle
                    tx0 >>= v.lx;
                    tx1 >>= v.lx;
                    ty0 >>= v.ly;
                    ty1 >>= v.ly;
                    touched = (uint32_t)((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
                    bb = make_uint2((uint32_t)x0 | ((uint32_t)y0 << 16), (uint32_t)x1 | ((uint32_t)y1 << 16));
                    tr = make_uint2((uint32_t)tx0 | ((uint32_t)ty0 << 16),
                                    (uint32_t)(tx1 - tx0 + 1) | ((uint32_t)(ty1 - ty0 + 1) << 16));
                    if (v.cells) {
                        // the cells of the pixel box's ends inside its first and last list
                        const int cw = cell_log(v.tw_log + v.lx, v.cells), ch = cell_log(v.th_log + v.ly, v.cells);
                        const int mx = (1 << (v.tw_log + v.lx - cw)) - 1, my = (1 << (v.th_log + v.ly - ch)) - 1;
                        tr.x |= ((uint32_t)((x0 >> cw) & mx) << 12) | ((uint32_t)((y0 >> ch) & my) << 28);
                        tr.y |= ((uint32_t)((x1 >> cw) & mx) << 12) | ((uint32_t)((y1 >> ch) & my) << 28);
                    }
                }
            }
            if (touched) {
                if (!sh_loaded) {
                    load_sh<ST, DEG>(s, n, g, k);
                    sh_loaded = true;
                }
                // colour at the direction camera centre -> Gaussian
                const float dx = dX.hi, dy = dY.hi, dz = dZ.hi;
                const float dn = 1.0f / sqrtf(__builtin_fmaf(dx, dx, __builtin_fmaf(dy, dy, dz * dz)));
                float rgb[3];
                sh_colour<DEG>(k, dx * dn, dy * dn, dz * dn, v.sh_degree, rgb);
                if (!sh_checked) {  // once per Gaussian, where the loads have landed
                    sh_fin = sh_finite<DEG>(k);
                    sh_checked = true;
                }
                // a non-finite SH coefficient of the degree in use drops the
                // Gaussian, as any other non-finite attribute does (and so
                // does a colour that overflows): every record's colour is finite
                const bool fin = ((sh_fin >> v.sh_degree) & 1u) && __builtin_isfinite(rgb[0]) &&
                                 __builtin_isfinite(rgb[1]) && __builtin_isfinite(rgb[2]);
                if (!fin) {
                    touched = tiles = 0;
                    fb = 0;
                    tr = make_uint2(0u, 0u);
                }
                r0 = make_float4(u.hi, w.hi, u.lo, w.lo);
                r1 = make_float4(-0.5f * LOG2E * ca, -LOG2E * cb, -0.5f * LOG2E * cc, L);
                r2 = make_float4(rgb[0], rgb[1], rgb[2], op);
            }
        }
        {
            // append near-singular visible Gaussians to the FP64 list (one atomic per wave)
            const bool lst = touched && fb;
            const uint64_t m = ballot(lst);
            if (m) {
                uint32_t base = 0;
                if ((threadIdx.x & 63) == (uint32_t)__builtin_ctzll(m))
                    base = atomicAdd(&o.cnt->fb_list, (uint32_t)__builtin_popcountll(m));
                base = readlane(base, __builtin_ctzll(m));
                const uint32_t pos = base + bits_below(m);
                if (lst && pos < o.fb_cap) o.fb_list[pos] = make_uint2(rec, (uint32_t)g);
            }
        }
        o.zkey[rec] = __float_as_uint(z32);
        if (touched) {
            Rec out;
            out.r0 = r0;
            out.r1 = r1;
            out.r2 = r2;
            out.bbox = bb;
            out.pad = make_uint2(0u, 0u);
            o.rec[rec] = out;
        }
        o.rect[rec] = tr;  // every record: whole-line, coalesced stores
        {
            // the wave's visible records, and one of them as a sample of the
            // view's depth distribution
            const uint64_t m = ballot(touched != 0u);
            const uint32_t wid = (uint32_t)__builtin_amdgcn_readfirstlane((int)(rec >> 6));
            const uint32_t src = m ? sample_lane(m, wid) : 0u;
            const uint32_t key = readlane(__float_as_uint(z32), (int)src);
            if ((threadIdx.x & 63) == 0) {
                o.vmask[wid] = m;
                o.sample[wid] = m ? key : 0xffffffffu;
            }
        }
        // per-block counts: wave sums, then one barrier (LDS slots alternate
        // between views so the next view cannot overwrite unread sums)
        const uint32_t s0 = wave_sum(touched), s1 = wave_sum(touched ? 1u + (fb << 16) : 0u), s2 = wave_sum(tiles);
        const int wv = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) {
            red[vi & 1][wv][0] = s0;
            red[vi & 1][wv][1] = s1;
            red[vi & 1][wv][2] = s2;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t t0 = 0, t1 = 0, t2 = 0;
#pragma unroll
            for (int j = 0; j < K1_THREADS / 64; ++j) {
                t0 += red[vi & 1][j][0];
                t1 += red[vi & 1][j][1];
                t2 += red[vi & 1][j][2];
            }
            const uint32_t blk = rec / K1_THREADS;
            o.blk_sum[blk] = t0;
            o.blk_vis[blk] = t1 & 0xffffu;
            o.blk_fb[blk] = t1 >> 16;
            o.blk_tiles[blk] = t2;
            o.blk_view[blk] = view_base + (uint32_t)vi;
        }
    }
}

// Conic of a listed near-singular Gaussian, recomputed in FP64 from the
// FP32 inputs: Sigma2D, its determinant and its inverse; the exponent
// coefficients of the record are overwritten (log2 opacity kept).  Run by
// k_bucket_sort or, before the radix passes, by k_compact: ahead of the tighter tile
// culling and the blend, which read the coefficients.
__device__ void conic_fp64(const uint2 e, const ViewParams* __restrict__ views, const uint32_t* __restrict__ blk_view,
                           Rec* __restrict__ recs) {
    {
        const uint32_t rec = e.x;
        const int64_t g = e.y;
        const ViewParams& v = views[blk_view[rec / K1_THREADS]];
        const SceneView& s = v.scene;
        const int64_t N = s.n;
        const float mx = s.mean[g], my = s.mean[N + g], mz = s.mean[2 * N + g];
        float q[4], ls[3];
        if (s.storage == 0) {
            const float4* a = reinterpret_cast<const float4*>(s.attr);
            const float4 r = a[g], m = a[N + g];
            q[0] = r.x; q[1] = r.y; q[2] = r.z; q[3] = r.w;
            ls[0] = m.x; ls[1] = m.y; ls[2] = m.z;
        } else {
            float f[8];
            unpack8(reinterpret_cast<const uint4*>(s.attr)[g], f, s.storage);
            q[0] = f[0]; q[1] = f[1]; q[2] = f[2]; q[3] = f[3];
            ls[0] = f[4]; ls[1] = f[5]; ls[2] = f[6];
        }
        double abc[3];
        cov2d_fp64(q, ls, mx, my, mz, v, abc);
        const double d64 = abc[0] * abc[2] - abc[1] * abc[1];
        float4 r = recs[rec].r1;
        r.x = -0.5f * LOG2E * (float)(abc[2] / d64);
        r.y = -LOG2E * (float)(-abc[1] / d64);
        r.z = -0.5f * LOG2E * (float)(abc[0] / d64);
        recs[rec].r1 = r;
    }
}

// Counts are staged through LDS for the scans: coalesced loads, SCAN_ITEMS
// consecutive counts per thread summed from LDS (one pad word per 32 keeps
// those strided reads free of bank conflicts), offsets written back through
// LDS and stored coalesced.
constexpr int SCAN_STAGE = SCAN_CHUNK + SCAN_CHUNK / 32;
__device__ __forceinline__ int spad(int i) { return i + (i >> 5); }

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor((unsigned long long)v, o, 64);
    return v;
}
__device__ __forceinline__ uint64_t block_sum_u64(uint64_t v, unsigned long long* lds) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    uint64_t t = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += lds[i];
    __syncthreads();
    return t;
}

// Multi-workgroup exclusive scans of per-block counts, chunk by chunk
// (SCAN_CHUNK counts per workgroup), in two kernels: chunk totals, then each
// chunk scanned from the sum of the totals before it.

// Totals of chunk blockIdx.x of `in` (and optionally of two more count arrays).
__global__ __launch_bounds__(SCAN_THREADS) void k_chunk_totals(const uint32_t* __restrict__ in, int n,
                                                               const uint32_t* __restrict__ in_a,
                                                               const uint32_t* __restrict__ in_b,
                                                               uint32_t* __restrict__ tot,
                                                               unsigned long long* __restrict__ tot_a,
                                                               uint32_t* __restrict__ tot_b) {
    __shared__ unsigned long long red64[SCAN_THREADS / 64];
    const int base = (int)blockIdx.x * SCAN_CHUNK;
    uint64_t s = 0, sa = 0, sb = 0;
#pragma unroll
    for (int r = 0; r < SCAN_ITEMS; ++r) {
        const int i = base + r * SCAN_THREADS + (int)threadIdx.x;
        if (i < n) {
            s += in[i];
            if (in_a) sa += in_a[i];
            if (in_b) sb += in_b[i];
        }
    }
    s = block_sum_u64(s, red64);
    if (in_a) sa = block_sum_u64(sa, red64);
    if (in_b) sb = block_sum_u64(sb, red64);
    if (threadIdx.x == 0) {
        tot[blockIdx.x] = (uint32_t)s;
        if (tot_a) tot_a[blockIdx.x] = sa;
        if (tot_b) tot_b[blockIdx.x] = (uint32_t)sb;
    }
}

// Exclusive scan of chunk blockIdx.x of `in` into `out`, starting from the
// sum of the totals of the chunks before it.
__device__ void scan_chunk(const uint32_t* __restrict__ in, int n, const uint32_t* __restrict__ tot,
                           uint32_t* __restrict__ out, uint32_t* red, unsigned long long* red64, uint32_t* stage) {
    uint64_t p = 0;
    for (int c = (int)threadIdx.x; c < (int)blockIdx.x; c += SCAN_THREADS) p += tot[c];
    const uint32_t prefix = (uint32_t)block_sum_u64(p, red64);
    const int base = (int)blockIdx.x * SCAN_CHUNK;
#pragma unroll
    for (int r = 0; r < SCAN_ITEMS; ++r) {
        const int i = r * SCAN_THREADS + (int)threadIdx.x;
        stage[spad(i)] = base + i < n ? in[base + i] : 0u;
    }
    __syncthreads();
    uint32_t loc[SCAN_ITEMS];
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) {
        loc[j] = sum;
        sum += stage[spad((int)threadIdx.x * SCAN_ITEMS + j)];
    }
    uint32_t total;
    const uint32_t ex = block_excl_scan<SCAN_THREADS>(sum, red, &total);
#pragma unroll
    for (int j = 0; j < SCAN_ITEMS; ++j) stage[spad((int)threadIdx.x * SCAN_ITEMS + j)] = prefix + ex + loc[j];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SCAN_ITEMS; ++r) {
        const int i = r * SCAN_THREADS + (int)threadIdx.x;
        if (base + i < n) out[base + i] = stage[spad(i)];
    }
}

// After preprocess (second kernel of the chunked scan): compaction offsets of
// the visible records; workgroup 0 also sets the totals V, D and FP64-fallback
// count and the overflow flag; every workgroup clears part of the per-frame
// accumulators of later kernels (digit totals, tile ranges).
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_visible(const uint32_t* __restrict__ blk_vis, int nblk,
                                                               const uint32_t* __restrict__ tot_vis,
                                                               const unsigned long long* __restrict__ tot_dup,
                                                               const uint32_t* __restrict__ tot_fb, int nchunks,
                                                               uint32_t* __restrict__ blk_off, Counters* cnt,
                                                               uint32_t cap, ZeroList zl) {
    __shared__ uint32_t red[SCAN_THREADS / 64];
    __shared__ unsigned long long red64[SCAN_THREADS / 64];
    __shared__ uint32_t stage[SCAN_STAGE];
    scan_chunk(blk_vis, nblk, tot_vis, blk_off, red, red64, stage);
    if (blockIdx.x == 0) {
        uint64_t V = 0, D = 0, F = 0;
        for (int c = (int)threadIdx.x; c < nchunks; c += SCAN_THREADS) {
            V += tot_vis[c];
            D += tot_dup[c];
            F += tot_fb[c];
        }
        V = block_sum_u64(V, red64);
        D = block_sum_u64(D, red64);
        F = block_sum_u64(F, red64);
        if (threadIdx.x == 0) {
            cnt->D = D > 0xffffffffull ? 0xffffffffu : (uint32_t)D;
            cnt->pairs = cnt->D;  // one tile per list: only bucketed plans share lists
            cnt->visible = (uint32_t)V;
            cnt->fallbacks = (uint32_t)F;
            cnt->overflow = D > (uint64_t)cap ? 1u : 0u;
            cnt->fb_listed = cnt->fb_list;  // every preprocess launch has appended
            cnt->fb_list = 0u;                // the next frame appends from zero
        }
    }
#pragma unroll
    for (int k = 0; k < ZeroList::N; ++k)
        for (uint32_t i = blockIdx.x * SCAN_THREADS + threadIdx.x; i < zl.n[k]; i += gridDim.x * SCAN_THREADS)
            zl.p[k][i] = 0u;
}

// Emission offsets: exclusive scan of the duplicate counts of the
// depth-sorted visible Gaussians, per 256-element block (second kernel of the
// chunked scan).
// With `cnt`, workgroup 0 also stores the sum of the counts as the frame's
// duplicate count D (the count once tiles are culled), unless the frame
// overflowed: D then keeps the whole rectangles' count the buffers are grown to.
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_dups(const uint32_t* __restrict__ blk_sum, int nblk,
                                                            const uint32_t* __restrict__ tot,
                                                            uint32_t* __restrict__ blk_off, int nchunks,
                                                            Counters* cnt) {
    __shared__ uint32_t red[SCAN_THREADS / 64];
    __shared__ unsigned long long red64[SCAN_THREADS / 64];
    __shared__ uint32_t stage[SCAN_STAGE];
    scan_chunk(blk_sum, nblk, tot, blk_off, red, red64, stage);
    if (cnt && blockIdx.x == 0) {
        uint64_t D = 0;
        for (int c = (int)threadIdx.x; c < nchunks; c += SCAN_THREADS) D += tot[c];
        D = block_sum_u64(D, red64);
        if (threadIdx.x == 0 && !cnt->overflow) cnt->D = cnt->pairs = (uint32_t)min(D, 0xffffffffull);
    }
}

// Tile rectangle (tx0 | ty0 << 16, nx | ny << 16) packed into one word as
// tx0 | ty0 << 8 | tx1 << 16 | ty1 << 24 (views of at most 256 x 256 tiles; the
// top four bits of a half may hold cells), and back.
__device__ __forceinline__ uint32_t pack_rect(uint2 r) {
    const uint32_t tx0 = r.x & 0xfffu, ty0 = (r.x >> 16) & 0xfffu;
    return tx0 | (ty0 << 8) | ((tx0 + (r.y & 0xfffu) - 1u) << 16) | ((ty0 + ((r.y >> 16) & 0xfffu) - 1u) << 24);
}
// The cells of the ends of a rectangle of lists, in the bits above a record's number:
// first column and row (in the first list), last column and row (in the last).
__device__ __forceinline__ uint32_t rect_cells(uint2 r, int cells) {
    const int c = cells;
    return (((r.x >> 12) & 3u) | (((r.x >> 28) & 3u) << c) | (((r.y >> 12) & 3u) << (2 * c)) |
            (((r.y >> 28) & 3u) << (3 * c)))
           << (cell_rec_bits(c) & 31);
}
__device__ __forceinline__ uint2 unpack_rect(uint32_t p) {
    const uint32_t tx0 = p & 0xffu, ty0 = (p >> 8) & 0xffu, tx1 = (p >> 16) & 0xffu, ty1 = p >> 24;
    return make_uint2(tx0 | (ty0 << 16), (tx1 - tx0 + 1u) | ((ty1 - ty0 + 1u) << 16));
}

// Visible records, in record order, as (depth key, record) pairs, and with
// `ext` the packed tile rectangle as a third word that the depth passes carry
// along.  Four records per thread (16-byte loads): a workgroup covers four
// preprocess blocks, whose first compaction offset it starts from.
__global__ __launch_bounds__(K1_THREADS) void k_compact(const uint32_t* __restrict__ zkey,
                                                        const uint2* __restrict__ rect,
                                                        const uint32_t* __restrict__ blk_off, int nblk,
                                                        uint32_t* __restrict__ key, uint32_t* __restrict__ val,
                                                        uint32_t* __restrict__ ext, const Counters* __restrict__ cnt,
                                                        const uint2* __restrict__ fb_list, uint32_t fb_cap,
                                                        const ViewParams* __restrict__ views,
                                                        const uint32_t* __restrict__ blk_view, Rec* __restrict__ recs) {
    __shared__ uint32_t red[K1_THREADS / 64];
    // the FP64 conics of the near-singular Gaussians (a few hundred per
    // frame), before anything reads the exponent coefficients
    const uint32_t nfb = min(cnt->fb_listed, fb_cap);
    for (uint32_t k = blockIdx.x * K1_THREADS + threadIdx.x; k < nfb; k += gridDim.x * K1_THREADS)
        conic_fp64(fb_list[k], views, blk_view, recs);
    const uint32_t nrec = (uint32_t)nblk * K1_THREADS;  // a multiple of 4
    const uint32_t r0 = (blockIdx.x * K1_THREADS + threadIdx.x) * 4u;
    uint4 z = make_uint4(0u, 0u, 0u, 0u), ra = z, rb = z;
    if (r0 < nrec) {  // a record is visible when its rectangle has tiles
        z = *reinterpret_cast<const uint4*>(zkey + r0);
        ra = *reinterpret_cast<const uint4*>(rect + r0);
        rb = *reinterpret_cast<const uint4*>(rect + r0 + 2);
    }
    // loaded with the inputs, not after the scan: one memory round trip less
    const uint32_t boff = (uint32_t)blockIdx.x * 4u < (uint32_t)nblk ? blk_off[blockIdx.x * 4] : 0u;
    const bool v0 = ra.y != 0u, v1 = ra.w != 0u, v2 = rb.y != 0u, v3 = rb.w != 0u;
    const uint32_t c = (uint32_t)v0 + (uint32_t)v1 + (uint32_t)v2 + (uint32_t)v3;
    uint32_t tot;
    const uint32_t ex = block_excl_scan<K1_THREADS>(c, red, &tot);
    if (c) {
        uint32_t pos = boff + ex;
        if (ext) {
            if (v0) { key[pos] = z.x; val[pos] = r0; ext[pos] = pack_rect(make_uint2(ra.x, ra.y)); ++pos; }
            if (v1) { key[pos] = z.y; val[pos] = r0 + 1; ext[pos] = pack_rect(make_uint2(ra.z, ra.w)); ++pos; }
            if (v2) { key[pos] = z.z; val[pos] = r0 + 2; ext[pos] = pack_rect(make_uint2(rb.x, rb.y)); ++pos; }
            if (v3) { key[pos] = z.w; val[pos] = r0 + 3; ext[pos] = pack_rect(make_uint2(rb.z, rb.w)); }
        } else {
            if (v0) { key[pos] = z.x; val[pos] = r0; ++pos; }
            if (v1) { key[pos] = z.y; val[pos] = r0 + 1; ++pos; }
            if (v2) { key[pos] = z.z; val[pos] = r0 + 2; ++pos; }
            if (v3) { key[pos] = z.w; val[pos] = r0 + 3; }
        }
    }
}

// Tiles in a tile rectangle (tx0 | ty0 << 16, nx | ny << 16), and in a packed one.
__device__ __forceinline__ uint32_t rect_tiles(uint2 r) { return (r.y & 0xffffu) * (r.y >> 16); }
__device__ __forceinline__ uint32_t rect_count(uint32_t p) {
    return (((p >> 16) & 0xffu) - (p & 0xffu) + 1u) * ((p >> 24) - ((p >> 8) & 0xffu) + 1u);
}

// Per 256 depth-sorted visible Gaussians: the sum of their tile counts (zero
// past the visible count); workgroups stride over the nblk blocks.  The
// rectangles come packed (sorted_packed) or as two words (sorted_rect).
__global__ __launch_bounds__(K1_THREADS) void k_sorted_sums(const uint2* __restrict__ sorted_rect,
                                                            const uint32_t* __restrict__ sorted_packed,
                                                            const Counters* __restrict__ cnt, int nblk,
                                                            uint32_t* __restrict__ blk_sum) {
    __shared__ uint32_t red[K1_THREADS / 64];
    const uint32_t V = cnt->overflow ? 0u : cnt->visible;
    for (uint32_t b = blockIdx.x; b < (uint32_t)nblk; b += gridDim.x) {
        if (b * K1_THREADS >= V) {  // uniform: empty block
            if (threadIdx.x == 0) blk_sum[b] = 0u;
            continue;
        }
        const uint32_t i = b * K1_THREADS + threadIdx.x;
        uint32_t t = 0;
        if (i < V) t = rect_tiles(sorted_packed ? unpack_rect(sorted_packed[i]) : sorted_rect[i]);
        const uint32_t s = block_sum<K1_THREADS>(t, red);
        if (threadIdx.x == 0) blk_sum[b] = s;
    }
}

// ---------------------------------------------------------------- duplicate
// One entry per (Gaussian, overlapped tile), Gaussians taken in depth order,
// tiles row-major over the Gaussian's tile rectangle: tile word = global tile
// id, value = record, and (when asked) the depth word, so that the entry's
// 64-bit key is (tile id << 32) | depth bits.  Load-balanced: the threads of a
// workgroup write consecutive entries of their 256 Gaussians' output range,
// each finding its Gaussian by marks at the first slots and a prefix maximum.
template <bool DEPTH>
__global__ __launch_bounds__(K1_THREADS) void k_duplicate(const uint32_t* __restrict__ sorted_rec,
                                                          const uint2* __restrict__ sorted_rect,
                                                          const uint32_t* __restrict__ sorted_packed,
                                                          const uint32_t* __restrict__ zkey,
                                                          const uint32_t* __restrict__ blk_off,
                                                          const uint32_t* __restrict__ blk_view,
                                                          const Counters* __restrict__ cnt, uint32_t cap,
                                                          const ViewParams* __restrict__ views,
                                                          uint32_t* __restrict__ tile_out,
                                                          uint32_t* __restrict__ val_out,
                                                          uint32_t* __restrict__ depth_out) {
    __shared__ uint32_t red[K1_THREADS / 64];
    __shared__ uint32_t pre[K1_THREADS + 1];  // inclusive prefix of tile counts, pre[0] = 0
    __shared__ uint32_t srec[K1_THREADS];
    __shared__ uint32_t sx0[K1_THREADS], stx[K1_THREADS], snx[K1_THREADS], stb[K1_THREADS];
    __shared__ float sinx[K1_THREADS];
    __shared__ uint32_t own[K1_THREADS];           // round-tagged owner marks of the output slots
    __shared__ uint32_t wmax[K1_THREADS / 64];
    static_assert(K1_THREADS == 256, "owner marks keep the Gaussian index in 8 bits");
    const uint32_t i = blockIdx.x * K1_THREADS + threadIdx.x;
    const uint32_t V = cnt->visible;
    uint32_t rec = 0, t = 0;
    uint2 tr = make_uint2(0u, 0u);
    if (i < V) {
        rec = sorted_rec[i];
        // tile rectangle in depth order: carried packed through the depth
        // passes, or gathered by the last one
        tr = sorted_packed ? unpack_rect(sorted_packed[i]) : sorted_rect[i];
        t = rect_tiles(tr);
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan<K1_THREADS>(t, red, &tot);
    if (cnt->overflow || tot == 0) return;  // uniform across the workgroup
    pre[threadIdx.x + 1] = ex + t;
    if (threadIdx.x == 0) pre[0] = 0;
    own[threadIdx.x] = 0u;
    srec[threadIdx.x] = rec;
    if (t) {
        const ViewParams& v = views[blk_view[rec / K1_THREADS]];
        const uint32_t nx = tr.y & 0xffffu;
        sx0[threadIdx.x] = tr.x & 0xffffu;
        snx[threadIdx.x] = nx;
        sinx[threadIdx.x] = 1.0f / (float)nx;
        stb[threadIdx.x] = v.tile_base;
        // tiles_x of the view, packed with the first row
        stx[threadIdx.x] = (tr.x >> 16) | ((uint32_t)v.tiles_x << 16);
    }
    __syncthreads();
    const uint32_t base = blk_off[blockIdx.x];
    // Output slots in rounds of 256.  The owner of slot j is the last
    // Gaussian e whose first slot is at or before j: every Gaussian marks its
    // first slot in the round it falls in with (round << 8) | e, and a
    // prefix maximum over the round's slots, started from the previous
    // round's last owner, gives each slot's owner.  Marks of earlier rounds
    // are smaller than any tag of the current one, so `own` is never cleared.
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t carry = 0;  // owner of the slot before the round
    for (uint32_t j0 = 0, m = 0; j0 < tot; j0 += K1_THREADS, ++m) {
        if (t && (ex >> 8) == m) own[ex & (K1_THREADS - 1)] = (m << 8) | threadIdx.x;
        __syncthreads();
        const uint32_t incl = wave_incl_max(own[threadIdx.x]);
        if (lane == 63) wmax[w] = incl;
        __syncthreads();
        uint32_t o = max(incl, (m << 8) | carry), all = (m << 8) | carry;
#pragma unroll
        for (uint32_t v = 0; v < K1_THREADS / 64; ++v) {
            const uint32_t x = wmax[v];
            if (v < w) o = max(o, x);
            all = max(all, x);
        }
        carry = all & 0xffu;
        const uint32_t j = j0 + threadIdx.x;
        if (j >= tot) continue;
        const uint32_t e = o & 0xffu;
        const uint32_t k = j - pre[e];
        const uint32_t nx = snx[e];
        // k / nx through the FP32 reciprocal, corrected to the exact quotient
        uint32_t q = (uint32_t)((float)k * sinx[e]);
        if (q * nx > k) --q;
        if ((q + 1) * nx <= k) ++q;
        const uint32_t ty = (stx[e] & 0xffffu) + q, tx = sx0[e] + (k - q * nx);
        const uint32_t tiles_x = stx[e] >> 16;
        const uint32_t r = srec[e];
        tile_out[base + j] = stb[e] + ty * tiles_x + tx;
        val_out[base + j] = r;
        if (DEPTH) depth_out[base + j] = zkey[r];
    }
}


// ------------------------------------------------- tighter tile culling
// Whether a Gaussian can reach the skip threshold (alpha >= 1/255) at some
// pixel centre of a tile: the exact maximum of its exponent
// e(d) = A dx^2 + B dx dy + C dy^2 + L over the rectangle of the tile's pixel
// centres inside the frame (as in the blend's block test: the centre when it
// lies inside, else the better of the two faces facing it, each maximised at a
// clamped stationary point), compared with the threshold less the blend's
// margin, so a dropped tile is one every pixel of it would skip.  Plain FP32
// operations only (IEEE division, no fused or approximate ones), in this
// order, so a CPU reference reproduces every decision bit for bit.
// (ox, oy): the tile's pixel origin; (cw, ch): its pixels inside the frame.
__device__ __forceinline__ bool tile_reaches(float uhi, float vhi, float ulo, float vlo, float A, float B, float C,
                                             float L, float ox, float oy, float cw, float ch) {
    const float u = (uhi - ox) + ulo, v = (vhi - oy) + vlo;
    const float dx0 = 0.5f - u, dx1 = (cw - 0.5f) - u;
    const float dy0 = 0.5f - v, dy1 = (ch - 0.5f) - v;
    if (!(A < 0.0f && C < 0.0f && B * B < (4.0f * A) * C)) return true;  // not concave: keep it
    float q = 0.0f;
    if (!(dx0 <= 0.0f && dx1 >= 0.0f && dy0 <= 0.0f && dy1 >= 0.0f)) {
        const float cx = dx1 < 0.0f ? dx1 : dx0;
        const float sy = fminf(fmaxf((-B * cx) / (2.0f * C), dy0), dy1);
        const float ex = (A * cx + B * sy) * cx + (C * sy) * sy;
        const float cy = dy1 < 0.0f ? dy1 : dy0;
        const float sx = fminf(fmaxf((-B * cy) / (2.0f * A), dx0), dx1);
        const float ey = (C * cy + B * sx) * cy + (A * sx) * sx;
        q = fmaxf(ex, ey);
    }
    const float r2 = fmaxf(dx0 * dx0, dx1 * dx1) + fmaxf(dy0 * dy0, dy1 * dy1);
    const float margin = 0.02f + (1e-5f * ((fabsf(A) + fabsf(B)) + fabsf(C))) * r2;
    return !(q + L < LOG2_ALPHA_MIN - margin);  // keeps NaN
}

// The tile-culled duplicates: the same enumeration of (Gaussian, tile in its
// rectangle) slots as k_duplicate, each kept only when tile_reaches says so.
// COUNT: per block of 256 depth-ordered Gaussians, the number of kept entries
// (block_cnt).  Otherwise the kept entries are written in slot order,
// compacted, from the block's offset (blk_off, the exclusive scan of the
// counts).  The records already hold the FP64 conics of the near-singular
// Gaussians (patched by k_compact), so both launches test the final
// coefficients.
template <bool COUNT, bool DEPTH>
__global__ __launch_bounds__(K1_THREADS) void k_duplicate_culled(
    const uint32_t* __restrict__ sorted_rec, const uint32_t* __restrict__ sorted_packed,
    const uint32_t* __restrict__ zkey, const uint32_t* __restrict__ blk_off, uint32_t* __restrict__ block_cnt,
    const uint32_t* __restrict__ blk_view, const Counters* __restrict__ cnt, const ViewParams* __restrict__ views,
    const Rec* __restrict__ recs, int tile_w, int tile_h, uint32_t* __restrict__ tile_out,
    uint32_t* __restrict__ val_out, uint32_t* __restrict__ depth_out) {
    __shared__ uint32_t red[K1_THREADS / 64];
    __shared__ uint32_t pre[K1_THREADS + 1];
    __shared__ uint32_t srec[K1_THREADS], spk[K1_THREADS], stb[K1_THREADS], swh[K1_THREADS];
    __shared__ float4 sr0[K1_THREADS], sr1[K1_THREADS];
    __shared__ uint32_t own[K1_THREADS];
    __shared__ uint32_t wmax[K1_THREADS / 64];
    const uint32_t i = blockIdx.x * K1_THREADS + threadIdx.x;
    const uint32_t V = cnt->overflow ? 0u : cnt->visible;
    uint32_t rec = 0, p = 0, t = 0;
    if (i < V) {
        rec = sorted_rec[i];
        p = sorted_packed[i];
        t = rect_count(p);
    }
    uint32_t tot;
    const uint32_t ex = block_excl_scan<K1_THREADS>(t, red, &tot);
    if (!COUNT && (cnt->overflow || tot == 0)) return;  // uniform across the workgroup
    pre[threadIdx.x + 1] = ex + t;
    if (threadIdx.x == 0) pre[0] = 0;
    own[threadIdx.x] = 0u;
    srec[threadIdx.x] = rec;
    spk[threadIdx.x] = p;
    if (t) {
        const ViewParams& v = views[blk_view[rec / K1_THREADS]];
        stb[threadIdx.x] = v.tile_base;
        swh[threadIdx.x] = (uint32_t)v.width | ((uint32_t)v.height << 16);
        sr0[threadIdx.x] = recs[rec].r0;
        sr1[threadIdx.x] = recs[rec].r1;
    }
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t base = COUNT ? 0u : blk_off[blockIdx.x];
    uint32_t kept_before = 0;  // kept entries of this block in earlier rounds
    uint32_t carry = 0;
    for (uint32_t j0 = 0, m = 0; j0 < tot; j0 += K1_THREADS, ++m) {
        if (t && (ex >> 8) == m) own[ex & (K1_THREADS - 1)] = (m << 8) | threadIdx.x;
        __syncthreads();
        const uint32_t incl = wave_incl_max(own[threadIdx.x]);
        if (lane == 63) wmax[w] = incl;
        __syncthreads();
        uint32_t o = max(incl, (m << 8) | carry), all = (m << 8) | carry;
#pragma unroll
        for (uint32_t vv = 0; vv < K1_THREADS / 64; ++vv) {
            const uint32_t x = wmax[vv];
            if (vv < w) o = max(o, x);
            all = max(all, x);
        }
        carry = all & 0xffu;
        const uint32_t j = j0 + threadIdx.x;
        bool keep = false;
        uint32_t tile = 0, r = 0;
        if (j < tot) {
            const uint32_t e = o & 0xffu;
            const uint32_t k = j - pre[e];
            const uint32_t pk = spk[e];
            const uint32_t x0 = pk & 0xffu, y0 = (pk >> 8) & 0xffu;
            const uint32_t nx = ((pk >> 16) & 0xffu) - x0 + 1u;
            const uint32_t q = k / nx;
            const uint32_t ty = y0 + q, tx = x0 + (k - q * nx);
            const uint32_t wh = swh[e];
            const int W = (int)(wh & 0xffffu), H = (int)(wh >> 16);
            const int px = (int)tx * tile_w, py = (int)ty * tile_h;
            const float4 a = sr0[e], c = sr1[e];
            keep = tile_reaches(a.x, a.y, a.z, a.w, c.x, c.y, c.z, c.w, (float)px, (float)py,
                                (float)min(tile_w, W - px), (float)min(tile_h, H - py));
            const int tiles_x = (W + tile_w - 1) / tile_w;
            tile = stb[e] + ty * (uint32_t)tiles_x + tx;
            r = srec[e];
        }
        uint32_t kept_round;
        const uint32_t kex = block_excl_scan<K1_THREADS>(keep ? 1u : 0u, red, &kept_round);
        if (!COUNT && keep) {
            const uint32_t pos = base + kept_before + kex;
            tile_out[pos] = tile;
            val_out[pos] = r;
            if (DEPTH) depth_out[pos] = zkey[r];
        }
        kept_before += kept_round;
    }
    if (COUNT && threadIdx.x == 0) block_cnt[blockIdx.x] = kept_before;
}

// ------------------------------------------------- bucketed depth sort
// The depth order of each view's visible records in four launches: records
// counted per (segment, bucket), the counts scanned, the records scattered to
// their buckets (in any order), and every bucket sorted in LDS by (depth key,
// record), which makes the order the stable one.  A bucket is a range of
// depth keys, every bucket holding about the same number of records: the
// boundaries come from the distribution of one sample per 64 records (a
// histogram of the samples' keys, and linear interpolation inside its bins; or,
// where many depths are nearly equal, order statistics of the samples).
// What bounds it: at 3M Gaussians the bytes (keys read twice, 16 bytes
// written and read per visible record) take about a third of the time, the
// launches and the workgroups' chains the rest; so nothing is ranked but in
// the last step, where a record meets only the few of its own bin.  Measured
// against the compaction and three radix passes of 9-bit digits (twelve
// launches with the scans): 20k Gaussians 73 -> 25 us, 1M 71 -> 32 us, 3M
// (1.5M visible) 108 -> 63 us, 96M records of 32 views 1.98 -> 1.55 ms.
constexpr int BUCKET_THREADS = 1024;
constexpr int BUCKET_SORT_THREADS = 512;

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return v;
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
    return v;
}
// Segment of workgroup `wg` of a pass: consecutive workgroup ids go
// round-robin to the 8 XCDs, so XCD x is given a contiguous run of segments
// (the runs of one digit written by neighbouring segments then meet in one
// L2 and leave it as whole cache lines).
__device__ __forceinline__ int xcd_segment(int wg, int nb) {
    const int per = nb >> 3, rem = nb & 7, x = wg & 7;
    return x * per + min(x, rem) + (wg >> 3);
}

__device__ __forceinline__ int bit_length(uint32_t v) { return 32 - __clz((int)v); }

// The view that owns number i of a numbering through the views (`base`: the
// view's first number).
template <class F>
__device__ __forceinline__ int view_of(uint32_t i, int nviews, F&& base) {
    int lo = 0, hi = nviews - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (base(mid) <= i) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Bucket of a depth key: the share of the samples below it, times the bucket
// count.  A non-decreasing function of the key.
struct KeyMap {
    uint32_t lo, hi, shift, scale;
};
__device__ __forceinline__ uint32_t key_bucket(uint32_t key, const uint32_t* cdf, const KeyMap& m, uint32_t nbkt) {
    const uint32_t d = min(max(key, m.lo), m.hi) - m.lo;
    const uint32_t bin = d >> m.shift;  // < BUCKET_BINS
    const uint32_t frac = d & ((1u << m.shift) - 1u);
    const uint32_t f16 = m.shift > 16 ? frac >> (m.shift - 16) : frac << (16 - m.shift);
    const uint32_t c0 = cdf[bin], c1 = cdf[bin + 1];  // at most BUCKET_SAMPLES = 2^14
    const uint32_t pos = (c0 << 16) + (c1 - c0) * f16;
    return min(__umulhi(pos, m.scale), nbkt - 1u);
}

// Bitonic sort of n2 64-bit words in LDS (a power of two from sort_min to SORT_MAX,
// padded with all ones by the caller) by the whole workgroup: a wave sorts
// sort_min of them in its registers (neighbours in a lane, lanes met by
// permutes), and the waves meet through LDS, where a word's place is its (wave,
// register, lane).  Of the 78 steps of 4096 words 6 (512 threads) or 10 (1024) are
// in LDS behind barriers.  A frame of 17k Gaussians at 960x540, 3500 of them at one
// depth, takes 131 us; with every step in LDS 155, by the radix passes 151, without
// a crowded bucket 86.
constexpr int SORT_MAX = 4096;
template <int NT>
__device__ constexpr uint32_t sort_min() {
    return 64 * (SORT_MAX / NT);
}
template <int NT>
__device__ void bitonic_sort(uint64_t* a, uint32_t n2) {
    constexpr int E = SORT_MAX / NT;  // words a lane
    constexpr uint32_t PER_WAVE = sort_min<NT>();
    const uint32_t lane = fresh(threadIdx.x) & 63u;
    const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool on = c * PER_WAVE < n2;  // uniform over the wave
    const uint32_t i0 = c * PER_WAVE + lane * E;  // number of the lane's first word
    uint64_t* const mine = a + c * PER_WAVE + lane;
    uint64_t x[E];
    auto lanes_step = [&](uint32_t j, bool up) {  // words j >= E apart in the wave
        const bool least = up == ((i0 & j) == 0u);
#pragma unroll
        for (int r = 0; r < E; ++r) {
            const uint64_t y = __shfl_xor((unsigned long long)x[r], (int)(j / E), 64);
            x[r] = (y < x[r]) == least ? y : x[r];
        }
    };
    auto lane_step = [&](int j, int r, bool up) {  // words r and r + j of the lane
        const uint64_t p = x[r], q = x[r + j];
        const bool swap = (p > q) == up;
        x[r] = swap ? q : p;
        x[r + j] = swap ? p : q;
    };
    auto lane_steps = [&](bool up) {
#pragma unroll
        for (int j = E / 2; j > 0; j >>= 1)
#pragma unroll
            for (int r = 0; r < E; ++r)
                if ((r & j) == 0) lane_step(j, r, up);
    };
    __syncthreads();
    if (on) {
#pragma unroll
        for (int r = 0; r < E; ++r) x[r] = mine[r * 64];  // any word to any place at first
#pragma unroll
        for (int k = 2; k < E; k <<= 1)
#pragma unroll
            for (int j = k / 2; j > 0; j >>= 1)
#pragma unroll
                for (int r = 0; r < E; ++r)
                    if ((r & j) == 0) lane_step(j, r, (r & k) == 0);
        lane_steps((i0 & E) == 0u);
#pragma unroll 1
        for (uint32_t k = 2 * E; k <= PER_WAVE; k <<= 1) {
            const bool up = (i0 & k) == 0u;
#pragma unroll 1
            for (uint32_t j = k / 2; j >= (uint32_t)E; j >>= 1) lanes_step(j, up);
            lane_steps(up);
        }
    }
#pragma unroll 1
    for (uint32_t k = 2 * PER_WAVE; k <= n2; k <<= 1) {
        const bool up = (i0 & k) == 0u;
#pragma unroll 1
        for (uint32_t j = k / 2; j >= PER_WAVE; j >>= 1) {
            __syncthreads();
            if (on) {
#pragma unroll
                for (int r = 0; r < E; ++r) mine[r * 64] = x[r];
            }
            __syncthreads();
            if (on) {
                const uint64_t* other = a + (c ^ (j / PER_WAVE)) * PER_WAVE + lane;
                const bool least = up == ((i0 & j) == 0u);
#pragma unroll
                for (int r = 0; r < E; ++r) {
                    const uint64_t y = other[r * 64];
                    x[r] = (y < x[r]) == least ? y : x[r];
                }
            }
        }
        if (on) {
#pragma unroll 1
            for (uint32_t j = PER_WAVE / 2; j >= (uint32_t)E; j >>= 1) lanes_step(j, up);
            lane_steps(up);
        }
    }
    __syncthreads();
    if (on) {
#pragma unroll
        for (int r = 0; r < E; ++r) a[i0 + r] = x[r];
    }
    __syncthreads();
}

// A view whose samples crowd (over `shares` times the mean + 8 of them in one bucket: a flat model seen face on, say) is parted by order statistics of the samples'
// (depth key, record) words instead: SPLIT_MAX - 1 of them at most, in the place
// of the distribution and marked by KeyMap::shift.  Equal depths are then parted
// by record, and no bucket is long however the depths lie.  Allocation-free
// frames of 17k / 200k Gaussians of one depth at 960x540 take 78 / 126 us; in one
// bucket 141 / 1987, by the radix passes 160 / 202 (with spread depths 66 / 106).
constexpr uint32_t SPLIT_MAX = BUCKET_BINS / 2;
constexpr uint32_t SPLIT_SAMPLES = 4096;
constexpr uint32_t KEYMAP_SPLIT = 0xffffffffu;
__device__ __forceinline__ uint32_t split_bucket(uint32_t key, uint32_t rec, const uint64_t* split) {
    const uint64_t x = ((uint64_t)key << 32) | rec;
    uint32_t pos = 0;
#pragma unroll
    for (uint32_t s = SPLIT_MAX / 2; s > 0; s >>= 1) pos += split[pos + s - 1] <= x ? s : 0u;
    return pos;
}

// Per segment of a view's records: the records of each bucket (rows) and the
// smallest and largest visible key.  In a plan of one round of workgroups each
// forms the view's sample distribution itself (the first one of the view also
// stores it for the scatter): the samples are 1/64 of the keys, and a launch of
// its own would cost more (FORM).  In larger plans a workgroup per view forms it
// first (FORM_ONLY), and the segments read it (READ): 32 views of 3M records in
// 5888 segments 226 us in two launches, 278 formed by all.
// All share the clearing of zl.  64 VGPRs: two workgroups per CU.
// Bound by latency (3M records: 512 workgroups of six rounds, 8192 samples
// each); the preprocess blocks' totals are summed segment by segment: one
// workgroup for all 11720 blocks of 3M records was the last to end.
// 3M records: 25 us with that workgroup, 18 without.
enum SampleMode { FORM, FORM_ONLY, READ };
constexpr uint32_t BUCKET_FORM_SEGMENTS = 512;  // a round: two workgroups on each of 256 compute units
// SPLIT: views with over `shares` times the mean + 8 samples in a bucket are parted
// by order statistics.
template <SampleMode MODE, bool SPLIT>
__global__ __launch_bounds__(BUCKET_THREADS, 8) void k_bucket_count(PreOut o, BucketMem b,
                                                                    const ViewParams* __restrict__ views, int nviews,
                                                                    uint32_t nseg, uint32_t seg_len, uint32_t shares,
                                                                    ZeroList zl) {
    constexpr int NT = BUCKET_THREADS, NW = NT / 64, SPT = BUCKET_SAMPLES / NT, RPT = 6;
    static_assert(BUCKET_BINS == 2 * NT, "two bins per thread");
    __shared__ __align__(8) uint32_t cdf[BUCKET_BINS + 1];
    __shared__ uint32_t hist[BUCKET_MAX];
    __shared__ uint32_t red[NW], red2[NW], tot32[2];
    __shared__ unsigned long long tot64[2];
    __shared__ uint64_t words[SPLIT && MODE != READ ? SPLIT_SAMPLES : 1];
    __shared__ uint32_t crowd[2], nwords;
    static_assert(SPLIT_SAMPLES <= SORT_MAX, "sorted at once");
    static_assert(SPLIT_MAX == NT && SPLIT_MAX * 2 <= BUCKET_BINS, "a thread per splitter, in the distribution's place");
    uint64_t* const split = reinterpret_cast<uint64_t*>(cdf);
    static_assert(NT / 4 >= SEG_MAX / K1_THREADS, "a thread of the first waves per preprocess block");
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (MODE != FORM_ONLY) {
#pragma unroll
        for (int k = 0; k < ZeroList::N; ++k)
            for (uint32_t i = blockIdx.x * NT + t; i < zl.n[k]; i += gridDim.x * NT) zl.p[k][i] = 0u;
        if (blockIdx.x >= nseg) return;  // no records at all: the clearing only
    }
    const int vi = MODE == FORM_ONLY ? (int)blockIdx.x
                                     : view_of(blockIdx.x, nviews, [&](int i) { return views[i].seg_base; });
    const ViewParams& v = views[vi];
    const uint32_t seg = MODE == FORM_ONLY ? 0u : blockIdx.x - v.seg_base, nbkt = v.nbkt;
    const uint32_t r0 = v.rec_base + seg * seg_len, r1 = min(r0 + seg_len, v.rec_base + v.n_pad);

    // the first records are on their way while the samples are sorted out
    uint32_t key[RPT];
    bool vis[RPT];
    auto load = [&](uint32_t i0) {
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const uint32_t i = i0 + (uint32_t)(k * NT + t);
            vis[k] = i < r1 && ((o.vmask[i >> 6] >> lane) & 1ull);
            key[k] = i < r1 ? o.zkey[i] : 0u;
        }
    };
    if (MODE != FORM_ONLY) load(r0);
    if (t < 2) {
        tot64[t] = 0ull;
        tot32[t] = 0u;
        crowd[t] = 0u;
    }
    // a preprocess block's counts, and their sums over the segment
    struct BlockCounts {
        uint32_t d, t, n, f;
    };
    auto block_counts = [&] {
        BlockCounts c{0, 0, 0, 0};
        if (MODE != FORM_ONLY && (uint32_t)t < (r1 - r0) / K1_THREADS) {
            const uint32_t i = r0 / K1_THREADS + (uint32_t)t;
            c = BlockCounts{o.blk_sum[i], o.blk_tiles[i], o.blk_vis[i], o.blk_fb[i]};
        }
        return c;
    };
    auto add_totals = [&](const BlockCounts& c) {
        if (MODE == FORM_ONLY || w >= NW / 4) return;
        const uint64_t d = wave_sum_u64(c.d), tl = wave_sum_u64(c.t);
        const uint32_t n = wave_sum(c.n), f = wave_sum(c.f);
        if (lane == 0) {
            atomicAdd(&tot64[0], (unsigned long long)d);
            atomicAdd(&tot64[1], (unsigned long long)tl);
            atomicAdd(&tot32[0], n);
            atomicAdd(&tot32[1], f);
        }
    };
    KeyMap m;
    uint32_t lo = 0xffffffffu, hi = 0u;
    if constexpr (MODE == READ) {
        const uint32_t* src = b.cdf + (size_t)vi * BUCKET_CDF_WORDS;
        m = KeyMap{src[BUCKET_BINS + 1], src[BUCKET_BINS + 2], src[BUCKET_BINS + 3], src[BUCKET_BINS + 4]};
        for (int i = t; i <= BUCKET_BINS; i += NT) cdf[i] = src[i];
        for (uint32_t i = t; i < nbkt; i += NT) hist[i] = 0u;
        const BlockCounts bc = block_counts();
        __syncthreads();
        add_totals(bc);
    } else {
        // the samples' distribution
        // (four samples per bucket: a bucket of twice the mean size is rare, and
        // one of more than BUCKET_SORT_CAP only costs time)
        const uint32_t nsamp_all = v.n_pad / 64;
        const uint32_t nsamp = min(nsamp_all, min((uint32_t)BUCKET_SAMPLES, max(2048u, 4u * nbkt)));
        const float stride = nsamp ? (float)nsamp_all / (float)nsamp : 0.0f;
        // (the 64 records that sample i stands for)
        auto wave_of = [&](uint32_t i) { return v.rec_base / 64 + min((uint32_t)((float)i * stride), nsamp_all - 1u); };
        uint32_t sk[SPT];
#pragma unroll
        for (int k = 0; k < SPT; ++k) {
            const uint32_t i = (uint32_t)(k * NT + t);
            sk[k] = 0xffffffffu;
            if (i < nsamp) sk[k] = o.sample[wave_of(i)];
            if (sk[k] != 0xffffffffu) {
                lo = min(lo, sk[k]);
                hi = max(hi, sk[k]);
            }
        }
        for (int i = t; i < BUCKET_BINS; i += NT) cdf[i] = 0u;
        for (uint32_t i = t; i < nbkt; i += NT) hist[i] = 0u;
        lo = wave_min(lo);
        hi = wave_max(hi);
        if (lane == 0) {
            red[w] = lo;
            red2[w] = hi;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            lo = min(lo, red[k]);
            hi = max(hi, red2[k]);
        }
        m.lo = lo <= hi ? lo : 0u;
        m.hi = lo <= hi ? hi : 0u;
        m.shift = (uint32_t)max(0, bit_length(m.hi - m.lo) - 11);
        static_assert(BUCKET_BINS == 1 << 11, "eleven bits of the samples' range");
#pragma unroll
        for (int k = 0; k < SPT; ++k)
            if (sk[k] != 0xffffffffu) atomicAdd(&cdf[(sk[k] - m.lo) >> m.shift], 1u);
        const BlockCounts bc = block_counts();
        __syncthreads();
        const uint32_t c0 = cdf[2 * t], c1 = cdf[2 * t + 1];
        uint32_t total;
        const uint32_t ex = block_excl_scan<NT>(c0 + c1, red, &total);
        cdf[2 * t] = ex;
        cdf[2 * t + 1] = ex + c0;
        if (t == 0) cdf[BUCKET_BINS] = total;
        m.scale = total ? (nbkt << 16) / total : 0u;
        const uint32_t mean = nbkt ? total / nbkt : 0u;
        const uint32_t most = shares * mean + 8u;
        // a bucket holds its share and parts of two bins at most
        if (SPLIT && max(c0, c1) > (most - mean) / 2u) crowd[0] = 1u;
        add_totals(bc);
        __syncthreads();
        if constexpr (SPLIT) {
            if (crowd[0]) {  // uniform
                for (uint32_t i = t; i < nsamp; i += NT) {
                    const uint32_t key = o.sample[wave_of(i)];
                    if (key != 0xffffffffu) atomicAdd(&hist[key_bucket(key, cdf, m, nbkt)], 1u);
                }
                __syncthreads();
                for (uint32_t i = t; i < nbkt; i += NT) {
                    if (hist[i] > most) crowd[1] = 1u;
                    hist[i] = 0u;
                }
                __syncthreads();
            }
            if (crowd[1]) {  // uniform
                const uint32_t every = (nsamp + SPLIT_SAMPLES - 1u) / SPLIT_SAMPLES, ns = (nsamp + every - 1u) / every;
                uint32_t n2 = sort_min<NT>(), have = 0;
                while (n2 < ns) n2 <<= 1;
                if (t == 0) nwords = 0u;
                __syncthreads();
                for (uint32_t k = t; k < n2; k += NT) {
                    uint64_t x = ~0ull;
                    if (k < ns) {
                        const uint32_t wid = wave_of(k * every), key = o.sample[wid];
                        if (key != 0xffffffffu) {
                            x = ((uint64_t)key << 32) | (wid * 64u + sample_lane(o.vmask[wid], wid));
                            ++have;
                        }
                    }
                    words[k] = x;
                }
                have = wave_sum(have);
                if (lane == 0) atomicAdd(&nwords, have);
                bitonic_sort<NT>(words, n2);
                const uint32_t parts = min(nbkt, SPLIT_MAX);
                split[t] = (uint32_t)t + 1u < parts && nwords ? words[((uint32_t)t + 1u) * nwords / parts] : ~0ull;
                m.shift = KEYMAP_SPLIT;
                __syncthreads();
            }
        }
        if (MODE == FORM_ONLY || seg == 0) {
            uint32_t* out = b.cdf + (size_t)vi * BUCKET_CDF_WORDS;
            for (uint32_t i = fresh(t); i <= BUCKET_BINS; i += NT) out[i] = cdf[i];
            if (t < 4) out[BUCKET_BINS + 1 + t] = t == 0 ? m.lo : t == 1 ? m.hi : t == 2 ? m.shift : m.scale;
        }
    }
    if (MODE == FORM_ONLY) return;

    // the segment's visible records
    lo = 0xffffffffu;
    hi = 0u;
    auto count = [&](auto&& bucket) {
        for (uint32_t i0 = r0; i0 < r1; i0 += NT * RPT) {
            if (i0 != r0) load(i0);
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                if (vis[k]) {
                    atomicAdd(&hist[bucket(key[k], i0 + (uint32_t)(k * NT + t))], 1u);
                    lo = min(lo, key[k]);
                    hi = max(hi, key[k]);
                }
        }
    };
    if (SPLIT && m.shift == KEYMAP_SPLIT) count([&](uint32_t k, uint32_t i) { return split_bucket(k, i, split); });
    else count([&](uint32_t k, uint32_t) { return key_bucket(k, cdf, m, nbkt); });
    lo = wave_min(lo);
    hi = wave_max(hi);
    __syncthreads();
    if (lane == 0) {
        red[w] = lo;
        red2[w] = hi;
    }
    __syncthreads();
    if (t == 0) {
        for (int k = 0; k < NW; ++k) {
            lo = min(lo, red[k]);
            hi = max(hi, red2[k]);
        }
        b.seg[blockIdx.x] = SegTotals{tot64[0], tot64[1], tot32[0], tot32[1], lo, hi};
    }
    uint32_t* row = b.rows + v.row_base + (size_t)seg * nbkt;
    for (uint32_t i = fresh(t); i < nbkt; i += NT) row[i] = hist[i];
}

// Exclusive prefixes down the columns of a row-major nrows x ncols array
// (rows `stride` words apart), in place, for the CW columns from c0 on, by
// 1024 threads: 1024 / CW groups of consecutive rows, a lane per column, the
// first U rows of a group kept in registers (all loads in flight at once, and
// usually all there are); a wave then scans the groups of a column or two.
// Per column its total (tot) and the totals of the chunk's columns before it
// (start_in), and the chunk's total.
template <uint32_t CW, uint32_t U>
__device__ __forceinline__ void column_scan(uint32_t* a, uint32_t nrows, uint32_t stride, uint32_t ncols, uint32_t c0,
                                            uint32_t* __restrict__ start_in, uint32_t* __restrict__ tot,
                                            uint32_t* __restrict__ chunk, uint32_t* lds) {
    constexpr uint32_t G = 1024 / CW, ROW = CW + 1;
    static_assert((CW == 16 && G == 64) || (CW == 32 && G == 32), "a wave scans the groups of one column or two");
    const uint32_t c = threadIdx.x % CW, g = threadIdx.x / CW;
    const bool in = c0 + c < ncols;
    const uint32_t per = (nrows + G - 1u) / G, b0 = min(nrows, g * per), b1 = in ? min(nrows, b0 + per) : b0;
    uint32_t* p = a + c0 + c;
    uint32_t x[U], sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < U; ++k) x[k] = b0 + k < b1 ? p[(size_t)(b0 + k) * stride] : 0u;
#pragma unroll
    for (uint32_t k = 0; k < U; ++k) sum += x[k];
    for (uint32_t r = b0 + U; r < b1; ++r) sum += p[(size_t)r * stride];
    lds[g * ROW + c] = sum;
    __syncthreads();
    {
        const uint32_t l = threadIdx.x & 63u, w = threadIdx.x >> 6;
        const uint32_t col = G == 64 ? w : 2 * w + (l >> 5), row = l % G;
        const uint32_t v = lds[row * ROW + col];
        uint32_t incl = wave_incl_scan(v);
        if (G == 32) {
            const uint32_t low = readlane(incl, 31);
            incl -= l >= 32u ? low : 0u;
        }
        lds[row * ROW + col] = incl - v;
        if (row == G - 1) lds[G * ROW + col] = incl;  // the column's total
    }
    __syncthreads();
    uint32_t run = lds[g * ROW + c];
#pragma unroll
    for (uint32_t k = 0; k < U; ++k) {
        if (b0 + k < b1) p[(size_t)(b0 + k) * stride] = run;
        run += x[k];
    }
    for (uint32_t r = b0 + U; r < b1; ++r) {
        const uint32_t y = p[(size_t)r * stride];
        p[(size_t)r * stride] = run;
        run += y;
    }
    if (threadIdx.x < 64) {
        const uint32_t v = threadIdx.x < CW ? lds[G * ROW + threadIdx.x] : 0u;
        const uint32_t incl = wave_incl_scan(v);
        if (threadIdx.x < CW && in) {
            start_in[c] = incl - v;
            tot[c] = v;
        }
        if (threadIdx.x == 63) *chunk = incl;
    }
}

// Cost of a unit of the tile placement when `total` is split into about
// nunits units (at most one more per view), and the units of a view.
__device__ __forceinline__ uint32_t unit_cost(uint64_t total, uint32_t nunits) {
    const uint64_t c = (uint64_t)(((double)total + (double)(nunits - 1)) / (double)nunits);
    return c < TILE_UNIT_MIN ? (uint32_t)TILE_UNIT_MIN : c > 0xffffffffull ? 0xffffffffu : (uint32_t)c;
}
__device__ __forceinline__ uint32_t units_for(uint64_t total, uint32_t cost) {
    return (uint32_t)(((double)total + (double)(cost - 1)) / (double)cost);
}

// A frame whose depth keys span 2^27 or more (about 16 octaves of depth).
__device__ __forceinline__ bool depth_wide(uint32_t lo, uint32_t hi) {
    return lo <= hi && ((hi - (lo & ~511u)) >> 27) != 0u;
}

// Column scans of the (segment, bucket) counts; the last workgroup sets the
// frame's counters and the views' first positions.
__global__ __launch_bounds__(1024) void k_bucket_scan(BucketMem b, const ViewParams* __restrict__ views, int nviews,
                                                      uint32_t nseg, uint32_t nchunks, Counters* cnt, uint32_t cap,
                                                      bool flag_wide, bool flag_crowd, uint32_t nunits) {
    __shared__ uint32_t lds[(1024 / COL_CHUNK + 1) * (COL_CHUNK + 1)];
    if (blockIdx.x < nchunks) {
        const uint32_t c0 = blockIdx.x * COL_CHUNK;
        const int vi = view_of(c0, nviews, [&](int i) { return views[i].bkt_base; });
        const ViewParams& v = views[vi];
        column_scan<COL_CHUNK, 16>(b.rows + v.row_base, v.nseg, v.nbkt, v.nbkt, c0 - v.bkt_base, b.start_in + c0, b.tot + c0,
                    b.chunk + blockIdx.x, lds);
        // (a thread reads the total that it wrote)
        if (flag_crowd && threadIdx.x < COL_CHUNK && c0 - v.bkt_base + threadIdx.x < v.nbkt &&
            b.tot[c0 + threadIdx.x] > max((uint32_t)BUCKET_SORT_CAP, v.n_pad / v.nbkt * CROWD_SHARES))
            atomicOr(&cnt->overflow, FLAG_CROWDED);
        return;
    }
    uint32_t lo = 0xffffffffu, hi = 0u;
    for (uint32_t i = threadIdx.x; i < nseg; i += 1024) {
        lo = min(lo, b.seg[i].lo);
        hi = max(hi, b.seg[i].hi);
    }
    // a wave per view: its totals
    for (int i = (int)(threadIdx.x >> 6); i < nviews; i += 16) {
        uint64_t d = 0, tl = 0;
        uint32_t n = 0, f = 0;
        for (uint32_t k = threadIdx.x & 63u; k < views[i].nseg; k += 64) {
            const SegTotals sg = b.seg[views[i].seg_base + k];
            d += sg.dups;
            tl += sg.tiles;
            n += sg.visible;
            f += sg.fallbacks;
        }
        d = wave_sum_u64(d);
        tl = wave_sum_u64(tl);
        n = wave_sum(n);
        f = wave_sum(f);
        if ((threadIdx.x & 63) == 0) {
            b.vc[i].dups = d;
            b.vc[i].tiles = tl;
            b.vc[i].visible = n;
            b.vc[i].fallbacks = f;
        }
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    if ((threadIdx.x & 63) == 0) {
        lds[threadIdx.x >> 6] = lo;
        lds[16 + (threadIdx.x >> 6)] = hi;
    }
    __syncthreads();
    if (threadIdx.x >= 64) return;
    lo = wave_min(lds[threadIdx.x & 15]);
    hi = wave_max(lds[16 + (threadIdx.x & 15)]);
    // a lane per view: their first positions, then their units of the tile
    // placement
    uint64_t D = 0, P = 0;
    uint32_t V = 0, F = 0;
    for (int i0 = 0; i0 < nviews; i0 += 64) {
        const int i = i0 + (int)threadIdx.x;
        uint64_t d = i < nviews ? b.vc[i].dups : 0ull, tl = i < nviews ? b.vc[i].tiles : 0ull;
        const uint32_t vis = i < nviews ? b.vc[i].visible : 0u, f = i < nviews ? b.vc[i].fallbacks : 0u;
        const uint32_t incl = wave_incl_scan(vis);
        if (i < nviews) b.vc[i].start = V + incl - vis;
        V += readlane(incl, 63);
        F += wave_sum(f);
#pragma unroll
        for (int k = 32; k > 0; k >>= 1) {
            d += __shfl_xor((unsigned long long)d, k, 64);
            tl += __shfl_xor((unsigned long long)tl, k, 64);
        }
        D += d;
        P += tl;
    }
    const uint32_t uc = unit_cost(D + (uint64_t)TILE_BASE_COST * V, nunits);
    uint32_t ub = 0;
    for (int i0 = 0; i0 < nviews; i0 += 64) {
        const int i = i0 + (int)threadIdx.x;
        const uint32_t nu =
            i < nviews ? units_for(b.vc[i].dups + (uint64_t)TILE_BASE_COST * b.vc[i].visible, uc) : 0u;
        const uint32_t incl = wave_incl_scan(nu);
        if (i < nviews) {
            b.vc[i].ubase = ub + incl - nu;
            b.vc[i].nu = nu;
            b.vc[i].ucost = uc;
        }
        ub += readlane(incl, 63);
    }
    if (threadIdx.x == 0) {
        cnt->D = D > 0xffffffffull ? 0xffffffffu : (uint32_t)D;
        cnt->pairs = P > 0xffffffffull ? 0xffffffffu : (uint32_t)P;
        cnt->visible = V;
        cnt->fallbacks = F;
        // cleared by the launch before; other workgroups may have set FLAG_CROWDED
        atomicOr(&cnt->overflow, (D > (uint64_t)cap ? 1u : 0u) | (flag_wide && depth_wide(lo, hi) ? FLAG_WIDE : 0u));
        cnt->fb_listed = cnt->fb_list;
        cnt->fb_list = 0u;  // the next frame appends from zero
    }
}

// Records of the bucket chunks of a view before chunk `c`: at most 128 chunks.
__device__ __forceinline__ uint32_t chunks_before(const uint32_t* __restrict__ chunk, uint32_t c) {
    static_assert(BUCKET_MAX / COL_CHUNK <= 128, "two chunk totals per lane");
    const uint32_t l = lane_id();
    return wave_sum((l < c ? chunk[l] : 0u) + (l + 64u < c ? chunk[l + 64u] : 0u));
}

// Every visible record of a segment to the next free place of its bucket.
template <bool SPLIT>
__global__ __launch_bounds__(BUCKET_THREADS, 8) void k_bucket_scatter(PreOut o, BucketMem b,
                                                                      const ViewParams* __restrict__ views, int nviews,
                                                                      uint32_t nseg, uint32_t seg_len,
                                                                      const Counters* __restrict__ cnt) {
    constexpr int NT = BUCKET_THREADS, RPT = 6;
    __shared__ __align__(8) uint32_t cdf[BUCKET_BINS + 1];
    __shared__ uint32_t next[BUCKET_MAX], cpre[BUCKET_MAX / COL_CHUNK];
    if (cnt->overflow & (FLAG_WIDE | FLAG_CROWDED)) return;  // uniform: rendered again
    const int t = threadIdx.x, lane = t & 63;
    const int wg = xcd_segment((int)blockIdx.x, (int)nseg);  // neighbouring segments, whose elements meet, in one L2
    const int vi = view_of((uint32_t)wg, nviews, [&](int i) { return views[i].seg_base; });
    const ViewParams& v = views[vi];
    const uint32_t seg = (uint32_t)wg - v.seg_base, nbkt = v.nbkt;
    const int cells = v.cells;
    const uint32_t r0 = v.rec_base + seg * seg_len, r1 = min(r0 + seg_len, v.rec_base + v.n_pad);
    // the first records are on their way while the buckets' positions are
    // formed (all records' rectangles: waiting for the mask would cost more)
    uint32_t key[RPT];
    uint2 rect[RPT];
    bool vis[RPT];
    auto load = [&](uint32_t i0) {
#pragma unroll
        for (int k = 0; k < RPT; ++k) {
            const uint32_t i = i0 + (uint32_t)(k * NT + t);
            vis[k] = i < r1 && ((o.vmask[i >> 6] >> lane) & 1ull);
            key[k] = i < r1 ? o.zkey[i] : 0u;
            rect[k] = i < r1 ? o.rect[i] : make_uint2(0u, 0u);
        }
    };
    load(r0);
    const uint32_t* src = b.cdf + (size_t)vi * BUCKET_CDF_WORDS;
    const KeyMap m{src[BUCKET_BINS + 1], src[BUCKET_BINS + 2], src[BUCKET_BINS + 3], src[BUCKET_BINS + 4]};
    for (int i = t; i <= BUCKET_BINS; i += NT) cdf[i] = src[i];
    if (t < 64) {
        // exclusive scan of the view's chunk totals
        const uint32_t nc = (nbkt + COL_CHUNK - 1) / COL_CHUNK, c0 = v.bkt_base / COL_CHUNK;
        const uint32_t x = 2u * t < nc ? b.chunk[c0 + 2 * t] : 0u, y = 2u * t + 1 < nc ? b.chunk[c0 + 2 * t + 1] : 0u;
        const uint32_t ex = wave_incl_scan(x + y) - x - y + b.vc[vi].start;
        cpre[2 * t] = ex;
        cpre[2 * t + 1] = ex + x;
    }
    __syncthreads();
    const uint32_t* row = b.rows + v.row_base + (size_t)seg * nbkt;
    for (uint32_t i = t; i < nbkt; i += NT) next[i] = cpre[i / COL_CHUNK] + b.start_in[v.bkt_base + i] + row[i];
    __syncthreads();
    auto scatter = [&](auto&& bucket) {
        for (uint32_t i0 = r0; i0 < r1; i0 += NT * RPT) {
            if (i0 != r0) load(i0);
#pragma unroll
            for (int k = 0; k < RPT; ++k)
                if (vis[k]) {
                    const uint32_t i = i0 + (uint32_t)(k * NT + t);
                    const uint32_t pos = atomicAdd(&next[bucket(key[k], i)], 1u);
                    b.elem[pos] = make_uint4(key[k], i, pack_rect(rect[k]), rect_cells(rect[k], cells));
                }
        }
    };
    if (SPLIT && m.shift == KEYMAP_SPLIT)
        scatter([&](uint32_t k, uint32_t i) { return split_bucket(k, i, reinterpret_cast<const uint64_t*>(cdf)); });
    else
        scatter([&](uint32_t k, uint32_t) { return key_bucket(k, cdf, m, nbkt); });
}

// One bucket sorted by (depth key, record).  Its elements are counted into
// bins of equal key ranges (of records, when all keys are equal), placed in
// LDS bin by bin, and each finds its rank among the few elements of its own
// bin.  Buckets with a crowded bin (many equal keys) take a bitonic sort
// instead.  Those of more than BUCKET_SORT_CAP elements are first placed bin by
// bin of their range of (key, record) words in the bucket's part of the
// outputs, and bins that fit together are sorted in LDS; a bin that does not
// fit goes window by window: as many of its smallest remaining elements as fit,
// found by counting over the bins of the remaining range (window by window alone
// its passes would grow with the square of the bucket).  That is the way of buckets
// of two to four shares, and of views of over 16M visible records, which have more
// than 4096 a bucket (34M: 8300, the launch 1.5 ms of 6.3).  The launch also recomputes
// the FP64 conics of the near-singular Gaussians, before anything reads the
// exponent coefficients.
__global__ __launch_bounds__(BUCKET_SORT_THREADS, 6) void k_bucket_sort(PreOut o, BucketMem b,
                                                                     const ViewParams* __restrict__ views, int nviews,
                                                                     const Counters* __restrict__ cnt,
                                                                     uint32_t* __restrict__ val,
                                                                     uint32_t* __restrict__ ext) {
    constexpr int NT = BUCKET_SORT_THREADS, NW = NT / 64, CAP = BUCKET_SORT_CAP, EPT = CAP / NT;
    constexpr int BINS = 2048, BPT = BINS / NT;
    static_assert(CAP <= SORT_MAX, "sorted at once");
    constexpr uint32_t CROWDED = 48;  // larger bins are left to the bitonic sort
    __shared__ uint64_t arr[CAP];
    __shared__ uint32_t bin[BINS + 1];
    __shared__ uint32_t red[NW], red2[NW];
    __shared__ uint64_t redlo[NW], redhi[NW];
    __shared__ uint32_t picked, fill;
    if (cnt->overflow & (FLAG_WIDE | FLAG_CROWDED)) return;  // uniform: rendered again
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    {
        const uint32_t nfb = min(cnt->fb_listed, o.fb_cap);
        for (uint32_t k = blockIdx.x * NT + t; k < nfb; k += gridDim.x * NT)
            conic_fp64(o.fb_list[k], views, o.blk_view, o.rec);
    }
    const int vi = view_of(blockIdx.x, nviews, [&](int i) { return views[i].bkt_base; });
    const ViewParams& v = views[vi];
    const uint32_t lb = blockIdx.x - v.bkt_base;
    if (lb >= v.nbkt) return;  // uniform: the views' buckets are numbered from multiples of COL_CHUNK
    const uint32_t n = b.tot[blockIdx.x];
    if (n == 0) {  // uniform
        if (t == 0) b.cost[blockIdx.x] = 0u;
        return;
    }
    // (scalar: the addresses formed from it are kept over the sort)
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(b.vc[vi].start + chunks_before(b.chunk + v.bkt_base / COL_CHUNK, lb / COL_CHUNK) + b.start_in[blockIdx.x]));
    const uint4* e = b.elem + first;
    // the bucket's placement cost, for the units of the tile placement
    auto store_cost = [&](uint32_t entries) {
        entries = block_sum<NT>(entries, red);
        if (t == 0) {
            const uint32_t c = entries + (uint32_t)TILE_BASE_COST * n;
            b.cost[blockIdx.x] = c;
            atomicAdd(&b.ccost[blockIdx.x / COL_CHUNK], (unsigned long long)c);
        }
    };
    val += first;
    ext += first;
    // with cells, a record is numbered inside its view, below the rectangle's cells
    const int cells = v.cells;
    const uint32_t rec0 = cells ? v.rec_base : 0u;
    if (n <= (uint32_t)CAP) {
        uint32_t key[EPT], rec[EPT], rc[EPT], be[EPT];
        uint32_t klo = 0xffffffffu, khi = 0u, rlo = 0xffffffffu, rhi = 0u;
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const uint32_t i = (uint32_t)(k * NT + t);
            key[k] = rec[k] = rc[k] = be[k] = 0u;
            if (i < n) {
                const uint4 x = e[i];
                key[k] = x.x;
                rec[k] = x.y;
                rc[k] = x.z;
                be[k] = x.w;
                klo = min(klo, x.x);
                khi = max(khi, x.x);
                rlo = min(rlo, x.y);
                rhi = max(rhi, x.y);
            }
        }
        {
            uint32_t entries = 0;
#pragma unroll
            for (int k = 0; k < EPT; ++k) entries += (uint32_t)(k * NT + t) < n ? rect_count(rc[k]) : 0u;
            store_cost(entries);
        }
#pragma unroll
        for (int k = 0; k < BPT; ++k) bin[k * NT + t] = 0u;
        klo = wave_min(klo);
        khi = wave_max(khi);
        if (lane == 0) {
            red[w] = klo;
            red2[w] = khi;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            klo = min(klo, red[k]);
            khi = max(khi, red2[k]);
        }
        const bool ties = klo == khi;
        if (ties) {  // uniform: bins of the record range
            __syncthreads();
            rlo = wave_min(rlo);
            rhi = wave_max(rhi);
            if (lane == 0) {
                red[w] = rlo;
                red2[w] = rhi;
            }
            __syncthreads();
            for (int k = 0; k < NW; ++k) {
                rlo = min(rlo, red[k]);
                rhi = max(rhi, red2[k]);
            }
        }
        const uint32_t lo = ties ? rlo : klo, by_rec = ties ? ~0u : 0u;
        const uint32_t sh = (uint32_t)max(0, bit_length((ties ? rhi : khi) - lo) - 11);
        static_assert(BINS == 1 << 11, "eleven bits of the bucket's range");
        uint32_t at[EPT];  // bin << 16 | arrival number in it
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const uint32_t i = (uint32_t)(k * NT + t);
            at[k] = 0u;
            if (i < n) {
                const uint32_t bi = (((rec[k] & by_rec) | (key[k] & ~by_rec)) - lo) >> sh;
                at[k] = (bi << 16) | atomicAdd(&bin[bi], 1u);
            }
        }
        __syncthreads();
        uint32_t c[BPT], sum = 0, big = 0;
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            c[k] = bin[t * BPT + k];
            sum += c[k];
            big = max(big, c[k]);
        }
        big = wave_max(big);
        uint32_t total;
        uint32_t ex = block_excl_scan<NT>(sum, red, &total);
        if (lane == 0) red2[w] = big;
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            bin[t * BPT + k] = ex;
            ex += c[k];
        }
        if (t == 0) bin[BINS] = n;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NW; ++k) big = max(big, red2[k]);
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const uint32_t i = (uint32_t)(k * NT + t);
            if (i < n) arr[bin[at[k] >> 16] + (at[k] & 0xffffu)] = ((uint64_t)key[k] << 32) | rec[k];
        }
        if (big <= CROWDED) {  // uniform
            __syncthreads();
#pragma unroll
            for (int k = 0; k < EPT; ++k) {
                const uint32_t i = (uint32_t)(k * NT + t);
                if (i < n) {
                    const uint64_t me = ((uint64_t)key[k] << 32) | rec[k];
                    const uint32_t q0 = bin[at[k] >> 16], q1 = bin[(at[k] >> 16) + 1];
                    uint32_t pos = q0;
                    for (uint32_t q = q0; q < q1; ++q) pos += arr[q] < me ? 1u : 0u;
                    val[pos] = (rec[k] - rec0) | be[k];
                    ext[pos] = rc[k];
                }
            }
            return;
        }
        uint32_t n2 = sort_min<NT>();
        while (n2 < n) n2 <<= 1;
        for (uint32_t i = n + t; i < n2; i += NT) arr[i] = ~0ull;
        bitonic_sort<NT>(arr, n2);
        for (uint32_t i = t; i < n; i += NT) {
            const uint32_t r = (uint32_t)arr[i];
            const uint2 rr = o.rect[r];
            val[i] = (r - rec0) | rect_cells(rr, cells);
            ext[i] = pack_rect(rr);
        }
        return;
    }
    // more elements than fit: [lo, top] is the range of (key, record) words in
    // which they lie; a record's number takes the bits that the view's need,
    // so that the bins part it early
    const int rb = bit_length(v.n_pad);
    const uint32_t rmask = (1u << rb) - 1u;
    auto join = [&](uint32_t key, uint32_t rec) { return ((uint64_t)key << rb) | (rec - v.rec_base); };
    auto rec_of = [&](uint64_t x) { return ((uint32_t)x & rmask) + v.rec_base; };
    auto word = [&](uint32_t i) {
        const uint4 x = e[i];
        return join(x.x, x.y);
    };
    auto each = [&](auto&& f) {  // over the elements' words, eight loads in flight
        for (uint32_t i0 = t; i0 < n; i0 += NT * 8) {
            uint64_t x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = word(min(i0 + (uint32_t)(k * NT), n - 1));
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i0 + (uint32_t)(k * NT) < n) f(x[k]);
        }
    };
    uint64_t lo = ~0ull, top = 0ull;
    uint32_t entries = 0;
    for (uint32_t i = t; i < n; i += NT) entries += rect_count(e[i].z);
    each([&](uint64_t x) {
        lo = x < lo ? x : lo;
        top = x > top ? x : top;
    });
    store_cost(entries);
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) {
        const uint64_t l2 = __shfl_xor((unsigned long long)lo, k, 64), t2 = __shfl_xor((unsigned long long)top, k, 64);
        lo = l2 < lo ? l2 : lo;
        top = t2 > top ? t2 : top;
    }
    if (lane == 0) {
        redlo[w] = lo;
        redhi[w] = top;
    }
    __syncthreads();
    for (int k = 0; k < NW; ++k) {
        lo = redlo[k] < lo ? redlo[k] : lo;
        top = redhi[k] > top ? redhi[k] : top;
    }
    // placed bin by bin in (val, ext), as (record, key)
    const int sh0 = max(0, 64 - __clzll((long long)(top - lo)) - 11);
    __syncthreads();
    for (int k = t; k < BINS; k += NT) bin[k] = 0u;
    __syncthreads();
    each([&](uint64_t x) { atomicAdd(&bin[(uint32_t)((x - lo) >> sh0)], 1u); });
    __syncthreads();
    {
        uint32_t c[BPT], sum = 0, total;
#pragma unroll
        for (int k = 0; k < BPT; ++k) sum += c[k] = bin[t * BPT + k];
        uint32_t ex = block_excl_scan<NT>(sum, red, &total);
#pragma unroll
        for (int k = 0; k < BPT; ++k) {
            bin[t * BPT + k] = ex;
            ex += c[k];
        }
    }
    __syncthreads();
    each([&](uint64_t x) {
        const uint32_t pos = atomicAdd(&bin[(uint32_t)((x - lo) >> sh0)], 1u);  // leaves the bin's end
        val[pos] = rec_of(x);
        ext[pos] = (uint32_t)(x >> rb);
    });
    auto placed = [&](uint32_t i) { return join(ext[i], val[i]); };
    auto put = [&](uint32_t pos, uint64_t x) {
        const uint32_t r = rec_of(x);
        const uint2 rr = o.rect[r];
        val[pos] = (r - rec0) | rect_cells(rr, cells);
        ext[pos] = pack_rect(rr);
    };
    // sorts arr[0, m) and writes it to `at`
    auto sort_out = [&](uint32_t m, uint32_t at) {
        uint32_t n2 = sort_min<NT>();
        while (n2 < m) n2 <<= 1;
        for (uint32_t i = m + t; i < n2; i += NT) arr[i] = ~0ull;
        bitonic_sort<NT>(arr, n2);
        for (uint32_t i = t; i < m; i += NT) put(at + i, arr[i]);
    };
    uint64_t* part = reinterpret_cast<uint64_t*>(b.elem + first);  // the elements are read no more
    for (uint32_t done = 0; done < n;) {
        __syncthreads();  // the placed words, and the use of arr and picked before
        if (t == 0) picked = fill = 0u;
        __syncthreads();
        uint32_t take = 0;  // bins whose end still fits
        for (int k = 0; k < BPT; ++k)
            if (bin[t * BPT + k] <= done + (uint32_t)CAP) take = (uint32_t)(t * BPT + k) + 1u;
        atomicMax(&picked, take);
        __syncthreads();
        const uint32_t nb = picked, end = nb ? bin[nb - 1] : 0u;
        if (end > done) {  // uniform
            const uint32_t m = end - done;
            uint32_t big = 0;
            for (int k = 0; k < BPT; ++k) {
                const uint32_t bi = (uint32_t)(t * BPT + k), e1 = bin[bi];
                if (e1 > done && e1 <= end) big = max(big, e1 - (bi ? bin[bi - 1] : 0u));
            }
            atomicMax(&fill, big);
            uint64_t me[EPT];
#pragma unroll
            for (int k = 0; k < EPT; ++k) me[k] = placed(done + min((uint32_t)(k * NT + t), m - 1));
#pragma unroll
            for (int k = 0; k < EPT; ++k)
                if ((uint32_t)(k * NT + t) < m) arr[k * NT + t] = me[k];
            __syncthreads();
            if (fill <= 4u * CROWDED) {  // uniform: ranks inside the bins; the bitonic sort is of 4096 here
#pragma unroll 1
                for (int k = 0; k < EPT; ++k)
                    if ((uint32_t)(k * NT + t) < m) {
                        const uint64_t x = arr[k * NT + t];
                        const uint32_t r = rec_of(x);
                        const uint2 rr = o.rect[r];
                        const uint32_t bi = (uint32_t)((x - lo) >> sh0);
                        const uint32_t q0 = (bi ? bin[bi - 1] : 0u) - done, q1 = bin[bi] - done;
                        uint32_t pos = q0;
#pragma unroll 4
                        for (uint32_t q = q0; q < q1; ++q) pos += arr[q] < x ? 1u : 0u;
                        val[done + pos] = (r - rec0) | rect_cells(rr, cells);
                        ext[done + pos] = pack_rect(rr);
                    }
            } else {
                sort_out(m, done);
            }
            done = end;
            continue;
        }
        // the next bin alone holds too many: its words out of the way, then
        // window by window; `bin` keeps the ends, arr also holds the counts
        uint32_t* cnt2 = reinterpret_cast<uint32_t*>(arr);
        const uint32_t d0 = done, m0 = bin[nb] - done;
        for (uint32_t i = t; i < m0; i += NT) part[d0 + i] = placed(d0 + i);
        uint64_t wlo = lo + ((uint64_t)nb << sh0), whi = wlo + (((uint64_t)1 << sh0) - 1);
        const uint64_t wtop = whi;
        while (done < d0 + m0) {
            const int sh = max(0, 64 - __clzll((long long)(whi - wlo)) - 11);
            __syncthreads();
            for (int k = t; k < BINS; k += NT) cnt2[k] = 0u;
            if (t == 0) picked = fill = 0u;
            __syncthreads();
            for (uint32_t i = t; i < m0; i += NT) {
                const uint64_t x = part[d0 + i];
                if (x >= wlo && x <= whi) atomicAdd(&cnt2[(uint32_t)((x - wlo) >> sh)], 1u);
            }
            __syncthreads();
            uint32_t sum = 0;
            for (int k = 0; k < BPT; ++k) sum += cnt2[t * BPT + k];
            uint32_t total, acc = block_excl_scan<NT>(sum, red, &total);
            uint32_t fits = 0;  // bins whose inclusive count still fits
            for (int k = 0; k < BPT; ++k) {
                acc += cnt2[t * BPT + k];
                if (acc <= (uint32_t)CAP) fits = (uint32_t)(t * BPT + k) + 1u;
            }
            atomicMax(&picked, fits);
            __syncthreads();
            const uint32_t wb = picked;
            if (wb == 0) {  // uniform: the first bin alone holds too many; look inside it
                const uint64_t last = wlo + (((uint64_t)1 << sh) - 1);
                whi = last < whi ? last : whi;
                continue;
            }
            uint64_t last = wlo + (((uint64_t)wb << sh) - 1);
            if (wb >= (uint32_t)BINS || last > whi) last = whi;
            for (uint32_t i = t; i < m0; i += NT) {
                const uint64_t x = part[d0 + i];
                if (x >= wlo && x <= last) arr[atomicAdd(&fill, 1u)] = x;
            }
            __syncthreads();
            const uint32_t m = fill;
            sort_out(m, done);
            done += m;
            wlo = last + 1;
            whi = wtop;
        }
    }
}

// ------------------------------------------------------------- radix sort
// One pass sorts (key, value[, extra]) triples stably by an 8-bit (or
// narrower) digit of the key.  The count comes from the device counters
// (which = 0: duplicates D, 1: visible Gaussians V) and is split into nb
// contiguous segments, one per workgroup, of a whole number of 2048-key
// chunks.  upsweep: digit histogram per segment; scan: exclusive offsets over
// (digit, segment); downsweep: rank (wave ballots + per-wave LDS counters)
// and scatter.


__device__ __forceinline__ uint32_t sort_count(const Counters* cnt, int which, uint32_t cap) {
    if (which == 1) return min(cnt->visible, cap);
    return cnt->overflow ? 0u : min(cnt->D, cap);
}
__device__ __forceinline__ uint64_t segment_len(uint32_t D, int nb) {
    const uint64_t per = ((uint64_t)D + nb - 1) / nb;
    return (per + SORT_CHUNK - 1) / SORT_CHUNK * SORT_CHUNK;
}
// The segment of workgroup wg: the segments that hold keys are spread over
// the XCDs in contiguous runs, the empty ones keep their own index.
__device__ __forceinline__ int pass_segment(uint32_t D, int nb, int wg) {
    const uint64_t per = segment_len(D, nb);
    const int nact = per ? (int)min((uint64_t)nb, ((uint64_t)D + per - 1) / per) : 0;
    return wg < nact ? xcd_segment(wg, nact) : wg;
}
__device__ __forceinline__ void segment(uint32_t D, int nb, int b, uint32_t* beg, uint32_t* end) {
    const uint64_t per = segment_len(D, nb);
    const uint64_t s = min((uint64_t)D, per * (uint64_t)b);
    *beg = (uint32_t)s;
    *end = (uint32_t)min((uint64_t)D, s + per);
}

// Digit counts of one segment: hist[d * nb + b] = keys of digit d in segment
// b, in 16 sub-histograms in LDS (one per wave and lane residue mod 4, rows of
// 257 words so that the copies of one digit sit in different banks): the
// leading digit of the whole depth key is nearly constant, and its keys then
// meet at most 16 to an address.
__global__ __launch_bounds__(SORT_THREADS) void k_sort_upsweep(const uint32_t* __restrict__ keys,
                                                               const Counters* __restrict__ cnt, int which,
                                                               uint32_t cap, int shift, int bits,
                                                               uint32_t* __restrict__ hist, int nb) {
    static_assert(SORT_THREADS == 256, "one digit per thread");
    constexpr int NDIG = 256, LPW = 4, NH = SORT_THREADS / 64 * LPW, ROW = NDIG + 1;
    __shared__ uint32_t h[NH * ROW];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < NH * ROW; i += SORT_THREADS) h[i] = 0u;
    __syncthreads();
    uint32_t beg, end;
    const uint32_t D = sort_count(cnt, which, cap);
    const int seg = pass_segment(D, nb, (int)blockIdx.x);
    segment(D, nb, seg, &beg, &end);
    const uint32_t mask = (1u << bits) - 1u;
    uint32_t* hrow = h + (w * LPW + (lane & (LPW - 1))) * ROW;
    // each wave walks blocks of 8 rows of 64 keys (8 loads in flight per lane)
    constexpr int U = 8;
    for (uint32_t blk = beg + (uint32_t)w * 64 * U; blk < end; blk += SORT_THREADS * U) {
        uint32_t kk[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = blk + u * 64 + lane;
            kk[u] = keys[i < end ? i : beg];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (blk + u * 64 + lane < end) atomicAdd(&hrow[(kk[u] >> shift) & mask], 1u);
    }
    __syncthreads();
    const int d = threadIdx.x;
    uint32_t x = 0;
#pragma unroll
    for (int k = 0; k < NH; ++k) x += h[k * ROW + d];
    if (d <= (int)mask) hist[(size_t)d * nb + seg] = x;
}

// One workgroup per digit: the digit's exclusive offsets over the segments
// (within the digit) and its total.  The four waves take consecutive quarters of the digit's row
// (NJ * 64 segments each) and learn the totals of the quarters before theirs
// through LDS.
template <int NJ>
__global__ __launch_bounds__(256) void k_sort_scan(uint32_t* __restrict__ hist, uint32_t* __restrict__ dtot, int nb) {
    __shared__ uint32_t qsum[4];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int d = blockIdx.x;
    uint32_t* row = hist + (size_t)d * nb;
    const int j0 = w * NJ * 64;
    uint32_t x[NJ];  // 4 * NJ * 64 >= nb
    uint32_t mine = 0;
#pragma unroll
    for (int q = 0; q < NJ; ++q) {
        const int j = j0 + q * 64 + lane;
        x[q] = j < nb ? row[j] : 0u;
        mine += x[q];
    }
    const uint32_t ws = wave_sum(mine);
    if (lane == 0) qsum[w] = ws;
    __syncthreads();
    if (threadIdx.x == 0) dtot[d] = qsum[0] + qsum[1] + qsum[2] + qsum[3];
    uint32_t running = 0;
    for (int v = 0; v < w; ++v) running += qsum[v];
#pragma unroll
    for (int q = 0; q < NJ; ++q) {
        if (j0 + q * 64 >= nb) break;
        const int j = j0 + q * 64 + lane;
        const uint32_t inc = wave_incl_scan(x[q]);
        if (j < nb) row[j] = running + inc - x[q];
        running += readlane(inc, 63);
    }
}

// Chunks of 2048 keys are ranked (per-wave ballot match + per-wave digit
// counters), staged in LDS in chunk-local digit order, and written out so that
// consecutive threads store consecutive positions of each digit run.
// SUMS (last depth pass): each Gaussian's tile rectangle is gathered once
// here and written in depth order, so that k_sorted_sums and k_duplicate read
// it contiguously instead of gathering by record.
template <bool EXTRA, bool SUMS>
__global__ __launch_bounds__(SORT_THREADS) void k_sort_downsweep(
    const uint32_t* __restrict__ skey, const uint32_t* __restrict__ sval, const uint32_t* __restrict__ sext,
    uint32_t* __restrict__ dkey, uint32_t* __restrict__ dval, uint32_t* __restrict__ dext,
    const Counters* __restrict__ cnt, int which, uint32_t cap, int shift, int bits,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ dtot, int nb,
    const uint2* __restrict__ rsrc, uint2* __restrict__ rdst) {
    constexpr int NDIG = 256, NT = SORT_THREADS;
    static_assert(NDIG == NT, "one digit per thread");
    constexpr int NW = NT / 64;
    constexpr int ROUNDS = SORT_CHUNK / NT;
    __shared__ uint32_t base[NDIG];    // global position of the next key of each digit
    __shared__ uint32_t lstart[NDIG];  // chunk-local start of each digit
    __shared__ uint32_t wcnt[NW][NDIG];
    __shared__ uint32_t red[NW];
    __shared__ uint32_t lkey[SORT_CHUNK];
    __shared__ uint32_t lval[SORT_CHUNK];
    __shared__ uint32_t lext[EXTRA ? SORT_CHUNK : 1];
    __shared__ uint2 lrect[SUMS ? SORT_CHUNK : 1];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const uint32_t mask = (1u << bits) - 1u;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    uint32_t beg, end;
    const uint32_t D = sort_count(cnt, which, cap);
    const int seg = pass_segment(D, nb, (int)blockIdx.x);
    segment(D, nb, seg, &beg, &end);
    // the keys of the next chunk are loaded while the current one is ranked
    // (the first chunk's while the digit starts are formed)
    uint32_t nk[ROUNDS], nv[ROUNDS], ne[ROUNDS];
    auto load_chunk = [&](uint32_t c) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t idx = c + (uint32_t)(w * (SORT_CHUNK / NW) + r * 64 + lane);
            const uint32_t ic = idx < end ? idx : c;  // clamped: loads never depend on a branch
            nk[r] = skey[ic];
            nv[r] = sval[ic];
            ne[r] = EXTRA ? sext[ic] : 0u;
        }
    };
    if (beg < end) load_chunk(beg);
    // a digit's first position: the totals of the digits below it (scanned
    // here from the per-digit totals) plus its offset in this segment
    {
        const uint32_t tt = t <= (int)mask ? dtot[t] : 0u;
        uint32_t all;
        const uint32_t st = block_excl_scan<NT>(tt, red, &all);
        base[t] = t <= (int)mask ? st + hist[(size_t)t * nb + seg] : 0u;
    }
    for (uint32_t chunk = beg; chunk < end; chunk += SORT_CHUNK) {
#pragma unroll
        for (int j = 0; j < NW; ++j) wcnt[j][t] = 0u;
        __syncthreads();
        uint32_t dig[ROUNDS], rank[ROUNDS], ek[ROUNDS], ev[ROUNDS], ee[ROUNDS];
        uint2 er[ROUNDS];
        bool ok[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            ek[r] = nk[r];
            ev[r] = nv[r];
            ee[r] = ne[r];
        }
        if (chunk + SORT_CHUNK < end) load_chunk(chunk + SORT_CHUNK);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const uint32_t idx = chunk + (uint32_t)(w * (SORT_CHUNK / NW) + r * 64 + lane);
            ok[r] = idx < end;
            const uint32_t key = ek[r];
            if constexpr (SUMS) er[r] = rsrc[ev[r]];
            const uint32_t d = (key >> shift) & mask;
            dig[r] = d;
            uint64_t m = ballot(ok[r]);
            for (int b = 0; b < bits; ++b) {
                const bool bit = (d >> b) & 1u;
                const uint64_t bl = ballot(bit);
                m &= bit ? bl : ~bl;
            }
            const uint32_t prior = (uint32_t)__builtin_popcountll(m & lt);
            uint32_t cur = 0;
            if (ok[r]) cur = wcnt[w][d];
            rank[r] = cur + prior;
            if (ok[r] && prior == 0) wcnt[w][d] = cur + (uint32_t)__builtin_popcountll(m);
        }
        __syncthreads();
        // digit t: chunk-local start, then per-wave local offsets
        uint32_t c = 0;
#pragma unroll
        for (int j = 0; j < NW; ++j) c += wcnt[j][t];
        uint32_t tot;
        const uint32_t ls = block_excl_scan<NT>(c, red, &tot);
        lstart[t] = ls;
        uint32_t acc = ls;
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            const uint32_t x = wcnt[j][t];
            wcnt[j][t] = acc;
            acc += x;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (ok[r]) {
                const uint32_t l = wcnt[w][dig[r]] + rank[r];
                lkey[l] = ek[r];
                lval[l] = ev[r];
                if (EXTRA) lext[l] = ee[r];
                if constexpr (SUMS) lrect[l] = er[r];
            }
        }
        __syncthreads();
        for (uint32_t l = (uint32_t)t; l < tot; l += NT) {
            const uint32_t k = lkey[l];
            const uint32_t d = (k >> shift) & mask;
            const uint32_t pos = base[d] + (l - lstart[d]);
            if (pos < D) {
                const uint32_t vv = lval[l];
                dkey[pos] = k;
                dval[pos] = vv;
                if (EXTRA) dext[pos] = lext[l];
                if constexpr (SUMS) rdst[pos] = lrect[l];
            }
        }
        __syncthreads();
        base[t] += c;
    }
}

// The frame's counters as the host sees them: the entries are counted in tiles,
// however many of them share a list.
__device__ __forceinline__ void store_counters(const Counters* cnt, FrameCounters* host_cnt) {
    FrameCounters c = *cnt;
    c.D = cnt->pairs;
    *host_cnt = c;
}

// ------------------------------------------------------------------ ranges

// Tile boundaries in the sorted tile words; the ranges array was cleared by
// k_scan_visible, so tiles without entries stay [0, 0).  The frame's counters
// are final here: one thread also stores them to the host-visible block the
// host reads after the frame (no separate copy).
__global__ __launch_bounds__(256) void k_ranges(const uint32_t* __restrict__ tile, const Counters* __restrict__ cnt,
                                                uint32_t cap, uint2* __restrict__ ranges, FrameCounters* host_cnt) {
    if (blockIdx.x == 0 && threadIdx.x == 0) store_counters(cnt, host_cnt);
    const uint32_t D = sort_count(cnt, 0, cap);
    // each wave takes 256 consecutive words per step, four per lane (one
    // 16-byte load); neighbours come from the adjacent lanes, and across the
    // step's edges from one extra load
    const int lane = threadIdx.x & 63;
    const uint32_t nwaves = gridDim.x * 4u;
    for (uint32_t c = ((blockIdx.x * 256u + threadIdx.x) >> 6) * 256u; c < D; c += nwaves * 256u) {
        const uint32_t i0 = c + (uint32_t)lane * 4u;
        uint32_t e[4];
        if (i0 + 3u < D) {
            const uint4 q = *reinterpret_cast<const uint4*>(tile + i0);
            e[0] = q.x; e[1] = q.y; e[2] = q.z; e[3] = q.w;
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) e[k] = i0 + k < D ? tile[i0 + k] : 0xffffffffu;
        }
        uint32_t prev = __shfl_up(e[3], 1, 64), next = __shfl_down(e[0], 1, 64);
        if (lane == 0) prev = c > 0u ? tile[c - 1u] : 0xffffffffu;
        if (lane == 63) next = c + 256u < D ? tile[c + 256u] : 0xffffffffu;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t i = i0 + (uint32_t)k;
            if (i < D) {
                const uint32_t t = e[k];
                const uint32_t p = k > 0 ? e[k - 1] : prev, n = k < 3 ? e[k + 1] : next;
                if (i == 0u || p != t) ranges[t].x = i;
                if (i + 1u == D || n != t) ranges[t].y = i + 1u;
            }
        }
    }
}

// ------------------------------------------------------ tile placement
// The most significant digit of the (tile | depth) key, the tile id, placed
// by counting instead of by radix passes over the duplicates: a view's
// Gaussians arrive in depth order, and entry (g, t) belongs at
//   start(t) + #{Gaussians before g, in depth order, whose rectangle holds t}.
// The depth order is cut into units of about equal cost (a Gaussian costs its
// entries plus TILE_BASE_COST), about `nunits` over all views; k_tile_count
// counts, per unit, the rectangles that hold each tile (a 2D difference grid:
// +1/-1 at the corners of each rectangle, then 2D prefix sums),
// k_tile_scan turns the counts into exclusive prefixes over the units, and
// k_tile_emit writes every entry straight to its sorted position.  A
// workgroup takes one unit and one group of at most TILE_CELLS cells of the
// grid (whole tile rows), so that any grid of at most 256 x 256 tiles fits its
// LDS and a few large near Gaussians are spread over several workgroups.
// Views of at most 256 x 256 tiles.
constexpr int TILE_THREADS = 256;
constexpr int TILE_WAVES = TILE_THREADS / 64;

// Rows of a workgroup's group of tiles, and the number of groups of a view.
__host__ __device__ __forceinline__ int tile_group_rows(int tiles_x) {
    return TILE_CELLS / tiles_x < 1 ? 1 : TILE_CELLS / tiles_x;
}

// The view of unit u, the unit's number in it and the cost of a unit: from
// the views' totals, or (flat: the radix depth order of a single view) from
// the frame's counters.
struct UnitOf {
    int view;
    uint32_t u;       // within the view
    uint32_t nu;      // units of the view
    uint32_t cost;    // of one unit
    uint32_t start, visible;
    uint64_t total;   // cost of the view
};
__device__ __forceinline__ bool unit_of(uint32_t u, const TileMem& m, const ViewCount* __restrict__ vc, int nviews,
                                        const Counters* __restrict__ cnt, bool flat, UnitOf* r) {
    if (flat) {
        r->view = 0;
        r->start = 0;
        r->visible = cnt->visible;
        r->total = (uint64_t)cnt->D + (uint64_t)TILE_BASE_COST * cnt->visible;
        r->cost = unit_cost(r->total, m.nunits);
        r->nu = units_for(r->total, r->cost);
        r->u = u;
        return u < r->nu;
    }
    const int vi = view_of(u, nviews, [&](int i) { return vc[i].ubase; });
    r->view = vi;
    r->start = vc[vi].start;
    r->visible = vc[vi].visible;
    r->total = vc[vi].dups + (uint64_t)TILE_BASE_COST * vc[vi].visible;
    r->cost = vc[vi].ucost;
    r->nu = vc[vi].nu;
    r->u = u - vc[vi].ubase;
    return r->u < r->nu;
}

// The position in a view's depth order at cost `t` of the units' split, by one
// wave: the bucket holding it from the costs of the chunks of buckets, then of
// the chunk's buckets, and by count inside it (its Gaussians lie at about one
// depth); `end` when the view costs no more than that.
__device__ __forceinline__ uint32_t unit_position(uint64_t t, uint32_t end, const BucketMem& b, const ViewParams& v) {
    const uint32_t l = lane_id();
    const uint32_t nc = (v.nbkt + COL_CHUNK - 1) / COL_CHUNK, ck0 = v.bkt_base / COL_CHUNK;
    auto scan64 = [&](unsigned long long x) {
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(x, o, 64);
            if ((int)l >= o) x += y;
        }
        return x;
    };
    const unsigned long long ca = 2 * l < nc ? b.ccost[ck0 + 2 * l] : 0ull;
    const unsigned long long cb = 2 * l + 1 < nc ? b.ccost[ck0 + 2 * l + 1] : 0ull;
    const unsigned long long before = scan64(ca + cb) - ca - cb;
    const uint64_t hit = ballot(t >= before && t < before + ca + cb);
    if (hit == 0) return end;
    const int src = __builtin_ctzll(hit);
    unsigned long long p = __shfl(before, src, 64);
    const unsigned long long first = __shfl(ca, src, 64);
    uint32_t ck = 2u * (uint32_t)src;
    if (t >= p + first) {
        p += first;
        ++ck;
    }
    const uint32_t base = chunks_before(b.chunk + ck0, ck);
    const uint32_t bi = ck * COL_CHUNK + l;
    const bool in = l < COL_CHUNK && bi < v.nbkt;
    const unsigned long long c = in ? b.cost[v.bkt_base + bi] : 0ull;
    const unsigned long long cp = p + scan64(c) - c;
    const bool mine = t >= cp && t < cp + c;
    uint32_t pos = 0;
    if (mine) {
        const uint32_t n = b.tot[v.bkt_base + bi];
        pos = base + b.start_in[v.bkt_base + bi] + min(n, (uint32_t)((float)(uint32_t)(t - cp) * ((float)n / (float)c)));
    }
    const uint64_t mm = ballot(mine);
    return mm ? readlane(pos, __builtin_ctzll(mm)) : end;
}

// Inclusive 2D prefix sums of an h1 x w1 grid (row-major, w1 <= 257) held in
// LDS, by a workgroup of 256 threads: rows (one wave per row, DPP scans), then
// columns (one thread per column, eight rows in flight).
__device__ void grid_prefix2d(uint32_t* g, int w1, int h1) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int y = w; y < h1; y += 4) {
        uint32_t carry = 0;
        for (int c0 = 0; c0 < w1; c0 += 64) {
            const int x = c0 + lane;
            const uint32_t v = x < w1 ? g[y * w1 + x] : 0u;
            const uint32_t sc = wave_incl_scan(v) + carry;
            if (x < w1) g[y * w1 + x] = sc;
            carry = readlane(sc, 63);
        }
    }
    __syncthreads();
    const int x = threadIdx.x;
    if (x < w1) {
        uint32_t run = 0;
        int y = 0;
        for (; y + 8 <= h1; y += 8) {
            uint32_t v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = g[(y + k) * w1 + x];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                run += v[k];
                g[(y + k) * w1 + x] = run;
            }
        }
        for (; y < h1; ++y) {
            run += g[y * w1 + x];
            g[y * w1 + x] = run;
        }
    }
    __syncthreads();
}

// Per unit and group of tile rows: how many of the unit's rectangles hold
// each tile (a row of m.rows).  The unit's range of the depth order is kept
// for the emission.
__global__ __launch_bounds__(TILE_THREADS) void k_tile_count(TileMem m, BucketMem b,
                                                             const ViewParams* __restrict__ views, int nviews,
                                                             const Counters* __restrict__ cnt, bool flat,
                                                             const uint32_t* __restrict__ packed) {
    constexpr int NT = TILE_THREADS;
    __shared__ uint32_t g[TILE_CELLS + 256];  // (tiles_x + 1) x rows: at most one spare column
    __shared__ uint32_t range[2];
    if (cnt->overflow) return;  // uniform
    UnitOf un;
    if (!unit_of(blockIdx.x, m, b.vc, nviews, cnt, flat, &un)) return;  // uniform
    const ViewParams& v = views[un.view];
    const int tiles_x = v.tiles_x, rpg = tile_group_rows(tiles_x);
    const int y0g = (int)blockIdx.y * rpg;
    if (y0g >= v.tiles_y) return;  // uniform
    const int nr = min(rpg, v.tiles_y - y0g), w1 = tiles_x + 1;
    const int t = threadIdx.x;
    for (int c = t; c < w1 * nr; c += NT) g[c] = 0u;
    if (t < 128) {  // the unit's first and last cost, a wave each
        const int k = __builtin_amdgcn_readfirstlane(t >> 6);
        const uint64_t at = ((uint64_t)un.u + (uint64_t)k) * un.cost;
        uint32_t pos = un.visible;
        if (at < un.total)
            pos = flat ? (uint32_t)((double)un.visible * (double)at / (double)un.total)
                       : unit_position(at, un.visible, b, v);
        if ((t & 63) == 0) range[k] = pos;
    }
    __syncthreads();
    const uint32_t g0 = un.start + range[0], g1 = un.start + max(range[0], range[1]);
    if (t == 0 && blockIdx.y == 0) m.urange[blockIdx.x] = make_uint2(g0, g1);
    constexpr int U = 8;  // loads in flight per thread
    for (uint32_t i0 = g0; i0 < g1; i0 += NT * U) {
        uint32_t pk[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint32_t i = i0 + (uint32_t)(k * NT + t);
            pk[k] = i < g1 ? packed[i] : 0u;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint32_t i = i0 + (uint32_t)(k * NT + t);
            const int x0 = (int)(pk[k] & 0xffu), x1 = (int)((pk[k] >> 16) & 0xffu) + 1;
            const int ya = max((int)((pk[k] >> 8) & 0xffu) - y0g, 0), yb = min((int)(pk[k] >> 24) - y0g + 1, nr);
            if (i < g1 && ya < yb) {
                // corners in the extra column or row only affect cells that
                // nothing reads (rectangles clamped to the frame's edges
                // would all meet there)
                atomicAdd(&g[ya * w1 + x0], 1u);
                if (x1 < tiles_x) atomicAdd(&g[ya * w1 + x1], 0xffffffffu);
                if (yb < nr) {
                    atomicAdd(&g[yb * w1 + x0], 0xffffffffu);
                    if (x1 < tiles_x) atomicAdd(&g[yb * w1 + x1], 1u);
                }
            }
        }
    }
    __syncthreads();
    grid_prefix2d(g, w1, nr);
    uint32_t* row = m.rows + (size_t)blockIdx.x * m.stride + (size_t)y0g * tiles_x;
    const int lane = t & 63, w = t >> 6;
    for (int y = w; y < nr; y += TILE_WAVES)
        for (int x = lane; x < tiles_x; x += 64) row[y * tiles_x + x] = g[y * w1 + x];
}

// Dense-first dispatch order of a frame's tiles for the blend: tiles by
// decreasing list length in 64 buckets of a quarter octave each (lengths up
// to 2^16 apart), so the longest lists start first and short ones fill the
// end of the launch instead of long ones running on after the rest are done.
// Within a bucket the order is whatever the atomics give: every tile's
// pixels are computed on their own, so the order changes only the timing.
__device__ __forceinline__ uint32_t length_bucket(uint32_t n) {
    const uint32_t x = n + 1u;
    const int msb = 31 - __builtin_clz(x);
    const uint32_t frac = msb >= 2 ? (x >> (msb - 2)) & 3u : (x << (2 - msb)) & 3u;
    return 63u - min(63u, 4u * (uint32_t)msb + frac);
}

// Per chunk of TILE_CHUNK tiles of a view: the exclusive prefixes of the units'
// counts (in place), the tiles' totals and their prefixes inside the chunk.
__global__ __launch_bounds__(1024) void k_tile_scan(TileMem m, BucketMem b, const ViewParams* __restrict__ views,
                                                    int nviews, const Counters* __restrict__ cnt, bool flat) {
    __shared__ uint32_t lds[(1024 / TILE_CHUNK + 1) * (TILE_CHUNK + 1)];
    if (cnt->overflow) return;  // uniform
    const int vi = view_of(blockIdx.x, nviews, [&](int i) { return views[i].tchunk_base; });
    const ViewParams& v = views[vi];
    uint32_t ub = 0, nu;
    if (flat) {
        UnitOf un;
        (void)unit_of(0, m, b.vc, nviews, cnt, true, &un);
        nu = un.nu;
    } else {
        ub = b.vc[vi].ubase;
        nu = b.vc[vi].nu;
    }
    const uint32_t n_tiles = (uint32_t)(v.tiles_x * v.tiles_y), c0 = (blockIdx.x - v.tchunk_base) * TILE_CHUNK;
    column_scan<TILE_CHUNK, 32>(m.rows + (size_t)ub * m.stride, nu, m.stride, n_tiles, c0, m.start_in + v.tile_base + c0,
                m.tot + v.tile_base + c0, m.chunk + blockIdx.x, lds);
}

// The emission.  A wave takes the tile rows of its group whose number is its
// own modulo the wave count, walks the unit's Gaussians 64 at a time and
// queues those with such a row.  A queue of 64 is placed at once, a lane per
// Gaussian: every lane sets its bit in the lane mask of each of its tiles
// (64-bit LDS atomics), and then its rank in a tile is the number of lower
// bits; the highest one moves the tile's next position on and clears the
// mask.  Gaussians of many tiles are spread over the lanes.  The first
// `nfront` workgroups write the ranges (and with `order` the blend's dispatch
// order) instead; workgroup 0 copies the counters for the host.
// Bound by latency: a queue is two dependent passes over LDS, and the stores,
// scattered over the lists, run into the units' neighbours only in one L2
// (contiguous units per XCD: 72 us at 3M/1080p with a list per tile, spread
// units 77).  Units of a 1/1536 of the work keep ~6 workgroups of a few queues
// on each CU: 3M/1080p, count + scan + emission with 512 / 1024 / 1536 / 2048
// units 92 / 68 / 62 / 65 us.  An LDS counting sort of a unit's entries with
// coalesced stores took 114 us where this took 72.  With four tiles per list
// list the placement of 3M/1080p takes 57 us (count 10, scan 12.5, emission 34;
// rounds of 256 Gaussians scattered into a list per tile: 117 us), that
// of 3M/4K 57 (two radix passes with duplicates, ranges and order: 305), that
// of 32 views 0.83 ms (two radix passes: 2.55).  Gaussians of more than 16
// tiles are spread over the lanes: from 32 on 75 us instead of 72.
// Few units leave the chip idle, and each lasts as long as its waves' chains of
// queues: up to TILE_WIDE_RECORDS records eight waves share a unit's rows instead
// of four.  Launches with 4 / 8 waves: 20k records 9.8 / 8.9 us, 100k 11.2 / 8.6,
// 200k 16.1 / 10.5, 400k 14.4 / 11.1, 800k 14.1 / 13.2, 1M 13.8 / 16.1, 3M 29.7 /
// 32.4, 32 views of 3M 434 / 681 (16 waves: 20k 9.2, 200k 9.2, 400k 11.6, 800k 19.6).
constexpr uint32_t TILE_WIDE_RECORDS = 800u << 10;
template <bool DEBUG, int NW>
__global__ __launch_bounds__(NW * 64) void k_tile_emit(
    TileMem m, BucketMem b, const ViewParams* __restrict__ views, int nviews, const Counters* __restrict__ cnt,
    bool flat, uint32_t nfront, uint32_t nchunks, uint2* __restrict__ ranges, uint32_t* __restrict__ order,
    FrameCounters* host_cnt, const uint32_t* __restrict__ rec, const uint32_t* __restrict__ packed,
    uint32_t* __restrict__ val_out, uint32_t* __restrict__ tile_out, uint32_t* __restrict__ depth_out,
    const uint32_t* __restrict__ zkey) {
    constexpr int NT = NW * 64;
    static_assert((NW & (NW - 1)) == 0, "rows modulo the waves");
    constexpr int FRONT_CHUNKS = TILE_FRONT_TILES / TILE_CHUNK;
    constexpr uint32_t MANY = 16;  // tiles from which a Gaussian is spread over the lanes
    __shared__ unsigned long long mask[TILE_CELLS];
    __shared__ uint32_t cur[TILE_CELLS];
    __shared__ uint32_t qp[NW][128], qr[NW][128];
    __shared__ uint32_t red[NW], cpre[TILE_CELLS / TILE_CHUNK + 2];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const uint32_t ov = cnt->overflow;
    if (blockIdx.x < nfront) {  // uniform
        if (blockIdx.y) return;
        if (blockIdx.x == 0 && t == 0) store_counters(cnt, host_cnt);
        const uint32_t f0 = blockIdx.x * FRONT_CHUNKS;
        uint32_t before = 0;
        if (!ov)
            for (uint32_t c = t; c < f0; c += NT) before += m.chunk[c];
        before = block_sum<NT>(before, red);
        static_assert(FRONT_CHUNKS == 128 && TILE_CELLS >= 256, "two chunks per lane");
        uint32_t* const cp = cur + 128;      // entries before each chunk
        uint32_t* const all = cur;           // all tiles per length bucket,
        uint32_t* const mine = cur + 64;     // those of the workgroups before this one; then the next places
        if (t < 64) {
            const uint32_t c = f0 + 2u * t;
            const uint32_t x = !ov && c < nchunks ? m.chunk[c] : 0u, y = !ov && c + 1 < nchunks ? m.chunk[c + 1] : 0u;
            const uint32_t ex = before + wave_incl_scan(x + y) - x - y;
            cp[2 * t] = ex;
            cp[2 * t + 1] = ex + x;
            all[t] = mine[t] = 0u;
        }
        __syncthreads();
        constexpr int K = TILE_FRONT_TILES / NT;
        for (int k = 0; k < K; ++k) {
            const uint32_t lc = (uint32_t)(k * NT + t) / TILE_CHUNK, c = f0 + lc;
            if (c >= nchunks) break;
            const int vi = view_of(c, nviews, [&](int i) { return views[i].tchunk_base; });
            const ViewParams& v = views[vi];
            const uint32_t lt = (c - v.tchunk_base) * TILE_CHUNK + (uint32_t)(t & (TILE_CHUNK - 1));
            if (lt < (uint32_t)(v.tiles_x * v.tiles_y)) {
                const uint32_t n = ov ? 0u : m.tot[v.tile_base + lt];
                const uint32_t s = n ? cp[lc] + m.start_in[v.tile_base + lt] : 0u;
                ranges[v.tile_base + lt] = make_uint2(s, s + n);
            }
        }
        if (!order) return;
        // the dispatch order of this workgroup's tiles (a single view: tile
        // ids are chunked without gaps): every front workgroup counts all
        // tiles' lengths, as contended device atomics cost more (34 us)
        const uint32_t n_tiles = (uint32_t)(views[0].tiles_x * views[0].tiles_y);
        const uint32_t o0 = blockIdx.x * TILE_FRONT_TILES, o1 = min(o0 + TILE_FRONT_TILES, n_tiles);
#pragma unroll 8
        for (uint32_t i = t; i < n_tiles; i += NT) {
            const uint32_t bk = length_bucket(ov ? 0u : m.tot[i]);
            atomicAdd(&all[bk], 1u);
            if (i < o0) atomicAdd(&mine[bk], 1u);
        }
        __syncthreads();
        if (t < 64) mine[t] += wave_incl_scan(all[t]) - all[t];
        __syncthreads();
        for (uint32_t i = o0 + t; i < o1; i += NT)
            order[atomicAdd(&mine[length_bucket(ov ? 0u : m.tot[i])], 1u)] = i;
        return;
    }
    if (ov) return;  // uniform
    // XCD x takes a contiguous run of the units: the entries that neighbouring
    // units write to one tile's list are adjacent and meet in one L2
    UnitOf un;
    const uint32_t wg = blockIdx.x - nfront;
    uint32_t nact;
    if (flat) {
        (void)unit_of(0, m, b.vc, nviews, cnt, true, &un);
        nact = un.nu;
    } else {
        nact = b.vc[nviews - 1].ubase + b.vc[nviews - 1].nu;
    }
    if (wg >= nact) return;  // uniform
    const uint32_t unit = (uint32_t)xcd_segment((int)wg, (int)nact);
    (void)unit_of(unit, m, b.vc, nviews, cnt, flat, &un);
    const ViewParams& v = views[un.view];
    const int tiles_x = v.tiles_x, rpg = tile_group_rows(tiles_x), y0g = (int)blockIdx.y * rpg;
    if (y0g >= v.tiles_y) return;  // uniform
    const int nr = min(rpg, v.tiles_y - y0g);
    const uint2 ur = m.urange[unit];
    const uint32_t ncell = (uint32_t)(nr * tiles_x), tl0 = (uint32_t)(y0g * tiles_x);  // the group's tiles in the view
    const uint32_t c_first = tl0 / TILE_CHUNK, nc = (tl0 + ncell - 1) / TILE_CHUNK - c_first + 1;
    {
        uint32_t before = 0;
        for (uint32_t c = t; c < v.tchunk_base + c_first; c += NT) before += m.chunk[c];
        before = block_sum<NT>(before, red);
        static_assert(TILE_CELLS / TILE_CHUNK + 2 <= 128, "two chunks per lane");
        if (t < 64) {
            const uint32_t* ch = m.chunk + v.tchunk_base + c_first;
            const uint32_t x = 2u * t < nc ? ch[2 * t] : 0u, y = 2u * t + 1 < nc ? ch[2 * t + 1] : 0u;
            const uint32_t ex = before + wave_incl_scan(x + y) - x - y;
            if (2u * t < nc) cpre[2 * t] = ex;
            if (2u * t + 1 < nc) cpre[2 * t + 1] = ex + x;
        }
        __syncthreads();
        const uint32_t* row = m.rows + (size_t)unit * m.stride + tl0;
        const uint32_t* sin = m.start_in + v.tile_base + tl0;
#pragma unroll 8
        for (uint32_t i = t; i < ncell; i += NT) {
            cur[i] = row[i] + sin[i] + cpre[(tl0 + i) / TILE_CHUNK - c_first];
            mask[i] = 0ull;
        }
    }
    __syncthreads();
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // this wave's rows of the rectangle p: the first one in the group, and the
    // last row of the rectangle inside it
    auto rows_of = [&](uint32_t p, int* first, int* last) {
        const int ya = max((int)((p >> 8) & 0xffu) - y0g, 0);
        *first = ya + ((w - ya) & (NW - 1));
        *last = min((int)(p >> 24) - y0g, nr - 1);
    };
    const uint32_t D = cnt->D;
    // with cells, of the view's lists: bits of a record's number, cells a side
    const int cells = v.cells, rb = cell_rec_bits(cells) & 31, side = 1 << cells;
    const uint32_t all = (1u << side) - 1u;
    auto put = [&](uint32_t cell, uint32_t pos, uint32_t r) {
        if (pos >= D) return;
        val_out[pos] = r;
        if (DEBUG) {
            tile_out[pos] = v.tile_base + tl0 + cell;
            depth_out[pos] = zkey[r];
        }
    };
    auto place = [&](uint32_t n) {  // the first n queued Gaussians
        const bool on = (uint32_t)lane < n;
        const uint32_t p = on ? qp[w][lane] : 0u, r = on ? qr[w][lane] : 0u;
        const int x0 = (int)(p & 0xffu), nx = (int)((p >> 16) & 0xffu) - x0 + 1;
        // with cells: masks of the rectangle's columns (from bit 0 in its first
        // list, 8 in its last) and rows (from 4 and 12), all elsewhere
        const uint32_t rec = cells ? r & ((1u << rb) - 1u) : r, ends = r >> rb, last_cell = (uint32_t)side - 1u;
        const uint32_t cm = cells ? ((all << (ends & last_cell)) & all) |
                                        (((all << ((ends >> cells) & last_cell)) & all) << 4) |
                                        (((2u << ((ends >> (2 * cells)) & last_cell)) - 1u) << 8) |
                                        (((2u << (ends >> (3 * cells))) - 1u) << 12)
                                  : 0u;
        const int yt = (int)((p >> 8) & 0xffu) - y0g, yb = (int)(p >> 24) - y0g;
        auto row_cells = [=](uint32_t m, int y, int top, int bottom) {
            return !cells ? 0u : ((y == top ? m >> 4 : all) & (y == bottom ? m >> 12 : all)) << (rb + side);
        };
        auto col_cells = [=](uint32_t m, int x, int n) {
            return !cells ? 0u : ((x == 0 ? m : all) & (x + 1 == n ? m >> 8 : all) & all) << rb;
        };
        int f, last;
        rows_of(p, &f, &last);
        const int ny = (last - f) / NW + 1;
        const uint32_t c0 = (uint32_t)(f * tiles_x + x0), nt = on ? (uint32_t)(nx * ny) : 0u;
        const int skip = NW * tiles_x - nx + 1;  // from a row's last tile to the next row's first
        const uint64_t bit = 1ull << lane;
        const uint64_t many = ballot(nt > MANY);
        {
            uint32_t c = c0;
            int x = 0;
            for (uint32_t k = 0; k < (nt > MANY ? 0u : nt); ++k) {
                atomicOr(&mask[c], bit);
                const bool end = ++x == nx;
                c += end ? (uint32_t)skip : 1u;
                x = end ? 0 : x;
            }
        }
        for (uint64_t q = many; q; q &= q - 1) {
            const int l = __builtin_ctzll(q);
            const uint32_t lc0 = readlane(c0, l), lnt = readlane(nt, l), lnx = readlane((uint32_t)nx, l);
            const float inv = 1.0f / (float)lnx;
            for (uint32_t k = lane; k < lnt; k += 64) {
                uint32_t y = (uint32_t)((float)k * inv);  // k / lnx, corrected
                if (y * lnx > k) --y;
                if ((y + 1) * lnx <= k) ++y;
                atomicOr(&mask[lc0 + y * (uint32_t)(NW * tiles_x) + (k - y * lnx)], 1ull << l);
            }
        }
        wave_sync();
        // a tile of one Gaussian is settled at once; of several, when all
        // lanes have read its mask
        uint32_t later = 0;  // bit k: this lane settles its k-th tile
        {
            uint32_t c = c0;
            int x = 0, yy = f;
            uint32_t re = rec | row_cells(cm, yy, yt, yb);
            for (uint32_t k = 0; k < (nt > MANY ? 0u : nt); ++k) {
                const uint64_t mm = mask[c];
                const uint32_t pos = cur[c], rank = bits_below(mm), tot = (uint32_t)__builtin_popcountll(mm);
                put(c, pos + rank, re | col_cells(cm, x, nx));
                if (tot == 1u) {
                    cur[c] = pos + 1u;
                    mask[c] = 0ull;
                } else if (rank + 1u == tot) {
                    later |= 1u << k;
                }
                const bool end = ++x == nx;
                c += end ? (uint32_t)skip : 1u;
                x = end ? 0 : x;
                if (end) re = rec | row_cells(cm, yy += NW, yt, yb);
            }
        }
        for (uint64_t q = many; q; q &= q - 1) {
            const int l = __builtin_ctzll(q);
            const uint32_t lc0 = readlane(c0, l), lnt = readlane(nt, l), lnx = readlane((uint32_t)nx, l);
            const uint32_t lr = readlane(rec, l), lcm = readlane(cm, l);
            const int lf = (int)readlane((uint32_t)f, l), lyt = (int)readlane((uint32_t)yt, l);
            const int lyb = (int)readlane((uint32_t)yb, l);
            const uint64_t below = (1ull << l) - 1ull;
            const float inv = 1.0f / (float)lnx;
            for (uint32_t k = lane; k < lnt; k += 64) {
                uint32_t y = (uint32_t)((float)k * inv);
                if (y * lnx > k) --y;
                if ((y + 1) * lnx <= k) ++y;
                const uint32_t c = lc0 + y * (uint32_t)(NW * tiles_x) + (k - y * lnx);
                put(c, cur[c] + (uint32_t)__builtin_popcountll(mask[c] & below),
                    lr | row_cells(lcm, lf + (int)y * NW, lyt, lyb) | col_cells(lcm, (int)(k - y * lnx), (int)lnx));
            }
        }
        wave_sync();
        for (; later; later &= later - 1) {
            const uint32_t k = (uint32_t)__builtin_ctz(later);
            uint32_t y = 0, xk = k;
            while (xk >= (uint32_t)nx) {
                xk -= (uint32_t)nx;
                ++y;
            }
            const uint32_t c = c0 + y * (uint32_t)(NW * tiles_x) + xk;
            cur[c] += (uint32_t)__builtin_popcountll(mask[c]);
            mask[c] = 0ull;
        }
        for (uint64_t q = many; q; q &= q - 1) {
            const int l = __builtin_ctzll(q);
            const uint32_t lc0 = readlane(c0, l), lnt = readlane(nt, l), lnx = readlane((uint32_t)nx, l);
            const float inv = 1.0f / (float)lnx;
            for (uint32_t k = lane; k < lnt; k += 64) {
                uint32_t y = (uint32_t)((float)k * inv);
                if (y * lnx > k) --y;
                if ((y + 1) * lnx <= k) ++y;
                const uint32_t c = lc0 + y * (uint32_t)(NW * tiles_x) + (k - y * lnx);
                // the highest lane of the tile settles it (a tile whose
                // highest lane is another one is settled by that one)
                const uint64_t mm = mask[c];
                if (mm >> l == 1ull) {
                    cur[c] += (uint32_t)__builtin_popcountll(mm);
                    mask[c] = 0ull;
                }
            }
            wave_sync();
        }
        wave_sync();
    };
    uint32_t queued = 0;
    uint32_t np = 0, nrc = 0;
    if (ur.x + lane < ur.y) {
        np = packed[ur.x + lane];
        nrc = rec[ur.x + lane];
    }
    for (uint32_t i0 = ur.x; i0 < ur.y; i0 += 64) {
        const bool in = i0 + lane < ur.y;
        const uint32_t p = np, r = nrc;
        if (i0 + 64 + lane < ur.y) {  // the next ones on their way
            np = packed[i0 + 64 + lane];
            nrc = rec[i0 + 64 + lane];
        }
        int f, last;
        rows_of(p, &f, &last);
        const bool hit = in && f <= last;
        const uint64_t hm = ballot(hit);
        if (hit) {
            const uint32_t s = queued + bits_below(hm);
            qp[w][s] = p;
            qr[w][s] = r;
        }
        queued += (uint32_t)__builtin_popcountll(hm);
        if (queued >= 64) {
            wave_sync();
            place(64);
            const uint32_t a = qp[w][64 + lane], c = qr[w][64 + lane];
            wave_sync();
            qp[w][lane] = a;
            qr[w][lane] = c;
            queued -= 64;
        }
    }
    wave_sync();
    if (queued) place(queued);
}

// The dispatch order as a launch of its own, for frames whose ranges come
// from k_ranges: one workgroup.
__global__ __launch_bounds__(1024) void k_tile_order(const uint2* __restrict__ ranges, uint32_t n_tiles,
                                                     uint32_t* __restrict__ order) {
    __shared__ uint32_t hist[64];
    if (threadIdx.x < 64) hist[threadIdx.x] = 0u;
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < n_tiles; t += 1024) {
        const uint2 r = ranges[t];
        atomicAdd(&hist[length_bucket(r.y - r.x)], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const uint32_t c = hist[threadIdx.x];
        hist[threadIdx.x] = wave_incl_scan(c) - c;
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < n_tiles; t += 1024) {
        const uint2 r = ranges[t];
        order[atomicAdd(&hist[length_bucket(r.y - r.x)], 1u)] = t;
    }
}

// ------------------------------------------------------------------- blend

constexpr float ALPHA_MAX = 0.99f;
constexpr float T_MIN = 1e-4f;
constexpr float LOG2_ALPHA_MAX = -0.0145f;  // just below log2(0.99)

__device__ __forceinline__ uint8_t to_u8(float x) {
    return (uint8_t)floorf(__builtin_fmaf(fminf(fmaxf(x, 0.0f), 1.0f), 255.0f, 0.5f));
}

struct BlendArgs {
    const ViewParams* views;
    int nviews;
    uint32_t n_lists, first;  // lists; the first one of the launch (a multiple of 8)
    int block_log;
    const uint2* ranges;
    const uint32_t* vals;  // the lists: records, or in a view with cells its records below masks of cells
    const Rec* rec;
    uint32_t nrec;
    unsigned long long* work;
    int cull;  // drop entries below the skip threshold on the whole block (never changes a pixel)
    const uint32_t* order;  // dense-first dispatch order of the lists of a single view (null: XCD chunks)
};

// A wave's LDS slice: the list entries whose pixel box meets its block, and the
// staged Gaussians: at most 7 left from the batch before and 64 new ones,
// rounded up to whole groups of eight.
struct Stage {
    float4 row[72];    // v relative to the block's origin, B, C, L
    float4 col[72];    // r, g, b, -1
    float nu[72];      // minus u relative to the block's origin
    float4 a[18];      // A, four entries each
    uint32_t q[128];   // records
};

// Does the Gaussian with exponent e(d) = A dx^2 + B dx dy + C dy^2 + L
// (negative-definite quadratic part) stay below the skip threshold on the
// whole rectangle [dx0, dx1] x [dy0, dy1] of offsets?  The maximum of a
// concave quadratic over a rectangle is at the unconstrained maximum when
// that lies inside, else on an edge facing the centre, where it is a 1D
// concave quadratic maximised at a clamped stationary point.  The test is
// conservative: it answers yes only with a margin far above the FP32
// rounding of this bound and of the per-pixel exponent, so a Gaussian it
// removes would have been skipped at every pixel of the rectangle.
// *low: the exponent stays below log2(ALPHA_MAX) (with the same margin: a
// concave quadratic is at most L), so the cap on alpha changes nothing.
__device__ __forceinline__ bool below_threshold(float A, float B, float C, float L, float dx0, float dx1, float dy0,
                                                float dy1, bool* low) {
    *low = false;
    if (!(A < 0.0f && C < 0.0f && B * B < 4.0f * A * C)) return false;  // not concave: keep it
    float q = 0.0f;
    if (!(dx0 <= 0.0f && dx1 >= 0.0f && dy0 <= 0.0f && dy1 >= 0.0f)) {
        const float ra = __builtin_amdgcn_rcpf(2.0f * A), rc = __builtin_amdgcn_rcpf(2.0f * C);
        auto edge_x = [&](float cx) {  // dx = cx fixed, best dy
            const float dy = fminf(fmaxf(-B * cx * rc, dy0), dy1);
            return (A * cx + B * dy) * cx + C * dy * dy;
        };
        auto edge_y = [&](float cy) {  // dy = cy fixed, best dx
            const float dx = fminf(fmaxf(-B * cy * ra, dx0), dx1);
            return (C * cy + B * dx) * cy + A * dx * dx;
        };
        // the maximum lies on a face visible from the centre (visibility is
        // affine-invariant, so it holds in the quadratic's own metric): the
        // x-face and the y-face on the centre's side suffice
        q = fmaxf(edge_x(dx1 < 0.0f ? dx1 : dx0), edge_y(dy1 < 0.0f ? dy1 : dy0));
    }
    const float r2 = fmaxf(dx0 * dx0, dx1 * dx1) + fmaxf(dy0 * dy0, dy1 * dy1);
    const float margin = 0.02f + 1e-5f * (fabsf(A) + fabsf(B) + fabsf(C)) * r2;
    *low = L + margin < LOG2_ALPHA_MAX;
    return q + L < LOG2_ALPHA_MIN - margin;  // false for NaN
}

// One block of 8x8 pixels of a list's, by one wave, a pixel per lane.  It walks
// the depth-sorted list 64 entries at a time and queues those whose pixel box meets the block;
// 64 queued ones at a time are fetched whole, those whose exponent can reach
// the skip threshold somewhere on the block (with culling on) are staged in
// LDS (ballot + mbcnt), and the 64 lanes composite them front to back in groups
// of eight, what is left of a group waiting for the next batch.  Each pixel's
// operations (and their rounding) are the same for every tile shape, and the
// entries culling drops are ones every pixel of the block skips.  The wave
// leaves as soon as all of its pixels have terminated.
//
// Bound by vector issue, so what has the form of a product with a constant
// over the block goes to the matrix cores, which run beside it: the
// v_mfma_f32_4x4x1_16b form is one FMA per element, rounded once, that takes a
// column of four values (of the lane's own 4x1 block, or of another one by the
// broadcast controls) against the lane's own value.  Per pair one of them adds
// the weighted colour and takes the weight from T (rows r, g, b, -1); per four
// pairs one each forms dx = px - u and spreads A over the lanes and the row
// terms B dy and C dy^2 + L, which lane l forms for entry l mod 8 and pixel row
// l / 8, over the lanes of their row.  With A read by a broadcast, that leaves
// 8 vector instructions per (pixel, Gaussian) pair (9 where alpha may reach
// ALPHA_MAX) besides 1.75 on the matrix cores, where colour, T, dx, permutes
// and the test for a stop took 14: 1454 instead of 2157 a wave at 3M/4K, the
// vector units issuing 92 % of the time.  Eight waves a SIMD need the 64
// registers of the launch bounds: with 90 (five waves) 602 us at 3M/4K instead
// of 521.  An entry's cells spare the gather of a box per entry and block, which
// kept the L1 busy (521 -> 426 us; a wave of 16 tiles' lists looks at 15 lists
// of 64 entries); pairs of words, with exact blocks, cost the placement more
// than they save (13 us at 3M/1080p).
// With a workgroup per tile, the launch at 3M/1080p, 3M/4K, 1M/720p and over 32
// views took 144, 418, 97 us and 2.39 ms; with the vector form before, 170, 497,
// 110 us and 2.87 ms.
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The staged entries 0 .. whole - 1 of a wave, in groups of eight, on its
// pixels.  A half group is first composited as if no pixel stopped in it: T only
// falls, so if no live pixel ends below T_MIN none did.  Else (a pixel stops
// once: a quarter of the half groups at 3M/1080p) it is composited again with
// the test at every pair.  A pixel that is done, an alpha below the threshold
// and a stop have a weight of zero, which leaves the (finite) colour sums and T
// exactly as they are.
template <bool CAP, bool COUNT>
__device__ __forceinline__ void blend_groups(const Stage& S, int lane, float pyr, f32x4 px4, uint32_t cnt,
                                             uint32_t whole, uint64_t& live, f32x4& acc, uint32_t& n_eval,
                                             uint32_t& n_contrib) {
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    lane = (int)fresh((uint32_t)lane);
    for (uint32_t j0 = 0; j0 < whole; j0 += 8) {
        if (live == 0) break;
        const uint32_t j = j0 + (uint32_t)(lane & 7);
        const float4 t = S.row[j];
        const float nu = S.nu[j];
        // column of entry k = lanes 4k .. 4k + 3
        const float col = reinterpret_cast<const float*>(&S.col[j0])[lane & 31];
        // the row terms: the very products and sums of the per-pixel exponent
        const float dy = pyr - t.x;
        const float rp = t.y * dy;
        const float rq = __builtin_fmaf(t.z * dy, dy, t.w);
#define TIGAS_ALPHA(I)                                                                                             \
    const float x##I = __builtin_amdgcn_exp2f(__builtin_fmaf(__builtin_fmaf(a4[I], dx[I], P[I]), dx[I], Q[I]));    \
    const float y##I = CAP ? fminf(ALPHA_MAX, x##I) : x##I;                                                        \
    const float al##I = __builtin_amdgcn_inverse_ballot_w64(ballot(y##I >= ALPHA_MIN) & live) ? y##I : 0.0f;
#define TIGAS_ADD(H, I, C, W) nxt = __builtin_amdgcn_mfma_f32_4x4x1f32(col, W, C, 4, 4 * (H) + (I), 0);
#define TIGAS_CHECKED(H, I, C)                                                                                     \
    {                                                                                                              \
        const float w = al##I * C[3];                                                                              \
        const uint64_t stop = ballot(C[3] - w < T_MIN) & ballot(al##I != 0.0f) & live;                             \
        live &= ~stop;                                                                                             \
        const bool add = __builtin_amdgcn_inverse_ballot_w64(live);                                                \
        if (COUNT && j0 + 4 * (H) + (I) < cnt) n_contrib += add && al##I != 0.0f ? 1u : 0u;                        \
        if (COUNT && j0 + 4 * (H) + (I) < cnt)                                                                     \
            n_eval += __builtin_amdgcn_inverse_ballot_w64(live | stop) ? 1u : 0u;                                  \
        TIGAS_ADD(H, I, C, add ? w : 0.0f)                                                                         \
    }
#define TIGAS_HALF(H)                                                                                              \
    {                                                                                                              \
        const f32x4 dx = __builtin_amdgcn_mfma_f32_4x4x1f32(nu, 1.0f, px4, 4, H, 0);                               \
        const f32x4 P = __builtin_amdgcn_mfma_f32_4x4x1f32(rp, 1.0f, zero, 1, H, 0);                               \
        const f32x4 Q = __builtin_amdgcn_mfma_f32_4x4x1f32(rq, 1.0f, zero, 1, H, 0);                               \
        const float4 af = S.a[j0 / 4 + (H)];                                                                       \
        const f32x4 a4 = {af.x, af.y, af.z, af.w};                                                                 \
        TIGAS_ALPHA(0)                                                                                             \
        TIGAS_ALPHA(1)                                                                                             \
        TIGAS_ALPHA(2)                                                                                             \
        TIGAS_ALPHA(3)                                                                                             \
        f32x4 nxt;                                                                                                 \
        TIGAS_ADD(H, 0, acc, al0 * acc[3])                                                                         \
        TIGAS_ADD(H, 1, nxt, al1 * nxt[3])                                                                         \
        TIGAS_ADD(H, 2, nxt, al2 * nxt[3])                                                                         \
        TIGAS_ADD(H, 3, nxt, al3 * nxt[3])                                                                         \
        if (ballot(nxt[3] < T_MIN) & live) {                                                                       \
            TIGAS_CHECKED(H, 0, acc)                                                                               \
            TIGAS_CHECKED(H, 1, nxt)                                                                               \
            TIGAS_CHECKED(H, 2, nxt)                                                                               \
            TIGAS_CHECKED(H, 3, nxt)                                                                               \
        } else if (COUNT) {                                                                                        \
            const uint32_t nv = min(4u, cnt - min(cnt, j0 + 4 * (H)));                                             \
            n_eval += __builtin_amdgcn_inverse_ballot_w64(live) ? nv : 0u;                                         \
            n_contrib += (al0 != 0.0f) + (al1 != 0.0f) + (al2 != 0.0f) + (al3 != 0.0f);                            \
        }                                                                                                          \
        acc = nxt;                                                                                                 \
    }
        TIGAS_HALF(0)
        __builtin_amdgcn_sched_barrier(0);
        TIGAS_HALF(1)
#undef TIGAS_HALF
#undef TIGAS_CHECKED
#undef TIGAS_ADD
#undef TIGAS_ALPHA
    }
}

template <bool COUNT, int PARTS>
__device__ __forceinline__ void blend_block(const BlendArgs& A, const ViewParams& v, uint32_t lt, uint32_t block,
                                            uint32_t part, Stage& S) {
    // the blocks of a list, row-major; those of an edge list may lie outside
    // the frame and have nothing to do
    // (scalars for what the whole wave shares, however the compiler loads it)
    auto scalar = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    const int lw = scalar(v.tw_log + v.lx), lh = scalar(v.th_log + v.ly);
    const int width = scalar(v.width), height = scalar(v.height);
    const uint32_t nx = (uint32_t)scalar(v.tiles_x), rec0 = (uint32_t)scalar((int)v.rec_base);
    const uint32_t ly = lt / nx, lx = lt - ly * nx;
    const int sx = scalar((int)((lx << lw) + ((block & ((1u << (lw - 3)) - 1u)) << 3)));
    const int sy = scalar((int)((ly << lh) + ((block >> (lw - 3)) << 3)));
    if (sx >= width || sy >= height) return;
    const int lane = (int)fresh(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(fresh(~0u), 0u)));
    // this wave's part of the block: all of it, the upper or lower half, or a
    // quarter; its lanes, and the rectangle of its pixel centres
    const int qx = PARTS == 4 ? (int)(part & 1u) * 4 : 0;
    const int qy = PARTS == 4 ? (int)(part >> 1) * 4 : PARTS == 2 ? (int)part * 4 : 0;
    const uint64_t own = PARTS == 1 ? ~0ull : (PARTS == 2 ? 0xffffffffull : 0x0f0f0f0full) << (qx + 8 * qy);
    const float cx0 = 0.5f + (float)qx, cx1 = PARTS == 4 ? cx0 + 3.0f : 7.5f;
    const float cy0 = 0.5f + (float)qy, cy1 = PARTS > 1 ? cy0 + 3.0f : 7.5f;
    const float pxr = (float)(lane & 7) + 0.5f, pyr = (float)(lane >> 3) + 0.5f;
    const float fsx = (float)sx, fsy = (float)sy;
    // the pixels still compositing, as a wave mask: the per-pair decisions are
    // combined in scalar registers and applied with one select
    uint64_t live = ballot(sx + (lane & 7) < width && sy + (lane >> 3) < height) & own;
    f32x4 acc = {0.0f, 0.0f, 0.0f, 1.0f};  // r, g, b, T
    const f32x4 px4 = {pxr, pxr, pxr, pxr};
    uint32_t n_eval = 0, n_contrib = 0;  // (pixel, Gaussian) evaluations / contributions, COUNT only
    // the wave's block clipped to the image: the only pixels it must cover
    const int bx1 = min(sx + 7, width - 1), by1 = min(sy + 7, height - 1);
    const uint2 rg = A.ranges[v.tile_base + lt];
    const uint32_t begin = (uint32_t)scalar((int)rg.x);
    const uint32_t end = (uint32_t)scalar((int)rg.y);
    auto wave_sync = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    uint32_t base = begin, queued = 0;
    // the cells of the list that hold the block
    const int cells = scalar(v.cells), rb = cell_rec_bits(cells) & 31;
    const uint32_t need = (1u << (rb + ((sx & ((1 << lw) - 1)) >> cell_log(lw, cells)))) |
                          (1u << ((rb + (1 << cells) + ((sy & ((1 << lh) - 1)) >> cell_log(lh, cells))) & 31));
    // (the lists' buffers have room for a read of 64 entries from any of them)
    uint32_t ahead = 0u;
    auto read = [&] {  // scalar base, 32-bit lane offset
        ahead = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(A.vals + base) + ((uint32_t)lane << 2));
    };
    if (base < end) read();
    auto scan = [&] {  // until a batch is queued or the list has ended
        while (queued < 64 && base < end) {
            uint32_t en = ahead;
            const uint64_t in = end - base >= 64 ? ~0ull : (1ull << (end - base)) - 1ull;
            base += 64;
            if (base < end) read();
            uint64_t m;
            if (cells) {
                m = in & ballot((en & need) == need);
                en = (en & ((1u << rb) - 1u)) + rec0;
            } else {
                bool hit = en < A.nrec && __builtin_amdgcn_inverse_ballot_w64(in);
                if (hit) {
                    const uint2 b = A.rec[en].bbox;
                    // x in the low halves, y in the high ones: compared where they are
                    hit = !(b.y << 16 < (uint32_t)sx << 16 || b.x << 16 > (uint32_t)bx1 << 16 ||
                            b.y < (uint32_t)sy << 16 || b.x >= (uint32_t)(by1 + 1) << 16);
                }
                m = ballot(hit);
            }
            if (__builtin_amdgcn_inverse_ballot_w64(m)) S.q[queued + bits_below(m)] = en;
            queued += (uint32_t)__builtin_popcountll(m);
        }
    };
    uint32_t nb = 0, rec = 0;  // records fetched, the lane's
    auto fetch = [&] {  // up to 64 queued records; the others move up
        wave_sync();
        nb = min(queued, 64u);
        queued -= nb;
        rec = S.q[lane];
        const uint32_t next = S.q[64 + lane];
        if ((uint32_t)lane < queued) S.q[lane] = next;
        wave_sync();
    };
    scan();
    fetch();
    float* const sa = reinterpret_cast<float*>(S.a);
    uint32_t left = 0;      // staged, waiting for a whole group
    uint64_t capped = 0;    // a staged Gaussian's alpha may reach ALPHA_MAX
    for (;;) {
        float4 f0, f1, f2;  // of the first nb lanes
        if ((uint32_t)lane < nb && rec < A.nrec) {
            f0 = A.rec[rec].r0;
            f1 = A.rec[rec].r1;
            f2 = A.rec[rec].r2;
        }
        // pixel centre relative to the block's origin, hi and lo parts combined here
        const float u = (f0.x - fsx) + f0.z, v0 = (f0.y - fsy) + f0.w;
        bool low;
        const bool below = below_threshold(f1.x, f1.y, f1.z, f1.w, cx0 - u, cx1 - u, cy0 - v0, cy1 - v0, &low);
        const bool hit = (uint32_t)lane < nb && !(A.cull && below);
        const uint64_t m = ballot(hit);
        capped = (left ? capped : 0) | (m & ~ballot(low));
        if (hit) {
            const uint32_t slot = left + bits_below(m);
            S.nu[slot] = -u;
            sa[slot] = f1.x;
            S.row[slot] = make_float4(v0, f1.y, f1.z, f1.w);
            S.col[slot] = make_float4(f2.x, f2.y, f2.z, __uint_as_float(fresh(__float_as_uint(-1.0f))));
        }
        const uint32_t cnt = left + (uint32_t)__builtin_popcountll(m);
        scan();
        const bool last = queued == 0;  // uniform
        if (!last) fetch();
        uint32_t whole = cnt & ~7u;
        if (last && whole < cnt) {  // entries that reach no pixel fill the last group
            whole += 8;
            const uint32_t slot = cnt + fresh(lane);
            if (slot < whole) {
                const float z = __uint_as_float(fresh(0u));
                S.nu[slot] = sa[slot] = z;
                S.row[slot] = make_float4(z, z, z, __uint_as_float(fresh(__float_as_uint(-1e30f))));
                S.col[slot] = make_float4(z, z, z, z);
            }
        }
        wave_sync();
        if (capped) blend_groups<true, COUNT>(S, lane, pyr, px4, cnt, whole, live, acc, n_eval, n_contrib);
        else blend_groups<false, COUNT>(S, lane, pyr, px4, cnt, whole, live, acc, n_eval, n_contrib);
        if (live == 0 || last) break;
        left = cnt - whole;
        if (left && whole) {
            const uint32_t ln = fresh(lane), l = ln & 7u;
            const float4 t = S.row[whole + l], c = S.col[whole + l];
            const float nu = S.nu[whole + l], ca = sa[whole + l];
            if (ln < left) {
                S.row[ln] = t;
                S.col[ln] = c;
                S.nu[ln] = nu;
                sa[ln] = ca;
            }
        }
        wave_sync();
    }
    if (COUNT) {
        const uint32_t se = wave_sum(n_eval), sc = wave_sum(n_contrib);
        if (lane == 0) {
            atomicAdd(&A.work[0], (unsigned long long)se);
            atomicAdd(&A.work[1], (unsigned long long)sc);
        }
    }
    const int ln = (int)fresh(lane), px = sx + (ln & 7), py = sy + (ln >> 3);
    if (px < width && py < height && __builtin_amdgcn_inverse_ballot_w64(own)) {
        const float r = __builtin_fmaf(acc[3], v.bg[0], acc[0]);
        const float g = __builtin_fmaf(acc[3], v.bg[1], acc[1]);
        const float b = __builtin_fmaf(acc[3], v.bg[2], acc[2]);
        const size_t pix = (size_t)py * (size_t)width + (size_t)px;
        if (v.fmt == 1) {
            float* out = reinterpret_cast<float*>(v.out_ptr) + pix * 3;
            out[0] = r;
            out[1] = g;
            out[2] = b;
        } else {
            uint8_t* out = reinterpret_cast<uint8_t*>(v.out_ptr) + pix * 3;
            out[0] = to_u8(r);
            out[1] = to_u8(g);
            out[2] = to_u8(b);
        }
    }
}

// One wave per workgroup: a workgroup of several holds its slots until its
// longest block is done, and one that pulled its tiles from a queue waited for
// it at every tile.  Launches of one wave against a workgroup per tile of 16x32:
// 3M/1080p 131 and 145 us, 3M/4K 378 and 423, 1M/720p 91 and 98, 20k/256x256 33
// and 39, 32 views 2.07 ms and 2.43 (a queue of four blocks an item 2.89).
// A workgroup per part of a block (2^block_log blocks for every list, the most of any view):
// list i of the dispatch order on XCD i mod 8 (consecutive workgroups go
// round-robin to the XCDs), so that a list's records are fetched into one L2.
// A single view's lists come dense first: the launch ends with short ones
// instead of a tail of long ones.
template <bool COUNT, int PARTS>
__global__ __launch_bounds__(64, COUNT ? 1 : 8) void k_blend(BlendArgs A) {
    __shared__ Stage stage;
    constexpr int PL = PARTS / 2;  // log2 of 1, 2, 4
    const uint32_t part = (blockIdx.x >> 3) & (PARTS - 1), slot = blockIdx.x >> (3 + PL);
    const uint32_t i = A.first + ((slot >> A.block_log) << 3) + (blockIdx.x & 7u);
    if (i >= A.n_lists) return;
    const uint32_t list = A.order ? A.order[i] : i, block = slot & ((1u << A.block_log) - 1u);
    const int vi = view_of(list, A.nviews, [&](int k) { return A.views[k].tile_base; });
    const ViewParams& v = A.views[vi];
    if (block >> (v.tw_log + v.lx + v.th_log + v.ly - 6)) return;
    blend_block<COUNT, PARTS>(A, v, list - v.tile_base, block, part, stage);
}

// One view's parameters, passed by value as a kernel argument, stored to
// device memory (the allocation-free entry point has no pinned host copy), and
// the clearing of the counters it keeps in its fixed scratch array: one launch
// instead of two (100k records at 960x540 82.8 -> 80.4 us).
__global__ void k_store_view(ViewParams v, ViewParams* __restrict__ dst, uint32_t* __restrict__ clear,
                             uint32_t nclear) {
    constexpr int W = (int)(sizeof(ViewParams) / 4);
    static_assert(sizeof(ViewParams) % 4 == 0, "view parameters are whole words");
    const uint32_t* src = reinterpret_cast<const uint32_t*>(&v);
    for (int i = threadIdx.x; i < W; i += blockDim.x) reinterpret_cast<uint32_t*>(dst)[i] = src[i];
    for (uint32_t i = threadIdx.x; i < nclear; i += blockDim.x) clear[i] = 0u;
}

__global__ void k_wave_scan_selftest(const uint32_t* in, uint32_t* out, int n) {
    const int i = blockIdx.x * 64 + threadIdx.x;
    const uint32_t x = i < n ? in[i] : 0u;
    const uint32_t s = wave_incl_scan(x);
    if (i < n) out[i] = s;
}

// ------------------------------------------------------------- launchers

#define TIGAS_LAUNCH_SHM(kernel, grid, block, shm, st, ...)                               \
    do {                                                                                  \
        KernelTimer* kt_ = g_kernel_timer;                                                \
        if (kt_) kt_->before(reinterpret_cast<const void*>(kernel), st);                 \
        hipLaunchKernelGGL(kernel, grid, block, shm, st, __VA_ARGS__);                    \
        if (kt_) kt_->after(st);                                                          \
    } while (0)
#define TIGAS_LAUNCH(kernel, grid, block, st, ...) TIGAS_LAUNCH_SHM(kernel, grid, block, 0, st, __VA_ARGS__)

template <int ST>
static void preprocess_deg(int deg, dim3 grid, const SceneView& s, const ViewParams* v, int nv, uint32_t rb,
                           uint32_t np, uint32_t vb, const PreOut& o, hipStream_t st) {
    switch (deg) {
        case 0: TIGAS_LAUNCH((k_preprocess<ST, 0>), grid, dim3(K1_THREADS), st, s, v, nv, rb, np, vb, o); break;
        case 1: TIGAS_LAUNCH((k_preprocess<ST, 1>), grid, dim3(K1_THREADS), st, s, v, nv, rb, np, vb, o); break;
        case 2: TIGAS_LAUNCH((k_preprocess<ST, 2>), grid, dim3(K1_THREADS), st, s, v, nv, rb, np, vb, o); break;
        default: TIGAS_LAUNCH((k_preprocess<ST, 3>), grid, dim3(K1_THREADS), st, s, v, nv, rb, np, vb, o); break;
    }
}

void launch_preprocess(const SceneView& s, const ViewParams* views_dev, const ViewParams* views_host, int nviews,
                       uint32_t rec_base, uint32_t n_pad, uint32_t view_base, const PreOut& o, hipStream_t st) {
    // the SH coefficients loaded are those of the highest degree any view uses
    int deg = 0;
    for (int i = 0; i < nviews; ++i) deg = views_host[i].sh_degree > deg ? views_host[i].sh_degree : deg;
    const dim3 grid(n_pad / K1_THREADS);
    if (s.storage == 0) preprocess_deg<0>(deg, grid, s, views_dev, nviews, rec_base, n_pad, view_base, o, st);
    else if (s.storage == 1) preprocess_deg<1>(deg, grid, s, views_dev, nviews, rec_base, n_pad, view_base, o, st);
    else preprocess_deg<2>(deg, grid, s, views_dev, nviews, rec_base, n_pad, view_base, o, st);
}


void launch_store_view(const ViewParams& v, ViewParams* dst, uint32_t* clear, uint32_t nclear, hipStream_t st) {
    TIGAS_LAUNCH(k_store_view, dim3(1), dim3(64), st, v, dst, clear, nclear);
}

void launch_scan_visible(const PreOut& o, int nblk, uint32_t* blk_off, Counters* cnt, uint32_t cap,
                         const ZeroList& zl, hipStream_t st) {
    const int nchunks = std::max(1, (nblk + SCAN_CHUNK - 1) / SCAN_CHUNK);
    TIGAS_LAUNCH(k_chunk_totals, dim3(nchunks), dim3(SCAN_THREADS), st, (const uint32_t*)o.blk_vis, nblk,
                 (const uint32_t*)o.blk_sum, (const uint32_t*)o.blk_fb, o.chunk_vis, o.chunk_dup, o.chunk_fb);
    TIGAS_LAUNCH(k_scan_visible, dim3(nchunks), dim3(SCAN_THREADS), st, (const uint32_t*)o.blk_vis, nblk,
                 (const uint32_t*)o.chunk_vis, (const unsigned long long*)o.chunk_dup, (const uint32_t*)o.chunk_fb,
                 nchunks, blk_off, cnt, cap, zl);
}

void launch_compact(const PreOut& o, int nblk, const uint32_t* blk_off, uint32_t* key, uint32_t* val, uint32_t* ext,
                    const ViewParams* views_dev, hipStream_t st) {
    if (nblk == 0) return;
    TIGAS_LAUNCH(k_compact, dim3((nblk + 3) / 4), dim3(K1_THREADS), st, o.zkey, (const uint2*)o.rect,
                 blk_off, nblk, key, val, ext, (const Counters*)o.cnt, (const uint2*)o.fb_list, o.fb_cap, views_dev,
                 (const uint32_t*)o.blk_view, o.rec);
}

void launch_duplicate(const PreOut& o, int nblk, const uint32_t* sorted_rec, const uint2* sorted_rect,
                      const uint32_t* sorted_packed,
                      uint32_t* blk_sum2, uint32_t* blk_off2, const Counters* cnt, uint32_t cap,
                      const ViewParams* views_dev, uint32_t* tile_out, uint32_t* val_out, uint32_t* depth_out,
                      hipStream_t st) {
    if (nblk == 0) return;
    TIGAS_LAUNCH(k_sorted_sums, dim3(std::min(nblk, 8192)), dim3(K1_THREADS), st, sorted_rect, sorted_packed, cnt, nblk,
                 blk_sum2);
    const int nchunks = std::max(1, (nblk + SCAN_CHUNK - 1) / SCAN_CHUNK);
    TIGAS_LAUNCH(k_chunk_totals, dim3(nchunks), dim3(SCAN_THREADS), st, (const uint32_t*)blk_sum2, nblk,
                 (const uint32_t*)nullptr, (const uint32_t*)nullptr, o.chunk_dups, (unsigned long long*)nullptr,
                 (uint32_t*)nullptr);
    TIGAS_LAUNCH(k_scan_dups, dim3(nchunks), dim3(SCAN_THREADS), st, (const uint32_t*)blk_sum2, nblk,
                 (const uint32_t*)o.chunk_dups, blk_off2, nchunks, (Counters*)nullptr);
    if (depth_out)
        TIGAS_LAUNCH(k_duplicate<true>, dim3(nblk), dim3(K1_THREADS), st, sorted_rec, sorted_rect, sorted_packed,
                     o.zkey, (const uint32_t*)blk_off2, o.blk_view, cnt, cap, views_dev, tile_out, val_out, depth_out);
    else
        TIGAS_LAUNCH(k_duplicate<false>, dim3(nblk), dim3(K1_THREADS), st, sorted_rec, sorted_rect, sorted_packed,
                     o.zkey, (const uint32_t*)blk_off2, o.blk_view, cnt, cap, views_dev, tile_out, val_out, depth_out);
}

void launch_duplicate_culled(const PreOut& o, int nblk, const uint32_t* sorted_rec, const uint32_t* sorted_packed,
                             uint32_t* blk_cnt, uint32_t* blk_off, Counters* cnt, const ViewParams* views_dev,
                             int tile_w, int tile_h, uint32_t* tile_out, uint32_t* val_out, uint32_t* depth_out,
                             hipStream_t st) {
    if (nblk == 0) return;
    TIGAS_LAUNCH((k_duplicate_culled<true, false>), dim3(nblk), dim3(K1_THREADS), st, sorted_rec, sorted_packed,
                 o.zkey, (const uint32_t*)nullptr, blk_cnt, (const uint32_t*)o.blk_view, (const Counters*)cnt,
                 views_dev, (const Rec*)o.rec, tile_w, tile_h, (uint32_t*)nullptr, (uint32_t*)nullptr,
                 (uint32_t*)nullptr);
    const int nchunks = std::max(1, (nblk + SCAN_CHUNK - 1) / SCAN_CHUNK);
    TIGAS_LAUNCH(k_chunk_totals, dim3(nchunks), dim3(SCAN_THREADS), st, (const uint32_t*)blk_cnt, nblk,
                 (const uint32_t*)nullptr, (const uint32_t*)nullptr, o.chunk_dups, (unsigned long long*)nullptr,
                 (uint32_t*)nullptr);
    // the kept count becomes the frame's duplicate count D
    TIGAS_LAUNCH(k_scan_dups, dim3(nchunks), dim3(SCAN_THREADS), st, (const uint32_t*)blk_cnt, nblk,
                 (const uint32_t*)o.chunk_dups, blk_off, nchunks, cnt);
    if (depth_out)
        TIGAS_LAUNCH((k_duplicate_culled<false, true>), dim3(nblk), dim3(K1_THREADS), st, sorted_rec, sorted_packed,
                     o.zkey, (const uint32_t*)blk_off, blk_cnt, (const uint32_t*)o.blk_view, (const Counters*)cnt,
                     views_dev, (const Rec*)o.rec, tile_w, tile_h, tile_out, val_out, depth_out);
    else
        TIGAS_LAUNCH((k_duplicate_culled<false, false>), dim3(nblk), dim3(K1_THREADS), st, sorted_rec, sorted_packed,
                     o.zkey, (const uint32_t*)blk_off, blk_cnt, (const uint32_t*)o.blk_view, (const Counters*)cnt,
                     views_dev, (const Rec*)o.rec, tile_w, tile_h, tile_out, val_out, depth_out);
}

void launch_bucket_sort(const PreOut& o, const BucketMem& b, const ViewParams* views_dev, int nviews, uint32_t nseg,
                        uint32_t nchunks, uint32_t seg_len, Counters* cnt, uint32_t cap, const ZeroList& zl,
                        bool flag_wide, bool flag_crowd, uint32_t split, uint32_t nunits, uint32_t* val, uint32_t* ext,
                        hipStream_t st) {
#define TIGAS_COUNT(M, GRID)                                                                                          \
    do {                                                                                                              \
        if (split)                                                                                                    \
            TIGAS_LAUNCH((k_bucket_count<M, true>), dim3(GRID), dim3(BUCKET_THREADS), st, o, b, views_dev, nviews,    \
                         nseg, seg_len, split, zl);                                                                          \
        else                                                                                                          \
            TIGAS_LAUNCH((k_bucket_count<M, false>), dim3(GRID), dim3(BUCKET_THREADS), st, o, b, views_dev, nviews,   \
                         nseg, seg_len, split, zl);                                                                          \
    } while (0)
    if (nseg <= BUCKET_FORM_SEGMENTS) {
        TIGAS_COUNT(FORM, std::max(nseg, 1u));
    } else {
        TIGAS_COUNT(FORM_ONLY, nviews);
        TIGAS_COUNT(READ, nseg);
    }
#undef TIGAS_COUNT
    TIGAS_LAUNCH(k_bucket_scan, dim3(nchunks + 1), dim3(1024), st, b, views_dev, nviews, nseg, nchunks, cnt, cap,
                 flag_wide, flag_crowd, nunits);
    if (nseg == 0) return;
    if (split)
        TIGAS_LAUNCH(k_bucket_scatter<true>, dim3(nseg), dim3(BUCKET_THREADS), st, o, b, views_dev, nviews, nseg,
                     seg_len, (const Counters*)cnt);
    else
        TIGAS_LAUNCH(k_bucket_scatter<false>, dim3(nseg), dim3(BUCKET_THREADS), st, o, b, views_dev, nviews, nseg,
                     seg_len, (const Counters*)cnt);
    TIGAS_LAUNCH(k_bucket_sort, dim3(nchunks * COL_CHUNK), dim3(BUCKET_SORT_THREADS), st, o, b, views_dev,
                 nviews, (const Counters*)cnt, val, ext);
}

int launch_sort(const SortBuffers& b, const SortPass* passes, int npasses, int which, uint32_t cap, int nblocks,
                int start, bool extra, Counters* cnt, const uint2* rect_src,
                uint2* rect_dst, hipStream_t st) {
    int cur = start;
    for (int p = 0; p < npasses; ++p) {
        const SortPass& ps = passes[p];
        TIGAS_LAUNCH(k_sort_upsweep, dim3(nblocks), dim3(SORT_THREADS), st, (const uint32_t*)b.key[cur], cnt, which,
                     cap, ps.shift, ps.bits, b.hist, nblocks);
        const int ndig = 1 << ps.bits;
        if (nblocks <= 1024) TIGAS_LAUNCH(k_sort_scan<4>, dim3(ndig), dim3(256), st, b.hist, b.dtot, nblocks);
        else TIGAS_LAUNCH((k_sort_scan<SORT_MAX_BLOCKS / 256>), dim3(ndig), dim3(256), st, b.hist, b.dtot, nblocks);
        const bool sums = rect_src && p + 1 == npasses;
#define TIGAS_DOWN(E, S)                                                                                        \
    TIGAS_LAUNCH((k_sort_downsweep<E, S>), dim3(nblocks), dim3(SORT_THREADS), st, b.key[cur], b.val[cur],       \
                 b.ext[cur], b.key[cur ^ 1], b.val[cur ^ 1], b.ext[cur ^ 1], cnt, which, cap, ps.shift, ps.bits, \
                 (const uint32_t*)b.hist, (const uint32_t*)b.dtot, nblocks, rect_src, rect_dst)
        if (extra && sums) TIGAS_DOWN(true, true);
        else if (extra) TIGAS_DOWN(true, false);
        else if (sums) TIGAS_DOWN(false, true);
        else TIGAS_DOWN(false, false);
#undef TIGAS_DOWN
        cur ^= 1;
    }
    return cur;
}

void launch_tile_order(const uint2* ranges, uint32_t n_tiles, uint32_t* order, hipStream_t st) {
    if (n_tiles) TIGAS_LAUNCH(k_tile_order, dim3(1), dim3(1024), st, ranges, n_tiles, order);
}

void launch_ranges(const uint32_t* tile_sorted, const Counters* cnt, uint32_t cap, uint2* ranges, FrameCounters* host_cnt,
                   hipStream_t st) {
    // one 1024-word step per workgroup at capacity, but no more workgroups
    // than a large frame needs (the capacity may have been sized by a much
    // larger frame)
    TIGAS_LAUNCH(k_ranges, dim3(std::min<uint32_t>(16384u, std::max<uint32_t>(1u, (cap + 1023) / 1024))), dim3(256), st,
                 tile_sorted, cnt, cap, ranges, host_cnt);
}

void launch_tiles(const TileMem& m, const BucketMem& b, const ViewParams* views_dev, const ViewParams* views_host,
                  int nviews, uint32_t nrec, const Counters* cnt, bool flat, uint32_t nchunks, const uint32_t* rec,
                  const uint32_t* packed, uint2* ranges, uint32_t* order,
                  FrameCounters* host_cnt, uint32_t* val_out,
                  uint32_t* tile_out, uint32_t* depth_out, const uint32_t* zkey, hipStream_t st) {
    int groups = 1;
    for (int i = 0; i < nviews; ++i) {
        const int rpg = tile_group_rows(views_host[i].tiles_x);
        groups = std::max(groups, (views_host[i].tiles_y + rpg - 1) / rpg);
    }
    const uint32_t units = m.nunits + (flat ? 0u : (uint32_t)nviews);
    const uint32_t nfront = std::max<uint32_t>(1u, (nchunks * TILE_CHUNK + TILE_FRONT_TILES - 1) / TILE_FRONT_TILES);
    TIGAS_LAUNCH(k_tile_count, dim3(units, groups), dim3(TILE_THREADS), st, m, b, views_dev, nviews, cnt, flat, packed);
    if (nchunks) TIGAS_LAUNCH(k_tile_scan, dim3(nchunks), dim3(1024), st, m, b, views_dev, nviews, cnt, flat);
    const uint32_t gx = (nfront + units + 7) / 8 * 8;  // a multiple of the XCDs: a column of the grid stays on one
    if (tile_out)
        TIGAS_LAUNCH((k_tile_emit<true, 4>), dim3(gx, groups), dim3(256), st, m, b, views_dev, nviews, cnt, flat,
                     nfront, nchunks, ranges, order, host_cnt, rec, packed, val_out, tile_out, depth_out, zkey);
    else if (nrec <= TILE_WIDE_RECORDS)
        TIGAS_LAUNCH((k_tile_emit<false, 8>), dim3(gx, groups), dim3(512), st, m, b, views_dev, nviews, cnt, flat,
                     nfront, nchunks, ranges, order, host_cnt, rec, packed, val_out, tile_out, depth_out, zkey);
    else
        TIGAS_LAUNCH((k_tile_emit<false, 4>), dim3(gx, groups), dim3(256), st, m, b, views_dev, nviews, cnt, flat,
                     nfront, nchunks, ranges, order, host_cnt, rec, packed, val_out, tile_out, depth_out, zkey);
}

// Up to these numbers of blocks a wave takes a quarter or a half of one.  The
// chip has 1024 SIMDs: with few blocks the launch lasts as long as the longest
// block's chain of pairs, and a part of it meets fewer Gaussians (a quarter
// 55 where the block meets 89, at 20k/256x256); with more of them the work that
// the parts do again costs more.  Launches of 1, 2 and 4 waves a block, 20k and
// 100k Gaussians over the frame: 256x256 (1024 blocks) 33 / 28 / 24 and 42 / 35 /
// 31 us; 320x320 (1600) 28 / 25 / 23 and 36 / 34 / 32; 384x384 (2304) 25.0 / 22.6 /
// 22.1 and 32.1 / 32.1 / 35.2; 448x448 (3136) 23.7 / 22.1 / 24.2 and 31.8 / 31.9 /
// 37.9; 512x512 (4096) 22.4 / 21.8 / 27.9 and 31.1 / 34.0 / 43.9.
constexpr uint64_t BLEND_QUARTERS = 1800, BLEND_HALVES = 3200;

void launch_blend(const ViewParams* views_dev, const ViewParams* views_host, int nviews, uint32_t n_lists,
                  const uint2* ranges, const uint32_t* vals, const PreOut& o, uint32_t nrec,
                  unsigned long long* work, bool cull, const uint32_t* order, hipStream_t st) {
    if (n_lists == 0) return;
    int bl = 0;  // log2 of a list's blocks
    uint64_t blocks = 0;  // inside the frames
    for (int i = 0; i < nviews; ++i) {
        const ViewParams& v = views_host[i];
        bl = std::max(bl, v.tw_log + v.lx + v.th_log + v.ly - 6);
        blocks += (uint64_t)((v.width + 7) / 8) * (uint64_t)((v.height + 7) / 8);
    }
    BlendArgs A{views_dev, nviews, n_lists, 0, bl, ranges, vals, o.rec, nrec, work, cull ? 1 : 0,
                order};
    const int pl = work || blocks > BLEND_HALVES ? 0 : blocks > BLEND_QUARTERS ? 1 : 2;
    // a launch has fewer than 2^32 threads: 2^26 blocks' waves, past which a batch of
    // 16 frames of 16384x16384 goes, or one of many lists beside a view with lists
    // of 128 blocks
    const uint32_t per = 1u << (25 - bl - pl);  // lists a launch at most
    for (; A.first < n_lists; A.first += per) {
        const dim3 grid((std::min(per, n_lists - A.first) + 7) / 8 * 8 << (bl + pl));
        if (work) TIGAS_LAUNCH((k_blend<true, 1>), grid, dim3(64), st, A);
        else if (pl == 2) TIGAS_LAUNCH((k_blend<false, 4>), grid, dim3(64), st, A);
        else if (pl == 1) TIGAS_LAUNCH((k_blend<false, 2>), grid, dim3(64), st, A);
        else TIGAS_LAUNCH((k_blend<false, 1>), grid, dim3(64), st, A);
    }
}

void launch_wave_scan_selftest(const uint32_t* in, uint32_t* out, int n, hipStream_t st) {
    TIGAS_LAUNCH(k_wave_scan_selftest, dim3((n + 63) / 64), dim3(64), st, in, out, n);
}

}  // namespace tigas
