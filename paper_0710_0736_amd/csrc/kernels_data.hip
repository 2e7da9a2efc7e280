// kernels_data.hip -- image data on refined lattices, the consistent-mass and
// by-simplex views of the image, and the colour-space pre-pass.  Each is one pass over the data
// (HBM bound).
#include <algorithm>

#include "acseg_internal.h"

namespace acseg {

namespace {

// Four adjacent elements at once; the address needs 4-byte alignment only.
typedef float gfloat4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kRowBlocks = 4096;  // grid-stride over rows: enough workgroups to fill the chip

// Piecewise-constant injection: row Y of plane c of the refined lattice copies
// pixel row Y >> r, each pixel value repeated over the 2^r nodes it owns along
// x (the last pixel owns one node).  One workgroup per row (grid-stride),
// coalesced writes; the pixel row is read from cache 2^r times.
__global__ __launch_bounds__(kBlock) void k_refine(const float* __restrict__ src, float* __restrict__ dst,
                                                   int W, int H, int r, int Wf, int Hf, int planes) {
    const int64_t n = (int64_t)W * H, nf = (int64_t)Wf * Hf;
    const int64_t rows = (int64_t)Hf * planes;
    for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
        const int c = (int)(row / Hf), Y = (int)(row - (int64_t)c * Hf);
        const float* s = src + c * n + (int64_t)(Y >> r) * W;
        float* d = dst + c * nf + (int64_t)Y * Wf;
        for (int X = threadIdx.x; X < Wf; X += kBlock) d[X] = s[X >> r];
    }
}

// The pixel nodes of a refined field: dst[c][y][x] = src[c][y 2^r][x 2^r].
__global__ __launch_bounds__(kBlock) void k_sample(const float* __restrict__ src, float* __restrict__ dst,
                                                   int W, int H, int r, int Wf, int Hf, int planes) {
    const int64_t n = (int64_t)W * H, nf = (int64_t)Wf * Hf;
    const int64_t rows = (int64_t)H * planes;
    for (int64_t row = blockIdx.x; row < rows; row += gridDim.x) {
        const int c = (int)(row / H), y = (int)(row - (int64_t)c * H);
        const float* s = src + c * nf + ((int64_t)y << r) * Wf;
        float* d = dst + c * n + (int64_t)y * W;
        for (int x = threadIdx.x; x < W; x += kBlock) d[x] = s[(int64_t)x << r];
    }
}

// sRGB (IEC 61966-2-1) to CIE 1976 L*a*b*, divided by 100.
//   linear c = v / 12.92 for v <= 0.04045, else ((v + 0.055) / 1.055)^2.4;
//   (X, Y, Z) = M (r, g, b) with the sRGB primaries' matrix M (D65);
//   f(t) = t^(1/3) for t > (6/29)^3, else t / (3 (6/29)^2) + 4/29;
//   L* = 116 f(Y/Yw) - 16, a* = 500 (f(X/Xw) - f(Y/Yw)), b* = 200 (f(Y/Yw) - f(Z/Zw)),
// with (Xw, Yw, Zw) = M (1, 1, 1), the row sums of M.
//
// The powers start from the hardware's exp2(e log2 v) and take one Newton step on the
// polynomial they solve, v^(12/5) = v^2 y with y^5 = v^2 and t^(1/3) = y with y^3 = t:
// the step squares the relative error of the start (a few 1e-7), so the result
// is exact to rounding, in about 15 instructions each where powf and cbrtf took the
// pass's time (1920 x 1080: 28 -> 14 us).
__device__ __forceinline__ float srgb_linear(float v) {
    const float a = (v + 0.055f) * (1.f / 1.055f);
    const float s = a * a;
    float y = __builtin_amdgcn_exp2f(0.4f * __builtin_amdgcn_logf(a));
    const float y2 = y * y, y4 = y2 * y2;
    // (an infinite v has no step to take)
    if (s < INFINITY) y = fmaf(fmaf(-y4, y, s), 0.2f * __builtin_amdgcn_rcpf(y4), y);
    return v <= 0.04045f ? v * (1.f / 12.92f) : s * y;
}
__device__ __forceinline__ float lab_f(float t) {
    constexpr float d = 6.f / 29.f;
    float y = __builtin_amdgcn_exp2f((1.f / 3.f) * __builtin_amdgcn_logf(t));
    const float y2 = y * y;
    if (t < INFINITY) y = fmaf(fmaf(-y2, y, t), (1.f / 3.f) * __builtin_amdgcn_rcpf(y2), y);
    return t > d * d * d ? y : t * (1.f / (3.f * d * d)) + 4.f / 29.f;
}

// One pixel's (L*, a*, b*) / 100.
__device__ __forceinline__ void lab_of(float vr, float vg, float vb, float& L, float& A, float& B) {
    constexpr float m00 = 0.4124f, m01 = 0.3576f, m02 = 0.1805f;
    constexpr float m10 = 0.2126f, m11 = 0.7152f, m12 = 0.0722f;
    constexpr float m20 = 0.0193f, m21 = 0.1192f, m22 = 0.9505f;
    constexpr float xw = m00 + m01 + m02, yw = m10 + m11 + m12, zw = m20 + m21 + m22;
    const float r = srgb_linear(vr), g = srgb_linear(vg), b = srgb_linear(vb);
    const float fx = lab_f((m00 * r + m01 * g + m02 * b) / xw);
    const float fy = lab_f((m10 * r + m11 * g + m12 * b) / yw);
    const float fz = lab_f((m20 * r + m21 * g + m22 * b) / zw);
    L = 1.16f * fy - 0.16f;
    A = 5.f * (fx - fy);
    B = 2.f * (fy - fz);
}

// Two pixels per thread and access.
template <bool AB>
__global__ __launch_bounds__(kBlock) void k_lab(const float* __restrict__ rgb, float* __restrict__ dst,
                                                int64_t count) {
    const int64_t step = 2 * (int64_t)gridDim.x * kBlock;
    for (int64_t p = 2 * ((int64_t)blockIdx.x * kBlock + threadIdx.x); p < count; p += step) {
        const bool two = p + 1 < count;
        float v[3][2], o[3][2];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float* s = rgb + k * count + p;
            if (two) {
                const gfloat2 t = *(const gfloat2*)s;
                v[k][0] = t.x;
                v[k][1] = t.y;
            } else {
                v[k][0] = v[k][1] = s[0];
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) lab_of(v[0][j], v[1][j], v[2][j], o[0][j], o[1][j], o[2][j]);
#pragma unroll
        for (int k = AB ? 1 : 0; k < 3; ++k) {
            float* d = dst + (k - (AB ? 1 : 0)) * count + p;
            d[0] = o[k][0];
            if (two) d[1] = o[k][1];
        }
    }
}

// The image as the consistent P1 mass matrix sees it: (M I)_p / m_p, every
// lattice cell split along its (x,y)-(x+1,y+1) diagonal.  A triangle T at node
// p with other vertices a, b adds |T|/12 (2 I_p + I_a + I_b) to (M I)_p and
// |T|/3 to the lumped mass m_p, so (M I)_p / m_p is the sum over the n_T
// triangles at p of (2 I_p + I_a + I_b), divided by 4 n_T (6 triangles inside;
// fewer on the boundary, at least one).
// SIMPLEX: projection by simplex instead.  Each triangle carries one value, the
// mean (I_p + I_a + I_b) / 3 of its vertices (its integral over |T|), and adds
// |T|/3 of it to node p's load, so the nodal value is the sum over the n_T
// triangles of (I_p + I_a + I_b), divided by 3 n_T.  Four nodes of a row per thread:
// three vector reads and four single ones instead of 28.  1920 x 1080 RGB: 35 -> 21 us.
template <bool SIMPLEX>
__global__ __launch_bounds__(kBlock) void k_mass_avg(const float* __restrict__ src, float* __restrict__ dst,
                                                     int W, int H, int planes) {
    const uint32_t n = (uint32_t)W * H;
    const uint32_t q = blockIdx.x * kBlock + threadIdx.x;  // column group q mod gx of row q / gx
    const uint32_t gx = ((uint32_t)W + 3) / 4;
    const int y = (int)(q / gx), x = 4 * (int)(q - (uint32_t)y * gx);
    if (y >= H) return;
    const uint32_t p = (uint32_t)y * W + x;
    const bool D = y > 0, U = y < H - 1;
    const uint32_t pd = D ? p - W : p, pu = U ? p + W : p;  // rows without a neighbour read their own
    for (int c = blockIdx.y; c < planes; c += gridDim.y) {
        const float* s = src + (int64_t)c * n;
        float* d = dst + (int64_t)c * n;
        if (x > 0 && x + 4 < W && D && U) {
            // four interior nodes: columns x - 1 .. x + 4 of row y, x - 1 .. x + 3 of
            // the row above, x .. x + 4 of the row below
            float r0[6], rd[5], ru[5];
            const gfloat4 m0 = *(const gfloat4*)(s + p), md = *(const gfloat4*)(s + pd), mu = *(const gfloat4*)(s + pu);
            r0[0] = s[p - 1];
            r0[5] = s[p + 4];
            rd[0] = s[pd - 1];
            ru[4] = s[pu + 4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                r0[1 + j] = m0[j];
                rd[1 + j] = md[j];
                ru[j] = mu[j];
            }
            gfloat4 o;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float ip2 = SIMPLEX ? r0[1 + j] : 2.f * r0[1 + j];
                float acc = (ip2 + rd[j] + rd[j + 1]) + (ip2 + rd[j] + r0[j]);
                acc += ip2 + rd[j + 1] + r0[j + 2];
                acc += ip2 + r0[j] + ru[j];
                acc += (ip2 + r0[j + 2] + ru[j + 1]) + (ip2 + ru[j] + ru[j + 1]);
                o[j] = acc / (float)((SIMPLEX ? 3 : 4) * 6);
            }
            *(gfloat4*)(d + p) = o;
            continue;
        }
        // a group at the boundary: columns x - 1 .. x + 4 of the three rows, those outside
        // the row its first or last (dropped below), all in flight before the first use
        // (512^2 in three planes: 22.7 us with the loads behind each node's conditions, 21.3 so)
        float r0[6], rd[6], ru[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const uint32_t o = (uint32_t)(min(max(x + j - 1, 0), W - 1) - x);
            r0[j] = s[p + o];
            rd[j] = s[pd + o];
            ru[j] = s[pu + o];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (x + j >= W) break;
            const bool L = x + j > 0, R = x + j < W - 1;
            const float ip2 = SIMPLEX ? r0[1 + j] : 2.f * r0[1 + j];
            float acc = 0.f;
            int nt = 0;
            if (L && D) {  // cell (x-1, y-1): both triangles have p as their (x+1, y+1) corner
                acc += (ip2 + rd[j] + rd[1 + j]) + (ip2 + rd[j] + r0[j]);
                nt += 2;
            }
            if (R && D) {  // cell (x, y-1): triangle (x, y-1), (x, y), (x+1, y)
                acc += ip2 + rd[1 + j] + r0[2 + j];
                nt += 1;
            }
            if (L && U) {  // cell (x-1, y): triangle (x-1, y), (x, y), (x, y+1)
                acc += ip2 + r0[j] + ru[1 + j];
                nt += 1;
            }
            if (R && U) {  // cell (x, y): both triangles have p as their (x, y) corner
                acc += (ip2 + r0[2 + j] + ru[2 + j]) + (ip2 + ru[1 + j] + ru[2 + j]);
                nt += 2;
            }
            d[p + j] = acc / (float)((SIMPLEX ? 3 : 4) * nt);
        }
    }
}

int row_blocks(int64_t rows) { return (int)std::max<int64_t>(1, std::min<int64_t>(rows, kRowBlocks)); }

}  // namespace

hipError_t launch_refine(int planes, int W, int H, int r, const float* src, float* dst, hipStream_t s) {
    const int Wf = ((W - 1) << r) + 1, Hf = ((H - 1) << r) + 1;
    hipLaunchKernelGGL(k_refine, dim3(row_blocks((int64_t)Hf * planes)), dim3(kBlock), 0, s, src, dst, W, H, r,
                       Wf, Hf, planes);
    return hipGetLastError();
}

hipError_t launch_sample(int planes, int W, int H, int r, const float* src, float* dst, hipStream_t s) {
    const int Wf = ((W - 1) << r) + 1, Hf = ((H - 1) << r) + 1;
    hipLaunchKernelGGL(k_sample, dim3(row_blocks((int64_t)H * planes)), dim3(kBlock), 0, s, src, dst, W, H, r,
                       Wf, Hf, planes);
    return hipGetLastError();
}

hipError_t launch_mass_avg(int planes, int W, int H, const float* src, float* dst, int simplex, hipStream_t s) {
    const int64_t groups = (int64_t)((W + 3) / 4) * H;
    const dim3 grid((unsigned)((groups + kBlock - 1) / kBlock), (unsigned)std::min(planes, 65535));
    if (simplex)
        hipLaunchKernelGGL(k_mass_avg<true>, grid, dim3(kBlock), 0, s, src, dst, W, H, planes);
    else
        hipLaunchKernelGGL(k_mass_avg<false>, grid, dim3(kBlock), 0, s, src, dst, W, H, planes);
    return hipGetLastError();
}

hipError_t launch_lab(int ab_only, int64_t count, const float* rgb, float* dst, hipStream_t s) {
    if (count == 0) return hipSuccess;
    const int blocks = (int)std::min<int64_t>((count + 2 * kBlock - 1) / (2 * kBlock), 8192);
    if (ab_only)
        hipLaunchKernelGGL(k_lab<true>, dim3(blocks), dim3(kBlock), 0, s, rgb, dst, count);
    else
        hipLaunchKernelGGL(k_lab<false>, dim3(blocks), dim3(kBlock), 0, s, rgb, dst, count);
    return hipGetLastError();
}

}  // namespace acseg
