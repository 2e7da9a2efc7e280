// kernels_fine.hip -- finest-level kernels of the Allen-Cahn segmentation step.
//
//   k_project   simplex projection of independent vectors
//   k_cmeans    colour means c_ik (eq. VV_fidelity, lumped mass), float64 sums
//   k_labels    argmax labels, composite and rounded composite
//   k_energy    discrete energy of eq. E
#include <algorithm>

#include "acseg_internal.h"

namespace acseg {

// ---------------------------------------------------------------------------
// Projection of independent vectors (component-major [N][count])
// ---------------------------------------------------------------------------

template <int N>
__global__ __launch_bounds__(kBlock) void k_project(const float* y, float* x, int64_t count) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= count) return;
    float v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = y[i * count + t];
    project_simplex<N>(v);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i * count + t] = v[i];
}

// ---------------------------------------------------------------------------
// Colour means: S_ik = sum_p w_p u_pi I_pk, S_i = sum_p w_p u_pi,
// SI_k = sum_p w_p I_pk, Sw = sum_p w_p; c_ik = S_ik / S_i.
// ---------------------------------------------------------------------------

// Four consecutive nodes of a plane; the address needs 4-byte alignment only.
typedef float gfloat4 __attribute__((ext_vector_type(4), aligned(4)));
typedef __attribute__((address_space(1))) gfloat4 gfloat4_1;
__device__ __forceinline__ void load4(const float* base, uint32_t i, bool full, uint32_t n, float (&v)[4]) {
    if (full) {
        const gfloat4 t = *(const gfloat4_1*)((const gchar*)base + (i << 2));
        v[0] = t.x;
        v[1] = t.y;
        v[2] = t.z;
        v[3] = t.w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = i + j < n ? gload(base, i + j) : 0.f;
    }
}

// Walks a W x H lattice four consecutive nodes at a time, over nb workgroups:
// f(p, x, y, full, inner) with (x, y) the first node's coordinates (the others may
// lie on the next rows), full: all four exist, inner: all four are interior nodes.
// One division per thread; the coordinates then advance by the stride's.
template <class F>
__device__ __forceinline__ void walk4(int W, int H, int nb, F&& f) {
    const uint32_t n = (uint32_t)W * H;
    const uint32_t step = 4u * nb * kBlock;
    uint32_t p = 4u * (blockIdx.x * kBlock + threadIdx.x);
    const int sy = (int)(step / (uint32_t)W), sx = (int)(step - (uint32_t)sy * W);
    int y = (int)(p / (uint32_t)W), x = (int)(p - (uint32_t)y * W);
#pragma unroll 2
    for (; p < n; p += step) {
        f(p, x, y, p + 3 < n, x > 0 && x + 4 < W && y > 0 && y < H - 1);
        x += sx;
        y += sy;
        if (x >= W) {
            x -= W;
            ++y;
        }
    }
}

struct CmeansArgs {
    const float* image;
    const float* u;  // explicit field, or NULL: bufs.b[ctl->cur]
    Bufs bufs;
    const Ctl* ctl;
    double* partials;  // [gridDim.y][cmeans_width(N, C)][gridDim.x]
    int W, H;
    int64_t u_stride;  // floats from one explicit field to the next (grid row y: u + y u_stride)
};

// The partial sums of one workgroup's nodes, into part[m][nb] at column blockIdx.x.
// Bound by memory: 4 (N + C) B per node are read once.  Four nodes per thread
// and access, and no division per node: 1920 x 1080 RGB at N = 4 (58 MB) took 29 us
// with one node per access and its coordinates by 64-bit division, 17 us now (3.4
// TB/s); 8 images of 1024^2 in one launch 61 us (3.8 TB/s).
template <int N, int C>
__device__ __forceinline__ void cmeans_sums(const float* image, const float* u, int W, int H, double* part, int nb) {
    constexpr int M = N * C + N + C + 2;  // S_ik, S_i, SI_k, Sw, non-finite count
    __shared__ double sh[kBlock / kWave][M];
    const uint32_t n = (uint32_t)W * H;
    double acc[M];
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m] = 0.0;
    walk4(W, H, nb, [&](uint32_t p, int x, int y, bool full, bool inner) __attribute__((always_inline)) {
        float I[C][4], v[N][4];
#pragma unroll
        for (int k = 0; k < C; ++k) load4(image + (int64_t)k * n, p, full, n, I[k]);
#pragma unroll
        for (int i = 0; i < N; ++i) load4(u + (int64_t)i * n, p, full, n, v[i]);
        double w[4];
        bool bad = false;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w[j] = 1.0;
            if (!inner) {
                int xj = x + j, yj = y;
                while (xj >= W) {
                    xj -= W;
                    ++yj;
                }
                w[j] = p + j < n ? mass_w(node_class(xj, yj, W, H)) : 0.0;
            }
#pragma unroll
            for (int k = 0; k < C; ++k) bad |= !isfinite(I[k][j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double Id[C];
#pragma unroll
            for (int k = 0; k < C; ++k) {
                Id[k] = (double)I[k][j];
                acc[N * C + N + k] = fma(w[j], Id[k], acc[N * C + N + k]);
            }
            acc[N * C + N + C] += w[j];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const double wu = w[j] * (double)v[i][j];
                acc[N * C + i] += wu;
#pragma unroll
                for (int k = 0; k < C; ++k) acc[i * C + k] = fma(wu, Id[k], acc[i * C + k]);
            }
        }
        acc[M - 1] += bad ? 1.0 : 0.0;
    });
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const double v = wave_sum(acc[m]);
        if (lane == 0) sh[wid][m] = v;
    }
    __syncthreads();
    if (threadIdx.x < M) {
        double s = 0.0;
        for (int w = 0; w < kBlock / kWave; ++w) s += sh[w][threadIdx.x];
        part[(int64_t)threadIdx.x * nb + blockIdx.x] = s;
    }
}

template <int N, int C>
__global__ __launch_bounds__(kBlock) void k_cmeans(CmeansArgs a) {
    constexpr int M = N * C + N + C + 2;
    const float* u = a.u ? a.u + blockIdx.y * a.u_stride : a.bufs.b[__builtin_amdgcn_readfirstlane(a.ctl->cur)];
    cmeans_sums<N, C>(a.image, u, a.W, a.H, a.partials + (int64_t)blockIdx.y * gridDim.x * M, gridDim.x);
}

struct CmeansFinArgs {
    const double* partials;
    int nb;
    Ctl* ctl;
    const double* c_prev64;
    double* c64;
    float* c_out;
    double* tot_out;  // reduced sums, or NULL
    int init;         // >= 0: the control block is set up here, with this current buffer
};

// Colour means from the reduced sums tot (LDS), lane i C + k of the first wave(s)
// finishing c_ik; ctl's flags.
template <int N, int C>
__device__ __forceinline__ void means_of(const double* tot, const double* c_prev64, Ctl* ctl, double* c64,
                                         float* c_out, int init = -1) {
    constexpr int M = N * C + N + C + 2;
    const double area = tot[N * C + N + C];
    if (threadIdx.x < N * C) {
        const int i = threadIdx.x / C, k = threadIdx.x - i * C;
        const double S = tot[N * C + i];
        const double c = S > 1e-12 * area ? tot[threadIdx.x] / S
                                          : (c_prev64 ? c_prev64[threadIdx.x] : tot[N * C + N + k] / area);
        if (c64) c64[threadIdx.x] = c;
        if (c_out) c_out[threadIdx.x] = (float)c;
    }
    if (threadIdx.x == 0) {
        int empty = 0;
        for (int i = 0; i < N; ++i) empty |= tot[N * C + i] > 1e-12 * area ? 0 : 1;
        const int bad = tot[M - 1] > 0.0 ? 1 : 0;
        if (init >= 0) {
            Ctl c = {};
            c.cur = init;
            c.empty_now = empty;
            c.nonfinite = bad;
            *ctl = c;
        } else {
            ctl->empty_now = empty;
            if (bad) ctl->nonfinite = 1;
        }
    }
}

// One block: finish the colour means from k_cmeans' partials.
template <int N, int C>
__global__ __launch_bounds__(kFinThreads) void k_cmeans_finish(CmeansFinArgs a) {
    constexpr int M = N * C + N + C + 2;
    __shared__ double tot[M];
    reduce_cols<M>(a.partials, a.nb, tot);
    if (a.tot_out && threadIdx.x < M) a.tot_out[threadIdx.x] = tot[threadIdx.x];
    means_of<N, C>(tot, a.c_prev64, a.ctl, a.c64, a.c_out, a.init);
}

// One workgroup per field of a k_cmeans launch over several fields: its
// reduced sums into tot[y][kCmeansMaxM].
template <int N, int C>
__global__ __launch_bounds__(kFinThreads) void k_cmeans_tot(const double* partials, int nb, double* tot) {
    constexpr int M = N * C + N + C + 2;
    __shared__ double t[M];
    reduce_cols<M>(partials + (int64_t)blockIdx.x * nb * M, nb, t);
    if (threadIdx.x < M) tot[(int64_t)blockIdx.x * kCmeansMaxM + threadIdx.x] = t[threadIdx.x];
}

// One thread: the means of fields first..first+count-1 from their reduced
// sums, in order, an empty phase keeping the previous field's mean (the first
// field's previous means: c64 of field first - 1, or the mean image colour
// when first is 0).
// (The sums and means pass through LDS: the one thread that walks the
// fields then waits on no memory.)  count <= kCmeansFields.
template <int N, int C>
__global__ __launch_bounds__(kBlock) void k_cmeans_chain(const double* tot, int first, int count, Ctl* ctl,
                                                         double* c64) {
    constexpr int M = N * C + N + C + 2;
    __shared__ double ts[kCmeansFields][M];
    __shared__ double cs[kCmeansFields + 1][N * C];
    for (int q = threadIdx.x; q < count * M; q += kBlock) {
        const int f = q / M, m = q - f * M;
        ts[f][m] = tot[(int64_t)(first + f) * kCmeansMaxM + m];
    }
    if (first > 0 && threadIdx.x < N * C) cs[0][threadIdx.x] = c64[(int64_t)(first - 1) * kNC + threadIdx.x];
    __syncthreads();
    // thread i C + k follows c_ik through the fields (a phase's chain does
    // not depend on the other phases)
    if (threadIdx.x < N * C) {
        const int i = threadIdx.x / C, k = threadIdx.x - i * C;
        for (int f = 0; f < count; ++f) {
            const double* t = ts[f];
            const double area = t[N * C + N + C], S = t[N * C + i];
            cs[f + 1][threadIdx.x] = S > 1e-12 * area
                                         ? t[i * C + k] / S
                                         : ((first + f) > 0 ? cs[f][threadIdx.x] : t[N * C + N + k] / area);
        }
    }
    if (threadIdx.x == 0) {
        const double* t = ts[count - 1];
        int empty = 0, bad = 0;
        for (int i = 0; i < N; ++i) empty |= t[N * C + i] > 1e-12 * t[N * C + N + C] ? 0 : 1;
        for (int f = 0; f < count; ++f) bad |= ts[f][M - 1] > 0.0 ? 1 : 0;
        ctl->empty_now = empty;
        if (bad) ctl->nonfinite = 1;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < count * N * C; q += kBlock) {
        const int f = q / (N * C), m = q - f * (N * C);
        c64[(int64_t)(first + f) * kNC + m] = cs[f + 1][m];
    }
}

// ---------------------------------------------------------------------------
// The same passes over the images of one (N, C) of a batch: grid row y is image
// imgs[y].  Every image takes the workgroups and the order it takes alone.
// (Three launches per image before and two after the time loop were 420 us of a
// batch of 8 images of 1024^2; one each per group are 71 us.)
// ---------------------------------------------------------------------------

template <int N, int C>
__global__ __launch_bounds__(kBlock) void k_cmeans_batch(const BatchImage* __restrict__ d,
                                                         const int* __restrict__ imgs) {
    const BatchImage& b = d[imgs[blockIdx.y]];
    if ((int)blockIdx.x >= b.nb) return;
    cmeans_sums<N, C>(b.image, b.bufs.b[0], b.W, b.H, b.part, b.nb);
}

template <int N, int C>
__global__ __launch_bounds__(kFinThreads) void k_cmeans_finish_batch(const BatchImage* __restrict__ d,
                                                                     const int* __restrict__ imgs, BatchMeans out,
                                                                     int steps, int fixed_c) {
    constexpr int M = N * C + N + C + 2;
    __shared__ double tot[M];
    const BatchImage& b = d[imgs[blockIdx.x]];
    reduce_cols<M>(b.part, b.nb, tot);
    if (threadIdx.x < M) b.tot[threadIdx.x] = tot[threadIdx.x];
    float* c_out = out.c[blockIdx.x];
    if (fixed_c && threadIdx.x < N * C) b.c64[2 * kNC + threadIdx.x] = (double)c_out[threadIdx.x];
    means_of<N, C>(tot, nullptr, b.ctl, b.c64 + kNC, steps == 0 && !fixed_c ? c_out : nullptr, 0);
}

// After the time loop: the field into the caller's buffer, and the means of the result.
template <int N, int C>
__global__ __launch_bounds__(kBlock) void k_batch_results(const BatchImage* __restrict__ d,
                                                          const int* __restrict__ imgs, BatchMeans out, int steps,
                                                          int fixed_c) {
    const BatchImage& b = d[imgs[blockIdx.y]];
    const int cur = __builtin_amdgcn_readfirstlane(b.ctl->cur);
    if (cur != 0 && b.bufs.b[cur] != b.bufs.b[0]) {
        const float* src = b.bufs.b[cur];
        float* dst = const_cast<float*>(b.bufs.b[0]);
        const int64_t count = (int64_t)N * b.W * b.H;
        for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < count; t += (int64_t)gridDim.x * kBlock)
            dst[t] = src[t];
    }
    float* c_out = out.c[blockIdx.y];
    if (blockIdx.x == 0 && c_out && steps > 0 && !fixed_c) {
        const int a = steps & 1;
        means_of<N, C>(b.tot + a * kCmeansMaxM, b.c64 + (a ^ 1) * kNC, b.ctl, nullptr, c_out);
    }
}

// ---------------------------------------------------------------------------
// Control-block helpers
// ---------------------------------------------------------------------------

__global__ void k_ctl_init(Ctl* ctl, int cur) {
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        Ctl c = {};
        c.cur = cur;
        *ctl = c;
    }
}

__global__ __launch_bounds__(kBlock) void k_copy_current(Bufs bufs, const Ctl* ctl, float* dst,
                                                         int64_t count, int steps) {
    if (steps >= 0 && ctl->steps_done != steps) return;
    const float* src = bufs.b[__builtin_amdgcn_readfirstlane(ctl->cur)];
    if (src == dst) return;
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < count;
         t += (int64_t)gridDim.x * kBlock)
        dst[t] = src[t];
}

__global__ void k_widen(const float* src, double* dst, int count) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < count) dst[t] = (double)src[t];
}

__global__ __launch_bounds__(kBlock) void k_fill(float* p, int64_t count, float v) {
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < count;
         t += (int64_t)gridDim.x * kBlock)
        p[t] = v;
}

// ---------------------------------------------------------------------------
// Post-processing
// ---------------------------------------------------------------------------

template <int N, int C>
__global__ __launch_bounds__(kBlock) void k_labels(const float* u, const float* c, uint8_t* labels,
                                                   float* composite, float* rounded, int64_t n) {
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= n) return;
    float v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = u[i * n + p];
    int best = 0;
#pragma unroll
    for (int i = 1; i < N; ++i)
        if (v[i] > v[best]) best = i;
    if (labels) labels[p] = (uint8_t)best;
#pragma unroll
    for (int k = 0; k < C; ++k) {
        if (composite) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < N; ++i) s += c[i * C + k] * v[i];
            composite[k * n + p] = s;
        }
        if (rounded) rounded[k * n + p] = c[best * C + k];
    }
}

// ---------------------------------------------------------------------------
// Energy of eq. E: interface eps/2 sum_edges c_e (u_p - u_q)^2, concave
// (h^2/eps) sum w u (1 - u), fitting lambda h^2 sum w u F(c).
// ---------------------------------------------------------------------------

struct EnergyArgs {
    const float* image;
    const float* u;
    const double* c64;
    double* partials;  // [3][gridDim.x]
    int W, H;
};

// Four nodes per thread and access, as k_cmeans; the lower neighbours come from a
// second read of the next row (cache).  1920 x 1080, N = 4: 34 -> 28 us.
// (N = 8, C = 4 needs the bound: free of it the compiler takes 257 registers, which leaves
// one wave per SIMD: 4096^2 927 us with one node per access, 1020 so, 705 with two waves.)
template <int N, int C>
__global__ __launch_bounds__(kBlock, (N * C >= 32 ? 2 : 1)) void k_energy(EnergyArgs a) {
    __shared__ double cs[N * C];
    __shared__ double sh[kBlock / kWave][3];
    if (threadIdx.x < N * C) cs[threadIdx.x] = a.c64[threadIdx.x];
    __syncthreads();
    const int W = a.W, H = a.H;
    const uint32_t n = (uint32_t)W * H;
    double e0 = 0.0, e1 = 0.0, e2 = 0.0;
    walk4(W, H, gridDim.x, [&](uint32_t p, int x, int y, bool full, bool inner) __attribute__((always_inline)) {
        float I[C][4];
#pragma unroll
        for (int k = 0; k < C; ++k) load4(a.image + (int64_t)k * n, p, full, n, I[k]);
        double w[4], ch[4], cv[4];  // mass, edge to the right, edge below (0: none)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            w[j] = ch[j] = cv[j] = 1.0;
            if (!inner) {
                int xj = x + j, yj = y;
                while (xj >= W) {
                    xj -= W;
                    ++yj;
                }
                const bool in = p + j < n;
                w[j] = in ? mass_w(node_class(xj, yj, W, H)) : 0.0;
                ch[j] = in && xj + 1 < W ? ((yj == 0 || yj == H - 1) ? 0.5 : 1.0) : 0.0;
                cv[j] = in && yj + 1 < H ? ((xj == 0 || xj == W - 1) ? 0.5 : 1.0) : 0.0;
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float* ui = a.u + (int64_t)i * n;
            float v[5], d[4];
            float v4[4];
            load4(ui, p, full, n, v4);
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = v4[j];
            v[4] = p + 4 < n ? gload(ui, p + 4) : 0.f;
            load4(ui, p + (uint32_t)W, p + W + 3 < n, n, d);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double uj = (double)v[j];
                // (selected, not weighted by 0: an infinite value has no edge past the lattice)
                const double dh = ch[j] != 0.0 ? uj - (double)v[j + 1] : 0.0;
                const double dv = cv[j] != 0.0 ? uj - (double)d[j] : 0.0;
                e0 = fma(ch[j] * dh, dh, e0);
                e0 = fma(cv[j] * dv, dv, e0);
                const double wu = w[j] * uj;
                e1 = fma(wu, 1.0 - uj, e1);
                double F = 0.0;
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    const double t = (double)I[k][j] - cs[i * C + k];
                    F = fma(t, t, F);
                }
                e2 = fma(wu, F, e2);
            }
        }
    });
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    e0 = wave_sum(e0);
    e1 = wave_sum(e1);
    e2 = wave_sum(e2);
    if (lane == 0) {
        sh[wid][0] = e0;
        sh[wid][1] = e1;
        sh[wid][2] = e2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double s = 0.0;
        for (int w = 0; w < kBlock / kWave; ++w) s += sh[w][threadIdx.x];
        a.partials[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = s;
    }
}

// One block: energy parts from k_energy's partials.
__global__ __launch_bounds__(kFinThreads) void k_energy_finish(const double* partials, int nb,
                                                          double eps, double lambda, double h,
                                                          double* energy) {
    __shared__ double tot[3];
    reduce_cols<3>(partials, nb, tot);
    if (threadIdx.x == 0) {
        const double h2 = h * h;
        energy[0] = 0.5 * eps * tot[0];
        energy[1] = h2 / eps * tot[1];
        energy[2] = lambda * h2 * tot[2];
        energy[3] = energy[0] + energy[1] + energy[2];
    }
}

// ---------------------------------------------------------------------------
// Launchers: runtime N, C -> template instances
// ---------------------------------------------------------------------------

static int grid_for(int64_t n, int max_blocks) {
    int64_t b = (n + kBlock * 4 - 1) / (kBlock * 4);
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return (int)b;
}

// Runtime N (2..8) and C (1..4) to template instances.
template <template <int, int> class F, class... A>
static hipError_t dispatch_nc(int N, int C, A&&... args) {
#define ACSEG_NC(n)                                          \
    case n:                                                  \
        switch (C) {                                         \
            case 1: return F<n, 1>::run(args...);            \
            case 2: return F<n, 2>::run(args...);            \
            case 3: return F<n, 3>::run(args...);            \
            case 4: return F<n, 4>::run(args...);            \
            default: return hipErrorInvalidValue;            \
        }
    switch (N) {
        ACSEG_NC(2) ACSEG_NC(3) ACSEG_NC(4) ACSEG_NC(5) ACSEG_NC(6) ACSEG_NC(7) ACSEG_NC(8)
        default: return hipErrorInvalidValue;
    }
#undef ACSEG_NC
}

template <template <int> class F, class... A>
static hipError_t dispatch_n(int N, A&&... args) {
    switch (N) {
        case 2: return F<2>::run(args...);
        case 3: return F<3>::run(args...);
        case 4: return F<4>::run(args...);
        case 5: return F<5>::run(args...);
        case 6: return F<6>::run(args...);
        case 7: return F<7>::run(args...);
        case 8: return F<8>::run(args...);
        default: return hipErrorInvalidValue;
    }
}

template <int N>
struct ProjectRun {
    static hipError_t run(int64_t count, const float* y, float* x, hipStream_t s) {
        const unsigned blocks = (unsigned)((count + kBlock - 1) / kBlock);
        hipLaunchKernelGGL(k_project<N>, dim3(blocks), dim3(kBlock), 0, s, y, x, count);
        return hipGetLastError();
    }
};

hipError_t launch_project(int N, int64_t count, const float* y, float* x, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    return dispatch_n<ProjectRun>(N, count, y, x, s);
}

int cmeans_width(int N, int C) { return N * C + N + C + 2; }

// Workgroups of a pass that sums over the lattice: eight nodes per thread until
// kCmeansBlocks of them (each ends with a reduction of its M sums).
int cmeans_blocks(int W, int H) {
    const int64_t b = ((int64_t)W * H + kBlock * 8 - 1) / (kBlock * 8);
    return (int)(b > kCmeansBlocks ? kCmeansBlocks : b);
}

template <int N, int C>
struct CmeansRun {
    static hipError_t run(const CmeansArgs& a, int blocks, hipStream_t s) {
        hipLaunchKernelGGL((k_cmeans<N, C>), dim3(blocks), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
};

hipError_t launch_cmeans(int N, int C, int W, int H, const float* image, const float* u,
                         Bufs bufs, const Ctl* ctl, double* partials, hipStream_t s) {
    const CmeansArgs a{image, u, bufs, ctl, partials, W, H, 0};
    return dispatch_nc<CmeansRun>(N, C, a, cmeans_blocks(W, H), s);
}

template <int N, int C>
struct CmeansFieldsRun {
    static hipError_t run(const CmeansArgs& a, int first, int count, double* tot, double* c64, Ctl* ctl,
                          hipStream_t s) {
        const int nb = cmeans_blocks(a.W, a.H);
        hipLaunchKernelGGL((k_cmeans<N, C>), dim3(nb, count), dim3(kBlock), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_cmeans_tot<N, C>), dim3(count), dim3(kFinThreads), 0, s, a.partials, nb,
                           tot + (int64_t)first * kCmeansMaxM);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_cmeans_chain<N, C>), dim3(1), dim3(kBlock), 0, s, tot, first, count, ctl, c64);
        return hipGetLastError();
    }
};

hipError_t launch_cmeans_fields(int N, int C, int W, int H, const float* image, const float* fields,
                                int first, int count, double* partials, double* tot, double* c64, Ctl* ctl,
                                hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (count > kCmeansFields) return hipErrorInvalidValue;
    const int64_t stride = (int64_t)N * W * H;
    const CmeansArgs a{image, fields + first * stride, Bufs{}, ctl, partials, W, H, stride};
    return dispatch_nc<CmeansFieldsRun>(N, C, a, first, count, tot, c64, ctl, s);
}

template <int N, int C>
struct CmeansFinishRun {
    static hipError_t run(const CmeansFinArgs& a, hipStream_t s) {
        hipLaunchKernelGGL((k_cmeans_finish<N, C>), dim3(1), dim3(kFinThreads), 0, s, a);
        return hipGetLastError();
    }
};

hipError_t launch_cmeans_finish(int N, int C, int W, int H, const double* partials, Ctl* ctl,
                                const double* c_prev64, double* c64, float* c_out, double* tot, int init,
                                hipStream_t s) {
    const CmeansFinArgs a{partials, cmeans_blocks(W, H), ctl, c_prev64, c64, c_out, tot, init};
    return dispatch_nc<CmeansFinishRun>(N, C, a, s);
}

// One block: colour means from already reduced sums.
template <int N, int C>
__global__ void k_means_from_tot(const double* tot, const double* c_prev64, Ctl* ctl, double* c64,
                                 float* c_out) {
    means_of<N, C>(tot, c_prev64, ctl, c64, c_out);
}

template <int N, int C>
struct MeansFromTotRun {
    static hipError_t run(const double* tot, const double* c_prev64, Ctl* ctl, double* c64,
                          float* c_out, hipStream_t s) {
        hipLaunchKernelGGL((k_means_from_tot<N, C>), dim3(1), dim3(64), 0, s, tot, c_prev64, ctl, c64,
                           c_out);
        return hipGetLastError();
    }
};

hipError_t launch_means_from_tot(int N, int C, const double* tot, const double* c_prev64,
                                 Ctl* ctl, double* c64, float* c_out, hipStream_t s) {
    return dispatch_nc<MeansFromTotRun>(N, C, tot, c_prev64, ctl, c64, c_out, s);
}

template <int N, int C>
struct BatchMeansRun {
    static hipError_t run(const BatchImage* d, const int* imgs, int nimg, const BatchMeans& out, int blocks,
                          int steps, int fixed_c, hipStream_t s) {
        hipLaunchKernelGGL((k_cmeans_batch<N, C>), dim3(blocks, nimg), dim3(kBlock), 0, s, d, imgs);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_cmeans_finish_batch<N, C>), dim3(nimg), dim3(kFinThreads), 0, s, d, imgs, out, steps,
                           fixed_c);
        return hipGetLastError();
    }
};

hipError_t launch_batch_means(int N, int C, const BatchImage* d, const int* imgs, int nimg, const BatchMeans& out,
                              int blocks, int steps, int fixed_c, hipStream_t s) {
    if (nimg < 1 || nimg > kBatchMeans) return hipErrorInvalidValue;
    return dispatch_nc<BatchMeansRun>(N, C, d, imgs, nimg, out, blocks, steps, fixed_c, s);
}

template <int N, int C>
struct BatchResultsRun {
    static hipError_t run(const BatchImage* d, const int* imgs, int nimg, const BatchMeans& out, int blocks,
                          int steps, int fixed_c, hipStream_t s) {
        hipLaunchKernelGGL((k_batch_results<N, C>), dim3(blocks, nimg), dim3(kBlock), 0, s, d, imgs, out, steps,
                           fixed_c);
        return hipGetLastError();
    }
};

// As many workgroups per image as a copy of the largest field takes alone, at least 128
// and 4096 over the images: with 128 always, one image of 4096^2, N = 8, whose steps took
// an odd number of launches (the field is then copied) took 2460 us for one step, 970 alone.
hipError_t launch_batch_results(int N, int C, const BatchImage* d, const int* imgs, int nimg, const BatchMeans& out,
                                int64_t most, int steps, int fixed_c, hipStream_t s) {
    if (nimg < 1 || nimg > kBatchMeans) return hipErrorInvalidValue;
    const int blocks = grid_for(most, std::max(128, 4096 / nimg));
    return dispatch_nc<BatchResultsRun>(N, C, d, imgs, nimg, out, blocks, steps, fixed_c, s);
}

hipError_t launch_ctl_init(Ctl* ctl, int cur, hipStream_t s) {
    hipLaunchKernelGGL(k_ctl_init, dim3(1), dim3(64), 0, s, ctl, cur);
    return hipGetLastError();
}

hipError_t launch_copy_current(Bufs bufs, const Ctl* ctl, float* dst, int64_t count, int steps,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_copy_current, dim3(grid_for(count, 4096)), dim3(kBlock), 0, s, bufs, ctl,
                       dst, count, steps);
    return hipGetLastError();
}

hipError_t launch_widen(const float* src, double* dst, int count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_widen, dim3((count + 63) / 64), dim3(64), 0, s, src, dst, count);
    return hipGetLastError();
}

hipError_t launch_fill(float* p, int64_t count, float v, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(count, 4096)), dim3(kBlock), 0, s, p, count, v);
    return hipGetLastError();
}

template <int N, int C>
struct LabelsRun {
    static hipError_t run(const float* u, const float* c, uint8_t* l, float* comp, float* rnd,
                          int64_t n, hipStream_t s) {
        const unsigned blocks = (unsigned)((n + kBlock - 1) / kBlock);
        hipLaunchKernelGGL((k_labels<N, C>), dim3(blocks), dim3(kBlock), 0, s, u, c, l, comp, rnd, n);
        return hipGetLastError();
    }
};

hipError_t launch_labels(int N, int C, int W, int H, const float* u, const float* c,
                         uint8_t* labels, float* composite, float* rounded, hipStream_t s) {
    return dispatch_nc<LabelsRun>(N, C, u, c, labels, composite, rounded, (int64_t)W * H, s);
}

template <int N, int C>
struct EnergyRun {
    static hipError_t run(const EnergyArgs& a, int blocks, hipStream_t s) {
        hipLaunchKernelGGL((k_energy<N, C>), dim3(blocks), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
};

hipError_t launch_energy(int N, int C, int W, int H, const float* image, const float* u,
                         const double* c64, double eps, double lambda, double h,
                         double* partials, double* energy, hipStream_t s) {
    const EnergyArgs a{image, u, c64, partials, W, H};
    const int blocks = cmeans_blocks(W, H);
    hipError_t e = dispatch_nc<EnergyRun>(N, C, a, blocks, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_energy_finish, dim3(1), dim3(kFinThreads), 0, s, partials, blocks, eps, lambda,
                       h, energy);
    return hipGetLastError();
}

}  // namespace acseg
