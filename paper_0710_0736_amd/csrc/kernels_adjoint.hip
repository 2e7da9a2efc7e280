// kernels_adjoint.hip -- gradients of a segmentation through its time steps.
//
// The paper does not differentiate its scheme; this is the derivative of the
// discrete step map of eq. alpha.  With the free sets I_p = {i : u^{n+1}_pi > 0}
// held fixed, u^{n+1} minimises the step's quadratic over
// {u_pi = 0 outside I_p, sum_{I_p} u_pi = 1}, so for a loss gradient ubar at
// u^{n+1} the gradient at the right-hand side b is z = (T H T)^+ T ubar, T the
// node-wise tangent projection (zero outside I_p, minus the mean over I_p;
// zero when |I_p| <= 1).  z is found by red-black block Gauss-Seidel on
//     z_p = T_p (ubar_p / (h^2 D_p) + kappa_p sum_q c_pq z_q)
// (the nodal minimiser of z.H z / 2 - ubar.z on the range of T_p, in the
// scaled units of the smoother), over-relaxed: z_p <- z_p + omega (that - z_p),
// which stays in the range of T_p.  The system is symmetric positive definite
// and red-black ordered (two-cyclic), so the sweeps converge for 0 < omega < 2
// and Young's optimum is 2 / (1 + sqrt(1 - rho^2)) with rho the block-Jacobi
// radius.  The first kAdjOmegaSweep sweeps of a solve are plain Gauss-Seidel
// (omega = 1); their successive changes shrink by its contraction rho^2, whose
// estimate, the ratio of the last two changes, then fixes omega for the rest
// of the solve, capped by
// the value for the bound rho <= q = max_p kappa_p sum_q c_pq (the T_p only
// shrink the coupling).  An early estimate errs low (fast transients), which
// under-relaxes: still faster than Gauss-Seidel.  For a contraction by r per
// sweep, the distance to the solution after a sweep that changed z by dz is
// at most dz r / (1 - r); so the solve stops when dz <= rtol max|z| (1 - r),
// with r the larger of the ratio of the last two changes and omega - 1 (the
// contraction of over-relaxed sweeps cannot be smaller), at most 0.999, or
// when dz has fallen to a few units of float32 rounding of max|z|.  The
// chain rule then runs through
//     b_pi = M_p [(1/tau + 2/eps) un_pi - lambda F_pi],  F_pi = sum_k (I_pk - c_ik)^2,
//     c_ik = S_ik / S_i,  H = M/tau + eps A,
// with M_p = h^2 w_p; an empty phase's (kept) mean is a constant.
#include <algorithm>

#include "acseg_internal.h"
#include "tile.hpp"

namespace acseg {

namespace {

// Maxima of V values over a workgroup of T threads, with one barrier: every
// thread returns them in v.
template <int V, int T>
__device__ __forceinline__ void block_max_v(float (&v)[V]) {
    __shared__ float sh[T / kWave][V];
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
#pragma unroll
    for (int j = 0; j < V; ++j) v[j] = wave_max(v[j]);
    if (lane == 0)
#pragma unroll
        for (int j = 0; j < V; ++j) sh[wid][j] = v[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < V; ++j) {
        float r = sh[0][j];
        for (int w = 1; w < T / kWave; ++w) r = fmaxf(r, sh[w][j]);
        v[j] = r;
    }
}

// Two red-black sweeps of the adjoint solve per launch.  A workgroup stages 64 x 32
// nodes of z, the scaled loss gradient ubar_p / (h^2 D_p) and the free sets in
// registers, two columns and two rows per lane, and owns the 56 x 24 in their
// middle: every half-sweep loses one ring of exact values.  Column neighbours come
// by data-parallel moves, rows of adjacent groups through LDS, as in the smoothing
// launches of the forward pass.  The
// launch that starts at sweep s reads z from buffer (s / 2) & 1 (a.z, a.z2)
// and writes the other, so tiles never see each other's new values.  Each
// sweep leaves per-workgroup partials (max |dz| over the tile's black nodes,
// max |z|) in the set of its index mod 6, so a launch never overwrites a set
// it reads.  Every launch after the first evaluates the stopping rule on the
// partials of the sweeps before it and skips the rest of the solve once the
// rule holds.
// Bound by latency at 512^2 (220 workgroups: 4.8 us until the staged values and the
// stopping rule are there, 3 to 4 us for the half-sweeps): N = 4 takes 17.3 us with
// tiles of 64 x 8 nodes in LDS, 12.2 us in registers, 11.8 us with the tile's loads
// issued before the stopping rule.  1920 x 1080: 93 -> 67 us (N = 8: 157 -> 128), by
// the 1.5 instead of 2.3 staged values per owned one.
constexpr int kAdjK = 2;  // sweeps per launch
constexpr int kAdjT = 512, kAdjG = kAdjT / 32;  // threads; groups of 32 lanes
constexpr int kAdjR = 2 * kAdjK;
constexpr int kAdjTX = 64 - 2 * kAdjR, kAdjTY = 2 * kAdjG - 2 * kAdjR;
constexpr int kAdjSlots = 6;
constexpr int kAdjOmegaSweep = 6;  // the sweep that fixes omega from the Gauss-Seidel contraction
constexpr float kAdjUlps = 8.f;    // changes this close to float32 rounding of max|z| stop the solve
static_assert(kAdjOmegaSweep % kAdjK == 0, "omega is fixed at the start of a launch");
static_assert(kAdjSlots >= kAdjK + 3, "a launch writes kAdjK sets and reads the three before them");

__host__ __device__ inline int adj_tiles(int W, int H) {
    return ((W + kAdjTX - 1) / kAdjTX) * ((H + kAdjTY - 1) / kAdjTY);
}

// The stopping rule after `sweeps` sweeps, evaluated by a whole workgroup
// (every workgroup that evaluates it reads the same partials and reaches the
// same result).  For a sweep t >= 2: with dz_t the largest change of sweep
// t - 1 and r the contraction per sweep (the ratio of the last two changes;
// sweep 0 compared its black values with zero, so it gives none), never
// below omega - 1 of the sweep, at most 0.999, the rule holds at t when
// dz_t <= rtol max|z| (1 - r), or when dz_t is within kAdjUlps units in the
// last place of max|z|: there float32 rounding, not the contraction, sets
// the changes, and further sweeps do not bring z closer.  The solve stops
// after `sweeps` sweeps when the rule holds at `sweeps` or at `sweeps` - 1
// (the sweep in between only brings z closer).  `ratio` is the ratio at
// `sweeps`, for the choice of omega.
struct AdjRule {
    bool stop;
    float ratio;
};

template <int T = kBlock>
__device__ AdjRule adj_rule(const AdjArgs& a, int sweeps) {
    auto set = [&](int t) { return a.part_f + (((t % kAdjSlots) + kAdjSlots) % kAdjSlots) * 2 * kMgBlocks; };
    const float *p1 = set(sweeps - 1), *p2 = set(sweeps - 2), *p3 = set(sweeps - 3);
    float dz1 = 0.f, zm1 = 0.f, dz2 = 0.f, zm2 = 0.f, dz3 = 0.f;
    for (int b = threadIdx.x; b < a.nblocks; b += T) {
        dz1 = fmaxf(dz1, p1[b]);
        zm1 = fmaxf(zm1, p1[kMgBlocks + b]);
        dz2 = fmaxf(dz2, p2[b]);
        zm2 = fmaxf(zm2, p2[kMgBlocks + b]);
        dz3 = fmaxf(dz3, p3[b]);
    }
    float m[5] = {dz1, zm1, dz2, zm2, dz3};
    block_max_v<5, T>(m);
    dz1 = m[0];
    zm1 = m[1];
    dz2 = m[2];
    zm2 = m[3];
    dz3 = m[4];
    const float omega = a.actl->omega;
    auto holds = [&](int t, float dz, float zm, float dzp) {
        const float ratio = t > 2 ? (dzp > 0.f ? dz / dzp : 0.f) : 1.f;
        const float om = t - 1 >= kAdjOmegaSweep ? omega : 1.f;
        const float r = fminf(fmaxf(ratio, om - 1.f), 0.999f);
        return !(dz > fmaxf(a.rtol * (1.f - r), kAdjUlps * 0x1p-24f) * zm);
    };
    const float ratio = sweeps > 2 ? (dz2 > 0.f ? dz1 / dz2 : 0.f) : 1.f;
    const bool stop = holds(sweeps, dz1, zm1, dz2) || (sweeps - 1 >= 2 && holds(sweeps - 1, dz2, zm2, dz3));
    return {stop, ratio};
}

__device__ __forceinline__ float mass_wf(int cls) {
    return cls == 0 ? 1.f : (cls == 1 ? 0.5f : (cls == 2 ? (1.f / 3.f) : (1.f / 6.f)));
}

// The colour means' share of a step's gradient (c_ik = S_ik / S_i), applied
// one launch later: for the step whose cbar, means and sums a.cm_* point to,
// A_ik = cbar_ik / S_i (0 for an empty phase, whose kept mean is a constant)
// and B_i = sum_k A_ik c_ik; then dL/du^n_pi gains w_p (sum_k A_ik I_pk - B_i)
// and dL/dI_pk gains w_p sum_i A_ik u^n_pi.  Threads i < N fill A[N*C], B[N].
template <int N, int C>
__device__ void means_share(const AdjArgs& a, float* A, float* B) {
    if (threadIdx.x >= N) return;
    const int i = threadIdx.x;
    const double* tot = a.cm_tot;
    const double S = tot[N * C + i], area = tot[N * C + N + C];
    double b = 0.0;
    for (int k = 0; k < C; ++k) {
        const double Aik = S > 1e-12 * area ? a.cm_cbar[i * C + k] / S : 0.0;
        A[i * C + k] = (float)Aik;
        b += Aik * a.cm_c64[i * C + k];
    }
    B[i] = (float)b;
}

// The buffer that holds z after `sweeps` sweeps (a multiple of kAdjK).
__device__ __forceinline__ const float* adj_z_after(const AdjArgs& a, int sweeps) {
    return ((sweeps / kAdjK) & 1) ? a.z2 : a.z;
}

// One staged tile.
template <int N, int C>
struct AdjTile {
    float z[2][2][N], b[2][2][N];  // b: the loss gradient, scaled by adj_sweeps
    float u[2][2][N], I[2][2][C];
};

template <int N, int C, bool INT>
__device__ __forceinline__ void adj_load(AdjTile<N, C>& t, const AdjArgs& a, const float* zin, bool share, int gx,
                                         int gy) {
    const int W = a.W, H = a.H;
    const int64_t P = (int64_t)W * H;
    load_pairs<N, 2, INT>(t.b, a.ub, P, gx, gy, W, H);
    load_pairs<N, 2, INT>(t.u, a.u1, P, gx, gy, W, H);
    if (zin) {
        load_pairs<N, 2, INT>(t.z, zin, P, gx, gy, W, H);
    } else {
#pragma unroll
        for (int q = 0; q < 4 * N; ++q) t.z[q / (2 * N)][q / N % 2][q % N] = 0.f;
    }
    if (share) load_pairs<C, 2, INT>(t.I, a.image, P, gx, gy, W, H);
}

// The sweeps of one tile: dzm[j] / zmax[j] gain the largest change and value of the
// tile's black nodes in the launch's sweep j.  INT: every staged node is an interior node.
template <int N, int C, bool INT>
__device__ __forceinline__ void adj_sweeps(AdjTile<N, C>& t, const AdjArgs& a, int gx, int gy, float* zout, float omega,
                                           bool share, const float* cmA, const float* cmB, float* lds,
                                           float (&dzm)[kAdjK], float (&zmax)[kAdjK]) {
    constexpr int NPD = node_pad(N);
    const int W = a.W, H = a.H;
    const int64_t P = (int64_t)W * H;
    const int l = threadIdx.x & 31, g = threadIdx.x >> 5;
    const bool out = l >= kAdjR / 2 && l < 32 - kAdjR / 2 && g >= kAdjR / 2 && g < kAdjG - kAdjR / 2;
    float(&z)[2][2][N] = t.z;
    float(&b)[2][2][N] = t.b;
    int m[2][2][N];   // all ones where the phase is free and T_p not zero, else 0
    float nk[2][2], rk[2][2];  // the number of free phases and its reciprocal (0: T_p is zero)
    static_for<0, 4>([&](auto qc) __attribute__((always_inline)) {
        constexpr int r = decltype(qc)::value / 2, e = decltype(qc)::value % 2;
        const int x = gx + e, y = gy + r;
        const bool in = INT || (x >= 0 && x < W && y >= 0 && y < H);
        const int cls = INT ? 0 : node_class(x, y, W, H);
        const float rs = in ? sel4(a.coef.inv_d, cls) * a.inv_h2 : 0.f;
        const float wv = mass_wf(cls);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float v = b[r][e][i];
            if (share) {
                float m = -cmB[i];
#pragma unroll
                for (int c = 0; c < C; ++c) m = fmaf(cmA[i * C + c], t.I[r][e][c], m);
                v = fmaf(wv, m, v);
            }
            b[r][e][i] = v * rs;
        }
        float k = 0.f;
#pragma unroll
        for (int i = 0; i < N; ++i) k += t.u[r][e][i] > 0.f ? 1.f : 0.f;  // nodes outside the lattice read 0
#pragma unroll
        for (int i = 0; i < N; ++i) m[r][e][i] = k >= 2.f && t.u[r][e][i] > 0.f ? -1 : 0;
        nk[r][e] = k;
        rk[r][e] = k >= 2.f ? 1.f / k : 0.f;
    });
    // coupling and edge weights of the lane's nodes (0 outside the lattice)
    [[maybe_unused]] float kp[2][2], wh[2], wv[2];
    const float k0 = uniform_f(a.coef.kappa[0]);
    if constexpr (!INT) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            wh[q] = edge_w_h(gy + q, H);
            wv[q] = edge_w_v(gx + q, W);
        }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int x = gx + e, y = gy + r;
                const bool in = x >= 0 && x < W && y >= 0 && y < H;
                kp[r][e] = in ? sel4(a.coef.kappa, node_class(x, y, W, H)) : 0.f;
            }
    }
    // rows exchanged between groups, two buffers: slot g + 1 of `bot` is group g's
    // second row, slot g of `top` its first.  The outermost slots are filled once, below, with the
    // group's own rows: they only reach nodes of the dropped rings, but are read
    constexpr int kRow = 32 * NPD, kBuf = 2 * (kAdjG + 1) * kRow;
    float* const bot_w = lds + (g + 1) * kRow + l * NPD;
    float* const bot_r = lds + g * kRow + l * NPD;
    float* const top_w = lds + (kAdjG + 1 + g) * kRow + l * NPD;
    float* const top_r = lds + (kAdjG + 2 + g) * kRow + l * NPD;
    // as a black half-sweep leaves it
    lds_st<N>(top_w + kBuf, z[0][1]);
    lds_st<N>(bot_w + kBuf, z[1][0]);
    if (g == 0) {
        lds_st<N>(bot_r, z[0][0]);
        lds_st<N>(bot_r + kBuf, z[0][0]);
    }
    if (g == kAdjG - 1) {
        lds_st<N>(top_r, z[1][1]);
        lds_st<N>(top_r + kBuf, z[1][1]);
    }
    __syncthreads();
    static_for<0, 2 * kAdjK>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value, CB = k % 2, j = k / 2;
        float up[N], dn[N];
        lds_ld<N>(bot_r + (CB ^ 1) * kBuf, up);
        lds_ld<N>(top_r + (CB ^ 1) * kBuf, dn);
        static_for<0, 2>([&](auto rc) __attribute__((always_inline)) {
            constexpr int r = decltype(rc)::value, e = (r + CB) & 1;
            float v[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float side;
                if constexpr (e == 0)
                    side = dpp_move_f<0x138>(z[r][1][i]);  // wave_shr:1
                else
                    side = dpp_move_f<0x130>(z[r][0][i]);  // wave_shl:1
                const float hs = z[r][1 - e][i] + side;
                const float vs = z[1 - r][e][i] + (r == 0 ? up[i] : dn[i]);
                // the edge weights are powers of two: every tile rounds a node alike
                v[i] = INT ? fmaf(k0, hs + vs, b[r][e][i]) : fmaf(kp[r][e], fmaf(wh[r], hs, wv[e] * vs), b[r][e][i]);
            }
            // T_p
            auto masked = [&](int i, float w) __attribute__((always_inline)) {
                return __int_as_float(__float_as_int(w) & m[r][e][i]);
            };
            float sum = masked(0, v[0]);
#pragma unroll
            for (int i = 1; i < N; ++i) sum += masked(i, v[i]);
            // sum / nk as a division rounds it: the product and one correction
            float mean = sum * rk[r][e];
            mean = fmaf(fmaf(-nk[r][e], mean, sum), rk[r][e], mean);
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = masked(i, v[i] - mean);
            if (CB == 1 && out) {
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const float zo = z[r][e][i], zn = fmaf(omega, v[i] - zo, zo);
                    dzm[j] = fmaxf(dzm[j], fabsf(zn - zo));
                    zmax[j] = fmaxf(zmax[j], fabsf(zn));
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) z[r][e][i] = fmaf(omega, v[i] - z[r][e][i], z[r][e][i]);
        });
        if constexpr (k + 1 < 2 * kAdjK) {
            lds_st<N>(top_w + CB * kBuf, z[0][CB]);
            lds_st<N>(bot_w + CB * kBuf, z[1][1 - CB]);
            __syncthreads();
        }
    });
    if (out) store_pairs<N, 2, INT>(z, zout, P, gx, gy, W, H);
}

template <int N, int C>
__global__ __launch_bounds__(kAdjT, (N <= 2 ? 4 : 2)) void k_adj_sweep(AdjArgs a, int s0) {
    __shared__ __attribute__((aligned(16))) float lds[2 * 2 * (kAdjG + 1) * 32 * node_pad(N)];
    __shared__ float cmA[N * C], cmB[N];
    AdjCtl* ac = a.actl;
    // A solve that is long enough to have fixed omega may have ended well before its
    // budget: its launches look before they load (512^2 in pixel units, 269 of 700
    // launches at work: backward 6.2 -> 4.8 ms).  The first few load first.
    if (s0 > kAdjOmegaSweep && ac->done) return;
    const bool share = a.cm_cbar != nullptr;  // ubar = a.ub plus the later step's means share
    float omega = 1.f;                        // of both sweeps of the launch
    const int W = a.W, H = a.H;
    const float* zin = s0 > 0 ? adj_z_after(a, s0) : nullptr;
    float* zout = const_cast<float*>(adj_z_after(a, s0 + kAdjK));
    const int tiles_x = (W + kAdjTX - 1) / kAdjTX;
    const int ntiles = adj_tiles(W, H);
    float dzm[kAdjK], zmax[kAdjK];
#pragma unroll
    for (int j = 0; j < kAdjK; ++j) dzm[j] = zmax[j] = 0.f;
    // the workgroups of XCD x (id mod 8) take contiguous tiles
    const int first = (int)(blockIdx.x % kXcd * (gridDim.x / kXcd) + blockIdx.x / kXcd);
    int tile = first;
    do {
        const int x0 = (tile % tiles_x) * kAdjTX - kAdjR, y0 = (tile / tiles_x) * kAdjTY - kAdjR;
        const bool interior = x0 >= 1 && y0 >= 1 && x0 + 64 <= W - 1 && y0 + 2 * kAdjG <= H - 1;
        const int gx = x0 + 2 * (threadIdx.x & 31), gy = y0 + 2 * (threadIdx.x >> 5);
        AdjTile<N, C> t;
        if (interior)
            adj_load<N, C, true>(t, a, zin, share, gx, gy);
        else
            adj_load<N, C, false>(t, a, zin, share, gx, gy);  // reads clamped into the lattice, also without a tile
        if (tile == first) {
            if (s0 <= kAdjOmegaSweep && ac->done) return;
            if (share) means_share<N, C>(a, cmA, cmB);
            if (s0 >= 2) {
                const AdjRule rule = adj_rule<kAdjT>(a, s0);
                if (rule.stop) {
                    if (blockIdx.x == 0 && threadIdx.x == 0) {
                        ac->done = 1;
                        ac->sweeps = s0;
                    }
                    return;
                }
                if (s0 == kAdjOmegaSweep) {
                    // Gauss-Seidel so far: the ratio estimates rho^2
                    const float rho2 = fminf(rule.ratio, 0.99f);
                    omega = fminf(a.omega, fmaxf(1.f, 2.f / (1.f + sqrtf(1.f - rho2))));
                    if (blockIdx.x == 0 && threadIdx.x == 0) ac->omega = omega;  // read by later launches
                } else if (s0 > kAdjOmegaSweep) {
                    omega = ac->omega;
                }
            }
        }
        if (tile >= ntiles) break;
        __syncthreads();  // the means' share is in LDS; the previous tile's reads of the exchanged rows are done
        if (interior)
            adj_sweeps<N, C, true>(t, a, gx, gy, zout, omega, share, cmA, cmB, lds, dzm, zmax);
        else
            adj_sweeps<N, C, false>(t, a, gx, gy, zout, omega, share, cmA, cmB, lds, dzm, zmax);
        tile += gridDim.x;
    } while (tile < ntiles);
    float m[2 * kAdjK];
#pragma unroll
    for (int j = 0; j < kAdjK; ++j) {
        m[2 * j] = dzm[j];
        m[2 * j + 1] = zmax[j];
    }
    block_max_v<2 * kAdjK, kAdjT>(m);
    if (threadIdx.x == 0)
#pragma unroll
        for (int j = 0; j < kAdjK; ++j) {
            float* cur = a.part_f + ((s0 + j) % kAdjSlots) * 2 * kMgBlocks;
            cur[blockIdx.x] = m[2 * j];
            cur[kMgBlocks + blockIdx.x] = m[2 * j + 1];
        }
}

// One workgroup: the stopping rule after `sweeps` sweeps, for a caller that
// reads the convergence flag between chunks of sweep launches.
__global__ __launch_bounds__(kBlock) void k_adj_check(AdjArgs a, int sweeps) {
    AdjCtl* ac = a.actl;
    if (ac->done) return;
    if (adj_rule(a, sweeps).stop && threadIdx.x == 0) {
        ac->done = 1;
        ac->sweeps = sweeps;
    }
}

// The black half-sweep's change bounds the sweep's residual: the red values
// of the sweep were computed from the previous black ones, so with those
// reproduced to |dz| the red nodes are consistent to kappa-weighted |dz|.

// Direct terms of the chain rule at every node, in float32, summed in
// float64 into block partials of dL/dlambda, dL/deps, dL/dtau and cbar_ik;
// with the later step's means share of dL/dI (u^{n+1} is that step's u^n).
// The solve ended either where a sweep launch found the stopping rule met,
// or after the a.budget sweeps the caller enqueued: then every workgroup
// evaluates the rule there itself, and workgroup 0 records the outcome for
// the step's bookkeeping.  Partial q: 0 sum z M F, 1 sum z (-2/eps^2 M u^n -
// A u^{n+1}), 2 sum z M (u^{n+1} - u^n), 3 + iC + k sum 2 lambda M z (I - c);
// k_adj_reduce applies the signs and 1/tau^2.
// Two nodes per thread, every load that does not need the stopping rule before it: at
// 512^2, N = 4, 12.5 -> 10.7 us (33 MB); the rows above and below in an XCD's own L2
// make 1 us of that.  Registers hold three workgroups of 256 threads per CU at N = 4,
// hence at most 768 of them; four spill (23.7 us).  Above 12 sums two fit, and only N = 8, C = 4
// spills there (92 registers; 512^2, five steps back: 1357 us before the register tiles, 1077 now).
template <int N, int C>
__global__ __launch_bounds__(kBlock, (N * C <= 12 ? 3 : 2)) void k_adj_accum(AdjArgs a) {
    // both nodes of a pair round alike: only the multiply-adds that are written as such are fused
#pragma clang fp contract(off)
    constexpr int Q = 3 + N * C;
    constexpr int T = kBlock;
    __shared__ double sh[Q][T];
    __shared__ float cmA[N * C], cmB[N];
    const int W = a.W, H = a.H;
    const int64_t n = (int64_t)W * H;
    AdjCtl* ac = a.actl;
    const bool share = a.cm_cbar != nullptr;
    float c[N * C];
#pragma unroll
    for (int q = 0; q < N * C; ++q) c[q] = uniform_f((float)a.c64[q]);
    double acc[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q] = 0.0;
    const float h2 = (float)a.h2, ce = (float)(-2.0 / (a.eps * a.eps)), lam2 = (float)(2.0 * a.lambda);
    const float aa = (float)(1.0 / a.tau + 2.0 / a.eps);
    const float* zf = nullptr;
    const int wp = (W + 1) / 2, np = wp * H;  // pairs of nodes in x
    // the workgroups of XCD x (id mod 8) take the x-th eighth of the pairs, so the rows
    // above and below are in its L2
    const int per = ((np + T - 1) / T + kXcd - 1) / kXcd;  // runs of T pairs per XCD
    for (int q = blockIdx.x / kXcd; q < per; q += gridDim.x / kXcd) {
        const int64_t first = (int64_t)T * (blockIdx.x % kXcd * per + q);
        if (first >= np) break;
        const int t0 = (int)first;
        const bool in = t0 + (int)threadIdx.x < np;
        const int t = in ? t0 + (int)threadIdx.x : np - 1;
        const int y = t / wp, x = 2 * (t - y * wp);
        // every load of the pair before its first store (the stores could
        // alias later loads, which would then wait for them)
        float Ik[1][2][C], ib[1][2][C], zv[1][2][N], unv[1][2][N], u1v[1][2][N], up[1][2][N], dn[1][2][N], lf[N], rt[N];
        load_pairs<C, 1, false>(Ik, a.image, n, x, y, W, H);
        load_pairs<C, 1, false>(ib, a.Ibar, n, x, y, W, H);
        load_pairs<N, 1, false>(unv, a.u0, n, x, y, W, H);
        load_pairs<N, 1, false>(u1v, a.u1, n, x, y, W, H);
        load_pairs<N, 1, false>(up, a.u1, n, x, y - 1, W, H);
        load_pairs<N, 1, false>(dn, a.u1, n, x, y + 1, W, H);
        const uint32_t p = (uint32_t)(y * W + x);
        const uint32_t pl = x > 0 ? p - 1 : p, pr = x + 2 < W ? p + 2 : p;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            lf[i] = gload(a.u1 + i * n, pl);
            rt[i] = gload(a.u1 + i * n, pr);
        }
        if (!zf) {
            if (share) means_share<N, C>(a, cmA, cmB);  // read after the barrier below
            int sweeps = a.budget;
            bool conv = ac->done != 0;
            if (conv)
                sweeps = ac->sweeps;
            else if (sweeps >= 2)
                conv = adj_rule<T>(a, sweeps).stop;
            __syncthreads();
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                ac->fin_done = conv ? 1 : 0;
                ac->fin_sweeps = sweeps;
            }
            zf = adj_z_after(a, sweeps);
        }
        load_pairs<N, 1, false>(zv, zf, n, x, y, W, H);
        if (!in) continue;
        float ubo[1][2][N];
        static_for<0, 2>([&](auto ec) __attribute__((always_inline)) {
            constexpr int e = decltype(ec)::value;
            if (e == 1 && x + 1 >= W) return;
            const int cls = node_class(x + e, y, W, H);
            const float w = mass_wf(cls), Mp = h2 * w;
            const float ast = sel4(a.diagA, cls);
            const float wh = edge_w_h(y, H), wv = edge_w_v(x + e, W);
            float tq[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) tq[q] = 0.f;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float z = zv[0][e][i], un = unv[0][e][i], u1 = u1v[0][e][i];
                const float l = e == 0 ? (x > 0 ? lf[i] : 0.f) : u1v[0][0][i];
                const float r = e == 0 ? u1v[0][1][i] : (x + 2 < W ? rt[i] : 0.f);
                const float Au1 = fmaf(ast, u1, -fmaf(wh, l + r, wv * (up[0][e][i] + dn[0][e][i])));
                const float zM = z * Mp, lz = lam2 * zM;
                float F = 0.f;
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    const float d = Ik[0][e][k] - c[i * C + k];
                    F = fmaf(d, d, F);
                    tq[3 + i * C + k] = lz * d;
                    ib[0][e][k] = fmaf(-lz, d, ib[0][e][k]);
                    if (share) ib[0][e][k] = fmaf(w * cmA[i * C + k], u1, ib[0][e][k]);
                }
                ubo[0][e][i] = aa * zM;
                tq[0] = fmaf(zM, F, tq[0]);
                tq[1] = fmaf(z, fmaf(ce * Mp, un, -Au1), tq[1]);
                tq[2] = fmaf(zM, u1 - un, tq[2]);
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) acc[q] += (double)tq[q];
        });
        store_pairs<N, 1, false>(ubo, a.ub_out, n, x, y, W, H);
        store_pairs<C, 1, false>(ib, a.Ibar, n, x, y, W, H);
    }
    // The sums over the workgroup: transposed through LDS, 32 lanes per sum (each sum of
    // doubles over a wave costs 20 instructions: the launch at 512^2, N = 4, took 12.0 us
    // with 3 + N C of them, 10.8 us without).
#pragma unroll
    for (int q = 0; q < Q; ++q) sh[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int q = threadIdx.x >> 5; q < Q; q += T / 32) {
        const int seg = threadIdx.x & 31;
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < T / 32; ++w) v += sh[q][32 * w + seg];
        v = half_wave_sum_last(v);
        if (seg == 31) a.part_d[(int64_t)q * gridDim.x + blockIdx.x] = v;
    }
}

// One workgroup: the step's totals from k_adj_accum's partials, into grads
// (accumulated) and cbar of the step, plus the solve's bookkeeping.  What is updated is
// loaded before the partials.
template <int N, int C>
__global__ __launch_bounds__(kFinThreads) void k_adj_reduce(AdjArgs a) {
    constexpr int Q = 3 + N * C;
    __shared__ double tot[Q];
    AdjCtl* ac = a.actl;
    Ctl* ctl = a.ctl;
    const int q = (int)threadIdx.x - kWave;  // the second wave's lanes: cbar_q
    const float cb = q >= 0 && q < N * C && a.cbar_out && a.cbar_accumulate ? a.cbar_out[q] : 0.f;
    int sw = 0, fin_done = 0, short_steps = 0, c_total = 0, c_max = 0, unconv = 0, done = 0;
    double g0 = 0.0, g1 = 0.0, g2 = 0.0;
    if (threadIdx.x == 0) {
        sw = ac->fin_sweeps, fin_done = ac->fin_done, short_steps = ac->short_steps;
        c_total = ctl->cycles_total, c_max = ctl->cycles_max, unconv = ctl->steps_unconv, done = ctl->steps_done;
        g0 = a.grads[0], g1 = a.grads[1], g2 = a.grads[2];
    }
    reduce_cols<Q>(a.part_d, a.nblocks_acc, tot);
    if (q >= 0 && q < N * C) {
        a.cbar64[q] = tot[3 + q];
        if (a.cbar_out) a.cbar_out[q] = cb + (float)tot[3 + q];
    }
    if (threadIdx.x != 0) return;
    a.grads[0] = g0 - tot[0];
    a.grads[1] = g1 + tot[1];
    a.grads[2] = g2 + tot[2] / (a.tau * a.tau);
    ctl->cycles_total = c_total + sw;
    ctl->cycles_max = sw > c_max ? sw : c_max;
    if (!fin_done) {
        // a budget below the cap was the caller's guess, not the solve's limit
        if (a.budget < a.max_sweeps)
            ac->short_steps = short_steps + 1;
        else
            ctl->steps_unconv = unconv + 1;
    }
    ctl->steps_done = done + 1;
    ac->done = 0;
    ac->sweeps = 0;
}

// The means share of the first step (the one left after the last
// accumulation pass): grad_u0 = a.ub + that share (when a.ub_out is set) and
// dL/dI gains its part, with u^n = a.u0.
template <int N, int C>
__global__ __launch_bounds__(kBlock) void k_adj_final(AdjArgs a) {
    __shared__ float cmA[N * C], cmB[N];
    means_share<N, C>(a, cmA, cmB);
    __syncthreads();
    const int W = a.W, H = a.H;
    const int64_t n = (int64_t)W * H;
    for (int t = blockIdx.x * kBlock + threadIdx.x; t < (int)n; t += gridDim.x * kBlock) {
        const int y = t / W, x = t - y * W;
        const uint32_t p = (uint32_t)t;
        const float w = mass_wf(node_class(x, y, W, H));
        float Ik[C], ib[C], unv[N], ubv[N];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            Ik[k] = gload(a.image + k * n, p);
            ib[k] = gload(a.Ibar + k * n, p);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            unv[i] = gload(a.u0 + i * n, p);
            ubv[i] = a.ub_out ? gload(a.ub + i * n, p) : 0.f;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float du = -cmB[i];
#pragma unroll
            for (int k = 0; k < C; ++k) {
                du = fmaf(cmA[i * C + k], Ik[k], du);
                ib[k] = fmaf(w * cmA[i * C + k], unv[i], ib[k]);
            }
            if (a.ub_out) gstore(a.ub_out + i * n, p, fmaf(w, du, ubv[i]));
        }
#pragma unroll
        for (int k = 0; k < C; ++k) gstore(a.Ibar + k * n, p, ib[k]);
    }
}

__global__ void k_adj_init(AdjCtl* ac, double* grads) {
    if (threadIdx.x == 0) {
        AdjCtl c = {};
        *ac = c;
        grads[0] = grads[1] = grads[2] = 0.0;
    }
}

// Workgroups of a node-parallel pass, one node per thread of `threads`, at
// most `cap`.
int adj_blocks(int64_t n, int threads, int cap) {
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + threads - 1) / threads, cap));
}

template <int N, int C>
hipError_t adj_nc(int op, const AdjArgs& a, int sweep, hipStream_t s) {
    const int64_t n = (int64_t)a.W * a.H;
    switch (op) {
        case kAdjSweep:
            hipLaunchKernelGGL((k_adj_sweep<N, C>), dim3(a.nblocks), dim3(kAdjT), 0, s, a, sweep);
            break;
        case kAdjCheck: hipLaunchKernelGGL(k_adj_check, dim3(1), dim3(kBlock), 0, s, a, sweep); break;
        case kAdjAccum:
            hipLaunchKernelGGL((k_adj_accum<N, C>), dim3(a.nblocks_acc), dim3(kBlock), 0, s, a);
            break;
        case kAdjReduce: hipLaunchKernelGGL((k_adj_reduce<N, C>), dim3(1), dim3(kFinThreads), 0, s, a); break;
        case kAdjFinal:
            hipLaunchKernelGGL((k_adj_final<N, C>), dim3(adj_blocks(n, kBlock, kMgBlocks)), dim3(kBlock), 0, s, a);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int N>
hipError_t adj_n(int C, int op, const AdjArgs& a, int sweep, hipStream_t s) {
    switch (C) {
        case 1: return adj_nc<N, 1>(op, a, sweep, s);
        case 2: return adj_nc<N, 2>(op, a, sweep, s);
        case 3: return adj_nc<N, 3>(op, a, sweep, s);
        case 4: return adj_nc<N, 4>(op, a, sweep, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

// a multiple of the XCDs (every workgroup leaves its partials, also without a tile)
int adj_sweep_blocks(int W, int H) { return std::min((adj_tiles(W, H) + kXcd - 1) / kXcd * kXcd, kMgBlocks); }
int adj_accum_blocks(int N, int C, int W, int H) {
    return (adj_blocks((int64_t)((W + 1) / 2) * H, kBlock, kAdjAccBlocks) + kXcd - 1) / kXcd * kXcd;
}
int adj_sweeps_per_launch() { return kAdjK; }

hipError_t launch_adj(int N, int C, int op, const AdjArgs& a, int sweep, hipStream_t s) {
    switch (N) {
        case 2: return adj_n<2>(C, op, a, sweep, s);
        case 3: return adj_n<3>(C, op, a, sweep, s);
        case 4: return adj_n<4>(C, op, a, sweep, s);
        case 5: return adj_n<5>(C, op, a, sweep, s);
        case 6: return adj_n<6>(C, op, a, sweep, s);
        case 7: return adj_n<7>(C, op, a, sweep, s);
        case 8: return adj_n<8>(C, op, a, sweep, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_adj_init(AdjCtl* ac, double* grads, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_init, dim3(1), dim3(kWave), 0, s, ac, grads);
    return hipGetLastError();
}

}  // namespace acseg
