// Generic FLuRKA attention path: every contraction is a strided, batched GEMM
// with fp32 arithmetic, joined by small row-wise kernels.  It serves the fp32
// storage type, shapes the MFMA kernels do not cover, and acts as an on-device
// cross-check for them.  Math per (batch, head), following Eq. 2 with the
// App. D row normaliser:
//   K' = E K, V' = F V;  PhiK = phi(K') (shifted);  S = PhiK^T V';  z = PhiK^T 1
//   P = phi(Q) (shifted per row);  out = (P S) / (P z)
#include "flurka_gemm_f32.h"

namespace flurka {

#define FLURKA_CHECK_LAUNCH()                                   \
    do {                                                        \
        if (hipGetLastError() != hipSuccess) return FLURKA_ERR_LAUNCH; \
    } while (0)

// ---------------------------------------------------------------------------
// GEMM launches (flurka_gemm_f32.h)
// ---------------------------------------------------------------------------
// C (and C2), contiguous, from the split partials; 4 consecutive elements per thread
__global__ __launch_bounds__(256) void gemm_f32_sum_kernel(void* C, void* C2, const float* part, int splits, long count, int c_bf16) {
    const long i = 4 * ((long)blockIdx.x * 256 + threadIdx.x);
    if (i >= count) return;
    const long plane = count * (C2 ? 2 : 1);
    const float* p = part + (blockIdx.y ? count : 0) + i;
    void* const c = blockIdx.y ? C2 : C;
    if (i + 4 <= count) {
        float s[4] = {0.f, 0.f, 0.f, 0.f};
        for_parts<8, float4>(
            splits, [&](int u) { float4 x; __builtin_memcpy(&x, p + u * plane, 16); return x; },
            [&](const float4& x) { s[0] += x.x; s[1] += x.y; s[2] += x.z; s[3] += x.w; });
        if (c_bf16) {
            const uint2 v = {pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3])};
            __builtin_memcpy((uint16_t*)c + i, &v, 8);
        } else {
            __builtin_memcpy((float*)c + i, s, 16);
        }
        return;
    }
    for (int e = 0; i + e < count; ++e) {
        float s = 0.f;
        for (int u = 0; u < splits; ++u) s += p[u * plane + e];
        store_elem(c, i + e, s, c_bf16);
    }
}

template <bool AKF, bool BKF, int TA, int TB, int TM, int TN>
static flurka_status launch_gemm_tile(const GemmArgs& g, int splits, hipStream_t s) {
    const long tiles = (long)((g.N + TN - 1) / TN) * ((g.M + TM - 1) / TM);
    const auto kern = gemm_f32_kernel<AKF, BKF, TA, TB, TM, TN>;
    constexpr int ldsb = GemmF32Lds<AKF, BKF, TA, TB, TM, TN>::bytes;
    KernelFacts facts;
    if (!kernel_facts((const void*)kern, 256, ldsb, &facts)) return FLURKA_ERR_LAUNCH;      // raises the LDS limit
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles, (unsigned)splits, (unsigned)(g.batches * (g.C2 ? 2 : 1))), dim3(256), ldsb, s, g);
    FLURKA_CHECK_LAUNCH();
    return FLURKA_OK;
}

template <bool AKF, bool BKF, int TA, int TB>
static flurka_status launch_gemm_layout(GemmArgs g, float* part, size_t part_floats, hipStream_t s) {
    // Larger tiles halve the operand traffic per product; smaller ones give more workgroups.  A tile edge of
    // 128 is taken where the result, with its reduction split as far as that goes, still has a workgroup
    // for every compute unit.
    const long cus = chip_cus();
    const long batches = (long)g.batches * (g.C2 ? 2 : 1);
    const int steps = (g.K + F_GK - 1) / F_GK;
    auto tiles = [&](int tm, int tn) { return (long)((g.M + tm - 1) / tm) * ((g.N + tn - 1) / tn) * batches; };
    auto max_splits = [&]() -> long {           // ranges of at least two steps, as many as the scratch holds
        if (!part) return 1;
        long q = steps / 2 < 32 ? steps / 2 : 32;
        const long room = (long)(part_floats / ((size_t)g.c_count * (g.C2 ? 2 : 1)));
        if (q > room) q = room;
        return q < 1 ? 1 : q;
    };
    const long most = max_splits();
    const int tm = g.M > 64 && tiles(128, 64) * most >= cus ? 128 : 64;
    const int tn = tm == 128 && g.N > 64 && tiles(128, 128) * most >= cus ? 128 : 64;
    // two workgroups per compute unit where splitting allows it
    long splits = (2 * cus + tiles(tm, tn) - 1) / tiles(tm, tn);
    if (tiles(tm, tn) >= 2 * cus || splits < 1) splits = 1;
    if (splits > most) splits = most;
    g.steps_per_split = (int)((steps + splits - 1) / splits);
    splits = (steps + g.steps_per_split - 1) / g.steps_per_split;
    g.part = splits > 1 ? part : nullptr;
    flurka_status st = tm == 64 ? launch_gemm_tile<AKF, BKF, TA, TB, 64, 64>(g, (int)splits, s)
                       : tn == 64 ? launch_gemm_tile<AKF, BKF, TA, TB, 128, 64>(g, (int)splits, s)
                                  : launch_gemm_tile<AKF, BKF, TA, TB, 128, 128>(g, (int)splits, s);
    if (st != FLURKA_OK || splits == 1) return st;
    hipLaunchKernelGGL(gemm_f32_sum_kernel, dim3((unsigned)((g.c_count + 1023) / 1024), g.C2 ? 2u : 1u), dim3(256), 0, s, g.C,
                       g.C2, (const float*)g.part, (int)splits, g.c_count, g.c_bf16);
    FLURKA_CHECK_LAUNCH();
    return FLURKA_OK;
}

flurka_status launch_gemm_f32(GemmArgs g, int batches, float* part, size_t part_floats, hipStream_t s) {
    g.batches = batches;
    g.c_count = (long)batches * g.M * g.N;
    if (g.C2 && 2L * batches > 65535) {        // more batches than a grid dimension takes: one GEMM at a time
        GemmArgs g2 = g;
        g2.A = g.A2; g2.B = g.B2; g2.C = g.C2;
        g.A2 = g.B2 = nullptr; g.C2 = nullptr;
        g2.A2 = g2.B2 = nullptr; g2.C2 = nullptr;
        const flurka_status st = launch_gemm_f32(g, batches, part, part_floats, s);
        return st != FLURKA_OK ? st : launch_gemm_f32(g2, batches, part, part_floats, s);
    }
    // the layouts and storage types the path has: an fp32 x bf16 product has its bf16 operand on the right
    // except where E stands on the left (transposed, in dK = E^T dK')
    const bool akf = g.sAki == 1, bkf = g.sBki == 1;
    if (akf && bkf)
        return g.a_bf16 ? launch_gemm_layout<true, true, 1, 1>(g, part, part_floats, s)
               : g.b_bf16 ? launch_gemm_layout<true, true, 3, 1>(g, part, part_floats, s)
                          : launch_gemm_layout<true, true, 3, 3>(g, part, part_floats, s);
    if (akf)
        return g.a_bf16 ? launch_gemm_layout<true, false, 1, 1>(g, part, part_floats, s)
               : g.b_bf16 ? launch_gemm_layout<true, false, 3, 1>(g, part, part_floats, s)
                          : launch_gemm_layout<true, false, 3, 3>(g, part, part_floats, s);
    return g.a_bf16 ? launch_gemm_layout<false, false, 1, 3>(g, part, part_floats, s)
           : g.b_bf16 ? launch_gemm_layout<false, false, 3, 1>(g, part, part_floats, s)
                      : launch_gemm_layout<false, false, 3, 3>(g, part, part_floats, s);
}

static flurka_status launch_gemm(const GemmArgs& g, int batches, hipStream_t s) { return launch_gemm_f32(g, batches, nullptr, 0, s); }

// ---------------------------------------------------------------------------
// Row-wise kernels.  One 64-lane wavefront per row, four rows per block.
// ---------------------------------------------------------------------------
// e_rj <- e_rj - |k'_r|^2 / 2.   rows = BH*k rows of length m in e, of length d in Kp.
__global__ __launch_bounds__(256) void key_exponent_kernel(float* e, const float* Kp, long rows, int d, int m) {
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const float* kr = Kp + row * d;
    float sq = 0.f;
    for (int t = lane; t < d; t += 64) sq = fmaf(kr[t], kr[t], sq);
    sq = 0.5f * wave_sum(sq);
    float* er = e + row * m;
    for (int j = lane; j < m; j += 64) er[j] -= sq;
}

// c[bh, j] = max_r e[bh, r, j]: one exponent shift per feature (any positive rescaling of a
// feature's column of phi(K') is undone by the same factor on that feature of phi(Q))
__global__ void column_max_kernel(float* c, const float* e, int k, int m, long total) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const long bh = idx / m;
    const int j = (int)(idx % m);
    const float* p = e + bh * (long)k * m + j;
    float mx = -INFINITY;
    for (int r = 0; r < k; ++r) mx = fmaxf(mx, p[(long)r * m]);
    c[idx] = mx;
}

// PhiK <- exp(e - c_j)
__global__ __launch_bounds__(256) void key_exp_kernel(float* e, const float* c, long rows, int k, int m) {
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const float* cc = c + (row / k) * m;
    float* er = e + row * m;
    for (int j = lane; j < m; j += 64) er[j] = expf(er[j] - cc[j]);
}

__global__ void fill_f32_kernel(float* p, float v, long count) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = v;
}

__device__ __forceinline__ float elu1(float x) { return x > 0.f ? x + 1.f : expf(x); }
__device__ __forceinline__ float elu1_grad(float x) { return x > 0.f ? 1.f : expf(x); }

// dst[bh, i, :] = elu(src[bh, row0 + i, :]) + 1 for i < nr.
__global__ void elu1_rows_kernel(float* dst, const void* src, int src_bf16, long total,
                                 int nr, int d, long src_rows_per_bh, int row0) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int t = (int)(idx % d);
    const long r = idx / d;
    const long bh = r / nr, i = r % nr;
    dst[idx] = elu1(load_elem(src, (bh * src_rows_per_bh + row0 + i) * d + t, src_bf16));
}

// z[bh, j] = sum_r PhiK[bh, r, j]
__global__ void column_sum_kernel(float* z, const float* Phi, int k, int m, long total) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const long bh = idx / m;
    const int j = (int)(idx % m);
    const float* p = Phi + bh * (long)k * m + j;
    float s = 0.f;
    for (int r = 0; r < k; ++r) s += p[(long)r * m];
    z[idx] = s;
}

// P[row, :] <- exp(v - max_j v), v_j = U[row, j] + c[bh, j]   (rows = BH*nr).  With `rowmax` (the
// lse segment, forward only) the maximum of row (bh, row0 + i) is left there for fwd_finish_kernel.
__global__ __launch_bounds__(256) void row_exp_kernel(float* U, const float* c, long rows, int nr, int m,
                                                      float* rowmax, int n, int row0) {
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    float* u = U + row * m;
    const float* cc = c + (row / nr) * m;
    float mx = -INFINITY;
    for (int j = lane; j < m; j += 64) mx = fmaxf(mx, u[j] + cc[j]);
    mx = wave_max(mx);
    for (int j = lane; j < m; j += 64) u[j] = expf(u[j] + cc[j] - mx);
    if (rowmax && lane == 0) rowmax[(row / nr) * n + row0 + row % nr] = mx;
}

// D = P.z ; out = N / D  (rows = BH*nr; output row = bh*n + row0 + i); lse = row maximum + ln D
// (`has_max`: row_exp_kernel left the maximum in lse; otherwise it is 0)
__global__ __launch_bounds__(256) void fwd_finish_kernel(const float* P, const float* N, const float* z,
                                                         void* out, int out_bf16, long rows, int nr,
                                                         int n, int row0, int mf, int d, float* lse,
                                                         int has_max) {
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const long bh = row / nr, i = row % nr;
    const float* p = P + row * mf;
    const float* zz = z + bh * mf;
    float D = 0.f;
    for (int j = lane; j < mf; j += 64) D = fmaf(p[j], zz[j], D);
    D = wave_sum(D);
    const float* nrow = N + row * d;
    const long o = (bh * n + row0 + i) * d;
    for (int t = lane; t < d; t += 64) store_elem(out, o + t, nrow[t] / D, out_bf16);
    if (lane == 0) {
        float* l = lse + bh * n + row0 + i;
        *l = (has_max ? *l : 0.f) + logf(D);
    }
}

// Backward row preparation:  D = P.z, out = N/D, dD = -(G.out)/D, N <- dN = G/D.
__global__ __launch_bounds__(256) void bwd_row_prep_kernel(const float* P, float* N, const float* z,
                                                           const void* G, int g_bf16, float* dD,
                                                           long rows, int nr, int n, int row0, int mf, int d) {
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const long bh = row / nr, i = row % nr;
    const float* p = P + row * mf;
    const float* zz = z + bh * mf;
    float D = 0.f;
    for (int j = lane; j < mf; j += 64) D = fmaf(p[j], zz[j], D);
    D = wave_sum(D);
    const float inv = 1.f / D;
    float* nrow = N + row * d;
    const long go = (bh * n + row0 + i) * d;
    float dot = 0.f;
    for (int t = lane; t < d; t += 64) {
        const float g = load_elem(G, go + t, g_bf16);
        dot = fmaf(g, nrow[t] * inv, dot);
        nrow[t] = g * inv;
    }
    dot = wave_sum(dot);
    if (lane == 0) dD[row] = -dot * inv;
}

// T <- dP (*) P with dP = T + dD_i z_j   (performer: dU of the query side)
__global__ void bwd_du_kernel(float* T, const float* P, const float* dD, const float* z,
                              long total, int nr, int mf) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const long row = idx / mf;
    const int j = (int)(idx % mf);
    const long bh = row / nr;
    T[idx] = (T[idx] + dD[row] * z[bh * mf + j]) * P[idx];
}

// elu1: dQ = (T + dD_i z_j) * phi'(Q)
__global__ void bwd_dq_elu_kernel(const float* T, const float* dD, const float* z, const void* Q,
                                  void* dQ, int bf16, long total, int nr, int n, int row0, int d) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const long row = idx / d;
    const int t = (int)(idx % d);
    const long bh = row / nr, i = row % nr;
    const long qi = (bh * n + row0 + i) * d + t;
    const float dP = T[idx] + dD[row] * z[bh * d + t];
    store_elem(dQ, qi, dP * elu1_grad(load_elem(Q, qi, bf16)), bf16);
}

// Key side, performer: dPhiK += dz_j; dUk = dPhiK * PhiK (in place); rs_r = sum_j dUk_rj
__global__ __launch_bounds__(256) void bwd_key_du_kernel(float* dPhi, const float* Phi, const float* dz,
                                                         float* rs, long rows, int k, int m) {
    const int lane = threadIdx.x & 63;
    const long row = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const long bh = row / k;
    float* dp = dPhi + row * m;
    const float* ph = Phi + row * m;
    const float* dzz = dz + bh * m;
    float s = 0.f;
    for (int j = lane; j < m; j += 64) {
        const float v = (dp[j] + dzz[j]) * ph[j];
        dp[j] = v;
        s += v;
    }
    s = wave_sum(s);
    if (lane == 0) rs[row] = s;
}

// dK'_r -= rs_r K'_r
__global__ void bwd_key_norm_kernel(float* dKp, const float* Kp, const float* rs, long total, int d) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    dKp[idx] -= rs[idx / d] * Kp[idx];
}

// elu1 key side: dK' = (dPhiK + dz_j) * phi'(K')
__global__ void bwd_key_elu_kernel(float* dKp, const float* dPhi, const float* dz, const float* Kp,
                                   long total, int k, int d) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const long bh = idx / ((long)k * d);
    const int t = (int)(idx % d);
    dKp[idx] = (dPhi[idx] + dz[bh * d + t]) * elu1_grad(Kp[idx]);
}

static inline dim3 grid1d(long total, int block) { return dim3((unsigned)((total + block - 1) / block)); }

// ---------------------------------------------------------------------------
// Pieces shared by forward and backward
// ---------------------------------------------------------------------------
// P (B,H,nr,mf) <- shifted phi(Q[row0 : row0+nr]);  N (B,H,nr,d) <- P S
static flurka_status query_features_and_numerator(const Problem& p, const void* Q, const void* omega,
                                                  const float* S, const float* c, float* P, float* N,
                                                  int row0, int nr, float* rowmax, hipStream_t s) {
    const long rows = (long)p.BH * nr;
    if (!p.elu) {
        GemmArgs g{};
        g.A = (const char*)Q + (size_t)row0 * p.d * (p.bf16 ? 2 : 4);
        g.B = omega; g.C = P;
        g.M = nr; g.N = p.m; g.K = p.d; g.Kin = p.d;
        g.sAm = p.d; g.sAki = 1; g.sAb = (long)p.H * p.n * p.d; g.sAh = (long)p.n * p.d;
        g.sBn = p.d; g.sBki = 1; g.sBb = 0; g.sBh = p.omega_per_head ? (long)p.m * p.d : 0;
        g.sCm = p.m; g.sCn = 1; g.sCb = (long)p.H * nr * p.m; g.sCh = (long)nr * p.m;
        g.H = p.H; g.a_bf16 = p.bf16; g.b_bf16 = p.bf16;
        flurka_status st = launch_gemm(g, p.BH, s);
        if (st != FLURKA_OK) return st;
        hipLaunchKernelGGL(row_exp_kernel, grid1d(rows, 4), dim3(256), 0, s, P, c, rows, nr, p.m, rowmax, p.n, row0);
        FLURKA_CHECK_LAUNCH();
    } else {
        const long total = rows * p.d;
        hipLaunchKernelGGL(elu1_rows_kernel, grid1d(total, 256), dim3(256), 0, s, P, Q, p.bf16, total,
                           nr, p.d, (long)p.n, row0);
        FLURKA_CHECK_LAUNCH();
    }
    GemmArgs g{};
    g.A = P; g.B = S; g.C = N;
    g.M = nr; g.N = p.d; g.K = p.mf; g.Kin = p.mf;
    g.sAm = p.mf; g.sAki = 1; g.sAb = (long)p.H * nr * p.mf; g.sAh = (long)nr * p.mf;
    g.sBn = 1; g.sBki = p.d; g.sBb = (long)p.H * p.mf * p.d; g.sBh = (long)p.mf * p.d;
    g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * nr * p.d; g.sCh = (long)nr * p.d;
    g.H = p.H;
    return launch_gemm(g, p.BH, s);
}

// K' = E K, V' = F V: (B,H,k,d) <- (k,n) (B,H,n,d).  `part`: scratch for a split reduction.
static flurka_status project(const Problem& p, const FwdArgs& a, float* Kp, float* Vp, float* part, size_t part_floats,
                             hipStream_t s) {
    GemmArgs g{};
    g.A = a.E; g.B = a.K; g.C = Kp;
    g.A2 = a.F; g.B2 = a.V; g.C2 = Vp;
    g.M = p.k; g.N = p.d; g.K = p.n; g.Kin = p.n;
    g.sAm = p.n; g.sAki = 1; g.sAb = 0; g.sAh = p.ef_per_head ? (long)p.k * p.n : 0;
    g.sBn = 1; g.sBki = p.d; g.sBb = (long)p.H * p.n * p.d; g.sBh = (long)p.n * p.d;
    g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * p.k * p.d; g.sCh = (long)p.k * p.d;
    g.H = p.H; g.a_bf16 = p.bf16; g.b_bf16 = p.bf16;
    if (p.ef_per_head) return launch_gemm_f32(g, p.BH, part, part_floats, s);
    // E, F shared: all heads side by side as one row of columns (head, t)
    g.N = p.BH * p.d; g.Nin = p.d; g.sBno = (long)p.n * p.d; g.sCno = (long)p.k * p.d;
    return launch_gemm_f32(g, 1, part, part_floats, s);
}

// PhiK (k x mf, shifted) from K' in ctx.  With `new_shift` the per-feature shifts c are computed
// and stored; otherwise the stored ones are reused (backward: same PhiK as the forward had).
static flurka_status key_features(const Problem& p, const void* omega, const float* Kp, float* c,
                                  float* Phi, int new_shift, hipStream_t s) {
    const long krows = (long)p.BH * p.k;
    if (!p.elu) {
        GemmArgs g{};
        g.A = Kp; g.B = omega; g.C = Phi;
        g.M = p.k; g.N = p.m; g.K = p.d; g.Kin = p.d;
        g.sAm = p.d; g.sAki = 1; g.sAb = (long)p.H * p.k * p.d; g.sAh = (long)p.k * p.d;
        g.sBn = p.d; g.sBki = 1; g.sBb = 0; g.sBh = p.omega_per_head ? (long)p.m * p.d : 0;
        g.sCm = p.m; g.sCn = 1; g.sCb = (long)p.H * p.k * p.m; g.sCh = (long)p.k * p.m;
        g.H = p.H; g.b_bf16 = p.bf16;
        flurka_status st = launch_gemm(g, p.BH, s);
        if (st != FLURKA_OK) return st;
        hipLaunchKernelGGL(key_exponent_kernel, grid1d(krows, 4), dim3(256), 0, s, Phi, Kp, krows, p.d, p.m);
        FLURKA_CHECK_LAUNCH();
        if (new_shift) {
            const long ct = (long)p.BH * p.m;
            hipLaunchKernelGGL(column_max_kernel, grid1d(ct, 256), dim3(256), 0, s, c, (const float*)Phi, p.k,
                               p.m, ct);
            FLURKA_CHECK_LAUNCH();
        }
        hipLaunchKernelGGL(key_exp_kernel, grid1d(krows, 4), dim3(256), 0, s, Phi, (const float*)c, krows,
                           p.k, p.m);
        FLURKA_CHECK_LAUNCH();
    } else {
        const long total = krows * p.d;
        hipLaunchKernelGGL(elu1_rows_kernel, grid1d(total, 256), dim3(256), 0, s, Phi, (const void*)Kp, 0,
                           total, p.k, p.d, (long)p.k, 0);
        FLURKA_CHECK_LAUNCH();
        if (new_shift) {
            const long ct = (long)p.BH * p.d;
            hipLaunchKernelGGL(fill_f32_kernel, grid1d(ct, 256), dim3(256), 0, s, c, 0.f, ct);
            FLURKA_CHECK_LAUNCH();
        }
    }
    return FLURKA_OK;
}

// PhiK, S, z, c from K', V' (in ctx)
static flurka_status generic_key_state(const Problem& p, const void* omega, float* ctx, float* Phi, hipStream_t s) {
    const CtxLayout L = ctx_layout(p);
    float* Vp = ctx + L.Vp;
    float* S = ctx + L.S;
    float* z = ctx + L.z;
    flurka_status st = key_features(p, omega, ctx + L.Kp, ctx + L.c, Phi, 1, s);
    if (st != FLURKA_OK) return st;
    // S = PhiK^T V'
    GemmArgs g{};
    g.A = Phi; g.B = Vp; g.C = S;
    g.M = p.mf; g.N = p.d; g.K = p.k; g.Kin = p.k;
    g.sAm = 1; g.sAki = p.mf; g.sAb = (long)p.H * p.k * p.mf; g.sAh = (long)p.k * p.mf;
    g.sBn = 1; g.sBki = p.d; g.sBb = (long)p.H * p.k * p.d; g.sBh = (long)p.k * p.d;
    g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * p.mf * p.d; g.sCh = (long)p.mf * p.d;
    g.H = p.H;
    st = launch_gemm(g, p.BH, s);
    if (st != FLURKA_OK) return st;
    const long zt = (long)p.BH * p.mf;
    hipLaunchKernelGGL(column_sum_kernel, grid1d(zt, 256), dim3(256), 0, s, z, (const float*)Phi, p.k, p.mf, zt);
    FLURKA_CHECK_LAUNCH();
    return FLURKA_OK;
}

// ---------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------
flurka_status generic_forward(const Problem& p, const FwdArgs& a, hipStream_t s) {
    const CtxLayout L = ctx_layout(p);
    const GenericWs W = generic_ws_layout(p, 0);
    flurka_status st;
    {
        StageScope sc(s, STAGE_PROJECT);
        // nothing of the workspace is in use yet: all of it may hold split partials
        if ((st = project(p, a, a.ctx + L.Kp, a.ctx + L.Vp, a.ws, generic_ws_floats(p, 0), s)) != FLURKA_OK) return st;
    }
    {
        StageScope sc(s, STAGE_KEY_STATE);
        st = f32_fused_supported(p) ? f32_key_state(p, a.omega, a.ctx, s)
                                    : generic_key_state(p, a.omega, a.ctx, a.ws + W.PhiK, s);
        if (st != FLURKA_OK) return st;
    }
    if (f32_fused_supported(p)) {
        StageScope sc(s, STAGE_QUERY);
        return f32_query_forward(p, a, s);
    }
    const int nc = generic_chunk_rows(p);
    float* P = a.ws + W.P;
    float* N = a.ws + W.N;
    StageScope sc(s, STAGE_QUERY);
    for (int row0 = 0; row0 < p.n; row0 += nc) {
        const int nr = (p.n - row0 < nc) ? (p.n - row0) : nc;
        st = query_features_and_numerator(p, a.Q, a.omega, a.ctx + L.S, a.ctx + L.c, P, N, row0, nr, a.ctx + L.lse, s);
        if (st != FLURKA_OK) return st;
        const long rows = (long)p.BH * nr;
        hipLaunchKernelGGL(fwd_finish_kernel, grid1d(rows, 4), dim3(256), 0, s, P, N, a.ctx + L.z, a.out,
                           p.bf16, rows, nr, p.n, row0, p.mf, p.d, a.ctx + L.lse, p.elu ? 0 : 1);
        FLURKA_CHECK_LAUNCH();
    }
    return FLURKA_OK;
}

// ---------------------------------------------------------------------------
// Backward (chain rule of the forward; notation as in the forward)
//   dN = G/D, dD = -(G.out)/D, dP = dN S^T + dD z^T, dS = P^T dN, dz = P^T dD
//   dPhiK = V' dS^T + 1 dz^T, dV' = PhiK dS
//   performer: dU = dphi*phi, dx = dU omega - rowsum(dU) x  (the rowsum term is
//              identically zero on the query side: out is invariant to a
//              rescaling of a row of P);  elu1: dx = dphi * phi'(x)
//   dK = E^T dK', dV = F^T dV', dE = sum_bh dK' K^T, dF = sum_bh dV' V^T
// ---------------------------------------------------------------------------
// The four sequence-length GEMMs from dK', dV' (fp32)
// `part`: scratch for split partials of dE, dF
static flurka_status grad_gemms_f32(const Problem& p, const BwdArgs& a, const float* dKp, const float* dVp, float* part,
                                    size_t part_floats, hipStream_t s);

// head sizes up to 128: the query and key side on the fused kernels (flurka_f32.hip)
static flurka_status fused_backward(const Problem& p, const BwdArgs& a, hipStream_t s) {
    const F32BwdWs W = f32_bwd_ws_layout(p);
    flurka_status st;
    {
        StageScope sc(s, STAGE_BWD_QUERY);
        if ((st = f32_query_backward(p, a, s)) != FLURKA_OK) return st;
    }
    {
        StageScope sc(s, STAGE_BWD_KEY);
        if ((st = f32_key_backward(p, a, s)) != FLURKA_OK) return st;
    }
    // what lies in front of dK', dV' is done with
    // (two fp32 operands: the fp32 matrix rate bounds the GEMM, splitting it only adds the sum: 67 us against 63)
    return grad_gemms_f32(p, a, a.ws + W.dKp, a.ws + W.dVp, a.ws, p.bf16 ? W.dKp : 0, s);
}

size_t generic_ws_floats(const Problem& p, int bwd) {
    const size_t unfused = generic_ws_layout(p, bwd).total;
    if (!f32_fused_supported(p)) return unfused;
    if (bwd) return f32_bwd_ws_layout(p).total;
    // split partials of the projection: fewer than 512 tiles of 128 x 128 are split, into at most 1024 in all
    const size_t partials = (size_t)1024 * 128 * 128;
    return unfused < partials ? unfused : partials;
}

flurka_status generic_backward(const Problem& p, const BwdArgs& a, hipStream_t s) {
    if (f32_fused_supported(p)) return fused_backward(p, a, s);
    const CtxLayout L = ctx_layout(p);
    const GenericWs W = generic_ws_layout(p, 1);
    const float* Kp = a.ctx + L.Kp;
    const float* Vp = a.ctx + L.Vp;
    float* Phi = a.ws + W.PhiK;
    const float* S = a.ctx + L.S;
    const float* cshift = a.ctx + L.c;
    const float* z = a.ctx + L.z;
    float* P = a.ws + W.P;
    float* T = a.ws + W.T;
    float* N = a.ws + W.N;
    float* dD = a.ws + W.dD;
    float* dS = a.ws + W.dS;
    float* dz = a.ws + W.dz;
    float* dPhi = a.ws + W.dPhiK;
    float* dKp = a.ws + W.dKp;
    float* dVp = a.ws + W.dVp;
    float* rs = a.ws + W.rs;
    const int es = p.bf16 ? 2 : 4;
    flurka_status st;
    const int nc = generic_chunk_rows(p);

    stage_begin(s);
    for (int row0 = 0; row0 < p.n; row0 += nc) {
        const int nr = (p.n - row0 < nc) ? (p.n - row0) : nc;
        const long rows = (long)p.BH * nr;
        st = query_features_and_numerator(p, a.Q, a.omega, S, cshift, P, N, row0, nr, nullptr, s);
        if (st != FLURKA_OK) return st;
        hipLaunchKernelGGL(bwd_row_prep_kernel, grid1d(rows, 4), dim3(256), 0, s, P, N, z, a.dOut, p.bf16,
                           dD, rows, nr, p.n, row0, p.mf, p.d);
        FLURKA_CHECK_LAUNCH();
        {   // T = dN S^T  (nr x mf)
            GemmArgs g{};
            g.A = N; g.B = S; g.C = T;
            g.M = nr; g.N = p.mf; g.K = p.d; g.Kin = p.d;
            g.sAm = p.d; g.sAki = 1; g.sAb = (long)p.H * nr * p.d; g.sAh = (long)nr * p.d;
            g.sBn = p.d; g.sBki = 1; g.sBb = (long)p.H * p.mf * p.d; g.sBh = (long)p.mf * p.d;
            g.sCm = p.mf; g.sCn = 1; g.sCb = (long)p.H * nr * p.mf; g.sCh = (long)nr * p.mf;
            g.H = p.H;
            if ((st = launch_gemm(g, p.BH, s)) != FLURKA_OK) return st;
        }
        if (!p.elu) {
            const long total = rows * p.mf;
            hipLaunchKernelGGL(bwd_du_kernel, grid1d(total, 256), dim3(256), 0, s, T, P, dD, z, total, nr, p.mf);
            FLURKA_CHECK_LAUNCH();
            GemmArgs g{};   // dQ = dU omega
            g.A = T; g.B = a.omega; g.C = (char*)a.dQ + (size_t)row0 * p.d * es;
            g.M = nr; g.N = p.d; g.K = p.m; g.Kin = p.m;
            g.sAm = p.m; g.sAki = 1; g.sAb = (long)p.H * nr * p.m; g.sAh = (long)nr * p.m;
            g.sBn = 1; g.sBki = p.d; g.sBb = 0; g.sBh = p.omega_per_head ? (long)p.m * p.d : 0;
            g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * p.n * p.d; g.sCh = (long)p.n * p.d;
            g.H = p.H; g.b_bf16 = p.bf16; g.c_bf16 = p.bf16;
            if ((st = launch_gemm(g, p.BH, s)) != FLURKA_OK) return st;
            if (a.dOmega) {
                // d omega_j (+)= sum over (batch[, head], i) of dU_ij q_i   (u_ij = omega_j . q_i - |q_i|^2/2)
                GemmArgs w{};
                w.A = T; w.B = (const char*)a.Q + (size_t)row0 * p.d * es; w.C = a.dOmega;
                w.M = p.m; w.N = p.d; w.Kin = nr;
                w.sAm = 1; w.sAki = p.m; w.sBn = 1; w.sBki = p.d; w.sCm = p.d; w.sCn = 1;
                w.b_bf16 = p.bf16; w.accumulate = row0 > 0;
                if (p.omega_per_head) {      // one result per head, reduction over (batch, i)
                    w.K = p.B * nr; w.sAko = (long)p.H * nr * p.m; w.sAh = (long)nr * p.m;
                    w.sBko = (long)p.H * p.n * p.d; w.sBh = (long)p.n * p.d; w.sCh = (long)p.m * p.d; w.H = p.H;
                    if ((st = launch_gemm(w, p.H, s)) != FLURKA_OK) return st;
                } else {                      // one result, reduction over (batch, head, i)
                    w.K = p.BH * nr; w.sAko = (long)nr * p.m; w.sBko = (long)p.n * p.d; w.H = 1;
                    if ((st = launch_gemm(w, 1, s)) != FLURKA_OK) return st;
                }
            }
        } else {
            const long total = rows * p.d;
            hipLaunchKernelGGL(bwd_dq_elu_kernel, grid1d(total, 256), dim3(256), 0, s, T, dD, z, a.Q, a.dQ,
                               p.bf16, total, nr, p.n, row0, p.d);
            FLURKA_CHECK_LAUNCH();
        }
        {   // dS (+)= P^T dN
            GemmArgs g{};
            g.A = P; g.B = N; g.C = dS;
            g.M = p.mf; g.N = p.d; g.K = nr; g.Kin = nr;
            g.sAm = 1; g.sAki = p.mf; g.sAb = (long)p.H * nr * p.mf; g.sAh = (long)nr * p.mf;
            g.sBn = 1; g.sBki = p.d; g.sBb = (long)p.H * nr * p.d; g.sBh = (long)nr * p.d;
            g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * p.mf * p.d; g.sCh = (long)p.mf * p.d;
            g.H = p.H; g.accumulate = row0 > 0;
            if ((st = launch_gemm(g, p.BH, s)) != FLURKA_OK) return st;
        }
        {   // dz (+)= P^T dD
            GemmArgs g{};
            g.A = P; g.B = dD; g.C = dz;
            g.M = p.mf; g.N = 1; g.K = nr; g.Kin = nr;
            g.sAm = 1; g.sAki = p.mf; g.sAb = (long)p.H * nr * p.mf; g.sAh = (long)nr * p.mf;
            g.sBn = 0; g.sBki = 1; g.sBb = (long)p.H * nr; g.sBh = nr;
            g.sCm = 1; g.sCn = 0; g.sCb = (long)p.H * p.mf; g.sCh = p.mf;
            g.H = p.H; g.accumulate = row0 > 0;
            if ((st = launch_gemm(g, p.BH, s)) != FLURKA_OK) return st;
        }
    }

    stage_end(s, STAGE_BWD_QUERY);

    stage_begin(s);
    const long krows = (long)p.BH * p.k;
    // PhiK exactly as the forward had it (same K', same shifts)
    if ((st = key_features(p, a.omega, Kp, const_cast<float*>(cshift), Phi, 0, s)) != FLURKA_OK) return st;
    {   // dPhiK = V' dS^T   (k x mf)
        GemmArgs g{};
        g.A = Vp; g.B = dS; g.C = dPhi;
        g.M = p.k; g.N = p.mf; g.K = p.d; g.Kin = p.d;
        g.sAm = p.d; g.sAki = 1; g.sAb = (long)p.H * p.k * p.d; g.sAh = (long)p.k * p.d;
        g.sBn = p.d; g.sBki = 1; g.sBb = (long)p.H * p.mf * p.d; g.sBh = (long)p.mf * p.d;
        g.sCm = p.mf; g.sCn = 1; g.sCb = (long)p.H * p.k * p.mf; g.sCh = (long)p.k * p.mf;
        g.H = p.H;
        if ((st = launch_gemm(g, p.BH, s)) != FLURKA_OK) return st;
    }
    {   // dV' = PhiK dS   (k x d)
        GemmArgs g{};
        g.A = Phi; g.B = dS; g.C = dVp;
        g.M = p.k; g.N = p.d; g.K = p.mf; g.Kin = p.mf;
        g.sAm = p.mf; g.sAki = 1; g.sAb = (long)p.H * p.k * p.mf; g.sAh = (long)p.k * p.mf;
        g.sBn = 1; g.sBki = p.d; g.sBb = (long)p.H * p.mf * p.d; g.sBh = (long)p.mf * p.d;
        g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * p.k * p.d; g.sCh = (long)p.k * p.d;
        g.H = p.H;
        if ((st = launch_gemm(g, p.BH, s)) != FLURKA_OK) return st;
    }
    if (!p.elu) {
        hipLaunchKernelGGL(bwd_key_du_kernel, grid1d(krows, 4), dim3(256), 0, s, dPhi, Phi, dz, rs, krows,
                           p.k, p.m);
        FLURKA_CHECK_LAUNCH();
        GemmArgs g{};   // dK' = dUk omega
        g.A = dPhi; g.B = a.omega; g.C = dKp;
        g.M = p.k; g.N = p.d; g.K = p.m; g.Kin = p.m;
        g.sAm = p.m; g.sAki = 1; g.sAb = (long)p.H * p.k * p.m; g.sAh = (long)p.k * p.m;
        g.sBn = 1; g.sBki = p.d; g.sBb = 0; g.sBh = p.omega_per_head ? (long)p.m * p.d : 0;
        g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * p.k * p.d; g.sCh = (long)p.k * p.d;
        g.H = p.H; g.b_bf16 = p.bf16;
        if ((st = launch_gemm(g, p.BH, s)) != FLURKA_OK) return st;
        if (a.dOmega) {
            // d omega_j += sum over (batch[, head], r) of dUk_rj k'_r
            GemmArgs w{};
            w.A = dPhi; w.B = Kp; w.C = a.dOmega;
            w.M = p.m; w.N = p.d; w.Kin = p.k;
            w.sAm = 1; w.sAki = p.m; w.sBn = 1; w.sBki = p.d; w.sCm = p.d; w.sCn = 1;
            w.accumulate = 1;
            if (p.omega_per_head) {
                w.K = p.B * p.k; w.sAko = (long)p.H * p.k * p.m; w.sAh = (long)p.k * p.m;
                w.sBko = (long)p.H * p.k * p.d; w.sBh = (long)p.k * p.d; w.sCh = (long)p.m * p.d; w.H = p.H;
                if ((st = launch_gemm(w, p.H, s)) != FLURKA_OK) return st;
            } else {
                w.K = p.BH * p.k; w.sAko = (long)p.k * p.m; w.sBko = (long)p.k * p.d; w.H = 1;
                if ((st = launch_gemm(w, 1, s)) != FLURKA_OK) return st;
            }
        }
        const long total = krows * p.d;
        hipLaunchKernelGGL(bwd_key_norm_kernel, grid1d(total, 256), dim3(256), 0, s, dKp, Kp, rs, total, p.d);
        FLURKA_CHECK_LAUNCH();
    } else {
        const long total = krows * p.d;
        hipLaunchKernelGGL(bwd_key_elu_kernel, grid1d(total, 256), dim3(256), 0, s, dKp, dPhi, dz, Kp, total,
                           p.k, p.d);
        FLURKA_CHECK_LAUNCH();
    }

    stage_end(s, STAGE_BWD_KEY);
    return grad_gemms_f32(p, a, dKp, dVp, a.ws, p.bf16 ? W.dKp : 0, s);
}

static flurka_status grad_gemms_f32(const Problem& p, const BwdArgs& a, const float* dKp, const float* dVp, float* part,
                                    size_t part_floats, hipStream_t s) {
    flurka_status st;
    // dK = E^T dK', dV = F^T dV'   (n x d per head)
    stage_begin(s);
    {
        GemmArgs g{};
        g.A = a.E; g.B = dKp; g.C = a.dK;
        g.A2 = a.F; g.B2 = dVp; g.C2 = a.dV;
        g.M = p.n; g.N = p.d; g.K = p.k; g.Kin = p.k;
        g.sAm = 1; g.sAki = p.n; g.sAb = 0; g.sAh = p.ef_per_head ? (long)p.k * p.n : 0;
        g.sBn = 1; g.sBki = p.d; g.sBb = (long)p.H * p.k * p.d; g.sBh = (long)p.k * p.d;
        g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * p.n * p.d; g.sCh = (long)p.n * p.d;
        g.H = p.H; g.a_bf16 = p.bf16; g.c_bf16 = p.bf16;
        int batches = p.BH;
        if (!p.ef_per_head) {    // E, F shared: all heads side by side as one row of columns (head, t)
            g.N = p.BH * p.d; g.Nin = p.d; g.sBno = (long)p.k * p.d; g.sCno = (long)p.n * p.d;
            batches = 1;
        }
        if ((st = launch_gemm(g, batches, s)) != FLURKA_OK) return st;
    }
    stage_end(s, STAGE_BWD_DKDV);
    // dE = sum_bh dK' K^T, dF = sum_bh dV' V^T   (k x n); reduction index = (bh, t)
    stage_begin(s);
    {
        GemmArgs g{};
        g.A = dKp; g.B = a.K; g.C = a.dE;
        g.A2 = dVp; g.B2 = a.V; g.C2 = a.dF;
        g.M = p.k; g.N = p.n; g.Kin = p.d;
        g.sAm = p.d; g.sAki = 1; g.sBn = p.d; g.sBki = 1; g.sCm = p.n; g.sCn = 1;
        g.b_bf16 = p.bf16; g.c_bf16 = p.bf16 && !p.grad_ef_f32;
        if (p.ef_per_head) {     // one (k x n) gradient per head, reduction index = (batch, t)
            g.K = p.B * p.d; g.sAko = (long)p.H * p.k * p.d; g.sAh = (long)p.k * p.d;
            g.sBko = (long)p.H * p.n * p.d; g.sBh = (long)p.n * p.d; g.sCh = (long)p.k * p.n; g.H = p.H;
            if ((st = launch_gemm_f32(g, p.H, part, part_floats, s)) != FLURKA_OK) return st;
        } else {                  // E, F shared: reduction index = (batch, head, t)
            g.K = p.BH * p.d; g.sAko = (long)p.k * p.d; g.sBko = (long)p.n * p.d; g.H = 1;
            if ((st = launch_gemm_f32(g, 1, part, part_floats, s)) != FLURKA_OK) return st;
        }
    }
    stage_end(s, STAGE_BWD_DEDF);
    return FLURKA_OK;
}

}  // namespace flurka
