// Fused kernels of the fp32-arithmetic path for head sizes up to 128 (gfx950): nothing of size n x m ever
// reaches memory.  They serve fp32 storage, and bf16 storage wherever the bf16 kernels (flurka_fast.hip,
// flurka_bwd.hip) do not apply, with results as exact as fp32 operands and fp32 sums give.
//
// Query side (work that grows with n): contractions on v_mfma_f32_32x32x16_bf16 with every fp32 operand
// split into three bf16 terms (8 + 8 + 8 = 24 mantissa bits, so the split is exact) and every bf16 operand
// as it is (flurka_gemm_f32.h: six of the nine products of two split operands, the rest is at most 2^-24 of the
// product).  Six bf16 products cost 6/16 of the same product on the fp32 matrix instruction, three
// (bf16 x fp32) 3/16.
// Key side (work that grows with k): fp32 matrix instructions; it is a few percent of the whole.
//
//   f32_key_state    S = PhiK^T V', z, c      workgroup = (head, 32 features), wavefront = key range
//   f32_query_fwd    out, lse                 wavefront = 32 queries, lane = query
//   f32_bwd_x        dQ, g, 1/D               wavefront = 32 queries, lane = query
//   f32_bwd_y        dS, dz (d omega)         wavefront = 32 features of one query range, lane = feature
//   f32_bwd_merge    sums the ranges
//   f32_bwd_key      dK', dV'                 workgroup = (head, 32 keys), lane = key
// Notation and formulas as in flurka_generic.hip; operand chaining as in flurka_fast.hip: an accumulator
// (row 8(g/4) + 4h + g%4 in element g of lane half h) is the next contraction's operand as it stands.
#include "flurka_gemm_f32.h"

namespace flurka {

#define FLURKA_CHECK_LAUNCH()                                   \
    do {                                                        \
        if (hipGetLastError() != hipSuccess) return FLURKA_ERR_LAUNCH; \
    } while (0)

constexpr float F32_LOG2E = FLURKA_LOG2E;

__device__ __forceinline__ float f32_elu1(float x) { return x > 0.f ? x + 1.f : expf(x); }

// ---- rows in memory -> operands ------------------------------------------------
// Head sizes are padded to D = 64 or 128 with zeros; rows in memory have d elements and start on element
// boundaries only.  No divergent branches: a group of coordinates past the end is read from a clamped
// place and replaced by zeros.  N consecutive elements from coordinate c0 of the row at element `off`
// (bf16: as packed pairs):
template <int N>
__device__ __forceinline__ void f32_load(const float* p, long off, int c0, int d, float (&v)[N]) {
    if (d % N == 0) {
        const bool in = c0 < d;
        __builtin_memcpy(v, p + off + (in ? c0 : 0), 4 * N);
#pragma unroll
        for (int e = 0; e < N; ++e) v[e] = in ? v[e] : 0.f;
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const float x = p[off + (c0 + e < d ? c0 + e : 0)];
            v[e] = c0 + e < d ? x : 0.f;
        }
    }
}
template <int N>
__device__ __forceinline__ void bf16_load(const uint16_t* p, long off, int c0, int d, uint32_t (&w)[N / 2]) {
    if (d % N == 0) {
        const bool in = c0 < d;
        __builtin_memcpy(w, p + off + (in ? c0 : 0), 2 * N);
#pragma unroll
        for (int e = 0; e < N / 2; ++e) w[e] = in ? w[e] : 0u;
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) {
            uint32_t x = p[off + (c0 + e < d ? c0 + e : 0)];
            x = c0 + e < d ? x : 0u;
            w[e >> 1] = (e & 1) ? (w[e >> 1] | (x << 16)) : x;
        }
    }
}
__device__ __forceinline__ void f32_load8(const float* p, long off, int c0, int d, float (&v)[8]) { f32_load<8>(p, off, c0, d, v); }
__device__ __forceinline__ uint4 bf16_load8(const uint16_t* p, long off, int c0, int d) {
    uint32_t w[4];
    bf16_load<8>(p, off, c0, d, w);
    return make_uint4(w[0], w[1], w[2], w[3]);
}
// 4 consecutive floats
__device__ __forceinline__ float4 f32_load4(const float* p, long off, int c0, int d) {
    float v[4];
    f32_load<4>(p, off, c0, d, v);
    return make_float4(v[0], v[1], v[2], v[3]);
}
// 4 consecutive elements of either storage type
__device__ __forceinline__ float4 any_load4(const void* p, long off, int c0, int d, int bf16) {
    if (!bf16) return f32_load4((const float*)p, off, c0, d);
    uint32_t w[2];
    bf16_load<4>((const uint16_t*)p, off, c0, d, w);
    return make_float4(pair_lo(w[0]), pair_hi(w[0]), pair_lo(w[1]), pair_hi(w[1]));
}

// 8 values as loaded, before the split
template <int T> struct Raw8 { float v[8]; };
template <> struct Raw8<1> { uint4 v; };

__device__ __forceinline__ void split3_8(const float (&v)[8], uint4 (&t)[3]) {
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split3_pair(v[2 * e], v[2 * e + 1], h[e], m[e], l[e]);
    t[0] = make_uint4(h[0], h[1], h[2], h[3]);
    t[1] = make_uint4(m[0], m[1], m[2], m[3]);
    t[2] = make_uint4(l[0], l[1], l[2], l[3]);
}
template <int T>
__device__ __forceinline__ Raw8<T> load_raw(const void* p, long off, int c0, int d) {
    Raw8<T> r;
    if constexpr (T == 1) r.v = bf16_load8((const uint16_t*)p, off, c0, d);
    else f32_load8((const float*)p, off, c0, d, r.v);
    return r;
}
template <int T>
__device__ __forceinline__ Terms<T> to_terms(const Raw8<T>& r) {
    Terms<T> x;
    if constexpr (T == 1) x.t[0] = r.v;
    else split3_8(r.v, x.t);
    return x;
}

// An accumulator tile's 16 values as operand terms for the two 16-slot halves of the next reduction.
__device__ __forceinline__ void split_acc(const float (&v)[16], uint4 (&t)[2][3]) {
#pragma unroll
    for (int sp = 0; sp < 2; ++sp) {
        uint32_t w[3][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) split3_pair(v[8 * sp + 2 * e], v[8 * sp + 2 * e + 1], w[0][e], w[1][e], w[2][e]);
#pragma unroll
        for (int i = 0; i < 3; ++i) t[sp][i] = make_uint4(w[i][0], w[i][1], w[i][2], w[i][3]);
    }
}

// position of feature / row f of a 32-row tile in a per-row vector kept in accumulator order (16h + g)
__device__ __forceinline__ int acc_slot(int f) { return 16 * ((f >> 2) & 1) + 4 * (f >> 3) + (f & 3); }

struct F32QueryArgs {
    const void* Q;
    const void* G;             // dOut          (backward)
    const void* omega;
    const float* S; const float* z; const float* c;     // ctx
    float* lse;                // ctx: written by the forward, read by the backward
    void* out;                 // out, or dQ
    float* delta;              // (BH, n) g_i   (backward)
    float* dinv;               // (BH, n) 1 / sum of the weights as formed with lse as the shift
    int n, H, d, mf, FT, blocks_per_head;
    long omega_head_stride;
};

// Feature tiles pass through two LDS buffers: the threads of the workgroup fetch tile ft + 1 into
// registers while tile ft is being worked on, split it and store it after; one barrier per tile.
//   W: TW terms of omega (absent for elu1), X: three terms of S or S / z, then c and z in accumulator order
template <int D, int TW>
struct FeatureStage {
    static constexpr int x_off = TW * Tile32<D>::bytes;
    static constexpr int v_off = x_off + 3 * Tile32<D>::bytes;
    static constexpr int bytes = v_off + 64 * 4;
};

template <int D, int TW, int NT, bool OVER_Z>
struct FeatureFetch {
    static constexpr int CH = Tile32<D>::chunks / NT;
    static_assert(Tile32<D>::chunks % NT == 0 && NT >= 64, "whole chunks per thread");
    Raw8<TW ? TW : 1> w[CH];
    float x[CH][8];
    float cv, zv;
    // rows past mf: finite omega, S = 0, z = 0, c = -inf: their weights are exactly 0
    __device__ __forceinline__ void load(const F32QueryArgs& a, long bh, int ft, int tid) {
        const long row0 = bh * a.mf;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int idx = tid + NT * i, r = idx / (D / 8), c0 = 8 * (idx % (D / 8));
            const int f = 32 * ft + r, fr = f < a.mf ? f : a.mf - 1;
            if constexpr (TW > 0) w[i] = load_raw<TW>(a.omega, (bh % a.H) * a.omega_head_stride + (long)fr * a.d, c0, a.d);
            f32_load8(a.S, (row0 + fr) * a.d, c0, a.d, x[i]);
            float scale = f < a.mf ? 1.f : 0.f;
            if (OVER_Z && f < a.mf) scale = 1.f / a.z[row0 + f];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[i][e] *= scale;
        }
        if (tid < 32) {
            const int f = 32 * ft + tid;
            cv = f < a.mf ? a.c[row0 + f] : -INFINITY;
            zv = f < a.mf ? a.z[row0 + f] : 0.f;
        }
    }
    __device__ __forceinline__ void store(unsigned char* buf, int tid) const {
        using L = FeatureStage<D, TW>;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int idx = tid + NT * i, r = idx / (D / 8), c = idx % (D / 8);
            if constexpr (TW > 0) {
                const Terms<TW> t = to_terms<TW>(w[i]);
#pragma unroll
                for (int k = 0; k < TW; ++k) *(uint4*)Tile32<D>::chunk(buf + k * Tile32<D>::bytes, r, c) = t.t[k];
            }
            uint4 t[3];
            split3_8(x[i], t);
#pragma unroll
            for (int k = 0; k < 3; ++k) *(uint4*)Tile32<D>::chunk(buf + L::x_off + k * Tile32<D>::bytes, r, c) = t[k];
        }
        if (tid < 32) {
            float* v = (float*)(buf + L::v_off);
            v[acc_slot(tid)] = cv;
            v[32 + acc_slot(tid)] = zv;
        }
    }
};

// this lane's 16 values of a per-row vector kept in accumulator order
__device__ __forceinline__ void acc_vector(const float* v, int half, float (&x)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) *(float4*)&x[4 * q] = *(const float4*)(v + 16 * half + 4 * q);
}

// elu1: coordinates 32 ft + 8q + 4 half + e of a row in accumulator order, as fp32
__device__ __forceinline__ void acc_coords(const void* p, long off, int ft, int half, int d, int bf16, float (&x)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) *(float4*)&x[4 * q] = any_load4(p, off, 32 * ft + 8 * q + 4 * half, d, bf16);
}

// rows of results: the lane's 4 consecutive values at coordinate c0 of the row at element `off`
__device__ __forceinline__ void store4(void* p, long off, int c0, int d, const float (&v)[4], int bf16) {
    if (c0 + 4 <= d) {
        if (bf16) {
            const uint2 w = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
            __builtin_memcpy((uint16_t*)p + off + c0, &w, 8);
        } else {
            __builtin_memcpy((float*)p + off + c0, v, 16);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e)
            if (c0 + e < d) store_elem(p, off + c0 + e, v[e], bf16);
    }
}

constexpr int F32_NW = 4;      // wavefronts of a query-side workgroup

// ---- infinities ----------------------------------------------------------------
// An infinite operand, or a finite one past the largest bf16 value, has no three-term form: its products come out
// NaN.  So do sums that overflow only because of the lazy row maximum.  The query-side kernels therefore look at
// their results (one instruction a value, after the loop), and a wavefront that holds one that is not finite forms
// its rows again without terms: PlainRow and plain_dot below, fp32 fused multiply-adds on the operands as they
// are, the formulas and the shift of flurka_generic.hip.  All lanes take part, lanes l and l ^ 32 sharing a row;
// rows that were finite keep what they have.  One tile of coordinates at a time and features formed again for
// each: the kernels' registers (and with them the wavefronts in flight) are not to grow for this (whole rows at a
// time: 181 instead of 118 registers in the elu dQ kernel; as calls: 248).  4 x 12 x 3001 x 64, 150 features: one
// infinite element of dOut 5.4 ms instead of 0.36, all of Q NaN 4.7.
__device__ __forceinline__ float pair_sum(float x) { return x + __shfl_xor(x, 32, 64); }
// product of two rows of d elements, each lane of a pair half of it
__device__ __forceinline__ float plain_dot(const void* p, long po, int p_bf16, const void* q, long qo, int q_bf16, int d, int half) {
    float s = 0.f;
#pragma unroll 1
    for (int c = 4 * half; c < d; c += 8) {
        const float4 x = any_load4(p, po, c, d, p_bf16), y = any_load4(q, qo, c, d, q_bf16);
        s = fmaf(x.x, y.x, s); s = fmaf(x.y, y.y, s); s = fmaf(x.z, y.z, s); s = fmaf(x.w, y.w, s);
    }
    return pair_sum(s);
}

// A NaN in a row of Q or dOut, or in z, makes everything NaN that the row gives: nothing to form again.
__device__ __forceinline__ bool row_has_nan(const void* p, long off, int d, int half, int bf16) {
    float s = 0.f;
#pragma unroll 1
    for (int c = 4 * half; c < d; c += 8) {
        const float4 x = any_load4(p, off, c, d, bf16);
        s += (x.x != x.x || x.y != x.y || x.z != x.z || x.w != x.w) ? 1.f : 0.f;
    }
    return pair_sum(s) > 0.f;
}
__device__ __forceinline__ bool z_has_nan(const F32QueryArgs& a, long bh, int lane) {
    bool nan = false;
#pragma unroll 1
    for (int j = lane; j < a.mf; j += 64) nan |= a.z[bh * a.mf + j] != a.z[bh * a.mf + j];
    return __any(nan);
}

struct PlainRow {
    const F32QueryArgs& a;
    long bh, qoff, omega_off;
    int half, bf16;
    float mx;                  // row maximum of the exponents
    __device__ __forceinline__ PlainRow(const F32QueryArgs& args, long bh_, long qoff_, int half_, int bf16_)
        : a(args), bh(bh_), qoff(qoff_), omega_off((bh_ % args.H) * args.omega_head_stride), half(half_), bf16(bf16_), mx(0.f) {}
    __device__ __forceinline__ float exponent(int j) const {
        return plain_dot(a.omega, omega_off + (long)j * a.d, bf16, a.Q, qoff, bf16, a.d, half) + a.c[bh * a.mf + j];
    }
    template <bool ELU>
    __device__ __forceinline__ float feature(int j) const {
        if constexpr (ELU) return f32_elu1(load_elem(a.Q, qoff + j, bf16));
        else return expf(exponent(j) - mx);
    }
    // sets mx; returns the denominator
    template <bool ELU>
    __device__ __forceinline__ float denominator() {
        if constexpr (!ELU) {
            mx = -INFINITY;
#pragma unroll 1
            for (int j = 0; j < a.mf; ++j) mx = fmaxf(mx, exponent(j));
        }
        float den = 0.f;
#pragma unroll 1
        for (int j = 0; j < a.mf; ++j) den = fmaf(feature<ELU>(j), a.z[bh * a.mf + j], den);
        return den;
    }
    // sum_j weight(j) M_j, this lane's coordinates of tile t in accumulator order
    template <class W>
    __device__ __forceinline__ void tile(const void* M, long off, int m_bf16, int t, W&& weight, float (&acc)[16]) const {
#pragma unroll
        for (int g = 0; g < 16; ++g) acc[g] = 0.f;
#pragma unroll 1
        for (int j = 0; j < a.mf; ++j) {
            const float w = weight(j);
            float x[16];
            acc_coords(M, off + (long)j * a.d, t, half, a.d, m_bf16, x);
#pragma unroll
            for (int g = 0; g < 16; ++g) acc[g] = fmaf(w, x[g], acc[g]);
        }
    }
    __device__ __forceinline__ void store_tile(int t, const float (&v)[16]) const {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const float x[4] = {v[4 * q4], v[4 * q4 + 1], v[4 * q4 + 2], v[4 * q4 + 3]};
            store4(a.out, qoff, 32 * t + 8 * q4 + 4 * half, a.d, x, bf16);
        }
    }
};

// ---------------------------------------------------------------------------
// Forward.  T = 1: bf16 storage, 3: fp32 storage.
// Per 32 x 32 (feature, query) tile at D = 64: 4 T' MFMAs for u (T' = 1 or 6 products), 24 for the
// numerator, 16 exponentials, 88 instructions that split the weights.
// ---------------------------------------------------------------------------
template <int D, int T, bool ELU>
__global__ __launch_bounds__(F32_NW * 64, D == 64 ? 2 : 1) void f32_query_fwd_kernel(F32QueryArgs a) {
    constexpr int TW = ELU ? 0 : T, KS = D / 16, TT = D / 32, NT = F32_NW * 64;
    using L = FeatureStage<D, TW>;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const Tile32<D> tl(lane);
    const long bh = blockIdx.x / a.blocks_per_head;
    const int row = ((int)(blockIdx.x % a.blocks_per_head) * F32_NW + wave) * 32 + l32;
    const bool live = row < a.n;
    const long qoff = (bh * a.n + (live ? row : a.n - 1)) * a.d;

    FeatureFetch<D, TW, NT, false> ff;
    ff.load(a, bh, 0, tid);
    Terms<T> q[KS];
    if constexpr (!ELU) {
#pragma unroll
        for (int s = 0; s < KS; ++s) q[s] = to_terms<T>(load_raw<T>(a.Q, qoff, 16 * s + 8 * half, a.d));
    }
    floatx16 acc[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[t] = zero16();
    float den = 0.f, mu = 0.f;
    ff.store(lds, tid);
    __syncthreads();
    for (int ft = 0; ft < a.FT; ++ft) {
        const unsigned char* buf = lds + (ft & 1) * L::bytes;
        if (ft + 1 < a.FT) ff.load(a, bh, ft + 1, tid);
        float p[16], zv[16];
        acc_vector((const float*)(buf + L::v_off) + 32, half, zv);
        if constexpr (ELU) {
            acc_coords(a.Q, qoff, ft, half, a.d, T == 1, p);
#pragma unroll
            for (int g = 0; g < 16; ++g) p[g] = f32_elu1(p[g]);
        } else {
            floatx16 u = zero16();
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                uint4 w[T];
#pragma unroll
                for (int k = 0; k < T; ++k) w[k] = tl.row_frag(buf + k * Tile32<D>::bytes, s);
                u = mfma_terms<T, T>(w, q[s].t, u);
            }
            acc_vector((const float*)(buf + L::v_off), half, p);
            float mx = -INFINITY;
#pragma unroll
            for (int g = 0; g < 16; ++g) { p[g] += u[g]; mx = fmaxf(mx, p[g]); }
            mx = half_max(mx);
            if (ft == 0) {
                mu = mx;
            } else if (mx > mu + FLURKA_LAZY_MAX) {
                const float sc = fast_exp2((mu - mx) * F32_LOG2E);
                mu = mx;
                den *= sc;
#pragma unroll
                for (int t = 0; t < TT; ++t)
#pragma unroll
                    for (int g = 0; g < 16; ++g) acc[t][g] *= sc;
            }
            const float shift = -mu * F32_LOG2E;
#pragma unroll
            for (int g = 0; g < 16; ++g) p[g] = fast_exp2(fmaf(p[g], F32_LOG2E, shift));
        }
#pragma unroll
        for (int g = 0; g < 16; ++g) den = fmaf(p[g], zv[g], den);
        uint4 pt[2][3];
        split_acc(p, pt);
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            // a tile's products form a sum of their own before they join the running one
            floatx16 part = zero16();
#pragma unroll
            for (int sp = 0; sp < 2; ++sp) {
                uint4 x[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) x[k] = tl.col_frag(buf + L::x_off + k * Tile32<D>::bytes, sp, t);
                part = mfma_terms<3, 3>(x, pt[sp], part);
            }
            acc[t] += part;
        }
        if (ft + 1 < a.FT) ff.store(lds + ((ft & 1) ^ 1) * L::bytes, tid);
        __syncthreads();
    }
    den = half_sum(den);
    float chk = den * 0.f;
#pragma unroll
    for (int t = 0; t < TT; ++t) chk = not_finite(acc[t], chk);
    bool bad = half_sum(chk) != 0.f;
    if (__any(bad)) {
        const bool q_nan = row_has_nan(a.Q, qoff, a.d, half, T == 1), z_nan = z_has_nan(a, bh, lane);
        bad = bad && !q_nan && !z_nan;
    }
    const float inv = 1.f / den;
    if (live && !bad) {
        if (half == 0) a.lse[bh * a.n + row] = mu + logf(den);
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[t][4 * q4 + e] * inv;
                store4(a.out, qoff, 32 * t + 8 * q4 + 4 * half, a.d, v, T == 1);
            }
    }
    if (__any(bad)) {
        PlainRow plain(a, bh, qoff, half, T == 1);
        const float pden = plain.template denominator<ELU>();
        const bool write = bad && live;
        if (write && half == 0) a.lse[bh * a.n + row] = plain.mx + logf(pden);
#pragma unroll 1
        for (int t = 0; t < TT; ++t) {
            float num[16];
            plain.tile(a.S, bh * a.mf * a.d, 0, t, [&](int j) { return plain.template feature<ELU>(j); }, num);
#pragma unroll
            for (int g = 0; g < 16; ++g) num[g] /= pden;
            if (write) plain.store_tile(t, num);
        }
    }
}

// ---------------------------------------------------------------------------
// Backward, lane = query: dQ, g_i and the row scale of the dS kernel.
// With W_ij = exp(u_ij + c_j - lse_i) (lse_i only serves as the shift: its rounding cancels in 1/sB),
// b = W z, t_ij = G_i . S_j / z_j and any ghat_i:
//     sB = sum_j b_ij,  r_ij = b_ij (t_ij - ghat_i),  g_i = ghat_i + sum_j r_ij / sB
//     dQ_i = (sum_j r_ij omega_j - (g_i - ghat_i) sum_j b_ij omega_j) / sB
// ghat_i = sum_j b_ij t_ij / sum_j b_ij over the first feature tile, which keeps r of the size of t - g; the
// caller's `out` is not read, it may be anything.  Both sums over omega take all three terms of their weights.
// elu1: T_ij = G_i . S_j, D = P . z, g = (P . T) / D, dQ = (T - g z) / D * phi'(Q).
// ---------------------------------------------------------------------------
template <int D, int T, bool ELU>
__global__ __launch_bounds__(F32_NW * 64, (D == 64 && (T == 1 || ELU)) ? 2 : 1) void f32_bwd_x_kernel(F32QueryArgs a) {
    constexpr int TW = ELU ? 0 : T, KS = D / 16, TT = D / 32, NT = F32_NW * 64;
    using L = FeatureStage<D, TW>;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const Tile32<D> tl(lane);
    const long bh = blockIdx.x / a.blocks_per_head;
    const int row = ((int)(blockIdx.x % a.blocks_per_head) * F32_NW + wave) * 32 + l32;
    const bool live = row < a.n;
    const long ri = bh * a.n + (live ? row : a.n - 1), qoff = ri * a.d;

    FeatureFetch<D, TW, NT, !ELU> ff;
    ff.load(a, bh, 0, tid);
    Terms<T> q[KS], g[KS];
    float gh = 0.f, nlam = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        g[s] = to_terms<T>(load_raw<T>(a.G, qoff, 16 * s + 8 * half, a.d));
        if constexpr (!ELU) q[s] = to_terms<T>(load_raw<T>(a.Q, qoff, 16 * s + 8 * half, a.d));
    }
    if constexpr (!ELU) nlam = -a.lse[ri] * F32_LOG2E;
    floatx16 accR[TT], accB[TT];                   // elu1: accR = the T tiles
#pragma unroll
    for (int t = 0; t < TT; ++t) { accR[t] = zero16(); accB[t] = zero16(); }
    float sR = 0.f, sB = 0.f;
    ff.store(lds, tid);
    __syncthreads();
    auto one_tile = [&](int ft, floatx16* keep) {
        const unsigned char* buf = lds + (ft & 1) * L::bytes;
        if (ft + 1 < a.FT) ff.load(a, bh, ft + 1, tid);
        floatx16 tp = zero16();
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            uint4 x[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) x[k] = tl.row_frag(buf + L::x_off + k * Tile32<D>::bytes, s);
            tp = mfma_terms<3, T>(x, g[s].t, tp);
        }
        float zv[16];
        acc_vector((const float*)(buf + L::v_off) + 32, half, zv);
        if constexpr (ELU) {
            float p[16];
            acc_coords(a.Q, qoff, ft, half, a.d, T == 1, p);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const float pe = f32_elu1(p[e]);
                sB = fmaf(pe, zv[e], sB);
                sR = fmaf(pe, tp[e], sR);
            }
            *keep = tp;
        } else {
            floatx16 u = zero16();
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                uint4 w[T];
#pragma unroll
                for (int k = 0; k < T; ++k) w[k] = tl.row_frag(buf + k * Tile32<D>::bytes, s);
                u = mfma_terms<T, T>(w, q[s].t, u);
            }
            float cv[16], b[16], r[16];
            acc_vector((const float*)(buf + L::v_off), half, cv);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                b[e] = fast_exp2(fmaf(u[e] + cv[e], F32_LOG2E, nlam)) * zv[e];
                sB += b[e];
            }
            if (ft == 0) {
                float bt = 0.f;
#pragma unroll
                for (int e = 0; e < 16; ++e) bt = fmaf(b[e], tp[e], bt);
                const float b0 = half_sum(sB);
                bt = half_sum(bt);
                gh = b0 > 0.f ? bt / b0 : 0.f;
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                r[e] = b[e] * (tp[e] - gh);
                sR += r[e];
            }
            // one weight after the other: omega's fragments are read twice, but the terms of only one are live
            auto add_omega = [&](const float (&v)[16], floatx16 (&acc)[TT]) {
                uint4 vt[2][3];
                split_acc(v, vt);
#pragma unroll
                for (int t = 0; t < TT; ++t) {
                    floatx16 part = zero16();
#pragma unroll
                    for (int sp = 0; sp < 2; ++sp) {
                        uint4 w[T];
#pragma unroll
                        for (int k = 0; k < T; ++k) w[k] = tl.col_frag(buf + k * Tile32<D>::bytes, sp, t);
                        part = mfma_terms<T, 3>(w, vt[sp], part);
                    }
                    acc[t] += part;
                }
            };
            add_omega(b, accB);
            __builtin_amdgcn_sched_barrier(0);
            add_omega(r, accR);
        }
        if (ft + 1 < a.FT) ff.store(lds + ((ft & 1) ^ 1) * L::bytes, tid);
        __syncthreads();
    };
    if constexpr (ELU) {
        // one feature tile per 32 coordinates, all of them kept (FT <= TT)
#pragma unroll
        for (int ft = 0; ft < TT; ++ft)
            if (ft < a.FT) one_tile(ft, &accR[ft]);
    } else {
        for (int ft = 0; ft < a.FT; ++ft) one_tile(ft, nullptr);
    }
    sB = half_sum(sB);
    sR = half_sum(sR);
    const float inv = 1.f / sB, dg = sR * inv;     // elu1: dg = g itself
    float chk = inv * 0.f + dg * 0.f;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        chk = not_finite(accR[t], chk);
        if constexpr (!ELU) chk = not_finite(accB[t], chk);
    }
    bool bad = half_sum(chk) != 0.f;
    if (__any(bad)) {
        const bool q_nan = row_has_nan(a.Q, qoff, a.d, half, T == 1), g_nan = row_has_nan(a.G, qoff, a.d, half, T == 1);
        const bool z_nan = z_has_nan(a, bh, lane);
        bad = bad && !q_nan && !g_nan && !z_nan;
    }
    if (live && !bad) {
        if (half == 0) {
            a.delta[ri] = ELU ? dg : gh + dg;
            a.dinv[ri] = inv;
        }
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int c0 = 32 * t + 8 * q4 + 4 * half;
                float v[4];
                if constexpr (ELU) {
                    const float4 x = any_load4(a.Q, qoff, c0, a.d, T == 1);
                    const float4 zz = f32_load4(a.z, bh * a.mf, c0, a.mf);
                    const float xs[4] = {x.x, x.y, x.z, x.w}, zs[4] = {zz.x, zz.y, zz.z, zz.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (accR[t][4 * q4 + e] - dg * zs[e]) * inv * (xs[e] > 0.f ? 1.f : expf(xs[e]));
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = (accR[t][4 * q4 + e] - dg * accB[t][4 * q4 + e]) * inv;
                }
                store4(a.out, qoff, c0, a.d, v, T == 1);
            }
    }
    if (__any(bad)) {
        PlainRow plain(a, bh, qoff, half, T == 1);
        const float pinv = 1.f / plain.template denominator<ELU>();
        const long soff = bh * a.mf * a.d;
        const bool write = bad && live;
        float gi = 0.f;
#pragma unroll 1
        for (int t = 0; t < TT; ++t) {
            float o[16], gv[16];
            plain.tile(a.S, soff, 0, t, [&](int j) { return plain.template feature<ELU>(j); }, o);
            acc_coords(a.G, qoff, t, half, a.d, T == 1, gv);
#pragma unroll
            for (int e = 0; e < 16; ++e) gi = fmaf(gv[e], o[e] * pinv, gi);
        }
        gi = pair_sum(gi);
        const float dD = -gi * pinv;
        if (write && half == 0) {
            a.delta[ri] = gi;
            // the dS kernel forms its weights with lse as the shift
            a.dinv[ri] = ELU ? pinv : pinv / expf(plain.mx - a.lse[ri]);
        }
        auto d_feature = [&](int j) {              // d loss / d feature j
            return plain_dot(a.G, qoff, T == 1, a.S, soff + (long)j * a.d, 0, a.d, half) * pinv + dD * a.z[bh * a.mf + j];
        };
        if constexpr (ELU) {
#pragma unroll 1
            for (int j = 0; j < a.mf; ++j) {
                const float x = load_elem(a.Q, qoff + j, T == 1), v = d_feature(j) * (x > 0.f ? 1.f : expf(x));
                if (write && half == 0) store_elem(a.out, qoff + j, v, T == 1);
            }
        } else {
#pragma unroll 1
            for (int t = 0; t < TT; ++t) {
                float dq[16];
                plain.tile(a.omega, plain.omega_off, T == 1, t, [&](int j) { return d_feature(j) * plain.template feature<ELU>(j); }, dq);
                if (write) plain.store_tile(t, dq);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Backward, lane = feature: dS_j = sum_i W_ij G_i, dz_j = - sum_i W_ij g_i over a range of queries, with
// W_ij = exp(u_ij + c_j - lse_i) / sB_i (elu1: phi(q)_ij / D_i); with DOM also
//     d omega_j = sum_i W_ij z_j (G_i . S_j / z_j - g_i) q_i.
// A workgroup is F32_NW feature tiles of one (head, range); blocks of Y_ROWS queries pass through LDS as
// operand terms, the next block being fetched into registers meanwhile.
// ---------------------------------------------------------------------------
struct F32YArgs {
    const void* Q; const void* G; const void* omega;
    const float* S; const float* z; const float* c; const float* lse; const float* delta; const float* dinv;
    float* dSpart;             // (BH, R, mf, d)
    float* dzpart;             // (BH, R, mf)
    float* dWpart;             // DOM: (BH, R, mf, d)
    int n, H, d, mf, FT, R, blocks_per_range;
    long omega_head_stride;
};

constexpr int F32_Y_ROWS = 64;

template <int D, int T>
struct F32YLds {
    static constexpr int g_off = 2 * T * Tile32<D>::bytes;       // Q terms of 2 row tiles, then dOut terms
    static constexpr int v_off = 2 * g_off;
    static constexpr int bytes = v_off + 3 * F32_Y_ROWS * 4;      // shift, 1/D, g per row
};

template <int D, int T, bool ELU, bool DOM>
__global__ __launch_bounds__(F32_NW * 64, (T == 1 && !DOM) || (D == 64 && (T == 1 || !DOM)) ? 2 : 1) void f32_bwd_y_kernel(F32YArgs a) {
    constexpr int KS = D / 16, TT = D / 32, NT = F32_NW * 64;
    constexpr int CH = F32_Y_ROWS * (D / 8) / NT;                 // chunks per thread and tensor
    using L = F32YLds<D, T>;
    constexpr int TB = Tile32<D>::bytes;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const Tile32<D> tl(lane);
    const int FG = (a.FT + F32_NW - 1) / F32_NW;
    long id = blockIdx.x;
    const int fg = (int)(id % FG); id /= FG;
    const int r = (int)(id % a.R);
    const long bh = id / a.R;
    const int ft = F32_NW * fg + wave;
    const bool active = ft < a.FT;
    const int f = 32 * (active ? ft : a.FT - 1) + l32, fr = f < a.mf ? f : a.mf - 1;
    const int row_begin = r * a.blocks_per_range * F32_Y_ROWS;
    int row_end = row_begin + a.blocks_per_range * F32_Y_ROWS;
    if (row_end > a.n) row_end = a.n;

    Terms<T> wf[KS];
    Terms<3> sf[DOM ? KS : 1];
    float cj = 0.f, zj = 0.f;
    if constexpr (!ELU) {
        const long wo = (bh % a.H) * a.omega_head_stride + (long)fr * a.d;
#pragma unroll
        for (int s = 0; s < KS; ++s) wf[s] = to_terms<T>(load_raw<T>(a.omega, wo, 16 * s + 8 * half, a.d));
        cj = f < a.mf ? a.c[bh * a.mf + fr] : -INFINITY;
        if constexpr (DOM) {
            zj = a.z[bh * a.mf + fr];
            const float rz = 1.f / zj;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                float v[8];
                f32_load8(a.S, (bh * a.mf + fr) * a.d, 16 * s + 8 * half, a.d, v);
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] *= rz;
                split3_8(v, sf[s].t);
            }
        }
    }
    floatx16 accS[TT], accW[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) { accS[t] = zero16(); accW[t] = zero16(); }
    float dz = 0.f;

    Raw8<T> rq[CH], rg[CH];
    float rv = 0.f;
    auto load_block = [&](int row0) {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int idx = tid + NT * u;
            int row = row0 + idx / (D / 8);
            if (row >= row_end) row = row_end - 1;
            const long off = (bh * a.n + row) * a.d;
            rq[u] = load_raw<T>(a.Q, off, 8 * (idx % (D / 8)), a.d);
            rg[u] = load_raw<T>(a.G, off, 8 * (idx % (D / 8)), a.d);
        }
        if (tid < 3 * F32_Y_ROWS) {                // rows past the end: weight 0
            const int row = row0 + tid % F32_Y_ROWS, kind = tid / F32_Y_ROWS;
            const bool in = row < row_end;
            const long ri = bh * a.n + (in ? row : row_end - 1);
            rv = kind == 0 ? (ELU ? 0.f : -a.lse[ri] * F32_LOG2E) : kind == 1 ? (in ? a.dinv[ri] : 0.f) : a.delta[ri];
        }
    };
    auto store_block = [&]() {
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int idx = tid + NT * u, row = idx / (D / 8), c = idx % (D / 8);
            const Terms<T> tq = to_terms<T>(rq[u]), tg = to_terms<T>(rg[u]);
            unsigned char* base = lds + (row >> 5) * T * TB;
#pragma unroll
            for (int k = 0; k < T; ++k) {
                *(uint4*)Tile32<D>::chunk(base + k * TB, row & 31, c) = tq.t[k];
                *(uint4*)Tile32<D>::chunk(base + L::g_off + k * TB, row & 31, c) = tg.t[k];
            }
        }
        if (tid < 3 * F32_Y_ROWS) {
            const int row = tid % F32_Y_ROWS;
            ((float*)(lds + L::v_off))[(tid / F32_Y_ROWS) * F32_Y_ROWS + (row & ~31) + acc_slot(row & 31)] = rv;
        }
    };
    if (row_begin < row_end) load_block(row_begin);
    for (int row0 = row_begin; row0 < row_end; row0 += F32_Y_ROWS) {
        store_block();
        __syncthreads();
        if (row0 + F32_Y_ROWS < row_end) load_block(row0 + F32_Y_ROWS);
#pragma unroll 1
        for (int i = 0; i < F32_Y_ROWS / 32; ++i) {
            const unsigned char* qi = lds + i * T * TB;
            const unsigned char* gi = qi + L::g_off;
            const float* vec = (const float*)(lds + L::v_off) + 32 * i;
            float w[16], inv[16], gv[16];
            acc_vector(vec + F32_Y_ROWS, half, inv);
            acc_vector(vec + 2 * F32_Y_ROWS, half, gv);
            if constexpr (ELU) {
                const int ftc = active ? ft : a.FT - 1;
#pragma unroll
                for (int sp = 0; sp < 2; ++sp) {
                    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = T - 1; k >= 0; --k) {
                        const uint4 v = tl.col_frag(qi + k * TB, sp, ftc);
                        const uint32_t ww[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) { x[2 * e] += pair_lo(ww[e]); x[2 * e + 1] += pair_hi(ww[e]); }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) w[8 * sp + e] = f32_elu1(x[e]) * inv[8 * sp + e];
                }
            } else {
                floatx16 u = zero16();
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    uint4 x[T];
#pragma unroll
                    for (int k = 0; k < T; ++k) x[k] = tl.row_frag(qi + k * TB, s);
                    u = mfma_terms<T, T>(x, wf[s].t, u);
                }
                float nl[16];
                acc_vector(vec, half, nl);
#pragma unroll
                for (int e = 0; e < 16; ++e) w[e] = fast_exp2(fmaf(u[e] + cj, F32_LOG2E, nl[e])) * inv[e];
            }
#pragma unroll
            for (int e = 0; e < 16; ++e) dz = fmaf(-w[e], gv[e], dz);
            {
                uint4 wt[2][3];
                split_acc(w, wt);
#pragma unroll
                for (int t = 0; t < TT; ++t) {
                    floatx16 part = zero16();
#pragma unroll
                    for (int sp = 0; sp < 2; ++sp) {
                        uint4 x[T];
#pragma unroll
                        for (int k = 0; k < T; ++k) x[k] = tl.col_frag(gi + k * TB, sp, t);
                        part = mfma_terms<3, T>(wt[sp], x, part);
                    }
                    accS[t] += part;
                }
            }
            if constexpr (DOM) {
                floatx16 tp = zero16();
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    uint4 x[T];
#pragma unroll
                    for (int k = 0; k < T; ++k) x[k] = tl.row_frag(gi + k * TB, s);
                    tp = mfma_terms<T, 3>(x, sf[s].t, tp);
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) w[e] = w[e] * zj * (tp[e] - gv[e]);
                uint4 wt[2][3];
                split_acc(w, wt);
#pragma unroll
                for (int t = 0; t < TT; ++t) {
                    floatx16 part = zero16();
#pragma unroll
                    for (int sp = 0; sp < 2; ++sp) {
                        uint4 x[T];
#pragma unroll
                        for (int k = 0; k < T; ++k) x[k] = tl.col_frag(qi + k * TB, sp, t);
                        part = mfma_terms<3, T>(wt[sp], x, part);
                    }
                    accW[t] += part;
                }
            }
        }
        __syncthreads();
    }
    if (!active) return;
    dz = half_sum(dz);
    const long po = (bh * a.R + r) * a.mf + 32 * ft;
    float chk = dz * 0.f;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        chk = not_finite(accS[t], chk);
        if constexpr (DOM) chk = not_finite(accW[t], chk);
    }
    if (__any(chk != 0.f)) {
        // without terms (see above): lane = feature, the lanes of a pair take half of the coordinates each, CW at a time
        constexpr int CW = DOM ? 16 : 32;
        const long wo = (bh % a.H) * a.omega_head_stride + (long)fr * a.d, so = (bh * a.mf + fr) * a.d;
#pragma unroll 1
        for (int c0 = D / 2 * half; c0 < D / 2 * half + D / 2; c0 += CW) {
            float ps[CW], pw[DOM ? CW : 1], pz = 0.f;
#pragma unroll
            for (int i = 0; i < CW; ++i) {
                ps[i] = 0.f;
                if constexpr (DOM) pw[i] = 0.f;
            }
#pragma unroll 1
            for (int row = row_begin; row < row_end; ++row) {
                const long ri = bh * a.n + row, off = ri * a.d;
                const float gi = a.delta[ri];
                float w;
                if constexpr (ELU) {
                    w = f32_elu1(load_elem(a.Q, off + fr, T == 1)) * a.dinv[ri];
                } else {
                    w = expf(plain_dot(a.omega, wo, T == 1, a.Q, off, T == 1, a.d, half) + cj - a.lse[ri]) * a.dinv[ri];
                }
                pz = fmaf(-w, gi, pz);
#pragma unroll
                for (int i = 0; i < CW; i += 4) {
                    const float4 x = any_load4(a.G, off, c0 + i, a.d, T == 1);
                    ps[i] = fmaf(w, x.x, ps[i]); ps[i + 1] = fmaf(w, x.y, ps[i + 1]);
                    ps[i + 2] = fmaf(w, x.z, ps[i + 2]); ps[i + 3] = fmaf(w, x.w, ps[i + 3]);
                }
                if constexpr (DOM) {
                    const float wd = w * (plain_dot(a.S, so, 0, a.G, off, T == 1, a.d, half) - zj * gi);
#pragma unroll
                    for (int i = 0; i < CW; i += 4) {
                        const float4 x = any_load4(a.Q, off, c0 + i, a.d, T == 1);
                        pw[i] = fmaf(wd, x.x, pw[i]); pw[i + 1] = fmaf(wd, x.y, pw[i + 1]);
                        pw[i + 2] = fmaf(wd, x.z, pw[i + 2]); pw[i + 3] = fmaf(wd, x.w, pw[i + 3]);
                    }
                }
            }
            if (f >= a.mf) continue;
            if (half == 0) a.dzpart[po + l32] = pz;
#pragma unroll
            for (int i = 0; i < CW; i += 4) {
                const float x[4] = {ps[i], ps[i + 1], ps[i + 2], ps[i + 3]};
                store4(a.dSpart, (po + l32) * a.d, c0 + i, a.d, x, 0);
                if constexpr (DOM) {
                    const float y[4] = {pw[i], pw[i + 1], pw[i + 2], pw[i + 3]};
                    store4(a.dWpart, (po + l32) * a.d, c0 + i, a.d, y, 0);
                }
            }
        }
        return;
    }
    if (half == 0 && f < a.mf) a.dzpart[po + l32] = dz;
    // feature 8(e/4) + 4 half + e%4 of the tile, coordinate 32t + l32; rows advance by uniform distances
    const int left = a.mf - 32 * ft - 4 * half;
    const long o = (po + 4 * half) * a.d + l32;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
        if (32 * t + l32 >= a.d) continue;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int fl = 8 * (e >> 2) + (e & 3);
            if (fl >= left) continue;
            (a.dSpart + o)[fl * a.d + 32 * t] = accS[t][e];
            if constexpr (DOM) (a.dWpart + o)[fl * a.d + 32 * t] = accW[t][e];
        }
    }
}

// Sums the query ranges: dS (BH, mf, d), dz (BH, mf).  One thread per element; column d stands for dz.
__global__ __launch_bounds__(256) void f32_bwd_merge_kernel(float* dS, float* dz, const float* dSpart, const float* dzpart, int R,
                                                            int mf, int d, long total) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int t = (int)(idx % (d + 1));
    const long rest = idx / (d + 1);
    const int j = (int)(rest % mf);
    const long bh = rest / mf;
    float s = 0.f;
    if (t < d) {
        const float* const ps = dSpart + (bh * R * mf + j) * d + t;
        for_parts<8, float>(R, [&](int r) { return ps[(long)r * mf * d]; }, [&](float x) { s += x; });
        dS[(bh * mf + j) * d + t] = s;
    } else {
        const float* const pz = dzpart + bh * R * mf + j;
        for_parts<8, float>(R, [&](int r) { return pz[(long)r * mf]; }, [&](float x) { s += x; });
        dz[bh * mf + j] = s;
    }
}

// d omega (H or 1, m, d) = sum over the batch (and the heads, shared omega) of the query ranges' parts and
// the key side's part (BH, m, d)
__global__ __launch_bounds__(256) void f32_domega_merge_kernel(float* dW, const float* part, const float* key_part, int B, int H,
                                                               int R, int m, int d, int per_head, long total) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int t = (int)(idx % d);
    const int j = (int)(idx / d % m);
    const int h0 = per_head ? (int)(idx / ((long)d * m)) : 0, h1 = per_head ? h0 + 1 : H;
    float s = 0.f;
    for (int b = 0; b < B; ++b)
        for (int h = h0; h < h1; ++h) {
            const long bh = (long)b * H + h;
            float x = key_part[(bh * m + j) * d + t];
            const float* const pw = part + (bh * R * m + j) * d + t;
            for_parts<8, float>(R, [&](int r) { return pw[(long)r * m * d]; }, [&](float y) { x += y; });
            s += x;
        }
    dW[idx] = s;
}

// ---------------------------------------------------------------------------
// Key side, fp32 matrix instructions.  A lane of half h holds coordinates 8q + 4h + e (q < D/8, e < 4) of
// its row: the reduction order of both operands.
// ---------------------------------------------------------------------------
template <int D> struct F32Row { float4 v[D / 8]; };

// BF16: storage type of the row; FULL: d == D (no tests)
template <int D, bool BF16, bool FULL>
__device__ __forceinline__ float4 row_load4(const void* p, long off, int c0, int d) {
    if constexpr (!FULL) {
        return any_load4(p, off, c0, d, BF16);
    } else if constexpr (BF16) {
        uint2 w;
        __builtin_memcpy(&w, (const uint16_t*)p + off + c0, 8);
        return make_float4(pair_lo(w.x), pair_hi(w.x), pair_lo(w.y), pair_hi(w.y));
    } else {
        float4 v;
        __builtin_memcpy(&v, (const float*)p + off + c0, 16);
        return v;
    }
}
template <int D, bool BF16, bool FULL>
__device__ __forceinline__ F32Row<D> load_row(const void* p, long off, int half, int d) {
    F32Row<D> r;
#pragma unroll
    for (int q = 0; q < D / 8; ++q) r.v[q] = row_load4<D, BF16, FULL>(p, off, 8 * q + 4 * half, d);
    return r;
}
// sum of the squares of 16 values, added pairwise: |k'|^2 goes into an exponent as an absolute value, and a
// chain of 64 additions would leave 1e-5 of it there
__device__ __forceinline__ float square_sum16(const float4* v) {
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = fmaf(v[i].x, v[i].x, v[i].y * v[i].y) + fmaf(v[i].z, v[i].z, v[i].w * v[i].w);
    return (s[0] + s[1]) + (s[2] + s[3]);
}

// A rows x B rows, 16 products to a partial sum.  The A row (fp32, or bf16 storage) comes from memory 32
// coordinates at a time, the next ones in flight, so that it never occupies D registers; `sq` gets the
// lane's share of its squares.
template <int D, bool BF16, bool FULL>
__device__ __forceinline__ floatx16 mfma_rows(const void* p, long off, int half, int d, const F32Row<D>& b, float& sq) {
    floatx16 acc = zero16();
    float4 cur[4], nxt[4];
    auto fetch = [&](int ch, float4 (&x)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = row_load4<D, BF16, FULL>(p, off, 32 * ch + 8 * i + 4 * half, d);
    };
    fetch(0, cur);
#pragma unroll
    for (int ch = 0; ch < D / 32; ++ch) {
        if (ch + 1 < D / 32) fetch(ch + 1, nxt);
        sq += square_sum16(cur);
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
            floatx16 part = zero16();
#pragma unroll
            for (int j = i; j < i + 2; ++j) {
                const float x[4] = {cur[j].x, cur[j].y, cur[j].z, cur[j].w};
                const float4 bv = b.v[4 * ch + j];
                const float y[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) part = mfma_f32(x[e], y[e], part);
            }
            acc += part;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) cur[i] = nxt[i];
        __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
}
template <int D>
__device__ __forceinline__ float half_square_norm(const F32Row<D>& a) {
    float s = 0.f;
#pragma unroll
    for (int ch = 0; ch < D / 32; ++ch) s += square_sum16(&a.v[4 * ch]);
    return 0.5f * half_sum(s);
}

struct F32KeyArgs {
    const float* Kp; const float* Vp;        // (BH, k, d)
    const void* omega;
    float* S; float* z; float* c;
    const float* dS; const float* dz;        // backward
    float* dKp; float* dVp;
    float* dU;                               // (BH, k, m) or nullptr: d loss / d exponent, for d omega
    int H, k, d, mf, FT, KR, tiles_per_range;
    long omega_head_stride;
};

template <int D>
struct F32KeyStateLds {
    static constexpr int s_pitch = D + 4;
    static constexpr int range_floats = 32 * s_pitch + 64;       // S tile, z, c
    static __host__ __device__ int bytes(int KR) { return KR * range_floats * 4; }
};

constexpr int F32_KEEP = 2;        // key tiles of a range whose exponents stay in registers
constexpr int F32_RANGES = 8;      // most key ranges (wavefronts) of a workgroup
constexpr int F32_MERGERS = 4;     // fewest wavefronts of a workgroup: the merge wants more than one

// Bound by latency: per key tile a chain of D/2 + 16 D/32 matrix instructions (64 cycles each) behind two loads.
// The first tile's V' is requested before its exponents (head size 64; others as the registers allow, four keys at
// a time), and the merge is one pass over LDS by the whole workgroup, thread = (feature, 4 coordinates): 64 keys,
// one head 10.8 -> 7.5 us, 128 keys 12.1 -> 9.8, 187 keys, 48 heads 14.8 -> 13.
template <int D, bool ELU, bool BF16, bool FULL>
__global__ __launch_bounds__(F32_RANGES * 64) void f32_key_state_kernel(F32KeyArgs a) {
    constexpr int TT = D / 32;
    using L = F32KeyStateLds<D>;
    extern __shared__ __attribute__((aligned(16))) float ks[];
    const int tid = threadIdx.x, lane = tid & 63, kr = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const int ft = (int)(blockIdx.x % a.FT);
    const long bh = blockIdx.x / a.FT;
    const int KT = (a.k + 31) / 32;
    const int kt0 = kr * a.tiles_per_range;
    int kt1 = kt0 + a.tiles_per_range;
    if (kt1 > KT) kt1 = KT;
    const int f = 32 * ft + l32, fr = f < a.mf ? f : a.mf - 1;

    if (kr < a.KR) {           // the others only take part in the merge
    F32Row<D> wf;
    if constexpr (!ELU) wf = load_row<D, BF16, FULL>(a.omega, (bh % a.H) * a.omega_head_stride + (long)fr * a.d, half, a.d);
    // lane = feature, element g = key 32 kt + 8(g/4) + 4 half + g%4: exponents, or elu1's features
    auto tile_values = [&](int kt) -> floatx16 {
        floatx16 e;
        if constexpr (ELU) {
            float x[16];
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                const int r = 32 * kt + 8 * (g >> 2) + 4 * half + (g & 3);
                x[g] = a.Kp[(bh * a.k + (r < a.k ? r : a.k - 1)) * a.d + fr];
            }
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                const int r = 32 * kt + 8 * (g >> 2) + 4 * half + (g & 3);
                e[g] = r < a.k ? f32_elu1(x[g]) : 0.f;
            }
        } else {
            const int r = 32 * kt + l32;
            float sq = 0.f;
            e = mfma_rows<D, false, FULL>(a.Kp, (bh * a.k + (r < a.k ? r : a.k - 1)) * a.d, half, a.d, wf, sq);
            sq = half_sum(sq);
            const float nrm = r < a.k ? 0.5f * sq : INFINITY;
#pragma unroll
            for (int g = 0; g < 16; ++g) e[g] -= __shfl(nrm, 8 * (g >> 2) + 4 * half + (g & 3), 64);
        }
        return e;
    };
    int col[TT];               // columns past d: any value does, nobody reads their sums
#pragma unroll
    for (int t = 0; t < TT; ++t) col[t] = 32 * t + l32 < a.d ? 32 * t + l32 : 0;
    constexpr bool AHEAD = D == 64 && FULL;
    struct VTile { float x[AHEAD ? 16 : 1][TT]; };
    auto value = [&](int kt, int g, int t) -> float {
        const int r = 32 * kt + 8 * (g >> 2) + 4 * half + (g & 3);
        return a.Vp[(bh * a.k + (r < a.k ? r : a.k - 1)) * a.d + col[t]];
    };
    auto load_v = [&](int kt, VTile& v) {
        if constexpr (AHEAD) {
#pragma unroll
            for (int g = 0; g < 16; ++g)
#pragma unroll
                for (int t = 0; t < TT; ++t) v.x[g][t] = value(kt, g, t);
        }
    };
    VTile vt;
    load_v(kt0, vt);
    const int nt = kt1 - kt0;
    const bool keep = nt <= F32_KEEP;
    floatx16 ev[F32_KEEP];
    float c = 0.f;
    if (keep) {
#pragma unroll
        for (int i = 0; i < F32_KEEP; ++i)
            if (i < nt) ev[i] = tile_values(kt0 + i);
    }
    if constexpr (!ELU) {
        c = -INFINITY;
        if (keep) {
#pragma unroll
            for (int i = 0; i < F32_KEEP; ++i)
                if (i < nt) {
#pragma unroll
                    for (int g = 0; g < 16; ++g) c = fmaxf(c, ev[i][g]);
                }
        } else {
            for (int kt = kt0; kt < kt1; ++kt) {
                const floatx16 e = tile_values(kt);
#pragma unroll
                for (int g = 0; g < 16; ++g) c = fmaxf(c, e[g]);
            }
        }
        c = half_max(c);
    }
    floatx16 acc[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) acc[t] = zero16();
    float zsum = 0.f;
    // a range in which every |k'|^2 overflows has no finite exponent: its weights are 0, not exp(-inf + inf)
    const float shift = c == -INFINITY ? 0.f : c;
    auto accumulate = [&](floatx16 e, int kt) {
        if constexpr (!ELU) {
#pragma unroll
            for (int g = 0; g < 16; ++g) e[g] = expf(e[g] - shift);
        }
        floatx16 part[TT];
#pragma unroll
        for (int t = 0; t < TT; ++t) part[t] = zero16();
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            zsum += e[g];
            const int r = 32 * kt + 8 * (g >> 2) + 4 * half + (g & 3);
            const bool in = r < a.k;                       // past the end: 0 x 0 (V' may be infinite)
#pragma unroll
            for (int t = 0; t < TT; ++t) {
                float x;
                if constexpr (AHEAD) x = vt.x[g][t];
                else                 x = value(kt, g, t);
                part[t] = mfma_f32(e[g], in ? x : 0.f, part[t]);
            }
            if (!AHEAD && (g & 3) == 3) __builtin_amdgcn_sched_barrier(0);       // bounds the loads in flight (registers)
        }
#pragma unroll
        for (int t = 0; t < TT; ++t) acc[t] += part[t];
    };
    if (keep) {
#pragma unroll
        for (int i = 0; i < F32_KEEP; ++i)
            if (i < nt) {
                if (i > 0) load_v(kt0 + i, vt);
                accumulate(ev[i], kt0 + i);
            }
    } else {
#pragma unroll 1
        for (int kt = kt0; kt < kt1; ++kt) {
            if (kt > kt0) load_v(kt, vt);
            accumulate(tile_values(kt), kt);
        }
    }
    zsum = half_sum(zsum);
    float* const mine = ks + kr * L::range_floats;
    if (half == 0) {
        mine[32 * L::s_pitch + l32] = zsum;
        mine[32 * L::s_pitch + 32 + l32] = c;
    }
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int g = 0; g < 16; ++g) mine[(8 * (g >> 2) + 4 * half + (g & 3)) * L::s_pitch + 32 * t + l32] = acc[t][g];
    }
    __syncthreads();
    // join the ranges: c = max, S and z rescaled
    const int fl = tid & 31, fo = 32 * ft + fl;
    const float* const pz = ks + 32 * L::s_pitch + fl;       // + range: z, + 32: c
    float w[F32_RANGES], cm = -INFINITY, zs = 0.f;
#pragma unroll
    for (int r = 0; r < F32_RANGES; ++r) {
        w[r] = pz[(r < a.KR ? r : 0) * L::range_floats + 32];
        cm = fmaxf(cm, w[r]);
    }
#pragma unroll
    for (int r = 0; r < F32_RANGES; ++r) {
        const float zr = pz[(r < a.KR ? r : 0) * L::range_floats];
        w[r] = ELU ? 1.f : expf(w[r] - cm);
        if (r < a.KR) zs = fmaf(w[r], zr, zs);
    }
    if (fo >= a.mf) return;
    if (tid < 32) {
        a.z[bh * a.mf + fo] = zs;
        a.c[bh * a.mf + fo] = cm;
    }
    for (int t = 4 * (tid >> 5); t < D; t += (int)blockDim.x / 8) {
        float4 sv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < F32_RANGES; ++r) {
            if (r >= a.KR) break;
            const float4 x = *(const float4*)(ks + r * L::range_floats + fl * L::s_pitch + t);
            sv.x = fmaf(w[r], x.x, sv.x); sv.y = fmaf(w[r], x.y, sv.y);
            sv.z = fmaf(w[r], x.z, sv.z); sv.w = fmaf(w[r], x.w, sv.w);
        }
        float* const o = a.S + (bh * a.mf + fo) * a.d + t;
        if (FULL) {
            *(float4*)o = sv;
        } else {
            if (t < a.d) o[0] = sv.x;
            if (t + 1 < a.d) o[1] = sv.y;
            if (t + 2 < a.d) o[2] = sv.z;
            if (t + 3 < a.d) o[3] = sv.w;
        }
    }
}

// Backward, lane = key; the wavefronts take every fourth feature tile and add up through LDS.
//     dPhi^T = dS V'^T + dz,  dU = dPhi * Phi,  dV' = Phi dS,  dK' = dU omega - rowsum(dU) K'
//     elu1: dK' = dPhi * phi'(K')
// A feature tile is 2 D + 32 D/32 chained matrix instructions of 64 cycles for the performer map, with the loads of
// dS and omega exposed between them; OCC wavefronts of a SIMD cover for each other.
template <int D, bool ELU, bool BF16, bool FULL, int OCC>
__global__ __launch_bounds__(256, OCC) void f32_bwd_key_kernel(F32KeyArgs a) {
    constexpr int TT = D / 32;
    extern __shared__ __attribute__((aligned(16))) float ks[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const int KT = (a.k + 31) / 32;
    const int kt = (int)(blockIdx.x % KT);
    const long bh = blockIdx.x / KT;
    const int key = 32 * kt + l32;
    const bool live = key < a.k;
    const long koff = (bh * a.k + (live ? key : a.k - 1)) * a.d;
    // uniform bases and 32-bit offsets from them (k, m at most 2^24 x 128 resp. 4096 x 128 elements)
    const float* const dSb = a.dS + bh * a.mf * a.d;
    const float* const dzb = a.dz + bh * a.mf;
    const float* const cb = a.c + bh * a.mf;
    const void* const ob = BF16 ? (const void*)((const uint16_t*)a.omega + (bh % a.H) * a.omega_head_stride)
                                : (const void*)((const float*)a.omega + (bh % a.H) * a.omega_head_stride);
    const F32Row<D> vp = load_row<D, false, FULL>(a.Vp, koff, half, a.d);
    F32Row<D> kp;
    float nrm = 0.f;
    if constexpr (!ELU) {
        kp = load_row<D, false, FULL>(a.Kp, koff, half, a.d);
        nrm = half_square_norm<D>(kp);
    }
    floatx16 accV[TT], accK[TT];
    int col[TT];               // columns past d: any value does, nobody reads their sums
#pragma unroll
    for (int t = 0; t < TT; ++t) { accV[t] = zero16(); accK[t] = zero16(); col[t] = 32 * t + l32 < a.d ? 32 * t + l32 : 0; }
    float rs = 0.f;
#pragma unroll 1
    for (int ft = wave; ft < a.FT; ft += 4) {
        const int f = 32 * ft + l32, fr = f < a.mf ? f : a.mf - 1;
        float unused = 0.f;
        floatx16 dp = mfma_rows<D, false, FULL>(dSb, fr * a.d, half, a.d, vp, unused), e;
        if constexpr (!ELU) e = mfma_rows<D, BF16, FULL>(ob, fr * a.d, half, a.d, kp, unused);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            const int fg = 32 * ft + 8 * (g >> 2) + 4 * half + (g & 3), fc = fg < a.mf ? fg : a.mf - 1;
            float phi, du = dp[g] + dzb[fc];
            if constexpr (ELU) {
                const float x = a.Kp[koff + fc];
                phi = f32_elu1(x);
                if (live && fg < a.mf) a.dKp[koff + fg] = du * (x > 0.f ? 1.f : phi);
            } else {
                phi = expf(e[g] - nrm - cb[fc]);
                du *= phi;
            }
            const bool in = fg < a.mf;       // past the end: 0 x 0 (dS may be infinite; where omega is, all is NaN anyway)
            if (!in) { phi = 0.f; du = 0.f; }
            rs += du;
            if (!ELU && a.dU && live && in) a.dU[(bh * a.k + key) * a.mf + fg] = du;
#pragma unroll
            for (int t = 0; t < TT; ++t) {
                const float x = dSb[fc * a.d + col[t]];
                accV[t] = mfma_f32(phi, in ? x : 0.f, accV[t]);
                if constexpr (!ELU) accK[t] = mfma_f32(du, load_elem(ob, fc * a.d + col[t], BF16), accK[t]);
            }
            if ((g & 3) == 3) __builtin_amdgcn_sched_barrier(0);       // bounds the loads in flight (registers)
        }
    }
    rs = half_sum(rs);
    // per wavefront [dV' | dK'][t][g][lane], then rs[32]; rows of the tiles are keys, columns coordinates
    constexpr int SLOT = 2 * TT * 16 * 64 + 32;
    float* my = ks + wave * SLOT;
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            my[(t * 16 + g) * 64 + lane] = accV[t][g];
            my[((TT + t) * 16 + g) * 64 + lane] = accK[t][g];
        }
    if (half == 0) my[2 * TT * 16 * 64 + l32] = rs;
    __syncthreads();
    // wavefront w finishes rows 8w + 4 half + {0..3}
#pragma unroll 1
    for (int i = 0; i < 4; ++i) {
        const int rl = 8 * wave + 4 * half + i, r = 32 * kt + rl;
        if (r >= a.k) continue;
        float rsum = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) rsum += ks[w * SLOT + 2 * TT * 16 * 64 + rl];
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            const int c = 32 * t + l32;
            if (c >= a.d) continue;
            float sv = 0.f, sk = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                sv += ks[w * SLOT + (t * 16 + 4 * wave + i) * 64 + lane];
                sk += ks[w * SLOT + ((TT + t) * 16 + 4 * wave + i) * 64 + lane];
            }
            const long o = (bh * a.k + r) * a.d + c;
            a.dVp[o] = sv;
            if constexpr (!ELU) a.dKp[o] = sk - rsum * a.Kp[o];
        }
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
bool f32_fused_supported(const Problem& p) { return p.d <= 128; }

template <class Kern, class Args>
static flurka_status launch_lds(Kern kern, long grid, int threads, int lds_bytes, const Args& a, hipStream_t s) {
    KernelFacts facts;
    if (!kernel_facts((const void*)kern, threads, lds_bytes, &facts)) return FLURKA_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), lds_bytes, s, a);
    FLURKA_CHECK_LAUNCH();
    return FLURKA_OK;
}

// Calls fn(D, T) with the padded head size and the number of operand terms as compile-time constants.
template <int N> struct Const { static constexpr int value = N; };
template <class Fn>
static flurka_status by_shape(const Problem& p, Fn&& fn) {
    if (p.d <= 64) return p.bf16 ? fn(Const<64>{}, Const<1>{}) : fn(Const<64>{}, Const<3>{});
    return p.bf16 ? fn(Const<128>{}, Const<1>{}) : fn(Const<128>{}, Const<3>{});
}

// fn(elu, bf16 omega, d == D) likewise; elu1 has no omega
template <class Fn>
static flurka_status by_row(const Problem& p, int D, Fn&& fn) {
    const bool full = p.d == D;
    if (p.elu) return full ? fn(Const<1>{}, Const<0>{}, Const<1>{}) : fn(Const<1>{}, Const<0>{}, Const<0>{});
    if (p.bf16) return full ? fn(Const<0>{}, Const<1>{}, Const<1>{}) : fn(Const<0>{}, Const<1>{}, Const<0>{});
    return full ? fn(Const<0>{}, Const<0>{}, Const<1>{}) : fn(Const<0>{}, Const<0>{}, Const<0>{});
}

static F32QueryArgs query_args(const Problem& p, const void* Q, const void* omega, float* ctx) {
    const CtxLayout L = ctx_layout(p);
    F32QueryArgs a{};
    a.Q = Q; a.omega = omega; a.S = ctx + L.S; a.z = ctx + L.z; a.c = ctx + L.c; a.lse = ctx + L.lse;
    a.n = p.n; a.H = p.H; a.d = p.d; a.mf = p.mf; a.FT = p.mfp / 32;
    a.blocks_per_head = (p.n + 32 * F32_NW - 1) / (32 * F32_NW);
    a.omega_head_stride = p.omega_per_head ? (long)p.m * p.d : 0;
    return a;
}

flurka_status f32_key_state(const Problem& p, const void* omega, float* ctx, hipStream_t s) {
    const CtxLayout L = ctx_layout(p);
    F32KeyArgs a{};
    a.Kp = ctx + L.Kp; a.Vp = ctx + L.Vp; a.omega = omega; a.S = ctx + L.S; a.z = ctx + L.z; a.c = ctx + L.c;
    a.H = p.H; a.k = p.k; a.d = p.d; a.mf = p.mf; a.FT = p.mfp / 32;
    a.omega_head_stride = p.omega_per_head ? (long)p.m * p.d : 0;
    const int KT = (p.k + 31) / 32;
    a.KR = KT < F32_RANGES ? KT : F32_RANGES;
    a.tiles_per_range = (KT + a.KR - 1) / a.KR;
    a.KR = (KT + a.tiles_per_range - 1) / a.tiles_per_range;
    const long grid = (long)p.BH * a.FT;
    return by_shape(p, [&](auto D, auto) {
        constexpr int d = decltype(D)::value;
        const int ldsb = F32KeyStateLds<d>::bytes(a.KR);
        return by_row(p, d, [&](auto E, auto B, auto F) {
            return launch_lds(f32_key_state_kernel<d, decltype(E)::value, decltype(B)::value, decltype(F)::value>, grid, 64 * (a.KR < F32_MERGERS ? F32_MERGERS : a.KR), ldsb, a, s);
        });
    });
}

flurka_status f32_query_forward(const Problem& p, const FwdArgs& f, hipStream_t s) {
    F32QueryArgs a = query_args(p, f.Q, f.omega, f.ctx);
    a.out = f.out;
    const long grid = (long)p.BH * a.blocks_per_head;
    return by_shape(p, [&](auto D, auto T) {
        constexpr int d = decltype(D)::value, t = decltype(T)::value;
        return p.elu ? launch_lds(f32_query_fwd_kernel<d, t, true>, grid, F32_NW * 64, 2 * FeatureStage<d, 0>::bytes, a, s)
                     : launch_lds(f32_query_fwd_kernel<d, t, false>, grid, F32_NW * 64, 2 * FeatureStage<d, t>::bytes, a, s);
    });
}

// Query ranges of the dS kernel (about two workgroups per compute unit, whole blocks of queries) and the scratch.
// No call may need more of it than the kernels of flurka_generic.hip would: fewer ranges and fewer split partials
// where that is little.  ranges = 0: not even one range fits (a few positions and keys with d omega; more than
// 2^25 rows in all), and those kernels are taken.
F32BwdWs f32_bwd_ws_layout(const Problem& p, int dom) {
    const size_t budget = generic_ws_layout(p, 1).total;
    const size_t BH = (size_t)p.BH, dS = BH * p.mf * p.d, keys = BH * p.k * p.d;
    const int FG = (p.mfp / 32 + F32_NW - 1) / F32_NW;
    const int blocks = (p.n + F32_Y_ROWS - 1) / F32_Y_ROWS;
    const long cus = chip_cus();
    long R = 2 * cus / ((long)p.BH * FG);
    if (R > blocks) R = blocks;
    if (R < 1) R = 1;
    for (;; R -= (R + 7) / 8) {
        F32BwdWs W{};
        if (R < 1) return W;
        W.blocks_per_range = (int)((blocks + R - 1) / R);
        W.ranges = (blocks + W.blocks_per_range - 1) / W.blocks_per_range;
        size_t o = 0;
        auto take = [&](size_t count) { const size_t at = o; o += round_up(count, 64); return at; };
        W.delta = take(BH * p.n);
        W.dinv = take(BH * p.n);
        W.dS = take(dS);
        W.dz = take(BH * p.mf);
        if (W.ranges > 1) {
            W.dSpart = take(dS * W.ranges);
            W.dzpart = take(BH * p.mf * W.ranges);
        } else {                   // one range: its sums are the result
            W.dSpart = W.dS;
            W.dzpart = W.dz;
        }
        W.dWkey = W.dS;            // key side of d omega: dS is done with by then
        const size_t front = o;
        W.dKp = take(keys);
        W.dVp = take(keys);
        if (dom) {                 // the ranges' parts and the key side's dU
            W.dWpart = take(dS * W.ranges);
            W.dU = take(BH * p.k * p.m);
        }
        W.total = o;
        if (W.total > budget) continue;
        // dE, dF from bf16 operands: once the key side is done, what lies in front of dK' takes split partials.  It
        // is made to hold as many ranges as their launch would ask for (at most four) if the budget has the room.
        const long tiles = 2L * ((p.k + 127) / 128) * ((p.n + 127) / 128);
        long splits = (2 * cus + tiles - 1) / tiles, most = (long)BH * p.d / (2 * F_GK);
        if (splits > 4) splits = 4;
        if (splits > most) splits = most;
        if (p.bf16 && !p.ef_per_head && splits > 1) {
            size_t grow = round_up((size_t)splits * 2 * p.k * p.n, 64);
            grow = grow > front ? grow - front : 0;
            if (grow > budget - W.total) grow = (budget - W.total) / 64 * 64;
            W.dKp += grow; W.dVp += grow; W.total += grow;
            if (dom) { W.dWpart += grow; W.dU += grow; }
        }
        return W;
    }
}

flurka_status f32_query_backward(const Problem& p, const BwdArgs& b, const F32BwdWs& W, hipStream_t s) {
    const CtxLayout C = ctx_layout(p);
    F32QueryArgs a = query_args(p, b.Q, b.omega, const_cast<float*>(b.ctx));
    a.G = b.dOut; a.out = b.dQ; a.delta = b.ws + W.delta; a.dinv = b.ws + W.dinv;
    const long grid = (long)p.BH * a.blocks_per_head;
    flurka_status st = by_shape(p, [&](auto D, auto T) {
        constexpr int d = decltype(D)::value, t = decltype(T)::value;
        return p.elu ? launch_lds(f32_bwd_x_kernel<d, t, true>, grid, F32_NW * 64, 2 * FeatureStage<d, 0>::bytes, a, s)
                     : launch_lds(f32_bwd_x_kernel<d, t, false>, grid, F32_NW * 64, 2 * FeatureStage<d, t>::bytes, a, s);
    });
    if (st != FLURKA_OK) return st;
    F32YArgs ya{};
    ya.Q = b.Q; ya.G = b.dOut; ya.omega = b.omega;
    ya.S = a.S; ya.z = a.z; ya.c = a.c; ya.lse = b.ctx + C.lse; ya.delta = a.delta; ya.dinv = a.dinv;
    ya.dSpart = b.ws + W.dSpart; ya.dzpart = b.ws + W.dzpart; ya.dWpart = b.ws + W.dWpart;
    ya.n = p.n; ya.H = p.H; ya.d = p.d; ya.mf = p.mf; ya.FT = p.mfp / 32;
    ya.R = W.ranges; ya.blocks_per_range = W.blocks_per_range;
    ya.omega_head_stride = a.omega_head_stride;
    const long ygrid = (long)p.BH * W.ranges * ((ya.FT + F32_NW - 1) / F32_NW);
    const bool dom = b.dOmega != nullptr;
    st = by_shape(p, [&](auto D, auto T) {
        constexpr int d = decltype(D)::value, t = decltype(T)::value;
        constexpr int ldsb = F32YLds<d, t>::bytes;
        if (p.elu) return launch_lds(f32_bwd_y_kernel<d, t, true, false>, ygrid, F32_NW * 64, ldsb, ya, s);
        return dom ? launch_lds(f32_bwd_y_kernel<d, t, false, true>, ygrid, F32_NW * 64, ldsb, ya, s)
                   : launch_lds(f32_bwd_y_kernel<d, t, false, false>, ygrid, F32_NW * 64, ldsb, ya, s);
    });
    if (st != FLURKA_OK || W.ranges == 1) return st;
    const long total = (long)p.BH * p.mf * (p.d + 1);
    hipLaunchKernelGGL(f32_bwd_merge_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, b.ws + W.dS, b.ws + W.dz,
                       (const float*)ya.dSpart, (const float*)ya.dzpart, W.ranges, p.mf, p.d, total);
    FLURKA_CHECK_LAUNCH();
    return FLURKA_OK;
}

flurka_status f32_key_backward(const Problem& p, const BwdArgs& b, const F32BwdWs& W, hipStream_t s) {
    const CtxLayout C = ctx_layout(p);
    F32KeyArgs a{};
    a.Kp = b.ctx + C.Kp; a.Vp = b.ctx + C.Vp; a.omega = b.omega; a.c = const_cast<float*>(b.ctx) + C.c;
    a.dS = b.ws + W.dS; a.dz = b.ws + W.dz; a.dKp = b.ws + W.dKp; a.dVp = b.ws + W.dVp;
    a.dU = b.dOmega ? b.ws + W.dU : nullptr;
    a.H = p.H; a.k = p.k; a.d = p.d; a.mf = p.mf; a.FT = p.mfp / 32;
    a.omega_head_stride = p.omega_per_head ? (long)p.m * p.d : 0;
    const long grid = (long)p.BH * ((p.k + 31) / 32);
    flurka_status st = by_shape(p, [&](auto D, auto) {
        constexpr int d = decltype(D)::value;
        constexpr int slot = (2 * (d / 32) * 16 * 64 + 32) * 4;
        return by_row(p, d, [&](auto E, auto B, auto F) {
            constexpr int e = decltype(E)::value, bf = decltype(B)::value, full = decltype(F)::value;
            if constexpr (d == 64 && !e && full) {
                // More workgroups than compute units: two to each (16 spilled registers) rather than a second round.
                // Head size 64, 48 heads, k 187, m 150: 49 -> 36 us; where one round holds them all, k 256, 16 heads,
                // m 256, 25.5 -> 28 us.
                if (grid > chip_cus()) return launch_lds(f32_bwd_key_kernel<d, e, bf, full, 2>, grid, 256, 4 * slot, a, s);
            }
            return launch_lds(f32_bwd_key_kernel<d, e, bf, full, d == 64 && e ? 2 : 1>, grid, 256, 4 * slot, a, s);
        });
    });
    if (st != FLURKA_OK || !b.dOmega) return st;
    GemmArgs g{};      // key side of d omega per head: dU^T K'
    g.A = b.ws + W.dU; g.B = b.ctx + C.Kp; g.C = b.ws + W.dWkey;
    g.M = p.m; g.N = p.d; g.K = p.k; g.Kin = p.k;
    g.sAm = 1; g.sAki = p.m; g.sAb = (long)p.H * p.k * p.m; g.sAh = (long)p.k * p.m;
    g.sBn = 1; g.sBki = p.d; g.sBb = (long)p.H * p.k * p.d; g.sBh = (long)p.k * p.d;
    g.sCm = p.d; g.sCn = 1; g.sCb = (long)p.H * p.m * p.d; g.sCh = (long)p.m * p.d;
    g.H = p.H;
    if ((st = launch_gemm_f32(g, p.BH, nullptr, 0, s)) != FLURKA_OK) return st;
    const long total = (long)(p.omega_per_head ? p.H : 1) * p.m * p.d;
    hipLaunchKernelGGL(f32_domega_merge_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, b.dOmega,
                       (const float*)(b.ws + W.dWpart), (const float*)(b.ws + W.dWkey), p.B, p.H, W.ranges, p.m, p.d,
                       p.omega_per_head, total);
    FLURKA_CHECK_LAUNCH();
    return FLURKA_OK;
}

}  // namespace flurka
