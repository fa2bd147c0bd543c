// Strided batched GEMM with fp32 operands, products and sums on the matrix cores of gfx950
// (v_mfma_f32_32x32x2_f32), for every contraction of the fp32-arithmetic path:
//     C[b,h] (M x N) (+)= A[b,h] (M x K) B[b,h] (K x N)
// Operands are addressed through element strides, so transposes, shared operands (batch stride 0) and a
// reduction index that runs over (outer, inner) pairs (K = Kout * Kin with separate strides) need no
// copies.  bf16 operands are widened to fp32 on their way into LDS; nothing is rounded.
#pragma once

#include "flurka_mfma.h"

namespace flurka {

struct GemmArgs {
    const void* A;
    const void* B;
    void* C;
    const void* A2;      // operands and result of a second GEMM of the same shape in the same launch
    const void* B2;      // (nullptr: none)
    void* C2;
    int M, N, K, Kin;
    long sAm, sAki, sAko, sAb, sAh;
    long sBn, sBki, sBko, sBb, sBh;
    long sCm, sCn, sCb, sCh;
    int H;
    int a_bf16, b_bf16, c_bf16;
    int accumulate;
    // filled in by launch_gemm_f32
    float* part;         // split partials [split][which][batch][M][N] (nullptr: the reduction is not split)
    int batches, steps_per_split;
};

// v_mfma_f32_32x32x2_f32, one wavefront: D(32x32) += A(32x2) B(2x32), all fp32.
// Operand layout, lane l: A row l%32, reduction slot l/32; B column l%32, slot l/32; D as for mfma32.
__device__ __forceinline__ floatx16 mfma_f32(float a, float b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

constexpr int F_GK = 32;                  // reduction step

// 4 consecutive elements starting at element i, as 16 bytes (fp32) or 8 bytes (bf16) that need no more
// than the element's own alignment
__device__ __forceinline__ uint4 ld4_raw(const void* p, long i, int bf16) {
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (bf16) __builtin_memcpy(&v, (const uint16_t*)p + i, 8);
    else      __builtin_memcpy(&v, (const float*)p + i, 16);
    return v;
}
__device__ __forceinline__ float4 raw_to_f32(const uint4& v, int bf16) {
    if (bf16) return make_float4(pair_lo(v.x), pair_hi(v.x), pair_lo(v.y), pair_hi(v.y));
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
// element e of a group, one at a time (edges of the operand)
__device__ __forceinline__ void raw_set(uint4& v, int e, uint32_t bits, int bf16) {
    uint32_t* w = &v.x;
    if (bf16) w[e >> 1] |= bits << (16 * (e & 1));
    else      w[e] = bits;
}
__device__ __forceinline__ uint32_t elem_bits(const void* p, long i, int bf16) {
    return bf16 ? (uint32_t)((const uint16_t*)p)[i] : ((const uint32_t*)p)[i];
}

// One operand tile of TR rows x 32 reduction slots.  KF: the reduction index is the contiguous one in
// memory; the tile is kept [row][slot] and fragments are read 16 bytes (4 slots) at a time.  Otherwise the
// rows are contiguous; the tile is kept [slot][row] and a fragment read is one dword per lane.  Either
// way a thread moves groups of 4 consecutive elements, and lane half h of the wavefront takes
// slots 8q + 4h + e (q, e = 0..3): the order of the slots is free as long as both operands agree.
// Pitches: 36 floats put 16 consecutive rows into 16 different groups of 4 banks; TR + 8 floats put the
// two halves' slots (4 rows of the tile apart) into different halves of the 64 banks.
template <bool KF, int TR>
struct F32Tile {
    static constexpr int pitch = KF ? F_GK + 4 : TR + 8;
    static constexpr int floats = KF ? TR * pitch : F_GK * pitch;
    static constexpr int groups = TR * F_GK / 4 / 256;       // per thread
    static __device__ __forceinline__ void place(int tid, int i, int& r, int& kk) {
        const int idx = tid + 256 * i;
        if (KF) { r = idx >> 3; kk = 4 * (idx & 7); }
        else    { kk = idx / (TR / 4); r = 4 * (idx % (TR / 4)); }
    }
    static __device__ __forceinline__ float* at(float* t, int r, int kk) { return KF ? t + r * pitch + kk : t + kk * pitch + r; }
};

// Tile TM x TN of C per workgroup of four wavefronts (2 x 2, each TM/2 x TN/2), 32-deep steps through one
// LDS buffer; the loads of the next step are in flight during the current one, and two or three
// workgroups share a compute unit.  A 32x32x2 fp32 MFMA takes 64 cycles and needs two dwords per lane, so
// LDS and issue slots are far from their limits: the kernel is bound by the fp32 matrix rate (the chip's
// 152 TFLOP/s measured on a large product) once there are enough tiles, by latency otherwise.  At
// 16 x (4096 x 256 x 64), fp32: 33 us = 65 TFLOP/s where the vector-unit kernel before it (64 x 64 x 16 tiles,
// one element per load) took 135 us.
// Every 16 products form a partial sum of their own that is then added to the running sum: the rounding
// error of a long reduction grows with K/16, not with K.
template <bool AKF, bool BKF, int TM, int TN>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
    using TA = F32Tile<AKF, TM>;
    using TB = F32Tile<BKF, TN>;
    __shared__ __attribute__((aligned(16))) float As[TA::floats];
    __shared__ __attribute__((aligned(16))) float Bs[TB::floats];
    constexpr int MT = TM / 64, NT = TN / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int wm = wave >> 1, wn = wave & 1;
    const int tiles_n = (g.N + TN - 1) / TN;
    const int m0 = (int)(blockIdx.x / tiles_n) * TM, n0 = (int)(blockIdx.x % tiles_n) * TN;
    const int which = (int)blockIdx.z / g.batches, bz = (int)blockIdx.z % g.batches;
    const int b = bz / g.H, h = bz % g.H;
    const void* const A = which ? g.A2 : g.A;
    const void* const B = which ? g.B2 : g.B;
    const long aoff = (long)b * g.sAb + (long)h * g.sAh;
    const long boff = (long)b * g.sBb + (long)h * g.sBh;
    const int k_begin = (int)blockIdx.y * g.steps_per_split * F_GK;
    int k_end = k_begin + g.steps_per_split * F_GK;
    if (k_end > g.K) k_end = g.K;
    const bool one_level = g.Kin >= g.K;
    // groups of 4 slots never straddle two outer indices, and the contiguous index has stride 1
    const bool a_vec = AKF ? (g.sAki == 1 && (one_level || g.Kin % 4 == 0)) : g.sAm == 1;
    const bool b_vec = BKF ? (g.sBki == 1 && (one_level || g.Kin % 4 == 0)) : g.sBn == 1;

    auto k_offset = [&](int k, long ski, long sko) -> long {
        if (one_level) return (long)k * ski;
        const int ko = k / g.Kin;
        return (long)ko * sko + (long)(k - ko * g.Kin) * ski;
    };
    auto load_group = [&](bool kf, const void* p, long off, int r, int k, int rmax, long sr, long ski, long sko, bool vec,
                          int bf16) -> uint4 {
        if (vec && (kf ? (r < rmax && k + 3 < k_end) : (r + 3 < rmax && k < k_end)))
            return ld4_raw(p, off + (long)r * sr + k_offset(k, ski, sko), bf16);
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int re = kf ? r : r + e, ke = kf ? k + e : k;
            if (re < rmax && ke < k_end) raw_set(v, e, elem_bits(p, off + (long)re * sr + k_offset(ke, ski, sko), bf16), bf16);
        }
        return v;
    };
    // Interior steps (every group of the tile exists and the step lies inside one outer index) take the
    // short way: fixed offsets per thread plus one uniform offset per step, no tests per group.
    const bool whole_steps = one_level || g.Kin % F_GK == 0;
    const bool a_short = a_vec && whole_steps && m0 + TM <= g.M, b_short = b_vec && whole_steps && n0 + TN <= g.N;
    long pa[TA::groups], pb[TB::groups];
#pragma unroll
    for (int i = 0; i < TA::groups; ++i) {
        int r, kk;
        TA::place(tid, i, r, kk);
        pa[i] = aoff + (long)(m0 + r) * g.sAm + (long)kk * g.sAki;
    }
#pragma unroll
    for (int i = 0; i < TB::groups; ++i) {
        int r, kk;
        TB::place(tid, i, r, kk);
        pb[i] = boff + (long)(n0 + r) * g.sBn + (long)kk * g.sBki;
    }
    uint4 ra[TA::groups], rb[TB::groups];
    auto fetch = [&](int k0) {
        const bool inside = k0 + F_GK <= k_end;
        if (inside && a_short) {
            const long ko = k_offset(k0, g.sAki, g.sAko);
            if (g.a_bf16) {
#pragma unroll
                for (int i = 0; i < TA::groups; ++i) ra[i] = ld4_raw(A, pa[i] + ko, 1);
            } else {
#pragma unroll
                for (int i = 0; i < TA::groups; ++i) ra[i] = ld4_raw(A, pa[i] + ko, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < TA::groups; ++i) {
                int r, kk;
                TA::place(tid, i, r, kk);
                ra[i] = load_group(AKF, A, aoff, m0 + r, k0 + kk, g.M, g.sAm, g.sAki, g.sAko, a_vec, g.a_bf16);
            }
        }
        if (inside && b_short) {
            const long ko = k_offset(k0, g.sBki, g.sBko);
            if (g.b_bf16) {
#pragma unroll
                for (int i = 0; i < TB::groups; ++i) rb[i] = ld4_raw(B, pb[i] + ko, 1);
            } else {
#pragma unroll
                for (int i = 0; i < TB::groups; ++i) rb[i] = ld4_raw(B, pb[i] + ko, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < TB::groups; ++i) {
                int r, kk;
                TB::place(tid, i, r, kk);
                rb[i] = load_group(BKF, B, boff, n0 + r, k0 + kk, g.N, g.sBn, g.sBki, g.sBko, b_vec, g.b_bf16);
            }
        }
    };
    floatx16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = zero16();

    if (k_begin < k_end) fetch(k_begin);
    for (int k0 = k_begin; k0 < k_end; k0 += F_GK) {
#pragma unroll
        for (int i = 0; i < TA::groups; ++i) {
            int r, kk;
            TA::place(tid, i, r, kk);
            *(float4*)TA::at(As, r, kk) = raw_to_f32(ra[i], g.a_bf16);
        }
#pragma unroll
        for (int i = 0; i < TB::groups; ++i) {
            int r, kk;
            TB::place(tid, i, r, kk);
            *(float4*)TB::at(Bs, r, kk) = raw_to_f32(rb[i], g.b_bf16);
        }
        __syncthreads();
        if (k0 + F_GK < k_end) fetch(k0 + F_GK);
#pragma unroll
        for (int ph = 0; ph < F_GK / 16; ++ph) {
            floatx16 part[MT][NT];
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) part[i][j] = zero16();
#pragma unroll
            for (int q = 2 * ph; q < 2 * ph + 2; ++q) {
                float fa[MT][4], fb[NT][4];
#pragma unroll
                for (int i = 0; i < MT; ++i) {
                    const int r = wm * (TM / 2) + 32 * i + l32;
                    if (AKF) *(float4*)fa[i] = *(const float4*)TA::at(As, r, 8 * q + 4 * half);
                    else
#pragma unroll
                        for (int e = 0; e < 4; ++e) fa[i][e] = *TA::at(As, r, 8 * q + 4 * half + e);
                }
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const int r = wn * (TN / 2) + 32 * j + l32;
                    if (BKF) *(float4*)fb[j] = *(const float4*)TB::at(Bs, r, 8 * q + 4 * half);
                    else
#pragma unroll
                        for (int e = 0; e < 4; ++e) fb[j][e] = *TB::at(Bs, r, 8 * q + 4 * half + e);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < MT; ++i)
#pragma unroll
                        for (int j = 0; j < NT; ++j) part[i][j] = mfma_f32(fa[i][e], fb[j][e], part[i][j]);
            }
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][j][e] += part[i][j][e];
        }
        __syncthreads();
    }
    // this lane holds column 32j + l32 and rows 32i + 8(e/4) + 4 half + e%4 of each MFMA tile
    float* const part_out = g.part ? g.part + ((long)((int)blockIdx.y * (g.C2 ? 2 : 1) + which) * g.batches + bz) * g.M * g.N : nullptr;
    void* const C = which ? g.C2 : g.C;
    const long coff = (long)b * g.sCb + (long)h * g.sCh;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int gm = m0 + wm * (TM / 2) + 32 * i + 8 * (e >> 2) + 4 * half + (e & 3);
                const int gn = n0 + wn * (TN / 2) + 32 * j + l32;
                if (gm >= g.M || gn >= g.N) continue;
                float v = acc[i][j][e];
                if (part_out) {
                    part_out[(long)gm * g.N + gn] = v;
                } else {
                    const long ci = coff + (long)gm * g.sCm + (long)gn * g.sCn;
                    if (g.accumulate) v += ((const float*)C)[ci];
                    store_elem(C, ci, v, g.c_bf16);
                }
            }
}

// `part`, `part_floats`: scratch for a split reduction (only for contiguous fp32 results: C[b,h][m][n] at
// ((b H + h) M + m) N + n); nullptr if the reduction must not be split.
flurka_status launch_gemm_f32(GemmArgs g, int batches, float* part, size_t part_floats, hipStream_t s);

}  // namespace flurka
