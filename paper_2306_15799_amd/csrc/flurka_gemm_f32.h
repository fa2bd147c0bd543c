// Strided batched GEMM of fp32 accuracy on the matrix cores of gfx950, for every contraction of the
// fp32-arithmetic path that runs over the sequence:
//     C[b,h] (M x N) (+)= A[b,h] (M x K) B[b,h] (K x N)
// Operands are addressed through element strides, so transposes, shared operands (batch stride 0), a
// reduction index that runs over (outer, inner) pairs (K = Kout * Kin) and result columns that run over
// (head, coordinate) pairs (N = Nout * Nin) need no copies.
//
// Beside a bf16 operand, which enters as it is, an fp32 operand enters as three bf16 terms (8 + 8 + 8 = 24
// mantissa bits: the split is exact, and so are the products).  Two fp32 operands are multiplied by the
// fp32 matrix instruction.
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
    int M, N, K, Kin, Nin;                       // Nin = 0: one level of columns
    long sAm, sAki, sAko, sAb, sAh;
    long sBn, sBki, sBko, sBb, sBh, sBno;        // sBno, sCno: between outer column indices
    long sCm, sCn, sCb, sCh, sCno;
    int H;
    int a_bf16, b_bf16, c_bf16;
    int accumulate;
    // filled in by launch_gemm_f32
    float* part;         // split partials [split][which], each laid out like C (nullptr: the reduction is not split)
    int batches, steps_per_split;
    long c_count;        // elements of C (split reductions: C is contiguous)
};

// ---- operand terms ----------------------------------------------------------
// T terms of 8 values, each an operand of mfma32.  T = 1: a bf16 operand as stored; T = 3: an fp32 operand.
template <int T> struct Terms { uint4 t[T]; };

// acc += A B over the terms, smallest products first.  Term i is at most 2^-9i of the value; of the products of
// two split operands the six with i + j <= 2 are formed, the rest is below 2^-26 of the product: less than
// the rounding of one fp32 addition.
template <int TA, int TB>
__device__ __forceinline__ floatx16 mfma_terms(const uint4 (&a)[TA], const uint4 (&b)[TB], floatx16 acc) {
#pragma unroll
    for (int s = 2; s >= 0; --s)
#pragma unroll
        for (int i = 0; i < TA; ++i)
            if (s - i >= 0 && s - i < TB) acc = mfma32(a[i], b[s - i], acc);
    return acc;
}

typedef short f32_short4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 f32_read_tr16(const unsigned char* p) {
    const f32_short4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((f32_short4 __attribute__((address_space(3)))*)p);
    return __builtin_bit_cast(uint2, v);
}

// ---- 32 x D bf16 tile in LDS ---------------------------------------------------
// Unpadded rows; 16-byte chunk c of row r sits at position c ^ swz(r), which makes both kinds of read
// conflict-free (see BwdXLds in flurka_bwd.hip, where this layout comes from):
//   row_frag   8 consecutive columns of row l32          (rows are the operand's free index)
//   col_frag   column 32t + l32 of 8 rows of a 16-row group, in accumulator order   (rows are reduced over):
//              slot 8h + e of lane half h is row 8(e/4) + 4h + e%4 of the group
template <int D>
struct Tile32 {
    static_assert(D == 64 || D == 128, "row swizzles are written for 128- and 256-byte rows");
    static constexpr int pitch = D * 2, bytes = 32 * pitch, chunks = 32 * D / 8;
    static __device__ __forceinline__ int swz(int r) {
        return D == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
    }
    static __device__ __forceinline__ unsigned char* chunk(unsigned char* t, int r, int c) { return t + r * pitch + 16 * (c ^ swz(r)); }
    int row_off, row_xor, tr_row, tr_low, tr_hi;
    __device__ __forceinline__ explicit Tile32(int lane) {
        const int half = lane >> 5, l32 = lane & 31, s16 = lane & 15, r4 = s16 >> 2;
        row_off = l32 * pitch;
        row_xor = 16 * (swz(l32) ^ half);
        tr_row = (4 * half + r4) * pitch + 8 * (s16 & 1);
        tr_low = 16 * ((2 * ((lane >> 4) & 1) + ((s16 >> 1) & 1)) ^ half);
        tr_hi = D == 128 ? r4 : (r4 >> 1);
    }
    __device__ __forceinline__ uint4 row_frag(const unsigned char* t, int s) const {
        return *(const uint4*)(t + row_off + ((32 * s) ^ row_xor));
    }
    __device__ __forceinline__ uint4 col_frag(const unsigned char* t, int sp, int tt) const {
        const unsigned char* fb = t + 16 * sp * pitch + tr_row;
        const int col = ((tt ^ tr_hi) << 6) + tr_low;
        const uint2 w0 = f32_read_tr16(fb + col);
        const uint2 w1 = f32_read_tr16(fb + 8 * pitch + (col ^ 32));
        return make_uint4(w0.x, w0.y, w1.x, w1.y);
    }
};

// ---- operand tiles of the GEMM -----------------------------------------------------
constexpr int F_GK = 32;                  // reduction step

// 4 consecutive elements starting at element i, as 16 bytes (fp32, T = 3) or 8 bytes (bf16, T = 1) that need
// no more than the element's own alignment
template <int T> struct Raw4 { uint4 v; };
template <> struct Raw4<1> { uint2 v; };
template <int T>
__device__ __forceinline__ Raw4<T> ld4_raw(const void* p, long i) {
    Raw4<T> r;
    if constexpr (T == 1) __builtin_memcpy(&r.v, (const uint16_t*)p + i, 8);
    else                  __builtin_memcpy(&r.v, (const float*)p + i, 16);
    return r;
}
// Element e of a group (edges of the operand): element i, or zero if !keep.  i is a valid index either way, so
// that the loads of a step go out together instead of one behind a branch each (a reduction of 187 had
// spent most of its six steps in the last one).
template <int T>
__device__ __forceinline__ void set_elem(Raw4<T>& r, int e, const void* p, long i, bool keep) {
    uint32_t* w = (uint32_t*)&r.v;
    if constexpr (T == 1) {
        uint32_t x = ((const uint16_t*)p)[i];
        x = keep ? x : 0u;
        w[e >> 1] = (e & 1) ? (w[e >> 1] | (x << 16)) : x;
    } else {
        const uint32_t x = ((const uint32_t*)p)[i];
        w[e] = keep ? x : 0u;
    }
}
template <int T>
__device__ __forceinline__ void keep_group(Raw4<T>& r, bool keep) {
    uint32_t* w = (uint32_t*)&r.v;
#pragma unroll
    for (int e = 0; e < (T == 1 ? 2 : 4); ++e) w[e] = keep ? w[e] : 0u;
}
template <int T>
__device__ __forceinline__ void split4(const Raw4<T>& r, uint2 (&t)[T]) {
    if constexpr (T == 1) {
        t[0] = r.v;
    } else {
        split3_pair(__uint_as_float(r.v.x), __uint_as_float(r.v.y), t[0].x, t[1].x, t[2].x);
        split3_pair(__uint_as_float(r.v.z), __uint_as_float(r.v.w), t[0].y, t[1].y, t[2].y);
    }
}

// One operand tile of TR free indices ("rows") x 32 reduction slots, T terms.
// KF: the reduction index is the contiguous one in memory; the tile is kept [row][slot], 80-byte rows (16
// consecutive rows start in 16 different groups of 4 banks), the four 4-slot groups of a 16-slot block in
// the order 0, 2, 1, 3, so that a lane half's 8 slots in accumulator order are 16 consecutive bytes.
// Otherwise the rows are contiguous; the tile is kept [slot][row] (Tile32) and fragments come out through
// transposing reads, in the same slot order.
template <bool KF, int TR, int T>
struct GemmTile {
    static constexpr int term = KF ? TR * 80 : Tile32<TR>::bytes;
    static constexpr int bytes = T * term;
    static constexpr int groups = TR * F_GK / 4 / 256;       // of 4 elements, per thread
    static __device__ __forceinline__ void place(int tid, int i, int& r, int& kk) {
        const int idx = tid + 256 * i;
        if (KF) { r = idx >> 3; kk = 4 * (idx & 7); }
        else    { kk = idx / (TR / 4); r = 4 * (idx % (TR / 4)); }
    }
    static __device__ __forceinline__ void store(unsigned char* t, int r, int kk, const Raw4<T>& x) {
        uint2 w[T];
        split4<T>(x, w);
        unsigned char* p;
        if (KF) {
            const int g = (kk >> 2) & 3;
            p = t + r * 80 + 32 * (kk >> 4) + 8 * (((g & 1) << 1) | (g >> 1));
        } else {
            p = Tile32<TR>::chunk(t, kk, r >> 3) + 2 * (r & 4);
        }
#pragma unroll
        for (int k = 0; k < T; ++k) *(uint2*)(p + k * term) = w[k];
    }
    // fragment of rows 32 rt + l32, 16-slot block s
    static __device__ __forceinline__ void frag(const unsigned char* t, int lane, int rt, int s, uint4 (&f)[T]) {
        if (KF) {
            const unsigned char* p = t + (32 * rt + (lane & 31)) * 80 + 32 * s + 16 * (lane >> 5);
#pragma unroll
            for (int k = 0; k < T; ++k) f[k] = *(const uint4*)(p + k * term);
        } else {
            const Tile32<TR> tl(lane);
#pragma unroll
            for (int k = 0; k < T; ++k) f[k] = tl.col_frag(t + k * term, s, rt);
        }
    }
};

// fp32 x fp32: operand tiles as they are, for v_mfma_f32_32x32x2_f32.  Six bf16 products would take less matrix
// time, but not less time in all (the kernel is then bound by LDS and the split: 48 us against 55 us at
// 16 x (256 x 64 x 4096)), and the bf16 instruction truncates where this one rounds: the projections of a long
// sequence come out 1e-6 too small instead of 2e-7 off either way.
// [row][slot] tile: 36 floats per row (16 consecutive rows start in 16 different groups of 4 banks), a
// fragment is 4 slots.  [slot][row] tile: TR + 8 floats (the two halves' slots, 4 rows apart, use different
// halves of the 64 banks), a fragment is one dword.  Lane half h takes slots 8q + 4h + e (q, e = 0..3).
template <bool KF, int TR>
struct GemmTileF32 {
    static constexpr int pitch = KF ? F_GK + 4 : TR + 8;
    static constexpr int bytes = (KF ? TR : F_GK) * pitch * 4;
    static constexpr int groups = TR * F_GK / 4 / 256;
    static __device__ __forceinline__ void place(int tid, int i, int& r, int& kk) { GemmTile<KF, TR, 3>::place(tid, i, r, kk); }
    static __device__ __forceinline__ void store(unsigned char* t, int r, int kk, const Raw4<3>& x) {
        *(uint4*)((float*)t + (KF ? r * pitch + kk : kk * pitch + r)) = x.v;
    }
    // slots 8q + 4 half .. + 3 of row 32 rt + l32
    static __device__ __forceinline__ void frag(const unsigned char* t, int lane, int rt, int q, float (&f)[4]) {
        const int r = 32 * rt + (lane & 31), k = 8 * q + 4 * (lane >> 5);
        if (KF) *(float4*)f = *(const float4*)((const float*)t + r * pitch + k);
        else
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = ((const float*)t)[(k + e) * pitch + r];
    }
};

// v_mfma_f32_32x32x2_f32, one wavefront: D(32x32) += A(32x2) B(2x32), all fp32.
// Operand layout, lane l: A row l%32, reduction slot l/32; B column l%32, slot l/32; D as for mfma32.
__device__ __forceinline__ floatx16 mfma_f32(float a, float b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

template <bool C, class X, class Y> struct PickType { typedef X type; };
template <class X, class Y> struct PickType<false, X, Y> { typedef Y type; };

// LDS of a workgroup: two buffers of both operand tiles
template <bool AKF, bool BKF, int TA, int TB, int TM, int TN>
struct GemmF32Lds {
    static constexpr bool native = TA == 3 && TB == 3;         // fp32 x fp32
    using LA = typename PickType<native, GemmTileF32<AKF, TM>, GemmTile<AKF, TM, TA>>::type;
    using LB = typename PickType<native, GemmTileF32<BKF, TN>, GemmTile<BKF, TN, TB>>::type;
    static constexpr int stage = LA::bytes + LB::bytes, bytes = 2 * stage;
    // steps between the request of an operand and its use: two where the registers for a second staging set
    // are there (128 x 128 tiles with an fp32 operand spill up to 56 registers with it and lose 3 to 7 us of 60)
    static constexpr int ahead = TM == 128 && TN == 128 && (TA == 3 || TB == 3) ? 1 : 2;
};

// Tile TM x TN of C per workgroup of four wavefronts (2 x 2, each TM/2 x TN/2), 32-deep steps through two
// LDS buffers, one barrier per step.  A step's operands are requested up to two steps before they are needed:
// it has only 6 to 32 matrix instructions per wavefront (200 to 2000 cycles) to cover a load with.  Bound by
// vector issue (splits, partial sums, the stores of short reductions) for bf16 operands, by the fp32 matrix
// rate for fp32 x fp32.
// Every 16 products (fp32 x fp32; else 32, every step) form a partial sum of their own that is then added to
// the running sum, so that the rounding error of a long reduction grows with K/16, not with K.
template <bool AKF, bool BKF, int TA, int TB, int TM, int TN>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(GemmArgs g) {
    using L = GemmF32Lds<AKF, BKF, TA, TB, TM, TN>;
    using LA = typename L::LA;
    using LB = typename L::LB;
    constexpr bool NATIVE = L::native;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
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
    const int Nin = g.Nin ? g.Nin : g.N;
    // groups of 4 never straddle two outer indices, and the contiguous index has stride 1
    const bool a_vec = AKF ? (g.sAki == 1 && (one_level || g.Kin % 4 == 0)) : g.sAm == 1;
    const bool b_vec = BKF ? (g.sBki == 1 && (one_level || g.Kin % 4 == 0)) : (g.sBn == 1 && (!g.Nin || g.Nin % 4 == 0));

    auto k_offset = [&](int k, long ski, long sko) -> long {
        if (one_level) return (long)k * ski;
        const int ko = k / g.Kin;
        return (long)ko * sko + (long)(k - ko * g.Kin) * ski;
    };
    auto a_row = [&](int r) -> long { return (long)r * g.sAm; };
    auto b_row = [&](int r) -> long {
        if (!g.Nin) return (long)r * g.sBn;
        const int no = r / Nin;
        return (long)no * g.sBno + (long)(r - no * Nin) * g.sBn;
    };
    // Three ways to load a step, the same for all threads of a workgroup:
    //   short     whole steps inside one outer index: fixed offsets per thread, one uniform offset per step
    //   groups    every group of 4 lies inside or outside of the operand as a whole: one load per group
    //   elements  anything else
    // Row indices are clamped (rows past the end only feed results nobody stores), reduction indices past the
    // end read a valid element and become zero.
    const bool whole_steps = one_level || g.Kin % F_GK == 0;
    const bool a_group = a_vec && (AKF ? g.K % 4 == 0 : (g.M % 4 == 0 || m0 + TM <= g.M));
    const bool b_group = b_vec && (BKF ? g.K % 4 == 0 : (g.N % 4 == 0 || n0 + TN <= g.N));
    const bool a_short = a_vec && whole_steps && (AKF || g.M % 4 == 0 || m0 + TM <= g.M);
    const bool b_short = b_vec && whole_steps && (BKF || g.N % 4 == 0 || n0 + TN <= g.N);
    long pa[LA::groups], pb[LB::groups];      // offsets of this thread's groups at reduction index 0
#pragma unroll
    for (int i = 0; i < LA::groups; ++i) {
        int r, kk;
        LA::place(tid, i, r, kk);
        const int rc = m0 + r < g.M ? m0 + r : (AKF ? g.M - 1 : 0);
        pa[i] = aoff + a_row(rc);
    }
#pragma unroll
    for (int i = 0; i < LB::groups; ++i) {
        int r, kk;
        LB::place(tid, i, r, kk);
        const int rc = n0 + r < g.N ? n0 + r : (BKF ? g.N - 1 : 0);
        pb[i] = boff + b_row(rc);
    }
    struct Stage { Raw4<TA> a[LA::groups]; Raw4<TB> b[LB::groups]; };
    auto fetch = [&](int k0, Stage& st) {
        const bool inside = k0 + F_GK <= k_end;
        if (inside && a_short) {
            const long ko = k_offset(k0, g.sAki, g.sAko);
#pragma unroll
            for (int i = 0; i < LA::groups; ++i) {
                int r, kk;
                LA::place(tid, i, r, kk);
                st.a[i] = ld4_raw<TA>(A, pa[i] + (long)kk * g.sAki + ko);
            }
        } else if (a_group) {
#pragma unroll
            for (int i = 0; i < LA::groups; ++i) {
                int r, kk;
                LA::place(tid, i, r, kk);
                const bool ok = k0 + kk < k_end;
                st.a[i] = ld4_raw<TA>(A, pa[i] + k_offset(ok ? k0 + kk : k0, g.sAki, g.sAko));
                keep_group<TA>(st.a[i], ok);
            }
        } else {
#pragma unroll
            for (int i = 0; i < LA::groups; ++i) {
                int r, kk;
                LA::place(tid, i, r, kk);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int re = m0 + (AKF ? r : r + e), ke = k0 + (AKF ? kk + e : kk);
                    set_elem<TA>(st.a[i], e, A, aoff + a_row(re < g.M ? re : g.M - 1) + k_offset(ke < k_end ? ke : k0, g.sAki, g.sAko),
                                 re < g.M && ke < k_end);
                }
            }
        }
        if (inside && b_short) {
            const long ko = k_offset(k0, g.sBki, g.sBko);
#pragma unroll
            for (int i = 0; i < LB::groups; ++i) {
                int r, kk;
                LB::place(tid, i, r, kk);
                st.b[i] = ld4_raw<TB>(B, pb[i] + (long)kk * g.sBki + ko);
            }
        } else if (b_group) {
#pragma unroll
            for (int i = 0; i < LB::groups; ++i) {
                int r, kk;
                LB::place(tid, i, r, kk);
                const bool ok = k0 + kk < k_end;
                st.b[i] = ld4_raw<TB>(B, pb[i] + k_offset(ok ? k0 + kk : k0, g.sBki, g.sBko));
                keep_group<TB>(st.b[i], ok);
            }
        } else {
#pragma unroll
            for (int i = 0; i < LB::groups; ++i) {
                int r, kk;
                LB::place(tid, i, r, kk);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int re = n0 + (BKF ? r : r + e), ke = k0 + (BKF ? kk + e : kk);
                    set_elem<TB>(st.b[i], e, B, boff + b_row(re < g.N ? re : g.N - 1) + k_offset(ke < k_end ? ke : k0, g.sBki, g.sBko),
                                 re < g.N && ke < k_end);
                }
            }
        }
    };
    auto put = [&](const Stage& st, unsigned char* buf) {
#pragma unroll
        for (int i = 0; i < LA::groups; ++i) {
            int r, kk;
            LA::place(tid, i, r, kk);
            LA::store(buf, r, kk, st.a[i]);
        }
#pragma unroll
        for (int i = 0; i < LB::groups; ++i) {
            int r, kk;
            LB::place(tid, i, r, kk);
            LB::store(buf + LA::bytes, r, kk, st.b[i]);
        }
    };
    floatx16 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = zero16();

    // step k0 out of `buf`; `mine` is free and takes the step `ahead` steps on, `next` holds the next step's
    // operands (ahead = 1: it is the same set), which go to `other` for it
    auto step = [&](int k0, unsigned char* buf, unsigned char* other, Stage& mine, const Stage& next) {
        const unsigned char* const As = buf;
        const unsigned char* const Bs = buf + LA::bytes;
        if (k0 + L::ahead * F_GK < k_end) fetch(k0 + L::ahead * F_GK, mine);
        floatx16 part[MT][NT];
        auto clear = [&]() {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) part[i][j] = zero16();
        };
        auto flush = [&]() {
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) acc[i][j] += part[i][j];
        };
        clear();
#pragma unroll
        for (int s = 0; s < F_GK / 16; ++s) {
            if constexpr (NATIVE) {
#pragma unroll
                for (int q = 2 * s; q < 2 * s + 2; ++q) {
                    float fa[MT][4], fb[NT][4];
#pragma unroll
                    for (int i = 0; i < MT; ++i) LA::frag(As, lane, wm * MT + i, q, fa[i]);
#pragma unroll
                    for (int j = 0; j < NT; ++j) LB::frag(Bs, lane, wn * NT + j, q, fb[j]);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int i = 0; i < MT; ++i)
#pragma unroll
                            for (int j = 0; j < NT; ++j) part[i][j] = mfma_f32(fa[i][e], fb[j][e], part[i][j]);
                }
                flush();
                if (s + 1 < F_GK / 16) clear();
            } else {
                uint4 fa[MT][TA], fb[NT][TB];
#pragma unroll
                for (int i = 0; i < MT; ++i) LA::frag(As, lane, wm * MT + i, s, fa[i]);
#pragma unroll
                for (int j = 0; j < NT; ++j) LB::frag(Bs, lane, wn * NT + j, s, fb[j]);
#pragma unroll
                for (int i = 0; i < MT; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) part[i][j] = mfma_terms<TA, TB>(fa[i], fb[j], part[i][j]);
            }
        }
        if constexpr (!NATIVE) flush();
        if (k0 + F_GK < k_end) {
            put(next, other);
            __syncthreads();     // `other` complete; everybody is done with `buf`, which the next step fills
        }
    };
    if (k_begin < k_end) {
        unsigned char* const b0 = lds;
        unsigned char* const b1 = lds + L::stage;
        if constexpr (L::ahead == 2) {
            Stage s0, s1;
            fetch(k_begin, s0);
            if (k_begin + F_GK < k_end) fetch(k_begin + F_GK, s1);
            put(s0, b0);
            __syncthreads();
            for (int k0 = k_begin; k0 < k_end; k0 += 2 * F_GK) {
                step(k0, b0, b1, s0, s1);
                if (k0 + F_GK < k_end) step(k0 + F_GK, b1, b0, s1, s0);
            }
        } else {
            Stage st;
            fetch(k_begin, st);
            put(st, b0);
            __syncthreads();
            int buf = 0;
            for (int k0 = k_begin; k0 < k_end; k0 += F_GK, buf ^= 1)
                step(k0, lds + buf * L::stage, lds + (buf ^ 1) * L::stage, st, st);
        }
    }
    // this lane holds column 32j + l32 and rows 32i + 8(e/4) + 4 half + e%4 of each MFMA tile.  Rows advance by
    // uniform distances; tiles inside the result store without a check per element (a short reduction spends as
    // long here as in its steps).
    float* const part_out = g.part ? g.part + ((long)blockIdx.y * (g.C2 ? 2 : 1) + which) * g.c_count : nullptr;
    void* const C = part_out ? (void*)part_out : which ? g.C2 : g.C;
    const bool c_bf16 = !part_out && g.c_bf16, accumulate = !part_out && g.accumulate;
    const long coff = (long)b * g.sCb + (long)h * g.sCh;
    const int row0 = m0 + wm * (TM / 2) + 4 * half;
    const bool whole = m0 + TM <= g.M;
    auto store_column = [&](auto* c, const floatx16 (&t)[MT][NT], int j, auto&& keep, auto&& put1) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                auto* cq = c + (long)(32 * i + 8 * q) * g.sCm;
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    const int r = 32 * i + 8 * q + e;
                    put1(cq + (long)e * g.sCm, cq + (long)(e + 1) * g.sCm, t[i][j][4 * q + e], t[i][j][4 * q + e + 1], keep(r), keep(r + 1));
                }
            }
    };
    auto all = [](int) { return true; };
    auto some = [&](int r) { return row0 + r < g.M; };
    auto two_bf16 = [](uint16_t* p0, uint16_t* p1, float x, float y, bool k0, bool k1) {
        const uint32_t v = pack_bf16(x, y);
        if (k0) *p0 = (uint16_t)v;
        if (k1) *p1 = (uint16_t)(v >> 16);
    };
    auto two_f32 = [](float* p0, float* p1, float x, float y, bool k0, bool k1) {
        if (k0) *p0 = x;
        if (k1) *p1 = y;
    };
    auto two_add = [](float* p0, float* p1, float x, float y, bool k0, bool k1) {
        if (k0) *p0 += x;
        if (k1) *p1 += y;
    };
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int gn = n0 + wn * (TN / 2) + 32 * j + l32;
        if (gn >= g.N) continue;
        const int no = g.Nin ? gn / Nin : 0;
        const long ci = coff + (long)no * g.sCno + (long)(gn - no * Nin) * g.sCn + (long)row0 * g.sCm;
        if (c_bf16) {
            if (whole) store_column((uint16_t*)C + ci, acc, j, all, two_bf16);
            else       store_column((uint16_t*)C + ci, acc, j, some, two_bf16);
        } else if (!accumulate) {
            if (whole) store_column((float*)C + ci, acc, j, all, two_f32);
            else       store_column((float*)C + ci, acc, j, some, two_f32);
        } else {
            store_column((float*)C + ci, acc, j, some, two_add);
        }
    }
}

// `part`, `part_floats`: scratch for a split reduction (only for contiguous fp32 results of `c_count` elements
// in all batches together); nullptr if the reduction must not be split.
flurka_status launch_gemm_f32(GemmArgs g, int batches, float* part, size_t part_floats, hipStream_t s);

}  // namespace flurka
