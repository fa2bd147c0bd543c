// Key-side state of FLuRKA attention on MFMA (gfx950):  S = PhiK^T V',  z = PhiK^T 1,  c.
//
// PhiK_rj = exp(e_rj - c_j),  e_rj = omega_j . k'_r - |k'_r|^2 / 2  (positive random features, Sec. 2
// "Kernel Methods"), or PhiK = elu(K') + 1.  exp() turns an absolute error of e into a relative error
// of the attention weights, and |e| reaches several hundred for long sequences, so e is formed to
// fp32 accuracy: K' (fp32) is split into three bf16 terms whose products with the bf16 omega are
// exact in the fp32 accumulator.  PhiK and V' enter the second contraction as two-term bf16 splits.
//
// Two kernels:
//   proj_finish   sums the projection's split-n partials into K', V' (fp32, ctx) and writes the
//                 operand images: K' as bf16 hi/mid/lo rows, V' as bf16 hi/lo, both in the order in which
//                 key_state's wavefronts read them (1 KiB of consecutive bytes per operand), and
//                 |k'|^2 / 2 per key
//   key_state     one workgroup per (head, 32 features), one wavefront per key range: first
//                 contraction on MFMA, column maximum, exp, second contraction on MFMA with PhiK taken
//                 from the accumulator registers as the A operand; the ranges' partial S, z, c meet in
//                 LDS, are joined there (log-sum-exp style) and leave as S, z, c (fp32, ctx) and as the
//                 bf16 images the query-stream kernel loads into LDS
// Both are bound by latency: a chain of loads, products, exponentials and the merge, on a chip that a few
// hundred keys per head do not fill.  So every operand of a wavefront is requested before the first is used,
// and the merge is one pass over LDS by the whole workgroup.  (Requests behind a branch per tile or per key, V' one
// dword at a time and a merge in transposed 32-coordinate pieces took, key_state alone: 64 keys, 4 heads 15.6 us,
// now 4.6; elu, 256 keys, 64 heads 19.9, now 6.8; 256 keys, 64 heads 14.4, now 11, where the eight workgroups of a
// head read its 160 KiB of images eight times out of L2.)
#include "flurka_fast.h"
#include "flurka_gemm.h"

namespace flurka {

#define FLURKA_CHECK_LAUNCH()                                   \
    do {                                                        \
        if (hipGetLastError() != hipSuccess) return FLURKA_ERR_LAUNCH; \
    } while (0)

static inline dim3 grid1d(long total, int block) { return dim3((unsigned)((total + block - 1) / block)); }

// x = hi + mid + lo with each term a bf16 (24 mantissa bits in total)
__device__ __forceinline__ void split3(float x, uint16_t& hi, uint16_t& mid, uint16_t& lo) {
    hi = f32_to_bf16(x);
    const float r1 = x - bf16_to_f32(hi);
    mid = f32_to_bf16(r1);
    lo = f32_to_bf16(r1 - bf16_to_f32(mid));
}

// ---------------------------------------------------------------------------
// proj_finish: one wavefront per (head, four consecutive keys 4g .. 4g+3); lane = coordinate t (and
// t + 64 for d = 128).  The four keys are the four floats of one 16-byte element of the projection's
// tile-ordered partial results, and consecutive t are consecutive elements: coalesced float4 loads.
// ---------------------------------------------------------------------------
struct FinishArgs {
    const float* part;      // tile-ordered split partials of the projection (see flurka_gemm.h)
    float* ctx;             // K' at ctx + Kp_off, V' at ctx + Vp_off
    long Kp_off, Vp_off;
    uint16_t* Kimg;         // 3 x (BH, kpad * d) bf16: hi, mid, lo, in key_state's operand order (nullptr for elu1)
    uint32_t* Vimg;         // 2 x (BH, kpad/2 * d) dwords: hi, lo; low half = even key (nullptr: K', V' only)
    float* nrm;             // (BH, kpad): |k'|^2/2, +inf for the padding keys (nullptr for elu1)
    int splits, tilesM, tilesN, k, kpad, d, BH;
    PartialTile tile;       // of the partial results
};

// Dword of the V' image that holds keys (2 p, 2 p + 1), coordinate t, inside a head: [32-key tile][16-key step]
// [32-coordinate tile][lane = 32 h + t % 32][4], the lane's four dwords being pairs 2h, 2h + 1, 2h + 4, 2h + 5 of the
// step: the order in which the accumulator hands PhiK^T on.  Pairs 2i and 2i + 1 are neighbours.
__device__ __forceinline__ int v_image_offset(int p, int t, int d) {
    const int q = p & 7;
    return ((((p >> 3) * (d / 32) + (t >> 5)) * 64) + 32 * ((q >> 1) & 1) + (t & 31)) * 4 + 2 * (q >> 2) + (q & 1);
}
// Element of the K' image that holds key r, coordinate t, inside a head: [32-key tile][16-coordinate step]
// [8-coordinate half][key][8]
__device__ __forceinline__ int k_image_offset(int r, int t, int d) {
    return ((((r >> 5) * (d / 16) + (t >> 4)) * 2 + ((t >> 3) & 1)) * 32 + (r & 31)) * 8 + (t & 7);
}

// value of lane ^ 1 and of lane ^ 2 (DPP quad permutations)
__device__ __forceinline__ uint32_t lane_xor1(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xb1, 0xf, 0xf, false); }
__device__ __forceinline__ uint32_t lane_xor2(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4e, 0xf, 0xf, false); }
// Four lanes t .. t + 3, each with one coordinate of four keys (k0 | k1, k2 | k3 as packed bf16): afterwards each has
// the four coordinates of one key, lane t % 4 = 0, 1, 2, 3 that of key 0, 2, 1, 3
__device__ __forceinline__ uint2 transpose_4x4(uint32_t p01, uint32_t p23, int lane) {
    const bool odd = lane & 1, upper = lane & 2;
    const uint32_t mine = odd ? p23 : p01, theirs = lane_xor1(odd ? p01 : p23);
    const uint32_t even_t = odd ? theirs : mine, odd_t = odd ? mine : theirs;      // coordinates t & ~1 and t | 1
    const uint32_t a = (even_t & 0xffffu) | (odd_t << 16), b = (even_t >> 16) | (odd_t & 0xffff0000u);
    const uint32_t keep = upper ? b : a, got = lane_xor2(upper ? a : b);
    return upper ? make_uint2(got, keep) : make_uint2(keep, got);
}

__global__ __launch_bounds__(256) void proj_finish_kernel(FinishArgs a) {
    const int lane = threadIdx.x & 63;
    const long wid = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int groups_per_head = a.kpad / 4;
    if (wid >= (long)a.BH * groups_per_head) return;
    const int bh = (int)(wid / groups_per_head);
    const int r0 = 4 * (int)(wid % groups_per_head);           // keys r0 .. r0 + 3
    const int hpt = a.tile.tn / a.d;                            // heads per column tile
    const int tn = bh / hpt, tm = r0 / a.tile.tm;
    const long tile_elems = a.tile.tm * a.tile.tn;
    const long img_plane = (long)a.BH * a.kpad * a.d;          // elements per K image plane
    const long vimg_plane = (long)a.BH * (a.kpad / 2) * a.d;
    float sq[4] = {0.f, 0.f, 0.f, 0.f};
    for (int t = lane; t < a.d; t += 64) {
        const int eo = partial_elem_offset(a.tile, r0 % a.tile.tm, (bh % hpt) * a.d + t);
        const float* const p0 = a.part + partial_tile_index(0, 0, tn, tm, a.splits, a.tilesN, a.tilesM) * tile_elems + eo;
        const float* const p1 = a.part + partial_tile_index(1, 0, tn, tm, a.splits, a.tilesN, a.tilesM) * tile_elems + eo;
        const long stride = (long)a.tilesN * a.tilesM * tile_elems;
        struct Pair { float4 k, v; };
        float4 ks = {0.f, 0.f, 0.f, 0.f}, vs = {0.f, 0.f, 0.f, 0.f};
        for_parts<4, Pair>(
            a.splits, [&](int s) { return Pair{*(const float4*)(p0 + s * stride), *(const float4*)(p1 + s * stride)}; },
            [&](const Pair& x) {
                ks.x += x.k.x; ks.y += x.k.y; ks.z += x.k.z; ks.w += x.k.w;
                vs.x += x.v.x; vs.y += x.v.y; vs.z += x.v.z; vs.w += x.v.w;
            });
        float kv[4] = {ks.x, ks.y, ks.z, ks.w}, vv[4] = {vs.x, vs.y, vs.z, vs.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int r = r0 + e;
            if (r < a.k) {
                const long off = ((long)bh * a.k + r) * a.d + t;
                a.ctx[a.Kp_off + off] = kv[e];
                a.ctx[a.Vp_off + off] = vv[e];
            } else {
                kv[e] = 0.f; vv[e] = 0.f;                      // rows of a tile past k hold nothing useful
            }
            sq[e] = fmaf(kv[e], kv[e], sq[e]);
        }
        if (a.Kimg) {
            uint32_t h0, m0, l0, h1, m1, l1;
            split3_pair(kv[0], kv[1], h0, m0, l0);
            split3_pair(kv[2], kv[3], h1, m1, l1);
            const int key = ((lane & 1) << 1) | ((lane >> 1) & 1);
            uint16_t* const o = a.Kimg + (long)bh * a.kpad * a.d + k_image_offset(r0 + key, t & ~3, a.d);
            *(uint2*)o = transpose_4x4(h0, h1, lane);
            *(uint2*)(o + img_plane) = transpose_4x4(m0, m1, lane);
            *(uint2*)(o + 2 * img_plane) = transpose_4x4(l0, l1, lane);
        }
        if (a.Vimg) {
            uint2 hp, lp;
            split2_pair(vv[0], vv[1], hp.x, lp.x);
            split2_pair(vv[2], vv[3], hp.y, lp.y);
            uint32_t* const o = a.Vimg + (long)bh * (a.kpad / 2) * a.d + v_image_offset(r0 / 2, t, a.d);
            *(uint2*)o = hp;
            *(uint2*)(o + vimg_plane) = lp;
        }
    }
    if (a.nrm) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float tot = wave_sum(sq[e]);
            const int r = r0 + e;
            if (lane == 0) a.nrm[(long)bh * a.kpad + r] = r < a.k ? 0.5f * tot : INFINITY;
        }
    }
}

// ---------------------------------------------------------------------------
// key_state: one wavefront per (head, feature tile, key range)
// ---------------------------------------------------------------------------
struct KeyStateArgs {
    const uint16_t* Kimg;   // performer
    const float* Kp;        // elu1: K' fp32 (BH, k, d)
    const uint16_t* Kb;     // elu1, EXACT: the keys themselves, bf16 (BH, k, d)
    const uint32_t* Vimg;
    const float* nrm;
    const uint16_t* omega;
    float* S; float* z; float* c;            // ctx
    uint16_t* St; float* zp; uint16_t* cw;   // images for the query stream (see the merge step below)
    long omega_head_stride;
    int BH, H, k, kpad, mf, mfp, FT, KR, tiles_per_range;   // mf features (ctx strides), mfp = mf rounded up to whole tiles (image strides)
};

// LDS of a workgroup: per key range the partial S tile (32 features x d, rows padded), z and c
template <int D>
struct KeyStateLds {
    static constexpr int s_pitch = D + 4;                                   // floats
    static constexpr int range_floats = 32 * s_pitch + 64;
    static __host__ __device__ int total(int KR) { return KR * range_floats * 4; }
};

// Key tiles of a range that stay in registers between maximum and accumulation.  Ranges of three or four tiles (513 to
// 1024 keys) keep them too where the registers allow (head size 64, random features): 48 heads of 64, m 256, key_state
// evaluating such ranges twice 29.9 us at k 768, 36.3 at 1024; kept 23.5 and 27.6.  In a kernel of its own: the shorter
// ranges need 20 registers less.
constexpr int KS_KEEP = 2, KS_KEEP_LONG = 4;
constexpr int KS_WAVES = 8;        // most wavefronts (key ranges) per workgroup: what the registers leave room for
constexpr int KS_MERGERS = 4;      // fewest wavefronts per workgroup: the merge wants more than one

// EXACT: the keys and values are bf16 numbers to begin with (kernel attention without a sequence
// projection): one term of K and one of V carry everything, the other operand terms are skipped.
// KEEP: key tiles of a range that are evaluated once.
template <int D, bool ELU, bool EXACT, int KEEP>
__global__ __launch_bounds__(KS_WAVES * 64) void key_state_kernel(KeyStateArgs a) {
    constexpr int KS = D / 16, TT = D / 32;
    constexpr int TERMS = EXACT ? 1 : 3;
    extern __shared__ __attribute__((aligned(16))) float ks_lds[];
    using L = KeyStateLds<D>;
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int kr = threadIdx.x >> 6;                       // this wavefront's key range
    // Workgroup ids go round the 8 XCDs; the FT workgroups of one head all read that head's K' and V'
    // images, so they take ids that are equal mod 8 and share one L2.
    const int slot = (int)(blockIdx.x >> 3);
    const int ft = slot % a.FT;
    const int bh = (slot / a.FT) * 8 + (int)(blockIdx.x & 7);
    if (bh >= a.BH) return;                                // head count rounded up to whole groups of 8
    const int KT = a.kpad / 32;
    const int kt0 = kr * a.tiles_per_range;
    int kt1 = kt0 + a.tiles_per_range;
    if (kt1 > KT) kt1 = KT;
    const long plane = (long)a.BH * a.kpad * D;
    const long vplane = (long)a.BH * (a.kpad / 2) * D;

    if (kr < a.KR) {           // the others only take part in the merge
    // B operand of the first contraction: omega rows of this feature tile
    uint4 wf[KS];
    if constexpr (!ELU) {
        // features past mf (a ragged last tile) take the last real row; their results are replaced below
        const int fr = 32 * ft + l32 < a.mf ? 32 * ft + l32 : a.mf - 1;
        const uint16_t* og = a.omega + (long)(bh % a.H) * a.omega_head_stride + (long)fr * D + 8 * half;
#pragma unroll
        for (int s = 0; s < KS; ++s) wf[s] = ld16(og + 16 * s);
    }

    // What one 32-key tile needs of memory for its exponents (performer) or features (elu1)
    struct KFrag { uint4 k[ELU ? 1 : TERMS * KS]; float4 n[ELU ? 1 : 4]; float x[ELU ? 16 : 1]; };
    auto load_k = [&](int kt, KFrag& f) {
        if constexpr (!ELU) {
            const uint16_t* kg = a.Kimg + (long)bh * a.kpad * D + ((long)kt * KS * 64 + lane) * 8;
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int u = 0; u < TERMS; ++u) f.k[TERMS * s + u] = ld16(kg + u * plane + 512 * s);
            const float* ng = a.nrm + (long)bh * a.kpad + 32 * kt + 4 * half;
#pragma unroll
            for (int q = 0; q < 4; ++q) f.n[q] = *(const float4*)(ng + 8 * q);
        } else {
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                int r = 32 * kt + 8 * (g >> 2) + 4 * half + (g & 3);
                if (r >= a.k) r = a.k - 1;
                const long idx = ((long)bh * a.k + r) * D + 32 * ft + l32;
                f.x[g] = EXACT ? bf16_to_f32(a.Kb[idx]) : a.Kp[idx];
            }
        }
    };
    // exponents or features of a tile: lane = feature 32*ft + l32, element g = key 32*kt + 8*(g/4) + 4*half + g%4
    auto tile_values = [&](int kt, const KFrag& f) -> floatx16 {
        floatx16 e = zero16();
        if constexpr (!ELU) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int u = 0; u < TERMS; ++u) e = mfma32(f.k[TERMS * s + u], wf[s], e);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                e[4 * q] -= f.n[q].x; e[4 * q + 1] -= f.n[q].y; e[4 * q + 2] -= f.n[q].z; e[4 * q + 3] -= f.n[q].w;
            }
        } else {
#pragma unroll
            for (int g = 0; g < 16; ++g) {
                const int r = 32 * kt + 8 * (g >> 2) + 4 * half + (g & 3);
                const float v = f.x[g] > 0.f ? f.x[g] + 1.f : __expf(f.x[g]);
                e[g] = r < a.k ? v : 0.f;                      // padding keys contribute nothing
            }
        }
        return e;
    };

    // B operands of the second contraction for one key tile: V' columns 32*tt + l32, key pairs in the
    // order in which the accumulator hands PhiK^T on
    struct VFrag { uint4 h[2][TT], l[EXACT ? 1 : 2][TT]; };
    auto load_v = [&](int kt, VFrag& f) {
        const uint32_t* vb = a.Vimg + (long)bh * (a.kpad / 2) * D + ((long)kt * 2 * TT * 64 + lane) * 4;
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                f.h[sp][tt] = *(const uint4*)(vb + (sp * TT + tt) * 256);
                if constexpr (!EXACT) f.l[sp][tt] = *(const uint4*)(vb + vplane + (sp * TT + tt) * 256);
            }
    };
    float c = 0.f;                                 // stays 0 for elu1
    floatx16 accS[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) accS[t] = zero16();
    float zsum = 0.f;
    constexpr float LOG2E = 1.4426950408889634f;
    // a range in which every |k'|^2 overflows has no finite exponent: its weights are 0, not exp(-inf + inf)
    float shift = 0.f;
    auto accumulate = [&](const floatx16& e, const VFrag& f) {
        uint32_t hi[8], lo[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float p0 = e[2 * q], p1 = e[2 * q + 1];
            if constexpr (!ELU) {
                p0 = fast_exp2((p0 - shift) * LOG2E);
                p1 = fast_exp2((p1 - shift) * LOG2E);
            }
            zsum += p0 + p1;
            split2_pair(p0, p1, hi[q], lo[q]);
        }
        // PhiK^T tile as A operand: row = this lane's feature, reduction slots = keys in accumulator order
        const uint4 ah[2] = {{hi[0], hi[1], hi[2], hi[3]}, {hi[4], hi[5], hi[6], hi[7]}};
        const uint4 al[2] = {{lo[0], lo[1], lo[2], lo[3]}, {lo[4], lo[5], lo[6], lo[7]}};
#pragma unroll
        for (int sp = 0; sp < 2; ++sp)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                accS[tt] = mfma32(ah[sp], f.h[sp][tt], accS[tt]);
                accS[tt] = mfma32(al[sp], f.h[sp][tt], accS[tt]);
                if constexpr (!EXACT) accS[tt] = mfma32(ah[sp], f.l[sp][tt], accS[tt]);
            }
    };
    // The registers of head size 128 do not hold the operands of K' and V' at once: the barriers to scheduling
    // keep the loads of one behind the products of the other there.
    constexpr bool V_EARLY = D <= 64;
    auto behind = [&]() { if constexpr (!V_EARLY) __builtin_amdgcn_sched_barrier(0); };
    auto raise = [&](const floatx16& e) {
#pragma unroll
        for (int g = 0; g < 16; ++g) c = fmaxf(c, e[g]);
    };
    auto set_shift = [&]() {
        c = half_max(c);
        shift = c == -INFINITY ? 0.f : c;
    };
    const int nt = kt1 - kt0;
    if constexpr (!ELU) c = -INFINITY;
    // Ranges of up to KEEP tiles (one or two is what the plan aims for) are evaluated once and kept in registers between
    // the maximum and the accumulation, the first tile's loads in flight together; longer ranges are evaluated twice.
    if (nt <= KEEP) {
        floatx16 ev[KEEP];
        KFrag kf;
        VFrag vf;
        load_k(kt0, kf);
        if constexpr (V_EARLY) load_v(kt0, vf);
        ev[0] = tile_values(kt0, kf);
        behind();
#pragma unroll
        for (int i = 1; i < KEEP; ++i)
            if (i < nt) {
                load_k(kt0 + i, kf);
                ev[i] = tile_values(kt0 + i, kf);
            }
        behind();
        if constexpr (!V_EARLY) load_v(kt0, vf);
        if constexpr (!ELU) {
            raise(ev[0]);
#pragma unroll
            for (int i = 1; i < KEEP; ++i)
                if (i < nt) raise(ev[i]);
            set_shift();
        }
        accumulate(ev[0], vf);
        behind();
#pragma unroll
        for (int i = 1; i < KEEP; ++i)
            if (i < nt) {
                load_v(kt0 + i, vf);
                accumulate(ev[i], vf);
            }
    } else {
        KFrag kf;
        if constexpr (!ELU) {
            for (int kt = kt0; kt < kt1; ++kt) {
                load_k(kt, kf);
                raise(tile_values(kt, kf));
            }
            set_shift();
        }
        for (int kt = kt0; kt < kt1; ++kt) {
            VFrag vf;
            load_k(kt, kf);
            if constexpr (V_EARLY) load_v(kt, vf);
            const floatx16 e = tile_values(kt, kf);
            behind();
            if constexpr (!V_EARLY) load_v(kt, vf);
            accumulate(e, vf);
            behind();
        }
    }
    zsum = half_sum(zsum);

    // this range's partial results into LDS: S tile [feature][t], then z[32], c[32]
    float* const mine = ks_lds + kr * L::range_floats;
    if (half == 0) {
        mine[32 * L::s_pitch + l32] = zsum;
        mine[32 * L::s_pitch + 32 + l32] = c;
    }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int g = 0; g < 16; ++g) {
            const int f = 8 * (g >> 2) + 4 * half + (g & 3);
            mine[f * L::s_pitch + 32 * tt + l32] = accS[tt][g];
        }
    }
    __syncthreads();

    // Merge of the key ranges, by the whole workgroup, thread = (feature, 4 coordinates):
    //   c_j = max_r c_jr,  S_j = sum_r exp(c_jr - c_j) S_jr,  z_j likewise
    //   St (d x mf) bf16: St[t][slot] = S[feature(slot)][t];  zp: z in accumulator order of a tile
    // For the random-feature map the query stream works with p'_ij = p_ij z_j, so that its denominator
    // is the plain sum of p': St holds S_j / z_j, and cw the exponent shift c_j + ln z_j as three bf16
    // terms (it enters the query kernel's first contraction as extra reduction slots against ones).
    // The slot -> feature order inside each group of 16 is the order in which the first MFMA of the
    // query-stream kernel hands P^T on as the B operand of the second (slot_of_feature_tile; natural for elu1).
    const int KR = a.KR, tid = threadIdx.x, nthreads = blockDim.x;
    const int fl = tid & 31, f = 32 * ft + fl;
    const bool real = f < a.mf;                  // a feature of the padding: weight exp(-1e30) = 0 in the query stream
    const float* const pz = ks_lds + 32 * L::s_pitch + fl;      // + range: z, + 32: c
    float w[KS_WAVES], cm = -INFINITY, zs = 0.f;
#pragma unroll
    for (int r = 0; r < KS_WAVES; ++r) {
        w[r] = pz[(r < KR ? r : 0) * L::range_floats + 32];
        cm = fmaxf(cm, w[r]);
    }
#pragma unroll
    for (int r = 0; r < KS_WAVES; ++r) {
        const float zr = pz[(r < KR ? r : 0) * L::range_floats];
        w[r] = r >= KR ? 0.f : ELU ? 1.f : expf(w[r] - cm);
        if (r < KR) zs = fmaf(w[r], zr, zs);
    }
    if (tid < 32) {
        if (real) {
            a.z[(long)bh * a.mf + f] = zs;
            a.c[(long)bh * a.mf + f] = cm;
        }
        // accumulator order of a 32-feature tile: position 16*h + g <-> feature 8*(g/4) + 4*h + g%4
        int pos = tid;
        if constexpr (!ELU) pos = 16 * ((tid >> 2) & 1) + 4 * (tid >> 3) + (tid & 3);
        a.zp[(long)bh * a.mfp + 32 * ft + pos] = zs;
        if constexpr (!ELU) {
            uint16_t hi, mid, lo;
            split3(real ? cm + logf(zs) : -1e30f, hi, mid, lo);
            uint2 pk;
            pk.x = (uint32_t)hi | ((uint32_t)mid << 16);
            pk.y = (uint32_t)lo;
            *(uint2*)(a.cw + ((long)bh * a.mfp + f) * 4) = pk;
        }
    }
    const float zinv = ELU ? 1.f : (real ? 1.f / zs : 0.f);
    uint16_t* const st = a.St + (long)bh * D * a.mfp + 32 * ft + (ELU ? fl : slot_of_feature_tile(fl));
    for (int t = 4 * (tid >> 5); t < D; t += nthreads / 8) {
        float4 sv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < KS_WAVES; ++r) {
            if (r >= KR) break;
            const float4 x = *(const float4*)(ks_lds + r * L::range_floats + fl * L::s_pitch + t);
            sv.x = fmaf(w[r], x.x, sv.x); sv.y = fmaf(w[r], x.y, sv.y);
            sv.z = fmaf(w[r], x.z, sv.z); sv.w = fmaf(w[r], x.w, sv.w);
        }
        if (real) *(float4*)(a.S + ((long)bh * a.mf + f) * D + t) = sv;
        const uint32_t p0 = pack_bf16(sv.x * zinv, sv.y * zinv), p1 = pack_bf16(sv.z * zinv, sv.w * zinv);
        st[(long)t * a.mfp] = (uint16_t)p0;
        st[(long)(t + 1) * a.mfp] = (uint16_t)(p0 >> 16);
        st[(long)(t + 2) * a.mfp] = (uint16_t)p1;
        st[(long)(t + 3) * a.mfp] = (uint16_t)(p1 >> 16);
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
KeyStatePlan key_state_plan(const Problem& p) {
    KeyStatePlan q;
    q.kpad = (p.k + 31) / 32 * 32;
    q.FT = p.mfp / 32;
    const int KT = q.kpad / 32;
    // Key ranges = wavefronts of a workgroup, at most KS_WAVES (the ranges' partial tiles meet in LDS): one key tile
    // each while the chip holds them all at once (two wavefronts per SIMD), two each otherwise.  Ranges of more tiles
    // than the kernel keeps are evaluated twice (maximum, then accumulation).
    int KR = KT < KS_WAVES ? KT : KS_WAVES;
    if ((long)p.BH * q.FT * KR > 8L * chip_cus() && KR > (KT + 1) / 2) KR = (KT + 1) / 2;
    q.tiles_per_range = (KT + KR - 1) / KR;
    q.KR = (KT + q.tiles_per_range - 1) / q.tiles_per_range;
    return q;
}

template <int D, bool ELU, bool EXACT, int KEEP = KS_KEEP>
static flurka_status launch_key_state_impl(const Problem& p, const KeyStateArgs& ka, hipStream_t s) {
    auto kern = key_state_kernel<D, ELU, EXACT, KEEP>;
    const int ldsb = KeyStateLds<D>::total(ka.KR);
    const int waves = ka.KR < KS_MERGERS ? KS_MERGERS : ka.KR;
    KernelFacts facts;
    if (!kernel_facts((const void*)kern, waves * 64, ldsb, &facts)) return FLURKA_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)((p.BH + 7) / 8 * 8 * ka.FT)), dim3(waves * 64), ldsb, s, ka);
    FLURKA_CHECK_LAUNCH();
    return FLURKA_OK;
}

template <int D>
static flurka_status launch_key_state(const Problem& p, const KeyStateArgs& ka, bool exact, hipStream_t s) {
    if (exact) return p.elu ? launch_key_state_impl<D, true, true>(p, ka, s) : launch_key_state_impl<D, false, true>(p, ka, s);
    if constexpr (D == 64) {
        // 513 to 1024 keys: three or four tiles a range
        if (!p.elu && ka.tiles_per_range > KS_KEEP && ka.tiles_per_range <= KS_KEEP_LONG)
            return launch_key_state_impl<D, false, false, KS_KEEP_LONG>(p, ka, s);
    }
    return p.elu ? launch_key_state_impl<D, true, false>(p, ka, s) : launch_key_state_impl<D, false, false>(p, ka, s);
}

flurka_status fast_proj_finish(const Problem& p, float* ctx, const float* partials, const PartialTile& tile, int tilesM, int tilesN,
                               int splits, bool images, const KeyStateBuffers& b, hipStream_t s) {
    const CtxLayout L = ctx_layout(p);
    const KeyStatePlan q = key_state_plan(p);
    StageScope sc(s, STAGE_K_PROJ_FINISH);
    FinishArgs fa{};
    fa.part = partials; fa.ctx = ctx; fa.tile = tile; fa.tilesM = tilesM; fa.tilesN = tilesN;
    fa.Kp_off = (long)L.Kp; fa.Vp_off = (long)L.Vp;
    fa.Kimg = (p.elu || !images) ? nullptr : b.Kimg; fa.Vimg = images ? b.Vimg : nullptr;
    fa.nrm = (p.elu || !images) ? nullptr : b.nrm;
    fa.splits = splits; fa.k = p.k; fa.kpad = q.kpad; fa.d = p.d; fa.BH = p.BH;
    const long waves = (long)p.BH * (q.kpad / 4);
    hipLaunchKernelGGL(proj_finish_kernel, grid1d(waves, 4), dim3(256), 0, s, fa);
    FLURKA_CHECK_LAUNCH();
    return FLURKA_OK;
}

flurka_status fast_key_state(const Problem& p, const void* omega, float* ctx, const float* partials,
                             const PartialTile& tile, int tilesM, int tilesN, int splits, const KeyStateBuffers& b, hipStream_t s) {
    const CtxLayout L = ctx_layout(p);
    const KeyStatePlan q = key_state_plan(p);
    {
        const flurka_status st = fast_proj_finish(p, ctx, partials, tile, tilesM, tilesN, splits, true, b, s);
        if (st != FLURKA_OK) return st;
    }
    {
        StageScope sc(s, STAGE_K_KEY_STATE);
        KeyStateArgs ka{};
        ka.Kimg = b.Kimg; ka.Kp = ctx + L.Kp; ka.Vimg = b.Vimg; ka.nrm = b.nrm;
        ka.omega = (const uint16_t*)omega;
        ka.S = ctx + L.S; ka.z = ctx + L.z; ka.c = ctx + L.c;
        ka.St = b.St; ka.zp = b.zp; ka.cw = b.cw;
        ka.omega_head_stride = p.omega_per_head ? (long)p.m * p.d : 0;
        ka.BH = p.BH; ka.H = p.H; ka.k = p.k; ka.kpad = q.kpad; ka.mf = p.mf; ka.mfp = p.mfp;
        ka.FT = q.FT; ka.KR = q.KR; ka.tiles_per_range = q.tiles_per_range;
        flurka_status st = p.d == 64 ? launch_key_state<64>(p, ka, false, s) : launch_key_state<128>(p, ka, false, s);
        if (st != FLURKA_OK) return st;
    }
    return FLURKA_OK;
}

// ---------------------------------------------------------------------------
// Kernel attention without a sequence projection (K' = K, V' = V): the keys and values are the caller's
// bf16 tensors.  identity_pack writes what key_state reads -- K in its operand order (one term), V with
// two consecutive keys per dword (one term), |k|^2 / 2 -- one wavefront per four keys, lane = coordinate.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void identity_pack_kernel(const uint16_t* K, const uint16_t* V, uint16_t* Kimg,
                                                            uint32_t* Vimg, float* nrm, int n, int d, int BH) {
    const int lane = threadIdx.x & 63;
    const long wid = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int groups_per_head = n / 4;
    if (wid >= (long)BH * groups_per_head) return;
    const int bh = (int)(wid / groups_per_head);
    const int r0 = 4 * (int)(wid % groups_per_head);
    float sq[4] = {0.f, 0.f, 0.f, 0.f};
    for (int t = lane; t < d; t += 64) {
        uint16_t kv[4], vv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const long off = ((long)bh * n + r0 + e) * d + t;
            kv[e] = K[off];
            vv[e] = V[off];
            const float x = bf16_to_f32(kv[e]);
            sq[e] = fmaf(x, x, sq[e]);
            const int r = r0 + e;
            if (Kimg) {
                Kimg[(long)bh * n * d + k_image_offset(r, t, d)] = kv[e];
            }
        }
#pragma unroll
        for (int pr = 0; pr < 2; ++pr)
            Vimg[(long)bh * (n / 2) * d + v_image_offset(r0 / 2 + pr, t, d)] = (uint32_t)vv[2 * pr] | ((uint32_t)vv[2 * pr + 1] << 16);
    }
    if (nrm) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float tot = wave_sum(sq[e]);
            if (lane == 0) nrm[(long)bh * n + r0 + e] = 0.5f * tot;
        }
    }
}

// p.k == p.n here: every position is a key.  Fills S, z, c in ctx and the St/zp/cw images.
flurka_status fast_identity_key_state(const Problem& p, const void* K, const void* V, const void* omega, float* S,
                                      float* z, float* c, const KeyStateBuffers& b, hipStream_t s) {
    const KeyStatePlan q = key_state_plan(p);
    {
        StageScope sc(s, STAGE_K_IDENTITY_PACK);
        const long waves = (long)p.BH * (p.n / 4);
        hipLaunchKernelGGL(identity_pack_kernel, grid1d(waves, 4), dim3(256), 0, s, (const uint16_t*)K, (const uint16_t*)V,
                           p.elu ? (uint16_t*)nullptr : b.Kimg, b.Vimg, p.elu ? (float*)nullptr : b.nrm, p.n, p.d, p.BH);
        FLURKA_CHECK_LAUNCH();
    }
    StageScope sc(s, STAGE_K_KEY_STATE);
    KeyStateArgs ka{};
    ka.Kimg = b.Kimg; ka.Kp = nullptr; ka.Kb = (const uint16_t*)K; ka.Vimg = b.Vimg; ka.nrm = b.nrm;
    ka.omega = (const uint16_t*)omega;
    ka.S = S; ka.z = z; ka.c = c;
    ka.St = b.St; ka.zp = b.zp; ka.cw = b.cw;
    ka.omega_head_stride = p.omega_per_head ? (long)p.m * p.d : 0;
    ka.BH = p.BH; ka.H = p.H; ka.k = p.k; ka.kpad = q.kpad; ka.mf = p.mf; ka.mfp = p.mfp;
    ka.FT = q.FT; ka.KR = q.KR; ka.tiles_per_range = q.tiles_per_range;
    return p.d == 64 ? launch_key_state<64>(p, ka, true, s) : launch_key_state<128>(p, ka, true, s);
}

}  // namespace flurka
