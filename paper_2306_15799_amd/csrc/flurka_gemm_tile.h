// bf16 MFMA GEMM main loop for gfx950 with output tiles of 64 x 128 to 128 x 256: the contractions over the
// sequence for which the 256 x 256 tile of flurka_gemm.h is too coarse.
//
// That tile keeps 256 KiB of sums per compute unit, so a reduction split over the whole chip leaves 64 MiB of fp32
// partial results whatever the size of the problem (13 us to write and 14 us to read again), and a small problem
// fills a fraction of the rows it pays for.  A smaller tile leaves a quarter to a half of that; what it costs is
// operand traffic between L2 and the compute units (a 128 x 128 tile needs twice the bytes per product).
//
// Structure: operands go from memory straight into LDS (no staging registers), NST buffers of one 64-deep step each;
// wavefronts hold 64 x 64 (32 x 64) of the tile.  A step is four 16-deep sub-steps.  While sub-step s multiplies, the
// fragments of the sub-step three later are read from LDS into one of four register sets (three products' time is
// shorter than an LDS read under load: with one sub-step of distance a step took 1250 cycles, 512 of them products),
// and the transfers of the step NST later go out between the products of sub-steps 1 to 3.  One barrier per step,
// behind sub-step 0: the next buffer has landed (this wavefront waits for its own transfers, the barrier for the
// others') and the current one has been read to the end, so that its transfers may go out.
//
// Bounds, measured on MI355X: 128 x 128 takes 0.57 - 0.6 us per step and workgroup with a compute unit to itself
// (operands 0.60 us alone, products 0.39 us alone: a compute unit takes in 54 - 57 GB/s of such tiles, however many
// transfers are in flight: 3, 4 and 5 buffers are equally fast), 128 x 256 0.95 us, against 1.78 us for four times
// the products with the 256 x 256 tile, which stays the faster one where the matrix rate is the bound.
#pragma once

#include "flurka_gemm.h"

namespace flurka {

// Descriptor of a byte range, as four scalar registers
__device__ __forceinline__ u32x4 tile_rsrc(const void* base, unsigned bytes) {
    const unsigned long p = (unsigned long)base;
    return u32x4{(unsigned)__builtin_amdgcn_readfirstlane((int)p), (unsigned)__builtin_amdgcn_readfirstlane((int)(p >> 32)) & 0xffffu,
                 (unsigned)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
}

// 16 bytes per lane from a buffer straight into LDS, lane l's at dst + 16 * l; addresses past the descriptor's
// range store zero.  Written as an instruction of its own because the compiler puts a wait for every transfer
// in flight before any LDS read that follows the builtin, which would leave nothing in flight; nothing comes
// back in registers, and wait_and_barrier below is what the reads of the data stand behind.
// What the compiler does between instructions of its own is done here: a write of m0 (the LDS address) and its use are
// one wait state apart, and a scalar register written by a vector instruction (v_readfirstlane, or v_readlane of a
// spilled one) and a vector memory instruction that reads it are five apart, whatever stands before the block: two
// scalar additions and s_nop 2.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"      // m0 is a register the allocator leaves alone: named all the same
template <int DST>
__device__ __forceinline__ void lds_dma16(const u32x4& r, unsigned lds_dst, int voff, int soff, int js) {
    // wave-uniform values all of them; said so for builds that do not find out
    lds_dst = __builtin_amdgcn_readfirstlane(lds_dst);
    soff = __builtin_amdgcn_readfirstlane(soff);
    js = __builtin_amdgcn_readfirstlane(js);
    int t;
    asm volatile("s_add_u32 m0, %1, %2\n\ts_add_u32 %0, %3, %4\n\ts_nop 2\n\tbuffer_load_dwordx4 %5, %6, %0 offen lds"
                 : "=&s"(t)
                 : "s"(lds_dst), "n"(DST), "s"(soff), "s"(js), "v"(voff), "s"(r)
                 : "scc", "m0", "memory");
}
#pragma clang diagnostic pop

// s_waitcnt vmcnt(N) lgkmcnt(0), then the workgroup barrier: this wavefront's transfers but the last N have
// landed and its LDS reads are done, and so are everybody else's once the barrier opens.
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

constexpr int T_BK = 64;
// Wavefronts of a workgroup: WM x WN, each 64 x 64 of the tile (32 x 64 of a 64-row one)
template <int TM, int TN>
struct TileShape {
    static constexpr int WR = TM == 64 ? 32 : 64, WC = 64, WM = TM / WR, WN = TN / WC, NW = WM * WN;
    static constexpr int JA = TM / (8 * NW), JB = TN / (8 * NW);        // 1 KiB transfers per wavefront and step
    static constexpr int a_bytes = TM * T_BK * 2, b_bytes = TN * T_BK * 2, stage = a_bytes + b_bytes;
    static constexpr int lds(int nst, bool tstore) { return nst * stage + (tstore ? NW * 4096 : 0); }
};

// What a lane fetches in transfer 0 of a wavefront: row-major operand, row of the tile and element of its 64;
// transposed operand, row (position) and column.  16-byte chunk c of a row sits at chunk position c ^ x:
//   row-major, 128-byte rows        x = (row / 2) % 8                      plain reads down a column of rows
//   transposed, 256-byte or longer  x = 4 * (row % 4) + (row / 4) % 4      transposing reads of 4 rows x 64 bytes
// Both leave a wavefront's LDS reads without bank conflicts, and both are the same for all transfers of a lane.
__device__ __forceinline__ int tile_a_row(int lane, int wave) { return 8 * wave + (lane >> 3); }
__device__ __forceinline__ int tile_a_elem(int lane, int wave) { return 8 * ((lane & 7) ^ (4 * (wave & 1) + (lane >> 4))); }
__device__ __forceinline__ int tile_b_row(int lane, int wave, int tn) { return tn == 128 ? 4 * wave + (lane >> 4) : 2 * wave + (lane >> 5); }
__device__ __forceinline__ int tile_b_col(int lane, int wave, int tn) {
    const int r = tile_b_row(lane, wave, tn), x = 4 * (r & 3) + ((r >> 2) & 3);
    return 8 * ((lane & (tn / 8 - 1)) ^ x);
}

// f(IC<0>{}), ..., f(IC<N - 1>{})
template <int N, class F, int... I>
__device__ __forceinline__ void unroll(F&& f) {
    if constexpr (sizeof...(I) == N) (f(IC<I>{}), ...);
    else unroll<N, F, I..., (int)sizeof...(I)>(static_cast<F&&>(f));
}

// Work items and their order: id mod 8 (the XCD) is the low part of (tile along the large operand, which, split),
// the tiles that share a tile of the large operand follow, so that they run on one XCD at about the same time and
// that tile leaves HBM once, and each XCD keeps to few ranges of the other operand.
struct TileItem { int split, tm, tn, which; bool valid; };
template <bool SHARE_A>
__host__ __device__ inline TileItem tile_item(const GemmParams& g, int id, int item_hi) {
    TileItem it;
    it.valid = id < item_hi;
    if (!it.valid) id = 0;
    const int xcd = id & 7; id >>= 3;
    const int shared = SHARE_A ? g.tilesN : g.tilesM;         // tiles that read the same large operand
    const int inner = id % shared; id /= shared;
    int u = 8 * id + xcd;                                     // (tile along the large operand, which, split)
    it.split = u % g.splits;  u /= g.splits;
    it.which = u & 1;
    int outer = u >> 1;
    // Only past the last real item of a workgroup.  Such an id still names a tile that exists: addresses and descriptor
    // ranges are formed for it too, and a range computed for heads past the last one would wrap to nearly 4 GiB,
    // which G_OOB lies inside of.
    if (outer >= (SHARE_A ? g.tilesM : g.tilesN)) { it.valid = false; outer = 0; }
    it.tm = SHARE_A ? outer : inner;
    it.tn = SHARE_A ? inner : outer;
    return it;
}

// A workgroup's items are streamed: the transfers run NST steps ahead of the products, into the next item.  nblocks
// is a multiple of 8 or the item count; item_lo is a multiple of 8.
template <class Pol, int NST>
__device__ __forceinline__ void gemm_tile_body(const GemmParams& g, const int block, const int nblocks,
                                               unsigned char* const lds, const int item_lo, const int item_hi) {
    constexpr int TM = Pol::TM, TN = Pol::TN;
    constexpr bool BT = Pol::B_TRANSPOSE;
    using L = TileShape<TM, TN>;
    static_assert(!BT || TN == 128 || (TN == 256 && L::NW == 8), "swizzle of the transposed rows");
    constexpr int FI = L::WR / 32, FJ = L::WC / 32;      // 32 x 32 tiles of a wavefront
    constexpr int JA = L::JA, JB = L::JB, NW = L::NW;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / L::WN, wn = wave % L::WN;
    const int half = lane >> 5, l32 = lane & 31, s16 = lane & 15, r4 = s16 >> 2;

    struct Item : TileItem { int step0, step1; };
    auto decode = [&](int id) -> Item {
        Item it;
        (TileItem&)it = tile_item<Pol::SHARE_A>(g, id, item_hi);
        it.step0 = it.split * g.steps_per_split;
        it.step1 = it.step0 + g.steps_per_split;
        if (it.step1 > g.total_steps) it.step1 = g.total_steps;
        return it;
    };

    // load side: item, step and addresses of the next transfer
    int lid = item_lo + block;
    Item li = decode(lid);
    typename Pol::Ctx lc = Pol::make(g, li.which, li.tm * TM, li.tn * TN, lane, wave);
    int lstep = li.step0;
    const unsigned lds0 = (unsigned)(unsigned long)(__attribute__((address_space(3))) unsigned char*)lds;
    int sA = 0, sB = 0, vA = G_OOB, vB[JB];
    // offsets of the load step
    auto load_step = [&]() {
        sA = Pol::a_soff(lc, lstep);
        sB = Pol::b_soff(lc, lstep);
        if constexpr (Pol::B_ROW_LIMIT) {
            if ((lstep + 1) * T_BK > lc.b_rows) {          // a ragged last step: only the rows that exist
#pragma unroll
                for (int j = 0; j < JB; ++j)
                    if (lstep * T_BK + tile_b_row(lane, wave, TN) + j * (NW * 512 / TN) >= lc.b_rows) vB[j] = G_OOB;
            }
        }
    };
    auto load_item = [&]() {
        vA = li.valid ? lc.voffA : G_OOB;
#pragma unroll
        for (int j = 0; j < JB; ++j) vB[j] = li.valid ? lc.voffB : G_OOB;
    };
    load_item();
    load_step();
    // one 1 KiB transfer of the load step: j < JA of A, then of B
    auto dma = [&](unsigned dst, auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (j < JA) lds_dma16<1024 * NW * j>(lc.rsA, dst, vA, sA, j * lc.a_js);
        else                  lds_dma16<L::a_bytes + 1024 * NW * (j - JA)>(lc.rsB, dst, vB[j - JA], sB, (j - JA) * lc.b_js);
    };
    auto dma_dst = [&](int buf) -> unsigned { return lds0 + buf * L::stage + wave * 1024; };
    auto load_advance = [&]() {
        if (!li.valid) return;
        if (++lstep == li.step1) {
            lid += nblocks;
            li = decode(lid);
            lc = Pol::make(g, li.which, li.tm * TM, li.tn * TN, lane, wave);
            lstep = li.step0;
            load_item();
        }
        load_step();
    };

    // fragment reads: fragment f < FI of A, then of B, of 16-deep sub-step s
    const int fa = (wm * L::WR + l32) * 128, fx = 16 * (((l32 >> 1) & 7) ^ half);             // + 32*i rows
    const int fb = L::a_bytes + (wn * L::WC + l32) * 128;                              // direct B
    const int bt = L::a_bytes + (8 * half + r4) * (2 * TN) + 8 * (s16 & 1);
    const int bt_c = wn * (L::WC / 8) + 2 * ((lane >> 4) & 1) + ((s16 >> 1) & 1), bt_x = 4 * r4 + 2 * half;
    uint4 FR[4][FI + FJ];
    auto frag = [&](int set, const unsigned char* p, int s, int f) {
        if (f < FI) {
            FR[set][f] = *(const uint4*)(p + fa + 4096 * f + (fx ^ (32 * s)));
        } else if constexpr (BT) {
            const int c = bt_c + 4 * (f - FI);
            const uint2 lo = gemm_read_tr16(p + bt + 32 * TN * s + 16 * (c ^ bt_x));
            const uint2 hi = gemm_read_tr16(p + bt + 32 * TN * s + 8 * TN + 16 * (c ^ (bt_x | 1)));
            FR[set][f] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        } else {
            FR[set][f] = *(const uint4*)(p + fb + 4096 * (f - FI) + (fx ^ (32 * s)));
        }
    };

    floatx16 acc[FI][FJ];
    constexpr int MF = FI * FJ, FN = FI + FJ, JN = JA + JB;
    // sub-step S: its products, between them the fragments of the sub-step three later (of buffer p) and
    // transfers LO .. HI - 1 of the load step to dst
    auto substep = [&](auto sc, const unsigned char* p, unsigned dst, auto loc, auto hic) {
        constexpr int S = decltype(sc)::value, NS = (S + 3) & 3, LO = decltype(loc)::value, HI = decltype(hic)::value;
        // the reads that the barrier behind sub-step 0 waits for go out early
        constexpr int FM = S == 0 ? (MF + 1) / 2 : MF;
        unroll<MF>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            acc[m / FJ][m % FJ] = mfma32(FR[S][m / FJ], FR[S][FI + m % FJ], acc[m / FJ][m % FJ]);
            constexpr int f0 = m < FM ? m * FN / FM : FN, f1 = m < FM ? (m + 1) * FN / FM : FN;
            unroll<f1 - f0>([&](auto f) { frag(NS, p, NS, f0 + decltype(f)::value); });
            constexpr int j0 = LO + m * (HI - LO) / MF, j1 = LO + (m + 1) * (HI - LO) / MF;
            unroll<j1 - j0>([&](auto j) { dma(dst, IC<j0 + decltype(j)::value>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };

    auto epilogue = [&](const Item& it) {
        if constexpr (Pol::PARTIAL_TILES) {
            float* tp = (float*)g.C[0] +
                        partial_tile_index(it.which, it.split, it.tn, it.tm, g.splits, g.tilesN, g.tilesM) * (TM * TN) +
                        (long)wave * (FI * FJ * 1024) + lane * 4;
#pragma unroll
            for (int i = 0; i < FI; ++i)
#pragma unroll
                for (int j = 0; j < FJ; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float4 v;
                        v.x = acc[i][j][4 * q]; v.y = acc[i][j][4 * q + 1]; v.z = acc[i][j][4 * q + 2]; v.w = acc[i][j][4 * q + 3];
                        *(float4*)(tp + ((i * FJ + j) * 4 + q) * 256) = v;
                    }
        } else {
            static_assert(!Pol::TRANSPOSED_STORE || FI == 2, "64 rows of a wavefront leave together");
            unsigned char* const tr = lds + NST * L::stage + wave * 4096;
#pragma unroll
            for (int j = 0; j < FJ; ++j) {
#pragma unroll
                for (int ii = 0; ii < 2; ++ii)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const floatx16& t = acc[ii][j];
                        uint2 v;
                        v.x = pack_bf16(t[4 * q], t[4 * q + 1]);
                        v.y = pack_bf16(t[4 * q + 2], t[4 * q + 3]);
                        *(uint2*)(tr + l32 * 128 + 16 * ((4 * ii + q) ^ ((l32 >> 1) & 7)) + 8 * half) = v;
                    }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = 8 * u + (lane >> 3), k = lane & 7;
                    const uint4 v = *(const uint4*)(tr + c * 128 + 16 * (k ^ ((c >> 1) & 7)));
                    Pol::store_rows(g, it.which, it.tm * TM + wm * L::WR, it.tn * TN + wn * L::WC + 32 * j + c, k, v);
                }
            }
        }
    };

    Item ci = li;
    int cid = lid, buf = 0;
    if (!ci.valid) return;
#pragma unroll
    for (int i = 0; i < NST; ++i) {
        unroll<JN>([&](auto j) { dma(dma_dst(i), j); });
        load_advance();
    }
    wait_and_barrier<(NST - 1) * JN>();
    unroll<3 * FN>([&](auto f) { frag(decltype(f)::value / FN, lds, decltype(f)::value / FN, decltype(f)::value % FN); });
    __builtin_amdgcn_sched_barrier(0);
    while (ci.valid) {
#pragma unroll
        for (int i = 0; i < FI; ++i)
#pragma unroll
            for (int j = 0; j < FJ; ++j) acc[i][j] = zero16();
        for (int step = ci.step0; step < ci.step1; ++step) {
            const int next = buf + 1 == NST ? 0 : buf + 1;
            const unsigned dst = dma_dst(buf);
            const unsigned char* const pn = lds + next * L::stage;
            substep(IC<0>{}, lds + buf * L::stage, dst, IC<0>{}, IC<0>{});
            wait_and_barrier<(NST - 2) * JN>();       // the next buffer is complete, this one read to the end
            substep(IC<1>{}, pn, dst, IC<0>{}, IC<JN / 3>{});
            substep(IC<2>{}, pn, dst, IC<JN / 3>{}, IC<2 * JN / 3>{});
            substep(IC<3>{}, pn, dst, IC<2 * JN / 3>{}, IC<JN>{});
            load_advance();
            buf = next;
        }
        epilogue(ci);
        cid += nblocks;
        ci = decode(cid);
    }
    wait_and_barrier<0>();          // transfers past the last item have landed (as zeros)
}

// ---------------------------------------------------------------------------
// Policies.  make(g, which, m0, n0, lane, wave) gives the descriptors, this lane's byte offsets and the byte
// stride between the 1 KiB transfers of a step:
//   row-major operand (A, direct B): transfer j of a wavefront is rows 8*NW*j + 8*wave .. + 7 of the tile
//   transposed B: transfer j is positions (512/TN)*(NW*j + wave) .. + 512/TN - 1 (4 at TN = 128, 2 at TN = 256)
// ---------------------------------------------------------------------------
struct TileCtx {
    u32x4 rsA, rsB;
    int voffA, voffB, a_js, b_js;
    int b_rows, b_step;
};
// K' = E K
template <int D, int TM_, int TN_>
struct TProjPolicy {
    static constexpr int TM = TM_, TN = TN_, NW = TileShape<TM, TN>::NW;
    static constexpr bool SHARE_A = false, B_TRANSPOSE = true, PARTIAL_TILES = true, TRANSPOSED_STORE = false, B_ROW_LIMIT = true;
    struct Ctx : TileCtx {};
    static __device__ __forceinline__ Ctx make(const GemmParams& g, int which, int m0, int n0, int lane, int wave) {
        Ctx c;
        const int bh0 = n0 / D;
        int heads = g.BH - bh0;
        if (heads > TN / D) heads = TN / D;
        c.rsA = tile_rsrc(g.A[which], (unsigned)g.k * (unsigned)g.n * 2u);
        c.rsB = tile_rsrc(g.B[which] + (long)bh0 * g.n * D, (unsigned)heads * (unsigned)g.n * (unsigned)(D * 2));
        c.voffA = ((m0 + tile_a_row(lane, wave)) * g.n + tile_a_elem(lane, wave)) * 2;
        c.a_js = NW * 16 * g.n;
        const int col = tile_b_col(lane, wave, TN);
        c.voffB = (((col / D) * g.n + tile_b_row(lane, wave, TN)) * D + col % D) * 2;
        c.b_js = (NW * 512 / TN) * D * 2;
        c.b_rows = g.n;
        return c;
    }
    static __device__ __forceinline__ int a_soff(const Ctx&, int step) { return step * (T_BK * 2); }
    static __device__ __forceinline__ int b_soff(const Ctx&, int step) { return step * (T_BK * D * 2); }
};

// Y = E X on the model-wide input
template <int TM_, int TN_>
struct TWidePolicy {
    static constexpr int TM = TM_, TN = TN_, NW = TileShape<TM, TN>::NW;
    static constexpr bool SHARE_A = false, B_TRANSPOSE = true, PARTIAL_TILES = true, TRANSPOSED_STORE = false, B_ROW_LIMIT = true;
    struct Ctx : TileCtx {};
    static __device__ __forceinline__ Ctx make(const GemmParams& g, int which, int m0, int n0, int lane, int wave) {
        Ctx c;
        const int tn = n0 / TN, b = tn / g.tiles_per_batch, c0 = (tn % g.tiles_per_batch) * TN;
        c.rsA = tile_rsrc(g.A[which], (unsigned)g.k * (unsigned)g.n * 2u);
        c.rsB = tile_rsrc(g.B[which] + (long)b * g.n * g.dm, (unsigned)g.n * (unsigned)g.dm * 2u);
        c.voffA = ((m0 + tile_a_row(lane, wave)) * g.n + tile_a_elem(lane, wave)) * 2;
        c.a_js = NW * 16 * g.n;
        // columns past dm (a ragged last tile) read the next position's values or zero, and nobody uses
        // those columns of the result
        c.voffB = (tile_b_row(lane, wave, TN) * g.dm + c0 + tile_b_col(lane, wave, TN)) * 2;
        c.b_js = (NW * 512 / TN) * g.dm * 2;
        c.b_step = T_BK * 2 * g.dm;
        c.b_rows = g.n;
        return c;
    }
    static __device__ __forceinline__ int a_soff(const Ctx&, int step) { return step * (T_BK * 2); }
    static __device__ __forceinline__ int b_soff(const Ctx& c, int step) { return step * c.b_step; }
};

// K' = Y W^K per head, Y as three bf16 terms
template <int TM_, int TN_>
struct TTransformPolicy {
    static constexpr int TM = TM_, TN = TN_, NW = TileShape<TM, TN>::NW;
    static constexpr bool SHARE_A = false, B_TRANSPOSE = false, PARTIAL_TILES = true, TRANSPOSED_STORE = false, B_ROW_LIMIT = false;
    struct Ctx : TileCtx { int steps_per_term; };
    static __device__ __forceinline__ Ctx make(const GemmParams& g, int which, int m0, int n0, int lane, int wave) {
        Ctx c;
        const int tn = n0 / TN, b = tn / g.tiles_per_batch, c0 = (tn % g.tiles_per_batch) * TN;
        const int row_bytes = 3 * g.dm * 2;
        c.rsA = tile_rsrc(g.A[which] + (long)b * g.k * 3 * g.dm, (unsigned)g.k * (unsigned)row_bytes);
        c.rsB = tile_rsrc(g.B[which], (unsigned)(g.tiles_per_batch * TN) * (unsigned)g.dm * 2u);
        c.voffA = (m0 + tile_a_row(lane, wave)) * row_bytes + 2 * tile_a_elem(lane, wave);
        c.a_js = NW * 8 * row_bytes;
        c.voffB = ((c0 + tile_a_row(lane, wave)) * g.dm + tile_a_elem(lane, wave)) * 2;
        c.b_js = NW * 16 * g.dm;
        c.steps_per_term = g.dm / T_BK;
        return c;
    }
    static __device__ __forceinline__ int a_soff(const Ctx&, int step) { return step * (T_BK * 2); }
    static __device__ __forceinline__ int b_soff(const Ctx& c, int step) { return (step % c.steps_per_term) * (T_BK * 2); }
};

// dK = E^T dK': rows = (head, t) of the (BH*D x kp) image, columns = positions, reduction = projected slots
template <int D, int TM_, int TN_>
struct TGradXPolicy {
    static constexpr int TM = TM_, TN = TN_, NW = TileShape<TM, TN>::NW;
    static constexpr bool SHARE_A = false, B_TRANSPOSE = true, PARTIAL_TILES = false, TRANSPOSED_STORE = true, B_ROW_LIMIT = false;
    struct Ctx : TileCtx {};
    static __device__ __forceinline__ Ctx make(const GemmParams& g, int which, int m0, int n0, int lane, int wave) {
        Ctx c;
        c.rsA = tile_rsrc(g.A[which], (unsigned)(g.BH * D) * (unsigned)g.kp * 2u);
        c.rsB = tile_rsrc(g.B[which], (unsigned)g.k * (unsigned)g.n * 2u);
        c.voffA = ((m0 + tile_a_row(lane, wave)) * g.kp + tile_a_elem(lane, wave)) * 2;
        c.a_js = NW * 16 * g.kp;
        c.voffB = (tile_b_row(lane, wave, TN) * g.n + n0 + tile_b_col(lane, wave, TN)) * 2;
        c.b_js = (NW * 512 / TN) * g.n * 2;
        c.b_step = T_BK * 2 * g.n;
        return c;
    }
    static __device__ __forceinline__ int a_soff(const Ctx&, int step) { return step * (T_BK * 2); }
    static __device__ __forceinline__ int b_soff(const Ctx& c, int step) { return step * c.b_step; }
    // rows r0 + 8*k .. + 7 (64 rows from r0 lie inside one head) of column col, as 8 bf16
    static __device__ __forceinline__ void store_rows(const GemmParams& g, int which, int r0, int col, int k,
                                                      const uint4& v) {
        if (col >= g.n || r0 >= g.BH * D) return;
        const int bh = r0 / D, t = r0 % D + 8 * k;
        *(uint4*)((uint16_t*)g.C[which] + ((long)bh * g.n + col) * D + t) = v;
    }
};

// dE = sum_bh dK' K^T, transposed: rows = positions (A = rows of K), columns = projected slots (B = rows of
// the (BH, kp, D) image), reduction = (head, t) pairs.  FINAL: not split, bf16 results to dE, dF.
template <int D, bool FINAL, int TM_, int TN_>
struct TGradEPolicy {
    static constexpr int TM = TM_, TN = TN_, NW = TileShape<TM, TN>::NW;
    static constexpr bool SHARE_A = true, B_TRANSPOSE = false, PARTIAL_TILES = !FINAL, TRANSPOSED_STORE = FINAL, B_ROW_LIMIT = false;
    struct Ctx : TileCtx { int a_batch, b_batch; };
    static __device__ __forceinline__ Ctx make(const GemmParams& g, int which, int m0, int n0, int lane, int wave) {
        Ctx c;
        c.rsA = tile_rsrc(g.A[which], (unsigned)g.BH * (unsigned)g.n * (unsigned)(D * 2));
        c.rsB = tile_rsrc(g.B[which], (unsigned)g.BH * (unsigned)g.kp * (unsigned)(D * 2));
        c.voffA = ((m0 + tile_a_row(lane, wave)) * D + tile_a_elem(lane, wave)) * 2;
        c.voffB = ((n0 + tile_a_row(lane, wave)) * D + tile_a_elem(lane, wave)) * 2;
        c.a_js = c.b_js = NW * 8 * D * 2;
        c.a_batch = g.n * D * 2;
        c.b_batch = g.kp * D * 2;
        return c;
    }
    static __device__ __forceinline__ int a_soff(const Ctx& c, int step) {
        constexpr int spb = D / T_BK;
        return (step / spb) * c.a_batch + (step % spb) * (T_BK * 2);
    }
    static __device__ __forceinline__ int b_soff(const Ctx& c, int step) {
        constexpr int spb = D / T_BK;
        return (step / spb) * c.b_batch + (step % spb) * (T_BK * 2);
    }
    // positions r0 + 8*k .. + 7 of slot col; n is a multiple of 32 here
    static __device__ __forceinline__ void store_rows(const GemmParams& g, int which, int r0, int col, int k,
                                                      const uint4& v) {
        if (col >= g.k || r0 + 8 * k >= g.n) return;
        *(uint4*)((uint16_t*)g.C[which] + (long)col * g.n + r0 + 8 * k) = v;
    }
};

// ids handed to workgroups: the (split, tile along the large operand, which) index padded to a multiple of 8
template <bool SHARE_A>
__host__ __device__ inline int tile_item_count(const GemmParams& g) {
    return SHARE_A ? 8 * g.tilesN * ((g.splits * g.tilesM * 2 + 7) / 8) : 8 * g.tilesM * ((g.splits * g.tilesN * 2 + 7) / 8);
}

template <class Pol, int NST>
__global__ __launch_bounds__(Pol::NW * 64) void gemm_tile_kernel(GemmParams g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    gemm_tile_body<Pol, NST>(g, (int)blockIdx.x, (int)gridDim.x, lds, 0, tile_item_count<Pol::SHARE_A>(g));
}

// Two GEMMs in one launch (see gemm_mfma_pair_kernel).
template <class PolA, class PolB, int NST>
__global__ __launch_bounds__(PolA::NW * 64) void gemm_tile_pair_kernel(GemmParams ga, GemmParams gb, PairPlan pl) {
    static_assert(PolA::NW == PolB::NW, "one workgroup size");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int b = (int)blockIdx.x;
    if (b < pl.blocks_a) {
        gemm_tile_body<PolA, NST>(ga, b, pl.blocks_a, lds, 0, pl.items_a);
        if (pl.main_b < pl.items_b) gemm_tile_body<PolB, NST>(gb, b, pl.blocks_a, lds, pl.main_b, pl.items_b);
    } else {
        gemm_tile_body<PolB, NST>(gb, b - pl.blocks_a, (int)gridDim.x - pl.blocks_a, lds, 0, pl.main_b);
    }
}

// As many workgroups as stay resident; more items than that are streamed.
template <class Pol, int NST>
static inline flurka_status launch_gemm_tile(const GemmParams& g, hipStream_t s) {
    auto kern = gemm_tile_kernel<Pol, NST>;
    constexpr int ldsb = TileShape<Pol::TM, Pol::TN>::lds(NST, Pol::TRANSPOSED_STORE);
    static_assert(ldsb <= 160 * 1024, "LDS of a compute unit");
    const int items = tile_item_count<Pol::SHARE_A>(g);
    int grid = resident_grid((const void*)kern, Pol::NW * 64, ldsb, items);
    if (grid < 1) return FLURKA_ERR_LAUNCH;
    if (grid < items) grid = grid / 8 * 8;
    if (grid < 8) return FLURKA_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(Pol::NW * 64), ldsb, s, g);
    if (hipGetLastError() != hipSuccess) return FLURKA_ERR_LAUNCH;
    return FLURKA_OK;
}

// Two workgroups of the pair share a compute unit (plan: 2 x compute units): one's products run while the other
// waits for a step's operands or drains the stores of its epilogue.
constexpr int T_PAIR_STAGES = 2;
template <class PolA, class PolB>
static inline flurka_status launch_gemm_tile_pair(const GemmParams& ga, const GemmParams& gb, const PairPlan& pl, int resident,
                                                  hipStream_t s) {
    auto kern = gemm_tile_pair_kernel<PolA, PolB, T_PAIR_STAGES>;
    constexpr int ldsb = TileShape<PolB::TM, PolB::TN>::lds(T_PAIR_STAGES, true);
    static_assert(PolA::TM == PolB::TM && PolA::TN == PolB::TN && PolB::TRANSPOSED_STORE, "one LDS size");
    static_assert(2 * ldsb <= 160 * 1024, "two workgroups per compute unit");
    KernelFacts facts;
    if (!kernel_facts((const void*)kern, PolA::NW * 64, ldsb, &facts)) return FLURKA_ERR_LAUNCH;
    // every workgroup strides over its items: a grid the device does not hold at once is slower, not wrong
    int blocks_b = resident - pl.blocks_a;
    if (blocks_b > pl.main_b) blocks_b = pl.main_b;
    hipLaunchKernelGGL(kern, dim3(pl.blocks_a + blocks_b), dim3(PolA::NW * 64), ldsb, s, ga, gb, pl);
    if (hipGetLastError() != hipSuccess) return FLURKA_ERR_LAUNCH;
    return FLURKA_OK;
}

}  // namespace flurka
