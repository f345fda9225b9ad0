// Implicit-GEMM quantized conv2d / dense with a short main loop: operands
// streamed straight into LDS as in conv_dma_kernel.h (same arithmetic, LDS
// image, swizzle and epilogue), for every channel count that is a multiple
// of 4.
//
// What bounds the layers of a network at these sizes is the K-step itself:
// per 64-byte step a wave of a 64 x 64 tile has 64 cycles of MFMA work, and
// conv_dma_kernel spends about 70 instructions on it, most of them scalar
// work of the loader (tap walk, ring index, liveness) in dependent chains and
// branches.  Here a step is the loads, the operand reads, the MFMAs and a
// handful of scalar instructions:
//   * the ring is unrolled, so LDS addresses are immediates;
//   * LINEAR form (a 1x1 filter whose taps are all inside the image, dense):
//     weights and activations advance by the same 64 bytes, one scalar
//     offset for every load;
//   * TAB form (any other filter): the workgroup first tabulates, per 16-byte
//     chunk of the reduction, the chunk's byte offset from the pixel's window
//     and the mask bits of its tap; a lane reads the entry of its chunk one
//     step ahead, so taps may change inside a K-step and any channel count
//     that is a multiple of 16 (per tap, after packing) streams at full rate;
//   * a stage past the end of the reduction has its descriptor's size set to
//     0 (LINEAR, weights) or an entry no pixel matches (TAB): the loads count
//     but touch no memory (the range check takes the scalar offset into
//     account, see kBufFlags).
// A step of a 64 x 64 tile is 19 instructions in LINEAR form and 27 in TAB
// form. Measured (hot): dense 4096^3 79 -> 58 us (256 x 256 tile), 1x1 1024 ->
// 256 at 14x14 batch 32 7.2 -> 5.7 us, 5x5 48 -> 64 at 35x35 batch 64 22.4 ->
// 12.0 us and 3x3 96 -> 96 28.5 -> 17.7 us (both from the gather kernel).
// Bytes of a chunk that lie past its pixel's channels (a channel count that
// is not a multiple of 64 in LINEAR form, of 16 in TAB form) are the next
// pixel's, or zeros past the end of x (the same range check), and meet zero
// weights.
#pragma once

#include "conv_dma_kernel.h"

namespace qnn {

namespace flow {

// LDS reads at an immediate offset from a lane's base address; see
// lds_read16 (the result may be used only after lds_wait / lds_settled).
template <int OFF>
__device__ __forceinline__ v4i read16(uint32_t addr)
{
    static_assert(OFF >= 0 && OFF < 65536, "ds_read offset range");
    v4i r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF) : "memory");
    return r;
}

typedef int v2i __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v2i read8(uint32_t addr)
{
    v2i r;
    asm volatile("ds_read_b64 %0, %1" : "=v"(r) : "v"(addr) : "memory");
    return r;
}

// Entry of a chunk of no tap: bit 15 of the row half is never set in a
// pixel's mask (filters of at most 15 rows and columns).
constexpr int kNoTap = 0x8000;

// Taps [0, n) at distance d from coordinate i0 that fall inside [0, size).
__device__ __forceinline__ uint32_t inside_mask(int i0, int n, int d, int size)
{
    if (d == 1) {
        const int lo = min(max(-i0, 0), n), hi = min(max(size - i0, 0), n);
        return ((1u << hi) - 1u) & ~((1u << lo) - 1u);
    }
    uint32_t m = 0;
    for (int r = 0; r < n; ++r)
        m |= (uint32_t)((unsigned)(i0 + r * d) < (unsigned)size) << r;
    return m;
}

// The chunk table's entries 0 .. n - 1, by all `threads` of a workgroup:
// {byte offset from the pixel's window, mask bits of the chunk's tap}.
__device__ __forceinline__ void fill_table(v2i *table, const ConvArgs &a, int n, int threads)
{
    for (int q = (int)threadIdx.x; q < n; q += threads) {
        v2i e = v2i{0, kNoTap};
        if (a.rowpack) {
            // K-step s: filter rows 2s and 2s + 1 of the padded image, 32 bytes each
            if (q < a.nk * 4)
                e = v2i{((q >> 2) * 2 + ((q >> 1) & 1)) * a.row_bytes + (q & 1) * 16, 0x10001};
        } else {
            const int t = fast_div(q, a.mCq, a.sCq);   // chunks per tap: Cq
            const int r = fast_div(t, a.mS, a.sS);
            const int s = t - r * a.S;
            if (r < a.R)
                e = v2i{(r * a.dh * a.W + s * a.dw) * a.C + (q - t * a.Cq) * 16, (1 << r) | (0x10000 << s)};
        }
        table[q] = e;
    }
}

}  // namespace flow

// Registers a wave may use: the largest wave tiles need half a SIMD's.
template <int WTC, int WTP, int THREADS>
constexpr int flow_occupancy()
{
    return THREADS >= 512 ? 2 : WTC * WTP >= 128 * 64 ? 1 : WTC * WTP >= 64 * 64 ? 2 : 3;
}

// TC x TP tile on WC x WP waves (times KS groups that take alternate K-steps
// of the same tile, each through its own ring of NS / KS stages; the second
// group's sums are added through LDS).  SHORT: at most NS K-steps, all in
// flight at once, no ring.  FUSE: the epilogue applies the residual add.
template <int TC, int TP, int WC, int WP, int NS, int KS, bool SHORT, bool TAB, bool FLIP, bool FUSE>
__global__ void __launch_bounds__(WC *WP * 64 * KS, (flow_occupancy<TC / WC, TP / WP, WC *WP * 64 * KS>()))
    conv_flow_kernel(ConvArgs a)
{
    constexpr int NW = WC * WP;
    constexpr int BK = 64;
    constexpr int WTC = TC / WC, WTP = TP / WP;
    constexpr int FC = WTC / 16, FP = WTP / 16;
    constexpr int STAGE = (TC + TP) * BK;
    // 96-channel tiles: of 96 channels, 64-wide tiles compute 128. 1x1 16 -> 96
    // at 112x112 batch 64 36.1 -> 30.1 us, 3x3 96 -> 96 at 35x35 batch 64 21.6 ->
    // 20.8 us, the Inception mixed-5 body 183 -> 176.5 us.
    // Blocks of 16 rows that each wave loads; where the waves don't divide the
    // channel blocks (96 channels), the last waves load two of them once more,
    // the same bytes to the same place, so that every wave counts alike
    constexpr int BLKA = TC / 16;
    constexpr int LA = (BLKA + NW - 1) / NW, LB = TP / (16 * NW);
    constexpr int LPS = LA + LB;
    constexpr int NSG = NS / KS;
    constexpr bool BIG = WTC * WTP >= 128 * 64;   // no registers for two sets of fragments
    constexpr int LDS_BYTES = NS * STAGE > TP * (TC + 16) ? NS * STAGE : TP * (TC + 16);
    static_assert(TC % 16 == 0 && BLKA >= NW && TP % (16 * NW) == 0, "every wave loads whole 16-row blocks");
    static_assert(TC % (16 * WC) == 0, "whole 16-channel blocks per wave");
    static_assert(KS == 1 || (KS == 2 && !SHORT && NW * FC * FP * 1024 <= LDS_BYTES), "two groups: ring form");
    static_assert(SHORT ? NS <= 4 : NSG == 4, "ring of four stages per group");
    static_assert(LPS * (SHORT ? NS - 1 : NSG - 2) < 64, "vmcnt range");
    static_assert(FC + FP + 1 <= 15, "reads of one step exceed the lgkmcnt range");

    __shared__ __attribute__((aligned(1024))) int8_t lds[LDS_BYTES];
    __shared__ __attribute__((aligned(16))) ChanRec recs[(TC + 63) / 64 * 64];
    extern __shared__ __attribute__((aligned(16))) int8_t dyn_lds[];   // TAB: the chunk table

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = KS == 1 ? 0 : wave_id / NW;
    const int wave = KS == 1 ? wave_id : wave_id % NW;
    const int wc = wave / WP, wpos = wave % WP;

    // XCD x takes the x-th eighth of the tile list; consecutive tiles are the
    // channel tiles of one pixel tile, or of a.gp pixel tiles interleaved
    // (weights larger than an L2: fewer passes over them)
    const int chunk = (a.ntiles + 7) >> 3;
    const int xcd = blockIdx.x & 7;
    const int tile = xcd * chunk + (blockIdx.x >> 3);
    if (tile >= min(a.ntiles, (xcd + 1) * chunk))
        return;
    int ct, pt;
    if (a.gp == 1) {
        pt = fast_div(tile, a.mTC, a.sTC);
        ct = tile - pt * a.tiles_c;
    } else {
        const int per = a.gp * a.tiles_c;
        const int g = tile / per, r = tile - g * per;
        const int gp = min(a.gp, a.ntiles / a.tiles_c - g * a.gp);
        ct = r / gp;
        pt = g * a.gp + r - ct * gp;
    }
    const int c0 = __builtin_amdgcn_readfirstlane(ct * TC), p0 = __builtin_amdgcn_readfirstlane(pt * TP);
    const int nk = a.nk;

    const int xbytes = a.N * a.H * a.W * a.C, wbytes = a.Kpad * a.fJpad;
    if (grp == 0 && wave == NW - 1) {
        // the tile's channel records, a kilobyte per load; older than this
        // wave's stage loads, so every stage wait covers them
        const __amdgpu_buffer_rsrc_t rc =
            __builtin_amdgcn_make_buffer_rsrc(a.krec ? (void *)a.krec : (void *)a.chan, (short)0, a.Kpad * (int)sizeof(ChanRec), kBufFlags);
#pragma unroll
        for (int q = 0; q < (TC + 63) / 64; ++q)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rc, (__attribute__((address_space(3))) void *)(recs + q * 64), 16,
                                                     (c0 + q * 64 + lane) * (int)sizeof(ChanRec), 0, 0, 0);
    }

    // lane L of a 16-row x 64-byte block's load: row L / 4, physical chunk
    // L % 4, logical chunk (L % 4) ^ sw64(row)
    const int r16 = lane >> 2;
    const int lch = (lane & 3) ^ sw64(r16);
    auto blkA = [&](int i) { return BLKA % NW == 0 || i < LA - 1 ? i * NW + wave : (i * NW + wave) % BLKA; };
    int voffA[LA];
#pragma unroll
    for (int i = 0; i < LA; ++i)
        voffA[i] = (c0 + blkA(i) * 16 + r16) * a.fJpad + lch * 16;
    int pbase[LB];
    uint32_t pmask[LB];
#pragma unroll
    for (int i = 0; i < LB; ++i) {
        const int m = p0 + (i * NW + wave) * 16 + r16;
        pbase[i] = TAB ? 0 : kOutOfRange;
        pmask[i] = 0;
        if (m < a.M) {
            if (!TAB && a.sh == 1 && a.sw == 1) {
                pbase[i] = m * a.C + lch * 16;   // 1x1, every pixel: the pixels are x's own rows
            } else {
                const int t = fast_div(m, a.mWo, a.sWo);
                const int ow = m - t * a.Wo;
                const int n = fast_div(t, a.mHo, a.sHo);
                const int oh = t - n * a.Ho;
                const int ih0 = oh * a.sh - a.pt, iw0 = ow * a.sw - a.pl;
                pbase[i] = ((n * a.H + ih0) * a.W + iw0) * a.C + (TAB ? 0 : lch * 16);
                if (TAB)
                    pmask[i] = a.rowpack ? 0x10001u
                                         : flow::inside_mask(ih0, a.R, a.dh, a.H) |
                                               (flow::inside_mask(iw0, a.S, a.dw, a.W) << 16);
            }
        }
    }

    // ---- chunk table (TAB): entry q = {byte offset, mask bits of its tap}
    uint32_t tbase = 0;
    flow::v2i ent[1] = {flow::v2i{0, flow::kNoTap}};
    if constexpr (TAB) {
        const int n = (nk + 2 * NS) * 4;   // entries of the stages past the end included
        flow::fill_table((flow::v2i *)dyn_lds, a, n, NW * KS * 64);
        __syncthreads();
        tbase = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) int8_t *)dyn_lds + (grp * 4 + lch) * 8;
        ent[0] = flow::read8(tbase);
    }

    // ---- loader: stage i of this group is K-step i * KS + grp ------------
    // byte offset of the next issue's K-step in a row, kept in a scalar
    // register (the compiler cannot see that it is uniform through the loop)
    int soff = __builtin_amdgcn_readfirstlane(grp * BK);
    const int send = nk * BK;
    auto issue = [&](int slot) __attribute__((always_inline)) {
        int8_t *base = lds + (slot * KS + grp) * STAGE + wave * 16 * BK;
        const bool live = soff < send;
        const __amdgpu_buffer_rsrc_t rw =
            __builtin_amdgcn_make_buffer_rsrc((void *)a.fw, (short)0, live ? wbytes : 0, kBufFlags);
        const __amdgpu_buffer_rsrc_t rx =
            __builtin_amdgcn_make_buffer_rsrc((void *)a.x, (short)0, TAB || live ? xbytes : 0, kBufFlags);
        int voffB[LB];
#pragma unroll
        for (int i = 0; i < LB; ++i) {
            if constexpr (TAB)
                voffB[i] = ((int)pmask[i] & ent[0].y) == ent[0].y ? pbase[i] + ent[0].x : kOutOfRange;
            else
                voffB[i] = pbase[i];
        }
#pragma unroll
        for (int i = 0; i < LA; ++i)
            dma16(rw, base + (blkA(i) - wave) * 16 * BK, voffA[i], soff);
#pragma unroll
        for (int i = 0; i < LB; ++i)
            dma16(rx, base + (TC + i * NW * 16) * BK, voffB[i], TAB ? 0 : soff);
        asm volatile("s_add_i32 %0, %0, %1" : "+s"(soff) : "n"(KS * BK) : "scc");
        if constexpr (TAB) {   // the entry of the next K-step, used after the caller's next wait
            tbase += KS * 32;
            ent[0] = flow::read8(tbase);
        }
    };
    auto settle_ent = [&]() __attribute__((always_inline)) {
        if constexpr (TAB) {
            lds_wait<0>();
            asm volatile("" : "+v"(ent[0]));
        }
    };

    // ---- fragments and MFMAs ------------------------------------------
    const int lrow = lane & 15, lchk = lane >> 4;
    const int co = (lchk ^ sw64(lrow)) << 4;
    const uint32_t l0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) int8_t *)lds + grp * STAGE + co;
    constexpr int SPAN = 49152;   // LDS bytes one base address covers with immediates
    constexpr int NB = (NS * STAGE + SPAN - 1) / SPAN;
    uint32_t aA[NB], aB[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        aA[b] = l0 + (wc * WTC + lrow) * BK + b * SPAN;
        aB[b] = l0 + (wpos * WTP + lrow) * BK + b * SPAN;
    }
    v4i acc[FC][FP];
#pragma unroll
    for (int i = 0; i < FC; ++i)
#pragma unroll
        for (int j = 0; j < FP; ++j)
            acc[i][j] = v4i{0, 0, 0, 0};
    v4i fa[2][FC], fb[2][FP];
    auto read_frags = [&](auto SLOT, v4i (&A)[FC], v4i (&B)[FP]) __attribute__((always_inline)) {
        constexpr int s0 = decltype(SLOT)::value * KS * STAGE;
        auto one = [&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            if constexpr (i < FP) {
                constexpr int o = s0 + TC * BK + i * 16 * BK;
                B[i] = flow::read16<o % SPAN>(aB[o / SPAN]);
            } else if constexpr (i < FP + FC) {
                constexpr int o = s0 + (i - FP) * 16 * BK;
                A[i - FP] = flow::read16<o % SPAN>(aA[o / SPAN]);
            }
        };
        one(std::integral_constant<int, 0>{});
        one(std::integral_constant<int, 1>{});
        one(std::integral_constant<int, 2>{});
        one(std::integral_constant<int, 3>{});
        one(std::integral_constant<int, 4>{});
        one(std::integral_constant<int, 5>{});
        one(std::integral_constant<int, 6>{});
        one(std::integral_constant<int, 7>{});
        one(std::integral_constant<int, 8>{});
        one(std::integral_constant<int, 9>{});
        one(std::integral_constant<int, 10>{});
        one(std::integral_constant<int, 11>{});
        static_assert(FC + FP <= 12, "fragment reads of one step");
    };
    auto settle_frags = [&](v4i (&A)[FC], v4i (&B)[FP]) __attribute__((always_inline)) {
        lds_settled(A);
        lds_settled(B);
    };
    auto mfma = [&](v4i (&A)[FC], v4i (&B)[FP]) __attribute__((always_inline)) {
        if constexpr (FLIP) {
#pragma unroll
            for (int j = 0; j < FP; ++j)
                B[j] ^= v4i{(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
        }
#pragma unroll
        for (int i = 0; i < FC; ++i)
#pragma unroll
            for (int j = 0; j < FP; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[i], B[j], acc[i][j], 0, 0, 0);
    };

    // the largest wave tiles: the MFMAs of A and B, a row of blocks at a time,
    // each A fragment replaced by the next stage's (slot SLOT) once its row
    // is issued, after the next stage's B fragments have been read into BN
    auto mfma_rotate = [&](auto SLOT, v4i (&A)[FC], v4i (&B)[FP], v4i (&BN)[FP]) __attribute__((always_inline)) {
        constexpr int s0 = decltype(SLOT)::value * KS * STAGE;
        if constexpr (FLIP) {
#pragma unroll
            for (int j = 0; j < FP; ++j)
                B[j] ^= v4i{(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
        }
        auto readB = [&](auto J) __attribute__((always_inline)) {
            constexpr int j = decltype(J)::value;
            if constexpr (j < FP) {
                constexpr int o = s0 + TC * BK + j * 16 * BK;
                BN[j] = flow::read16<o % SPAN>(aB[o / SPAN]);
            }
        };
        readB(std::integral_constant<int, 0>{});
        readB(std::integral_constant<int, 1>{});
        readB(std::integral_constant<int, 2>{});
        readB(std::integral_constant<int, 3>{});
        auto row = [&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            if constexpr (i < FC) {
#pragma unroll
                for (int j = 0; j < FP; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[i], B[j], acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                constexpr int o = s0 + i * 16 * BK;
                A[i] = flow::read16<o % SPAN>(aA[o / SPAN]);
            }
        };
        row(std::integral_constant<int, 0>{});
        row(std::integral_constant<int, 1>{});
        row(std::integral_constant<int, 2>{});
        row(std::integral_constant<int, 3>{});
        row(std::integral_constant<int, 4>{});
        row(std::integral_constant<int, 5>{});
        row(std::integral_constant<int, 6>{});
        row(std::integral_constant<int, 7>{});
        static_assert(!BIG || (FC <= 8 && FP <= 4), "rotated fragments: at most 8 x 4 blocks");
    };

    if constexpr (SHORT) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            settle_ent();
            issue(s);
        }
        auto step = [&](auto S) __attribute__((always_inline)) {
            constexpr int k = decltype(S)::value;
            if constexpr (k < NS) {
                stage_barrier<LPS *(NS - 1 - k)>();
                if (k < nk) {
                    read_frags(std::integral_constant<int, k>{}, fa[0], fb[0]);
                    lds_wait<0>();
                    settle_frags(fa[0], fb[0]);
                    mfma(fa[0], fb[0]);
                }
            }
        };
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
        asm volatile("" : "+v"(ent[0]));   // the last entry read is retired by the stage barriers
        __syncthreads();
    } else {
        // NSG - 1 stages in flight; the fragments of stage k + 1 are read
        // while the MFMAs of stage k run.  The barrier of step k certifies
        // that stage k + 1 has landed everywhere and that every wave has read
        // stage k, whose predecessor's slot takes stage k + NSG - 1.  Both
        // groups run the same number of steps, so every wave reaches every
        // barrier.
        const int nkl = (nk + KS - 1) / KS;
#pragma unroll
        for (int s = 0; s < NSG - 1; ++s) {
            settle_ent();
            issue(s);
        }
        stage_barrier<LPS *(NSG - 2)>();
        read_frags(std::integral_constant<int, 0>{}, fa[0], fb[0]);
        int k = 0;
        auto step = [&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            constexpr std::integral_constant<int, (s + 1) % NSG> kNext{};
            stage_barrier<LPS *(NSG - 3)>();   // and lgkmcnt 0: this step's fragments, the next entry
            constexpr int cur = BIG ? 0 : s & 1;
            settle_frags(fa[cur], fb[s & 1]);
            if constexpr (TAB)
                asm volatile("" : "+v"(ent[0]));
            issue((s + NSG - 1) % NSG);
            if constexpr (BIG) {
                mfma_rotate(kNext, fa[0], fb[s & 1], fb[(s + 1) & 1]);
            } else {
                read_frags(kNext, fa[(s + 1) & 1], fb[(s + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);   // the reads first: their latency runs under the MFMAs
                mfma(fa[s & 1], fb[s & 1]);
            }
        };
        for (; k + 4 <= nkl; k += 4) {
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
            step(std::integral_constant<int, 2>{});
            step(std::integral_constant<int, 3>{});
        }
        if (k < nkl)
            step(std::integral_constant<int, 0>{});
        if (k + 1 < nkl)
            step(std::integral_constant<int, 1>{});
        if (k + 2 < nkl)
            step(std::integral_constant<int, 2>{});
        // the reads of the step past the last one are still in flight: they
        // are retired before their registers are given to anything else
        lds_wait<0>();
        settle_frags(fa[0], fb[0]);
        lds_settled(fb[1]);
        if constexpr (!BIG)
            lds_settled(fa[1]);
        asm volatile("" : "+v"(ent[0]));
        wait_vmcnt<0>();   // the trailing loads also write LDS
        __syncthreads();
        if constexpr (KS > 1) {
            v4i *part = (v4i *)lds;
            if (grp == 1) {
#pragma unroll
                for (int i = 0; i < FC; ++i)
#pragma unroll
                    for (int j = 0; j < FP; ++j)
                        part[((wave * FC + i) * FP + j) * 64 + lane] = acc[i][j];
            }
            __syncthreads();
            if (grp == 1)
                return;   // the barriers below count only the first group
#pragma unroll
            for (int i = 0; i < FC; ++i)
#pragma unroll
                for (int j = 0; j < FP; ++j)
                    acc[i][j] += part[((wave * FC + i) * FP + j) * 64 + lane];
            __syncthreads();   // every partial read before the staging overwrites them
        }
    }
    store_tile<TC, TP, WC, WP, LDS_BYTES, FUSE, BIG, true>(a, acc, lds, c0, p0, recs);
}

// FlowTile -> tile, wave grid, stages, K-step groups, short form.
struct FlowCfg {
    int tc, tp, wc, wp, ns, ks;
    bool sh;
};
inline constexpr FlowCfg kFlowCfg[FLOW_COUNT] = {
    {64, 64, 2, 2, 4, 1, false},   {128, 64, 2, 2, 4, 1, false},  {64, 128, 2, 2, 4, 1, false},
    {128, 128, 2, 2, 4, 1, false}, {256, 128, 4, 2, 4, 1, false}, {128, 256, 2, 4, 4, 1, false},
    {256, 256, 2, 4, 4, 1, false}, {64, 64, 2, 2, 8, 2, false},   {128, 64, 2, 2, 8, 2, false},
    {128, 128, 2, 2, 8, 2, false}, {64, 64, 2, 2, 1, 1, true},    {64, 128, 2, 2, 1, 1, true},
    {128, 64, 2, 2, 1, 1, true},   {64, 64, 2, 2, 2, 1, true},    {64, 128, 2, 2, 2, 1, true},
    {128, 64, 2, 2, 2, 1, true},   {64, 64, 2, 2, 4, 1, true},    {64, 128, 2, 2, 4, 1, true},
    {128, 128, 2, 2, 4, 1, true},  {96, 64, 2, 2, 4, 1, false},   {96, 128, 2, 2, 4, 1, false},
    {96, 128, 2, 2, 1, 1, true},   {96, 128, 2, 2, 2, 1, true},
};
constexpr bool flow_fuse_cfg(int t)
{
    return kFlowCfg[t].tc / kFlowCfg[t].wc * (kFlowCfg[t].tp / kFlowCfg[t].wp) <= kFuseMaxWaveTile;
}

// Dynamic LDS of a launch: the chunk table.
inline uint32_t flow_table_bytes(const ConvArgs &a, const FlowCfg &c)
{
    return a.linear ? 0u : (uint32_t)(a.nk + 2 * c.ns) * 32u;
}

template <int T, bool FUSE>
hipError_t launch_flow_cfg(const ConvArgs &a, hipStream_t st)
{
    constexpr FlowCfg c = kFlowCfg[T];
    if constexpr (FUSE && !flow_fuse_cfg(T)) {
        return hipErrorInvalidValue;   // no fused-add instantiation
    } else {
        if (c.sh && a.nk > c.ns)
            return hipErrorInvalidValue;
        constexpr bool big = c.tc / c.wc * (c.tp / c.wp) >= 128 * 64;   // linear, without term 3 only
        if (big && (!a.linear || a.asum || a.pcorr))
            return hipErrorInvalidValue;
        const dim3 grid((a.ntiles + 7) / 8 * 8), block(c.wc * c.wp * 64 * c.ks);
        const uint32_t dyn = flow_table_bytes(a, c);
        if (a.linear && a.flip4)
            launch_main((conv_flow_kernel<c.tc, c.tp, c.wc, c.wp, c.ns, c.ks, c.sh, false, true, FUSE>), grid, block,
                        dyn, st, a);
        else if (a.linear)
            launch_main((conv_flow_kernel<c.tc, c.tp, c.wc, c.wp, c.ns, c.ks, c.sh, false, false, FUSE>), grid, block,
                        dyn, st, a);
        else if (a.flip4)
            launch_main((conv_flow_kernel<c.tc, c.tp, c.wc, c.wp, c.ns, c.ks, c.sh, !big, true, FUSE>), grid, block,
                        dyn, st, a);
        else
            launch_main((conv_flow_kernel<c.tc, c.tp, c.wc, c.wp, c.ns, c.ks, c.sh, !big, false, FUSE>), grid, block,
                        dyn, st, a);
        return hipGetLastError();
    }
}

template <int T, bool FUSE>
hipError_t launch_flow_from(const ConvArgs &a, int tile, hipStream_t st)
{
    if constexpr (T < FLOW_COUNT) {
        if (tile == T)
            return launch_flow_cfg<T, FUSE>(a, st);
        return launch_flow_from<T + 1, FUSE>(a, tile, st);
    } else {
        return hipErrorInvalidValue;
    }
}

// Launch with the residual add fused (a.res set, a.staged).
hipError_t launch_conv_flow_fused(const ConvArgs &a, int tile, hipStream_t st);

}  // namespace qnn
