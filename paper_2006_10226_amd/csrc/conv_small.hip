// Implicit-GEMM quantized conv2d / dense for few output pixels: small tiles,
// the reduction of a tile split over the eight waves of a workgroup.
//
// Arithmetic as in conv_mfma.hip (Sec. II-B Eq. (3), Sec. III-B/C); K-steps,
// packed weights and chunk table as in conv_flow_kernel.h.
//
// What bounds a layer of a few hundred pixels is a chain of latencies: a tile
// of 64 x 64 leaves most CUs idle and walks its K-steps one ring stage after
// another, and a reduction split over workgroups pays for partial sums that
// travel through memory and a counter (three dependent round trips). Here a
// tile has 16 to 64 channels and 16 to 64 pixels, so that hundreds of
// workgroups share the weights, and wave w takes the pairs of K-steps
// w, w + 8, ... with its operands loaded straight into registers, eight
// K-steps in flight: up to 64 K-steps cost one memory latency. The waves'
// partial sums meet in LDS and each 16 x 16 block is finished by one wave.
// Per layer at batch 1, hot: 3x3 256 -> 256 at 14x14 7.8 us with a six-way
// split over workgroups, 7.3 us with 64 x 64 short-loop tiles, 4.1 us here;
// 1x1 2048 -> 512 at 7x7 7.5, 5.8 and 3.0 us; a 64 x 2048 -> 1001 dense 8.5,
// 6.7 and 3.2 us. The ResNet-50 body at batch 1: 367 -> 249 us.
#include "conv_flow_kernel.h"

namespace qnn {

constexpr int kSmallWaves = 8;

// FC x FP blocks of 16 channels x 16 pixels per workgroup; TAB, FLIP as in
// conv_flow_kernel; FUSE: the epilogue applies the residual add.
//
// A load unit serves four neighbouring lanes at once if they read one 64-byte
// run, and the MFMA wants neighbouring lanes in different rows. Weights are
// therefore read in operand order (ConvArgs::wf, a contiguous kilobyte per
// block and K-step); activations come by LDS-direct loads of 64-byte runs
// into the wave's own LDS and are read back in operand order, which needs no
// barrier. Loading both straight in operand layout ran at a quarter of the
// rate (15 bytes a clock per CU instead of 55; the 3x3 layer above 5.3 us).
template <int FC, int FP, bool TAB, bool FLIP, bool FUSE>
__global__ void __launch_bounds__(kSmallWaves * 64, 2) conv_small_kernel(ConvArgs a)
{
    constexpr int NW = kSmallWaves, BK = 64;
    constexpr int U = 4 / FP;            // K-steps per set of loads; two sets in flight
    constexpr int LPS = U * (FC + FP);   // loads per set
    constexpr int NB = FC * FP;
    static_assert(FP == 1 || FP == 2 || FP == 4, "activation slots fill 8 KB per wave");
    // the waves' activation slots, then their partial sums
    __shared__ __attribute__((aligned(1024))) int8_t lds[NW * 8192];
    static_assert(NB <= 8, "partial sums fit the slots");
    extern __shared__ __attribute__((aligned(16))) int8_t dyn_lds[];   // TAB: the chunk table

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lchk = lane >> 4;

    // XCD x takes the x-th eighth of the tile list, pixel tiles fastest: its
    // L2 then holds its share of the weights only
    const int tiles_p = (a.M + 16 * FP - 1) / (16 * FP);
    const int chunk = (a.ntiles + 7) >> 3;
    const int xcd = blockIdx.x & 7;
    const int tile = xcd * chunk + (blockIdx.x >> 3);
    if (tile >= min(a.ntiles, (xcd + 1) * chunk))
        return;
    const int ct = tile / tiles_p;
    const int c0 = ct * 16 * FC, p0 = (tile - ct * tiles_p) * 16 * FP;
    const int nk = a.nk;

    // weights: block c0 / 16 + i of K-step s at ((c0 / 16 + i) * fJpad / 64 + s) KB
    int voffA[FC];
#pragma unroll
    for (int i = 0; i < FC; ++i)
        voffA[i] = (c0 + i * 16) * a.fJpad + lane * 16;
    // activations: lane L loads row L / 4, physical chunk L % 4 of a block
    const int r16 = lane >> 2, lch = (lane & 3) ^ sw64(r16);
    int pbase[FP];
    uint32_t pmask[FP];
#pragma unroll
    for (int j = 0; j < FP; ++j) {
        const int m = p0 + j * 16 + r16;
        pbase[j] = TAB ? 0 : kOutOfRange;
        pmask[j] = 0;
        if (m < a.M) {
            if (!TAB && a.sh == 1 && a.sw == 1) {
                pbase[j] = m * a.C + lch * 16;
            } else {
                const int t = fast_div(m, a.mWo, a.sWo);
                const int ow = m - t * a.Wo;
                const int n = fast_div(t, a.mHo, a.sHo);
                const int oh = t - n * a.Ho;
                const int ih0 = oh * a.sh - a.pt, iw0 = ow * a.sw - a.pl;
                pbase[j] = ((n * a.H + ih0) * a.W + iw0) * a.C + (TAB ? 0 : lch * 16);
                if (TAB)
                    pmask[j] = a.rowpack ? 0x10001u
                                         : flow::inside_mask(ih0, a.R, a.dh, a.H) |
                                               (flow::inside_mask(iw0, a.S, a.dw, a.W) << 16);
            }
        }
    }
    uint32_t tbase = 0;
    if constexpr (TAB) {
        flow::fill_table((flow::v2i *)dyn_lds, a, (nk + 1) / 2 * 8, NW * 64);
        __syncthreads();
        tbase = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) int8_t *)dyn_lds + lch * 8;
    }
    int8_t *const slots = lds + wave * 8192;
    const uint32_t rbase = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) int8_t *)slots + lrow * BK +
                           ((lchk ^ sw64(lrow)) << 4);

    // K-step of this wave's i-th: pairs of neighbouring steps, a pair every
    // 2 * NW steps
    auto kstep = [&](int i) { return (i >> 1) * (2 * NW) + wave * 2 + (i & 1); };
    v4i A[2][U][FC];
    // one set of loads (between two fences, so that exactly LPS
    // vector-memory operations lie between the waits that count them)
    auto load = [&](auto SET, int i0) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value;
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int ks = __builtin_amdgcn_readfirstlane(kstep(i0 + u));
            const bool live = ks < nk;   // steps past the end: size 0, zeros, no memory touched (kBufFlags)
            const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
                (void *)a.wf, (short)0, live ? a.Kpad * a.fJpad : 0, kBufFlags);
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
                (void *)a.x, (short)0, live ? a.N * a.H * a.W * a.C : 0, kBufFlags);
            flow::v2i e = flow::v2i{0, 0};
            if constexpr (TAB) {
                e = flow::read8(tbase + (live ? ks : 0) * 32);
                lds_wait<0>();
                asm volatile("" : "+v"(e));
            }
#pragma unroll
            for (int j = 0; j < FP; ++j) {
                int off = pbase[j];
                if constexpr (TAB)
                    off = ((int)pmask[j] & e.y) == e.y ? pbase[j] + e.x : kOutOfRange;
                dma16(rx, slots + ((set * U + u) * FP + j) * 1024, off, TAB ? 0 : (live ? ks * BK : 0));
            }
#pragma unroll
            for (int i = 0; i < FC; ++i)
                A[set][u][i] = __builtin_amdgcn_raw_buffer_load_b128(rw, voffA[i], live ? ks * 1024 : 0, 0);
        }
        asm volatile("" ::: "memory");
    };
    v4i acc[FC][FP];
#pragma unroll
    for (int i = 0; i < FC; ++i)
#pragma unroll
        for (int j = 0; j < FP; ++j)
            acc[i][j] = v4i{0, 0, 0, 0};
    // the MFMAs of a set; MORE: the other set's loads were issued after it
    auto mfma = [&](auto SET, bool more) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value;
        if (more)
            wait_vmcnt<LPS>();
        else
            wait_vmcnt<0>();
        asm volatile("" ::: "memory");
        v4i B[U][FP];
        auto rd = [&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value;
            B[q / FP][q % FP] = flow::read16<(set * U * FP + q) * 1024>(rbase);
        };
        rd(std::integral_constant<int, 0>{});
        rd(std::integral_constant<int, 1>{});
        rd(std::integral_constant<int, 2>{});
        rd(std::integral_constant<int, 3>{});
        lds_wait<0>();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lds_settled(B[u]);
            if constexpr (FLIP) {
#pragma unroll
                for (int j = 0; j < FP; ++j)
                    B[u][j] ^= v4i{(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080};
            }
#pragma unroll
            for (int i = 0; i < FC; ++i)
#pragma unroll
                for (int j = 0; j < FP; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[set][u][i], B[u][j], acc[i][j], 0, 0, 0);
        }
    };
    static_assert(U * FP == 4, "four activation blocks per set");
    const int mine = ((nk + 1) / 2 + NW - 1) / NW * 2;   // steps of every wave (uniform)
    constexpr std::integral_constant<int, 0> kS0{};
    constexpr std::integral_constant<int, 1> kS1{};
    load(kS0, 0);
    for (int i = 0; i < mine; i += 2 * U) {
        const bool second = i + U < mine;
        if (second)
            load(kS1, i + U);
        mfma(kS0, second);
        if (second) {
            const bool third = i + 2 * U < mine;
            if (third)
                load(kS0, i + 2 * U);
            mfma(kS1, third);
        }
    }

    // ---- the waves' partial sums; block q is finished by wave q % NW -------
    v4i *const part = (v4i *)lds;   // [wave][block][lane]; every wave is past its slots
    __syncthreads();
#pragma unroll
    for (int i = 0; i < FC; ++i)
#pragma unroll
        for (int j = 0; j < FP; ++j)
            part[(wave * NB + i * FP + j) * 64 + lane] = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int q0 = 0; q0 < NB; q0 += NW) {
        const int q = q0 + wave;
        if (q >= NB)
            return;
        const int i = q / FP, j = q - i * FP;
        const int m = p0 + j * 16 + lrow, ch = c0 + i * 16 + lchk * 4;
        if (m >= a.M || ch >= a.K)
            continue;
        const int n = min(4, a.K - ch);
        v4i rec[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            rec[e] = *(const v4i *)(a.chan + ch + e);   // ch + 3 < Kpad
        uint32_t res = 0;
        if constexpr (FUSE) {
            const uint8_t *rp = a.res + (size_t)m * a.r_ldc + a.r_coff + ch;
            if (a.res_vec && n == 4) {
                res = *(const uint32_t *)rp;
            } else {
                for (int e = 0; e < n; ++e)
                    res |= (uint32_t)rp[e] << (8 * e);
            }
        }
        v4i s = part[q * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w)
            s += part[(w * NB + q) * 64 + lane];
        if (a.pcorr) {
            const int cls = (int)a.pcls[m];
            if (cls != 255)
                s += *(const v4i *)(a.pcorr + (size_t)cls * a.Kpad + ch);
        }
        if (a.asum) {
            const int s3 = a.asum[m];
            s -= *(const v4i *)(a.zpw + ch) * v4i{s3, s3, s3, s3};
        }
        const size_t off = (size_t)m * a.y_ldc + a.y_coff + ch;
        const bool full = a.vec_store && n == 4;
        if (a.mode == OUT_INT32) {
            s += v4i{rec[0].y, rec[1].y, rec[2].y, rec[3].y};
            int32_t *yp = (int32_t *)a.y + off;
            if (full) {
                *(v4i *)yp = s;
            } else {
                for (int e = 0; e < n; ++e)
                    yp[e] = s[e];
            }
            continue;
        }
        uint32_t packed = requant4(a, s, rec);
        if constexpr (FUSE) {
            if (a.fadd.flt) {
                packed = residual_add4_f32(a, packed, res);
            } else {
                uint32_t o = 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t xb = (packed >> (8 * e)) & 0xffu, rb = (res >> (8 * e)) & 0xffu;
                    const int t = add_one(a.fadd, a.ydt == 1 ? (int)(int8_t)xb : (int)xb,
                                          a.rdt == 1 ? (int)(int8_t)rb : (int)rb);
                    o |= ((uint32_t)t & 0xffu) << (8 * e);
                }
                packed = o;
            }
        }
        uint8_t *yp = (uint8_t *)a.y + off;
        if (full) {
            *(uint32_t *)yp = packed;
        } else {
            for (int e = 0; e < n; ++e)
                yp[e] = (uint8_t)(packed >> (8 * e));
        }
    }
}

// SmallTile -> blocks of 16 channels, blocks of 16 pixels
struct SmallCfg {
    int fc, fp;
};
static constexpr SmallCfg kSmallCfg[SMALL_COUNT] = {{1, 1}, {2, 1}, {4, 1}, {1, 2}, {2, 2}, {2, 4}};

TileShape small_tile_shape(int tile) { return {kSmallCfg[tile].fc * 16, kSmallCfg[tile].fp * 16, 64}; }

size_t small_lds_bytes(int tile, int nk, bool linear)
{
    (void)tile;
    return (size_t)kSmallWaves * 8192 + (linear ? 0 : (size_t)((nk + 1) / 2) * 64);
}

template <int T, bool FUSE>
static hipError_t launch_small_cfg(const ConvArgs &a, hipStream_t st)
{
    constexpr SmallCfg c = kSmallCfg[T];
    const dim3 grid((a.ntiles + 7) / 8 * 8), block(kSmallWaves * 64);
    const uint32_t dyn = a.linear ? 0u : (uint32_t)((a.nk + 1) / 2) * 64u;
    if (a.linear && a.flip4) launch_main((conv_small_kernel<c.fc, c.fp, false, true, FUSE>), grid, block, dyn, st, a);
    else if (a.linear) launch_main((conv_small_kernel<c.fc, c.fp, false, false, FUSE>), grid, block, dyn, st, a);
    else if (a.flip4) launch_main((conv_small_kernel<c.fc, c.fp, true, true, FUSE>), grid, block, dyn, st, a);
    else launch_main((conv_small_kernel<c.fc, c.fp, true, false, FUSE>), grid, block, dyn, st, a);
    return hipGetLastError();
}

template <int T>
static hipError_t launch_small_from(const ConvArgs &a, int tile, hipStream_t st)
{
    if constexpr (T < SMALL_COUNT) {
        if (tile == T)
            return a.res ? launch_small_cfg<T, true>(a, st) : launch_small_cfg<T, false>(a, st);
        return launch_small_from<T + 1>(a, tile, st);
    } else {
        return hipErrorInvalidValue;
    }
}

hipError_t launch_conv_small(const ConvArgs &a, int tile, hipStream_t st)
{
    return launch_small_from<0>(a, tile, st);
}

}  // namespace qnn
