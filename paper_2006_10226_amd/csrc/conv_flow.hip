// Launches of the short-loop implicit-GEMM conv kernel (conv_flow_kernel.h)
// and its plan-time weight packing.
#include "conv_flow_kernel.h"

namespace qnn {

TileShape flow_tile_shape(int tile) { return {kFlowCfg[tile].tc, kFlowCfg[tile].tp, 64}; }
int flow_threads(int tile) { return kFlowCfg[tile].wc * kFlowCfg[tile].wp * 64 * kFlowCfg[tile].ks; }
int flow_stages(int tile) { return kFlowCfg[tile].ns; }
bool flow_short(int tile) { return kFlowCfg[tile].sh; }
int flow_groups(int tile) { return kFlowCfg[tile].ks; }
int flow_wave_tile(int tile)
{
    return kFlowCfg[tile].tc / kFlowCfg[tile].wc * (kFlowCfg[tile].tp / kFlowCfg[tile].wp);
}
size_t flow_lds_bytes(int tile, int nk, bool linear)
{
    const FlowCfg &c = kFlowCfg[tile];
    const size_t ring = (size_t)c.ns * (c.tc + c.tp) * 64, stage = (size_t)c.tp * (c.tc + 16);
    return (ring > stage ? ring : stage) + (c.tc + 63) / 64 * 64 * sizeof(ChanRec) + (linear ? 0 : (size_t)(nk + 2 * c.ns) * 32) +
           (flow_fuse_cfg(tile) ? 512 * sizeof(int32_t) : 0);
}

hipError_t launch_conv_flow(const ConvArgs &a, int tile, hipStream_t st)
{
    return a.res ? launch_conv_flow_fused(a, tile, st) : launch_flow_from<0, false>(a, tile, st);
}

// Weights with every tap's channels padded to whole 16-byte chunks:
// out[k][t * Cq * 16 + c] = w[k][t][c], zero elsewhere.  One thread per byte.
__global__ void __launch_bounds__(256) tap_pack_kernel(const int8_t *w, int K, int RS, int C, int C16, int Kpad,
                                                       int Jpad, int8_t *out)
{
    const long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (long long)Kpad * Jpad)
        return;
    const int k = (int)(g / Jpad), j = (int)(g - (long long)k * Jpad);
    const int t = j / C16, c = j - t * C16;
    out[g] = k < K && t < RS && c < C ? w[((size_t)k * RS + t) * C + c] : 0;
}

hipError_t launch_tap_pack(const int8_t *w, int K, int RS, int C, int C16, int Kpad, int Jpad, int8_t *out,
                           hipStream_t st)
{
    const long long n = (long long)Kpad * Jpad;
    hipLaunchKernelGGL(tap_pack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, w, K, RS, C, C16, Kpad,
                       Jpad, out);
    return hipGetLastError();
}

}  // namespace qnn
