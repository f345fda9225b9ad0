// Launches of the short-loop implicit-GEMM conv kernel (conv_flow_kernel.h).
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

}  // namespace qnn
