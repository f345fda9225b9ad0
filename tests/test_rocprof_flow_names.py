"""rocprof_summary names the short-loop and few-pixel kernels as plans do."""
import pytest

from paper_2006_10226_amd.rocprof_summary import group_of


@pytest.mark.parametrize("symbol,group", [
    ("void qnn::conv_flow_kernel<64, 128, 2, 2, 1, 1, true, false, false, true>(qnn::ConvArgs)",
     "conv_dma_flow tile=64x128x64 threads=256 stages=1s +add"),
    ("void qnn::conv_flow_kernel<128, 64, 2, 2, 8, 2, false, true, true, false>(qnn::ConvArgs)",
     "conv_dma_flow tile=128x64x64 threads=512 stages=8"),
    ("void qnn::conv_flow_kernel<256, 256, 2, 4, 4, 1, false, false, true, false>(qnn::ConvArgs)",
     "conv_dma_flow tile=256x256x64 threads=512 stages=4"),
    ("void qnn::conv_small_kernel<2, 4, true, false, false>(qnn::ConvArgs)",
     "conv_dma_small tile=32x64x64 threads=512 stages=1"),
])
def test_names(symbol, group):
    assert group_of(symbol) == group
