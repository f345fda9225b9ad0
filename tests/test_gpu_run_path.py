"""Plan.run's host path: the current stream's handle, and every argument that
it refuses."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from gpu_util import Q, dev, make_plan, run_oracle, assert_equal  # noqa: E402


def test_stream_handle():
    side = torch.cuda.Stream()
    assert Q._stream_handle() == torch.cuda.current_stream().cuda_stream
    assert Q._stream_handle(side) == side.cuda_stream
    with torch.cuda.stream(side):
        assert Q._stream_handle() == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert Q._stream_handle() == torch.cuda.current_stream().cuda_stream


def test_run_checks_and_results():
    c = W.conv_case(W.ConvLayer("c", 9, 8, 32, 48, 3, 3, 1, (1, 1, 1, 1)), 2, seed=1, zp_w="channel")
    p, keep = make_plan(c)
    x, ref = dev(c.x), run_oracle(c)
    out = torch.empty(p.y_ldc_shape, dtype=torch.uint8, device="cuda")
    assert p.workspace_size > 0 and p.residual is None
    for kw in (dict(), dict(out=out), dict(workspace=torch.zeros(p.workspace_size, dtype=torch.uint8, device="cuda"))):
        assert_equal(p.run(x, **kw).cpu().numpy(), ref, f"run {sorted(kw)}")
    bad = [(x[:1], {}), (x.view(torch.int8), {}), (x.cpu(), {}), (x.transpose(1, 2), {}), (x.view(2, 8, 9, 32), {}),
           (x, dict(out=out[:1])), (x, dict(out=out.view(torch.int8))), (x, dict(out=out.cpu())),
           (x, dict(workspace=torch.zeros(4, dtype=torch.uint8, device="cuda"))), (x, dict(residual=out))]
    for xb, kw in bad:
        with pytest.raises(ValueError):
            p.run(xb, **kw)
    p.close()
    with pytest.raises(Q.QnnError, match="NULL"):
        p.run(x)
