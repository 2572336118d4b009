"""Stores of goq_gemm's tile kernel: a tile is turned in LDS and stored in 16-byte pieces whose rows begin at any element,
with single elements where a piece crosses the last output.  Ragged widths of every remainder, both output types, memory
around Y, and the scales of the last tokens."""
import numpy as np
import pytest

import goq_inputs
from tests import gpu_util as gu
from tests.test_gpu_gemm_small import PACKERS, _inputs

pytestmark = pytest.mark.gpu
GUARD = 64                                         # elements before and after Y that nothing may touch


@pytest.mark.parametrize("act", ["A16"] + sorted(PACKERS))
@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("tokens,out", [(33, 129), (64, 134), (65, 131), (95, 4), (129, 257), (200, 255), (66, 136)])
def test_ragged_rows(oracle, act, bw, tokens, out):
    import paper_2605_26092_amd as goq
    torch = gu.torch_cuda()
    inn = 256
    print("rows %s bw=%d tokens=%d out=%d" % (act, bw, tokens, out), flush=True)
    q = oracle.quantize_geo(bw, goq_inputs.weights(out, inn, config_id=91, tensor_id=out), threads=8)
    Xd, sxd, X, sx = _inputs(goq, act, tokens, inn)
    top = np.abs(X.astype(np.float64)) * (1.0 if sx is None else sx[:, None])
    ref = oracle.gemm_a16(q, X, threads=8) if sx is None else oracle.gemm_a8(q, X, sx, threads=8, want_partials=True)[0]
    scale = top @ np.abs(oracle.dequant(q, want=("what",))["what"]).T
    packed = gu.pack_layer(goq, q)
    got = {}
    for ytype, dtype in ((goq.F32, torch.float32), (goq.F16, torch.float16)):
        whole = torch.full((tokens * out + 2 * GUARD,), 7.0, dtype=dtype, device="cuda")
        Y = whole[GUARD:-GUARD].view(tokens, out)
        goq.gemm(bw, getattr(goq, act), tokens, out, inn, packed, Xd, sxd, Y, ytype)
        torch.cuda.synchronize()
        assert (whole[:GUARD] == 7).all() and (whole[-GUARD:] == 7).all()
        got[ytype] = Y.clone()
    # fp32 sums of 256 products: the bound of the other tests of this kernel
    assert np.max(np.abs(got[goq.F32].cpu().numpy().astype(np.float64) - ref) / np.maximum(scale, 1e-30)) <= 1e-5
    assert torch.equal(got[goq.F16], got[goq.F32].half())
