"""goq_gemm with up to 32 tokens (the kernel that splits the depth over wavefronts) and just beyond: edges of its 16-token and
16-row tiles, wavefronts without a slab and with several, one, two and four row tiles per workgroup; the tile
kernel with every integer type; against the oracle, batch against single calls, and a token's bits between calls."""
import numpy as np
import pytest

import goq_inputs
from tests import gpu_util as gu
from tests.test_gemm_rules import ask, launch                      # (ask: a fixture)

pytestmark = pytest.mark.gpu

PACKERS = {"A8": None, "A4": (4, "pack_int4"), "A6": (6, "pack_int6"), "A3": (3, "pack_int3")}


def _inputs(goq, act, tokens, inn):
    """(device x, sx, host fp64 x or int8 x, host sx)"""
    if act == "A16":
        x = goq_inputs.activations_a16(tokens, inn, config_id=61, tensor_id=100 + tokens, outlier_frac=0.01)
        return gu.to_dev(x), None, x, None
    if act == "A8":
        x, sx = goq_inputs.activations_a8(tokens, inn, config_id=61, tensor_id=200 + tokens)
        return gu.to_dev(x), gu.to_dev(sx), x, sx
    bits, packer = PACKERS[act]
    x, sx = goq_inputs.activations_int(tokens, inn, bits, config_id=61, tensor_id=200 + tokens)
    return gu.to_dev(getattr(goq_inputs, packer)(x)), gu.to_dev(sx), x, sx


def _run(goq, bw, act, q, tokens, xd, sxd, ytype, partials=False):
    torch = gu.torch_cuda()
    out, inn = q["codes"].shape
    packed = gu.pack_layer(goq, q)
    Y = torch.full((tokens, out), float("nan"), dtype=torch.float32 if ytype == goq.F32 else torch.float16, device="cuda")
    P = torch.full((tokens, out, inn // 128, 2), -7777, dtype=torch.int32, device="cuda") if partials else None
    goq.gemm(bw, getattr(goq, act), tokens, out, inn, packed, xd, sxd, Y, ytype, partials=P)
    torch.cuda.synchronize()
    return Y, P


@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("tokens,out,inn", [(1, 1, 128), (2, 17, 896), (15, 16, 1024), (16, 63, 1152), (17, 65, 2176),
                                            (31, 48, 256), (32, 8209, 384), (33, 100, 640),
                                            (3, 32800, 128), (65, 257, 1024), (129, 100, 384), (257, 2432, 256), (257, 2433, 256),
                                            (257, 2433, 384), (1025, 1920, 128), (1025, 2049, 256)])
def test_few_tokens_a16(oracle, bw, tokens, out, inn):
    """fp32 results within 2e-6 of the sum of absolute products (2^-24 per rounding, at most some
    ten of them on a path from a product to y), fp16 results one rounding (2^-11) more."""
    import paper_2605_26092_amd as goq
    print("few tokens a16 bw=%d %dx%dx%d" % (bw, tokens, out, inn), flush=True)
    q = goq_inputs.canonical_random(bw, out, inn, config_id=60, tensor_id=tokens)
    xd, _, x, _ = _inputs(goq, "A16", tokens, inn)
    ref = oracle.gemm_a16(q, x, threads=8)
    scale = np.abs(x.astype(np.float64)) @ np.abs(oracle.dequant(q, want=("what",))["what"]).T + 1e-30
    y = _run(goq, bw, "A16", q, tokens, xd, None, goq.F32)[0].cpu().numpy().astype(np.float64)
    assert np.max(np.abs(y - ref) / scale) <= 2e-6
    h = _run(goq, bw, "A16", q, tokens, xd, None, goq.F16)[0].float().cpu().numpy().astype(np.float64)
    assert np.all(np.abs(h - ref) <= 2e-6 * scale + 2.0 ** -11 * np.abs(ref) + 2.0 ** -25)


@pytest.mark.parametrize("act", sorted(PACKERS))
@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("tokens,out,inn", [(3, 33, 128), (16, 20, 1152), (32, 8200, 256), (19, 64, 2304), (70, 130, 640)])
def test_few_tokens_integers(oracle, act, bw, tokens, out, inn):
    """int32 slab partials bit for bit; y from them; y without the partials the same bits."""
    import paper_2605_26092_amd as goq
    print("few tokens %s bw=%d %dx%dx%d" % (act, bw, tokens, out, inn), flush=True)
    q = goq_inputs.canonical_random(bw, out, inn, config_id=62, tensor_id=tokens)
    xd, sxd, x, sx = _inputs(goq, act, tokens, inn)
    ref, pref = oracle.gemm_a8(q, x, sx, threads=8, want_partials=True)
    Y, P = _run(goq, bw, act, q, tokens, xd, sxd, goq.F32, partials=True)
    assert np.array_equal(P.cpu().numpy(), pref)
    scale = (np.abs(x.astype(np.float64)) * sx[:, None]) @ np.abs(oracle.dequant(q, want=("what",))["what"]).T + 1e-30
    assert np.max(np.abs(Y.cpu().numpy().astype(np.float64) - ref) / scale) <= 2e-6
    assert gu.torch_cuda().equal(_run(goq, bw, act, q, tokens, xd, sxd, goq.F32)[0], Y)


@pytest.mark.parametrize("act", ["A16", "A8"])
def test_batch_of_few_and_many_tokens(act):
    """A batch that mixes problems of either kernel, of one and of two token tiles, and with enough
    rows for two row tiles per workgroup: the bits of single calls."""
    import paper_2605_26092_amd as goq
    torch = gu.torch_cuda()
    probs, single = [], []
    for i, (tokens, out, inn) in enumerate([(5, 8300, 256), (40, 200, 384), (32, 64, 2048), (1100, 1000, 128), (16, 70, 1280)]):
        q = goq_inputs.canonical_random(3, out, inn, config_id=63, tensor_id=i)
        packed = gu.pack_layer(goq, q)
        xd, sxd, _, _ = _inputs(goq, act, tokens, inn)
        ya, yb = (torch.full((tokens, out), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
        goq.gemm(3, getattr(goq, act), tokens, out, inn, packed, xd, sxd, ya, goq.F32)
        probs.append((tokens, out, inn, packed, xd, sxd, yb, goq.F32))
        single.append((ya, yb))
    goq.gemm_batch(3, getattr(goq, act), probs)
    torch.cuda.synchronize()
    for ya, yb in single:
        assert torch.equal(ya, yb)


@pytest.mark.parametrize("act", sorted(PACKERS))
@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("tokens,out,inn", [(1089, 1025, 128), (700, 2050, 384), (65, 130, 256), (1100, 9000, 128),
                                            (300, 4400, 1152)])
def test_many_tokens_integers(oracle, act, bw, tokens, out, inn):
    """The tile kernel with every integer type, ragged in both directions, one, three and nine slabs: int32
    slab partials bit for bit, with the extremes of the type in the first tokens, y from them, and y
    without the partials the same bits."""
    import paper_2605_26092_amd as goq
    print("many tokens %s bw=%d %dx%dx%d" % (act, bw, tokens, out, inn), flush=True)
    q = goq_inputs.canonical_random(bw, out, inn, config_id=64, tensor_id=tokens)
    q["codes"][:40] = 0                                            # all +1
    bits, packer = PACKERS[act] or (8, None)
    x, sx = goq_inputs.activations_int(tokens, inn, bits, config_id=64, tensor_id=200)
    top = 1 << (bits - 1)
    x[0], x[1], x[2, ::2] = -top, top - 1, -top
    xd = gu.to_dev(getattr(goq_inputs, packer)(x) if packer else x)
    rows = np.r_[0:8, tokens // 2:tokens // 2 + 8, tokens - 8:tokens]
    ref, pref = oracle.gemm_a8(q, x[rows], sx[rows], threads=8, want_partials=True)
    Y, P = _run(goq, bw, act, q, tokens, xd, gu.to_dev(sx), goq.F32, partials=True)
    assert np.array_equal(P.cpu().numpy()[rows], pref)
    scale = (np.abs(x[rows].astype(np.float64)) * sx[rows][:, None]) @ np.abs(oracle.dequant(q, want=("what",))["what"]).T + 1e-30
    assert np.max(np.abs(Y.cpu().numpy()[rows].astype(np.float64) - ref) / scale) <= 2e-6
    assert gu.torch_cuda().equal(_run(goq, bw, act, q, tokens, xd, gu.to_dev(sx), goq.F32)[0], Y)


@pytest.mark.parametrize("act", sorted(PACKERS))
@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("tokens", [30, 90])
def test_slabs_of_large_and_tiny_products(oracle, act, bw, tokens):
    """Slab sums at the full width the exactness claims name (W4: products up to 8, 32 or 128 beside odd
    multiples of 2^-7; running sums to 2^10, 2^12 or 2^14): the largest state against the most
    negative activation on one part of a slab, the smallest state against odd activations on the rest, in either
    order, within a group of eight and across groups, and large products that cancel.  int32 partials bit for bit."""
    import paper_2605_26092_amd as goq
    print("large and tiny products %s bw=%d tokens=%d" % (act, bw, tokens), flush=True)
    inn, k = 384, np.arange(128)
    parts = [k < 64, k >= 64, k < 120, k >= 8, k < 96, k >= 32, k % 8 == 0, k % 8 != 0, k % 8 != 7, k != 127, k != 0, k % 2 == 0, k % 32 < 16, k >= 0, k < 0]
    r = np.random.default_rng(5)
    half = 1 << (bw - 1)
    largest = [np.zeros(128, int), np.full(128, half), np.where(k % 2, half, 0), np.where(k < 64, 0, half)]   # +1, -1, cancelling
    tiny = [np.full(128, 2 * half - 1), np.where(k % 2, 2 * half - 1, half - 2), r.choice([half - 2, 2 * half - 2, 2 * half - 1], 128)]
    rows = [np.where(p, a, t) for p in parts for a in largest for t in tiny]
    q = goq_inputs.canonical_random(bw, len(rows), inn, config_id=65, tensor_id=tokens)
    q["codes"][:] = np.stack([np.concatenate([row, np.roll(row, 8), row[::-1]]) for row in rows])
    bits, packer = PACKERS[act] or (8, None)
    top = 1 << (bits - 1)
    x = np.empty((tokens, inn), np.int8)
    for t in range(tokens):
        p = np.concatenate([parts[t % len(parts)], np.roll(parts[t % len(parts)], 8), parts[t % len(parts)][::-1]])
        odd = 2 * r.integers(-(top // 2), top // 2, inn) + 1
        x[t] = np.where(p, -top if t % 2 else top - 1, odd if t % 3 else top - 1)
    sx = r.uniform(0.01, 0.02, tokens).astype(np.float32)
    _, pref = oracle.gemm_a8(q, x, sx, threads=8, want_partials=True)
    assert np.abs(pref).max() >= (top - 1) * 128 << (half - 1)     # the widest sums do occur
    xd = gu.to_dev(getattr(goq_inputs, packer)(x) if packer else x)
    Y, P = _run(goq, bw, act, q, tokens, xd, gu.to_dev(sx), goq.F32, partials=True)
    assert np.array_equal(P.cpu().numpy(), pref)
    assert gu.torch_cuda().equal(_run(goq, bw, act, q, tokens, xd, gu.to_dev(sx), goq.F32)[0], Y)


@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("tokens", [1, 5, 40])
def test_subnormal_activations(oracle, bw, tokens):
    """fp16 activations below 2^-14 alone, and beside ordinary ones in other slabs: no operand flushes
    them (fp32 sums of exact products: 2e-6 of the sum of absolute products, as above)."""
    import paper_2605_26092_amd as goq
    torch = gu.torch_cuda()
    out, inn = 130, 1152
    q = goq_inputs.canonical_random(bw, out, inn, config_id=66, tensor_id=tokens)
    x = (np.random.default_rng(7).integers(-1023, 1024, (tokens, inn)) * 2.0 ** -24)
    x[tokens // 2, 256:512] = 1.5
    x = x.astype(np.float16)
    ref = oracle.gemm_a16(q, x, threads=8)
    scale = np.abs(x.astype(np.float64)) @ np.abs(oracle.dequant(q, want=("what",))["what"]).T
    y = _run(goq, bw, "A16", q, tokens, gu.to_dev(x), None, goq.F32)[0].cpu().numpy().astype(np.float64)
    assert np.max(np.abs(y - ref) / scale) <= 2e-6
    if tokens == 1:
        packed, yv = gu.pack_layer(goq, q), torch.full((out,), float("nan"), dtype=torch.float32, device="cuda")
        goq.gemv(bw, goq.A16, out, inn, packed, gu.to_dev(x), None, yv, goq.F32)
        assert np.max(np.abs(yv.cpu().numpy().astype(np.float64) - ref[0]) / scale[0]) <= 2e-6


@pytest.mark.parametrize("act", ["A16"] + sorted(PACKERS))
@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("tokens,out,inn", [(5, 8209, 2176), (16, 8209, 1152), (16, 32785, 1152), (3, 32785, 2176), (20, 8209, 2176)])
def test_several_row_tiles_over_several_slabs(oracle, act, bw, tokens, out, inn):
    """Two and four row tiles per workgroup (more than 512 and, W3 with one token tile, more than 2048 row tiles), the
    last workgroup with one of them, and wavefronts that walk one, two and three slabs.  The oracle sees sampled
    rows of a layer that repeats every 1031 rows (a prime: a misplaced tile is another row); integers with partials bit
    for bit; the fp32 bound of test_few_tokens_a16."""
    import paper_2605_26092_amd as goq
    print("row tiles %s bw=%d %dx%dx%d" % (act, bw, tokens, out, inn), flush=True)
    base = goq_inputs.canonical_random(bw, 1031, inn, config_id=67, tensor_id=tokens)
    at = np.arange(out) % 1031
    q = {k: v[at] if isinstance(v, np.ndarray) else v for k, v in base.items()}
    rows = np.unique(np.r_[0:70, 1020:1040, out // 2:out // 2 + 70, out - 90:out])
    part = {k: np.ascontiguousarray(v[rows]) if isinstance(v, np.ndarray) else v for k, v in q.items()}
    xd, sxd, x, sx = _inputs(goq, act, tokens, inn)
    what = np.abs(oracle.dequant(part, want=("what",))["what"]).T
    Y, P = _run(goq, bw, act, q, tokens, xd, sxd, goq.F32, partials=act != "A16")
    if act == "A16":
        ref, scale = oracle.gemm_a16(part, x, threads=8), np.abs(x.astype(np.float64)) @ what
    else:
        ref, pref = oracle.gemm_a8(part, x, sx, threads=8, want_partials=True)
        scale = (np.abs(x.astype(np.float64)) * sx[:, None]) @ what
        assert np.array_equal(P.cpu().numpy()[:, rows], pref)
        assert gu.torch_cuda().equal(_run(goq, bw, act, q, tokens, xd, sxd, goq.F32)[0], Y)
    y = Y.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(y))
    assert np.max(np.abs(y[:, rows] - ref) / (scale + 1e-30)) <= 2e-6
    # every row: those a period apart are the same row
    assert np.array_equal(y[:, 1031:], y[:, :out - 1031])


@pytest.mark.parametrize("act", ["A16"] + sorted(PACKERS))
@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("tokens,layers", [(17, [(4000, 128), (520, 3072)]), (32, [(1000, 1152), (2050, 896), (1111, 2304)])])
def test_a_cu_to_each_workgroup(act, bw, tokens, layers):
    """Launches whose workgroups get a CU each (257 to 512 of them, one layer much deeper): the bits of single calls, which the
    other tests of this file hold to the oracle."""
    import paper_2605_26092_amd as goq
    from paper_2605_26092_amd import binding
    print("alone %s bw=%d %d tokens %s" % (act, bw, tokens, layers), flush=True)
    torch = gu.torch_cuda()
    problems, single = [], []
    for out, inn in layers:
        q = goq_inputs.canonical_random(bw, out, inn, config_id=73, tensor_id=out)
        xd, sxd, _, _ = _inputs(goq, act, tokens, inn)
        single.append(_run(goq, bw, act, q, tokens, xd, sxd, goq.F16)[0])
        Y = torch.full((tokens, out), float("nan"), dtype=torch.float16, device="cuda")
        problems.append((tokens, out, inn, gu.pack_layer(goq, q), xd, sxd, Y, goq.F16))
    goq.gemm_batch(bw, getattr(goq, act), binding.make_gemm_descs(problems))
    torch.cuda.synchronize()
    for p, y in zip(problems, single):
        assert torch.isfinite(y).all() and torch.equal(p[6], y)


@pytest.mark.parametrize("act", ["A16", "A8"])
@pytest.mark.parametrize("bw", [3, 4])
@pytest.mark.parametrize("out,inn,counts", [(200, 1152, (1, 5, 16, 20, 32)), (300, 640, (33, 64, 65, 130, 1000)), (16400, 384, (17, 32, 40, 300)), (20000, 256, (1, 7, 16, 33, 200))])
def test_bits_of_a_token(act, bw, out, inn, counts):
    """A token's outputs are the same bits in every call that one kernel serves, whatever else the call
    holds: few tokens, many, and the large or shallow layers whose few tokens go to the tiles."""
    import paper_2605_26092_amd as goq
    q = goq_inputs.canonical_random(bw, out, inn, config_id=68, tensor_id=out)
    if act == "A16":
        x, sx = goq_inputs.activations_a16(max(counts), inn, config_id=68, tensor_id=100, outlier_frac=0.01), None
    else:
        x, sx = goq_inputs.activations_a8(max(counts), inn, config_id=68, tensor_id=200)
    got = [_run(goq, bw, act, q, n, gu.to_dev(x[:n]), None if sx is None else gu.to_dev(sx[:n]), goq.F32)[0] for n in counts]
    for n, y in zip(counts, got):
        assert gu.torch_cuda().equal(y, got[-1][:n]), n


@pytest.mark.parametrize("bw,act", [(3, "A8"), (4, "A4"), (4, "A3")])
@pytest.mark.parametrize("tokens,out,inn", [(1023, 8191, 512), (993, 8190, 1152), (2017, 4090, 768)])
def test_tiles_of_128_tokens(oracle, bw, act, tokens, out, inn):
    """Launches that take 128-token tiles, ragged in both directions, with an odd and an even number of slabs and the extremes of the
    type in the first and last tokens: the bits of calls of 33 and of 100 tokens, which take narrower tiles, and the oracle's values."""
    import paper_2605_26092_amd as goq
    print("wide %s bw=%d %dx%dx%d" % (act, bw, tokens, out, inn), flush=True)
    torch = gu.torch_cuda()
    q = goq_inputs.canonical_random(bw, out, inn, config_id=69, tensor_id=tokens)
    q["codes"][:40] = 0                                            # all +1
    bits, packer = PACKERS[act] or (8, None)
    x, sx = goq_inputs.activations_int(tokens, inn, bits, config_id=69, tensor_id=200)
    top = 1 << (bits - 1)
    x[0], x[1], x[2, ::2], x[-1], x[-2] = -top, top - 1, -top, -top, top - 1
    dev = lambda r: (gu.to_dev(getattr(goq_inputs, packer)(x[r]) if packer else x[r]), gu.to_dev(sx[r]))
    Y, _ = _run(goq, bw, act, q, tokens, *dev(slice(None)), goq.F32)
    for r in (slice(0, 100), slice(tokens - 33, tokens), slice(tokens // 2, tokens // 2 + 100)):
        assert torch.equal(_run(goq, bw, act, q, r.stop - r.start, *dev(r), goq.F32)[0], Y[r]), r
    rows = np.r_[0:6, tokens - 6:tokens]
    ref, _ = oracle.gemm_a8(q, x[rows], sx[rows], threads=8, want_partials=True)
    scale = (np.abs(x[rows].astype(np.float64)) * sx[rows][:, None]) @ np.abs(oracle.dequant(q, want=("what",))["what"]).T + 1e-30
    assert np.max(np.abs(Y.cpu().numpy()[rows].astype(np.float64) - ref) / scale) <= 2e-6


@pytest.mark.parametrize("bw,act", [(3, "A16"), (4, "A16"), (3, "A8"), (4, "A8"), (4, "A4")])
@pytest.mark.parametrize("tokens,out,inn,order", [(165, 33001, 640, "2"), (16950, 1500, 512, "1")])
def test_tiles_in_ranges(oracle, ask, bw, act, tokens, out, inn, order):
    """Launches whose tiles are dealt to the XCDs in ranges of outputs and of tokens, ragged in both directions: every output is
    written, and sampled rows are the oracle's."""
    assert launch(ask, bw, act.lower(), tokens, [(out, inn)]) == (128 if act == "A4" and order == "1" else 64, [order])
    import paper_2605_26092_amd as goq
    print("ranges %s bw=%d %dx%dx%d" % (act, bw, tokens, out, inn), flush=True)
    q = goq_inputs.canonical_random(bw, out, inn, config_id=71, tensor_id=tokens)
    xd, sxd, x, sx = _inputs(goq, act, tokens, inn)
    Y, _ = _run(goq, bw, act, q, tokens, xd, sxd, goq.F32)
    assert gu.torch_cuda().isfinite(Y).all()
    rows = np.r_[0:3, 31:34, 63:66, 127:130, tokens // 2, tokens - 3:tokens]
    ref = oracle.gemm_a16(q, x[rows], threads=8) if sx is None else oracle.gemm_a8(q, x[rows], sx[rows], threads=8, want_partials=True)[0]
    scale = (np.abs(x[rows].astype(np.float64)) * (1.0 if sx is None else sx[rows][:, None])) @ np.abs(oracle.dequant(q, want=("what",))["what"]).T + 1e-30
    assert np.max(np.abs(Y[rows].cpu().numpy().astype(np.float64) - ref) / scale) <= 2e-6


@pytest.mark.parametrize("bw,act", [(3, "A16"), (3, "A8"), (4, "A8"), (4, "A4")])
@pytest.mark.parametrize("tokens,layers,order", [(165, [(33001, 640), (20001, 512)], "2"), (16950, [(1500, 640), (1000, 512)], "1")])
def test_ranges_of_a_second_layer(ask, bw, act, tokens, layers, order):
    """A batch whose second layer does not begin at a multiple of eight workgroups, so that its ranges belong to other XCDs than the
    first one's: the bits of single calls."""
    import paper_2605_26092_amd as goq
    from paper_2605_26092_amd import binding
    print("ranges of two %s bw=%d %d tokens %s" % (act, bw, tokens, layers), flush=True)
    tile, orders = launch(ask, bw, act.lower(), tokens, layers)
    assert orders == [order] * 2 and -(-tokens // tile) * -(-layers[0][0] // 128) % 8
    torch = gu.torch_cuda()
    problems, single = [], []
    for out, inn in layers:
        q = goq_inputs.canonical_random(bw, out, inn, config_id=74, tensor_id=out)
        xd, sxd, _, _ = _inputs(goq, act, tokens, inn)
        single.append(_run(goq, bw, act, q, tokens, xd, sxd, goq.F16)[0])
        Y = torch.full((tokens, out), float("nan"), dtype=torch.float16, device="cuda")
        problems.append((tokens, out, inn, gu.pack_layer(goq, q), xd, sxd, Y, goq.F16))
    goq.gemm_batch(bw, getattr(goq, act), binding.make_gemm_descs(problems))
    torch.cuda.synchronize()
    for p, y in zip(problems, single):
        assert torch.equal(p[6], y)
