"""The bf16-split variants (fp32 operands as three bf16 parts): what the tests
over all variants do not reach -- 1x1 filters with a stride, tile edges, values
that are not finite, and what their default plans may need.  Against
the oracle with its own tolerance; the split's products are exact to 2^-24 and
its sums rounded less often than an fp32 chain's, so no wider one is needed."""
import numpy as np
import pytest

import oracle
import paper_1909_02765_amd as ilpm

SPLIT = [v for v in range(ilpm.num_variants(ilpm.PATH_IGEMM)) if "_b3_" in ilpm.variant_name(ilpm.PATH_IGEMM, v)]


def _name(v):
    return ilpm.variant_name(ilpm.PATH_IGEMM, v)


@pytest.mark.parametrize("v", SPLIT, ids=_name)
def test_tiles_fit_their_variant(v):
    """Every plan's tile is within the variant's pixel slots and halo room and
    covers the output; `_even` variants plan even sides only (host only)."""
    info = ilpm.variant_info(ilpm.PATH_IGEMM, v)
    k, s = info["k"], info["stride"]
    px = int(_name(v).split("_px")[1].split("_")[0])
    rng = np.random.default_rng(v)
    for _ in range(200):
        h, w = (int(n) for n in np.exp(rng.uniform(np.log(1), np.log(400), 2)))
        stride = int(rng.integers(1, 4)) if k == 1 else s
        p = ilpm.plan_variant(20, h, w, 40, k, stride, k // 2, ilpm.PATH_IGEMM, v, 1)
        th, tw = p.tile_h, p.tile_w
        assert th >= 1 and tw >= 1 and th * tw <= px
        if _name(v).endswith("_even"):
            assert th % 2 == 0 and tw % 2 == 0
        tiles = -(-p.h_out // th) * -(-p.w_out // tw) * -(-40 // p.co_tile)
        assert p.grid == tiles * p.splits


def test_default_plans_stay_within_the_noalloc_array():
    """A default bf16-split plan never needs more than the no-alloc array."""
    seen = 0
    for c_in, h, w, c_out, k, s in [(640, 20, 20, 640, 3, 1), (320, 71, 97, 144, 3, 1), (512, 14, 14, 1024, 1, 2),
                                    (1024, 40, 40, 1024, 3, 1), (64, 400, 400, 64, 3, 1), (256, 60, 60, 256, 5, 1)]:
        p = ilpm.plan(c_in, h, w, c_out, k, s, k // 2)
        if p.path == ilpm.PATH_IGEMM and p.variant in SPLIT:
            seen += 1
            assert p.workspace_bytes <= ilpm.NOALLOC_SCRATCH_BYTES
    assert seen >= 3


# Shapes, and the workspace that the fp32 variants' plan of each needs.
BASE_WORKSPACE = [
    ((640, 20, 20, 640, 3, 1, 1), 0), ((388, 15, 16, 399, 3, 1, 1), 0), ((256, 115, 106, 32, 3, 1, 1), 0),
    ((400, 56, 90, 256, 3, 1, 1), 0), ((130, 78, 78, 182, 3, 1, 1), 0), ((208, 21, 23, 224, 1, 2, 0), 0),
    ((448, 33, 40, 112, 1, 2, 0), 0), ((240, 11, 11, 32, 1, 2, 0), 0), ((576, 89, 89, 176, 3, 2, 1), 0),
    ((329, 47, 47, 391, 3, 2, 1), 0), ((144, 61, 68, 32, 5, 1, 2), 0), ((592, 70, 91, 32, 5, 1, 2), 0),
    ((44, 84, 84, 52, 5, 2, 2), 0), ((30, 38, 38, 16, 5, 2, 2), 0), ((340, 53, 53, 341, 3, 1, 1), 7662952),
    ((377, 11, 11, 579, 3, 1, 1), 3362832), ((144, 43, 43, 624, 3, 2, 1), 2416128),
    ((606, 22, 22, 111, 5, 1, 2), 429792), ((247, 37, 56, 45, 5, 1, 2), 1491840)]


@pytest.mark.parametrize("shape,most", BASE_WORKSPACE, ids=str)
def test_default_plans_need_no_more_than_the_fp32_plans(shape, most):
    """What a caller may do with a shape (overlap calls of it on several
    streams, capture the first call, register a small workspace) does not
    shrink with the bf16-split plans: unsplit where the fp32 plan is, on both
    weight layouts and with either epilogue, and never more workspace."""
    for prepacked in (False, True):
        for epi in (0, ilpm.EPI_RELU | ilpm.EPI_MAXPOOL2):
            p = ilpm.plan_for(*shape, epi, prepacked)
            assert p.workspace_bytes <= most
            assert most > 0 or p.splits == 1


@pytest.mark.parametrize("shape", [(512, 105, 105, 368, 1, 1, 0), (320, 98, 145, 128, 3, 1, 1),
                                   (46, 171, 171, 51, 3, 1, 1), (79, 113, 113, 493, 3, 1, 1), (17, 45, 45, 72, 5, 1, 2)],
                         ids=str)
def test_plain_plans_pool_where_the_fp32_plans_do(shape):
    """Shapes whose fp32 plan pools in its kernel when the pooled epilogue is
    called with the plain plan: the default plain plan does too."""
    for prepacked in (False, True):
        p = ilpm.plan_for(*shape, 0, prepacked)
        assert p.path == ilpm.PATH_IGEMM and p.splits == 1
        assert p.tile_h % 2 == 0 and p.tile_w % 2 == 0
        if p.variant in SPLIT:
            assert _name(p.variant).endswith("_even")


@pytest.mark.parametrize("shape", [(512, 60, 60, 256, 1, 1, 0), (256, 56, 56, 128, 1, 1, 0), (256, 28, 28, 512, 1, 1, 0),
                                   (189, 122, 164, 222, 1, 1, 0), (19, 114, 114, 196, 1, 1, 0),
                                   (64, 224, 224, 64, 3, 1, 1)], ids=str)
def test_tiles_are_wide(shape):
    """Tiles of long rows: neighbouring lanes load and store neighbouring
    pixels, and a tile of short rows touches a 64-byte piece per row and
    channel for a few floats each (512->256 at 60^2: 47 us as 60x1 pixels, 13 as
    1x60)."""
    for prepacked in (False, True):
        for epi in (0, ilpm.EPI_RELU | ilpm.EPI_MAXPOOL2):
            p = ilpm.plan_for(*shape, epi, prepacked)
            assert p.variant in SPLIT
            assert p.tile_w >= min(28, p.w_out) and p.tile_w >= 4 * p.tile_h


# Layers on which the fp32 plan was measured faster than a bf16-split one that a
# cost model without the tiles' shape had chosen (us: fp32, bf16-split).
FP32_FASTER = [((304, 120, 120, 304, 1, 1, 0), 36.4, 180.5), ((64, 121, 97, 128, 1, 1, 0), 7.1, 29.9),
               ((24, 204, 204, 41, 1, 1, 0), 6.8, 12.8), ((48, 139, 139, 112, 1, 1, 0), 8.3, 14.4),
               ((28, 84, 84, 99, 1, 1, 0), 4.7, 8.8), ((128, 193, 309, 384, 1, 1, 0), 73.7, 96.9),
               ((18, 101, 73, 28, 5, 1, 2), 7.8, 10.2), ((23, 180, 305, 37, 3, 2, 1), 9.4, 12.1)]


@pytest.mark.parametrize("shape,fp32,split", FP32_FASTER, ids=str)
def test_fp32_plans_stay_where_they_are_faster(shape, fp32, split):
    p = ilpm.plan(*shape)
    assert p.path == ilpm.PATH_IGEMM and p.variant not in SPLIT


def test_overrides_take_the_split_variants():
    """The environment overrides narrow all matrix-core variants, bf16-split ones
    among them: the matrix-core family alone takes 1x1 filters with a stride
    (that only they run), plans the headline layer as it does by itself, and
    splits and tiles are those asked for."""
    from test_abi import plans_with_env
    strided, early, deep = (256, 56, 56, 512, 1, 2, 0), (64, 224, 224, 64, 3, 1, 1), (320, 71, 97, 144, 3, 1, 1)
    default = plans_with_env({}, [early])
    got = plans_with_env({"ILPM_FORCE_PATH": "igemm"}, [strided, early])
    assert got[0]["path"] == ilpm.PATH_IGEMM and "_b3_" in got[0]["name"] and got[0]["splits"] == 1
    assert got[1] == default[0] and "_b3_" in got[1]["name"]
    got = plans_with_env({"ILPM_SPLIT": "2"}, [strided, deep])
    assert all(g["splits"] == 2 for g in got) and "_b3_" in got[0]["name"]
    got = plans_with_env({"ILPM_TILE": "8x32"}, [early])
    assert got[0]["tile"] == [8, 32] and "_b3_" in got[0]["name"]
    got = plans_with_env({"ILPM_FORCE_PATH": "direct"}, [strided, early])
    assert all(g["path"] == ilpm.PATH_DIRECT for g in got)


@pytest.fixture
def gpu():
    import gpu_common
    gpu_common.torch_cuda()
    oracle.set_threads(16)
    return gpu_common


@pytest.mark.gpu
@pytest.mark.parametrize("v", SPLIT, ids=_name)
def test_edges_against_oracle(gpu, v):
    """One and several stages, the last one partial; one output channel more
    or less than the tile; one-pixel, one-row and one-column outputs; 1x1 with
    strides 1 to 3 and padding."""
    info = ilpm.variant_info(ilpm.PATH_IGEMM, v)
    k, cc, cot = info["k"], info["ci_chunk"], info["co_tile"]
    shapes = [(1, k, k, 1, 0), (cc, 3 + k, 70, cot + 1, 0), (2 * cc + 3, 40, k + 1, cot - 1, k // 2),
              (5 * cc - 1, 9, 11, 2 * cot, k)]
    for i, (c_in, h, w, c_out, pad) in enumerate(shapes):
        for stride in (1, 2, 3) if k == 1 else (info["stride"],):
            x, wt, b = gpu.random_case(9300 + 10 * i, c_in, h, w, c_out, k, bias=i % 2 == 0)
            ref, sab = oracle.conv2d_f64(x, wt, b, stride, pad)
            for splits in (1, 2):
                try:
                    plan = ilpm.plan_variant(c_in, h, w, c_out, k, stride, pad, ilpm.PATH_IGEMM, v, splits)
                except ilpm.IlpmError:
                    continue
                gpu.note(f"[split] {_name(v)} {(c_in, h, w, c_out, k, stride, pad)} splits {plan.splits}")
                got = gpu.run_conv(x, wt, b, stride, pad, plan=plan)
                gpu.assert_matches(got, ref, sab, c_in, k, f"{_name(v)} {shapes[i]} s{stride}")


@pytest.mark.gpu
@pytest.mark.parametrize("v", SPLIT, ids=_name)
def test_values_that_are_not_finite(gpu, v):
    """Infinities, NaN, values whose bf16 rounding overflows and subnormals:
    the outputs are infinite, NaN and finite where the VALU kernel's are, on
    both weight layouts alike, and the finite ones agree."""
    import torch
    info = ilpm.variant_info(ilpm.PATH_IGEMM, v)
    k, s = info["k"], info["stride"]
    x, wt, b = gpu.random_case(9400, 24, 16, 16, 40, k)
    x[0, 3, 4, 5], x[0, 7, 9, 9], x[0, 8, 2, 2], x[0, 1, 12, 12] = np.inf, np.nan, 3.4e38, 1e-42
    wt[5, 2] = -np.inf
    xd, wd, bd = gpu.dev(x), gpu.dev(wt), gpu.dev(b)
    base = ilpm.conv2d(xd, wd, bd, s, k // 2, plan=ilpm.plan_variant(24, 16, 16, 40, k, s, k // 2, ilpm.PATH_DIRECT, 0))
    for splits in (1, 2):
        try:
            plan = ilpm.plan_variant(24, 16, 16, 40, k, s, k // 2, ilpm.PATH_IGEMM, v, splits)
        except ilpm.IlpmError:
            continue
        gpu.note(f"[split not finite] {_name(v)} splits {plan.splits}")
        got = ilpm.conv2d(xd, wd, bd, s, k // 2, plan=plan)
        packed = ilpm.conv2d_prepacked(xd, ilpm.prepack_weights(wd, plan), 40, k, bd, s, k // 2, plan=plan)
        torch.cuda.synchronize()
        g, q, r = (t.cpu().numpy() for t in (got, packed, base))
        np.testing.assert_array_equal(np.isnan(g), np.isnan(r))
        np.testing.assert_array_equal(np.isposinf(g), np.isposinf(r))
        np.testing.assert_array_equal(np.isneginf(g), np.isneginf(r))
        np.testing.assert_array_equal(g, q)
        fin = np.isfinite(r)
        assert fin.sum() > 1000
        # Two fp32 sums of n products each: at most n * 2^-23 of the sum of
        # their magnitudes (here below n) apart, relative to the larger.
        n = 24 * k * k
        big = np.abs(r[fin]) > 1e6  # the outputs that 3.4e38 reaches
        np.testing.assert_allclose(g[fin][~big], r[fin][~big], rtol=0, atol=n * n * 2.0 ** -23)
        np.testing.assert_allclose(g[fin][big], r[fin][big], rtol=n * 2.0 ** -23)


@pytest.mark.gpu
@pytest.mark.parametrize("v", [v for v in SPLIT if not _name(v).endswith("_even")], ids=_name)
def test_small_values(gpu, v):
    """Inputs, or weights, scaled by 2^-90 to 2^-140: bf16 ends at 2^-133, so
    below 2^-109 an operand keeps an absolute error of 2^-134, and above it 24
    bits.  Per product |x||w| then at most 2^-22 of it (operands and dropped
    parts), 2^-134 of the other operand and, per addition, 2^-149."""
    info = ilpm.variant_info(ilpm.PATH_IGEMM, v)
    k, s = info["k"], info["stride"]
    x, wt, _ = gpu.random_case(9700, 40, 18, 21, info["co_tile"], k)
    ones_x, ones_w = np.ones_like(x), np.ones_like(wt)
    plan = ilpm.plan_variant(40, 18, 21, info["co_tile"], k, s, k // 2, ilpm.PATH_IGEMM, v, 1)
    for log2 in (-90, -108, -115, -120, -130, -140):
        for xs, ws in ((x * np.float32(2.0 ** log2), wt), (x, wt * np.float32(2.0 ** log2))):
            gpu.note(f"[split small values] {_name(v)} 2^{log2}")
            got = gpu.run_conv(xs, ws, None, s, k // 2, plan=plan).astype(np.float64)
            ref, sab = oracle.conv2d_f64(xs, ws, None, s, k // 2)
            other = 2.0 ** -134 * (oracle.conv2d_f64(np.abs(xs), ones_w, None, s, k // 2)[0] +
                                   oracle.conv2d_f64(ones_x, np.abs(ws), None, s, k // 2)[0])
            bound = sab.reshape(ref.shape) * 2.0 ** -20 + other + 40 * k * k * 2.0 ** -149
            assert np.all(np.abs(got.reshape(ref.shape) - ref) <= bound), f"2^{log2}"


@pytest.mark.gpu
@pytest.mark.parametrize("v", [v for v in SPLIT if _name(v).endswith("_even")], ids=_name)
def test_pooled_values_that_are_not_finite(gpu, v):
    """The same values through the 2x2 max-pool in the kernel, on both weight
    layouts: the bits of the unpooled result of the same plan, ReLU and the
    windows taken in the kernels' order (a NaN stays only as a window's first)."""
    import torch
    info = ilpm.variant_info(ilpm.PATH_IGEMM, v)
    k, s = info["k"], info["stride"]
    c_in, c_out = 2 * info["ci_chunk"] + 5, info["co_tile"] + 3
    x, wt, b = gpu.random_case(9450, c_in, 30, 34, c_out, k)
    x[0, 3, 4, 5], x[0, 7, 9, 9], x[0, 8, 2, 2], x[0, c_in - 1, 22, 23] = np.inf, np.nan, 3.4e38, -np.inf
    x[0, 2, 16, 16] = np.nan  # a window's first, of 1x1 filters too
    wt[5, 2] = -np.inf
    xd, wd, bd = gpu.dev(x), gpu.dev(wt), gpu.dev(b)
    plan = ilpm.plan_variant(c_in, 30, 34, c_out, k, s, k // 2, ilpm.PATH_IGEMM, v, 1)
    packed = ilpm.prepack_weights(wd, plan)
    gpu.note(f"[split pooled not finite] {_name(v)}")
    epi = ilpm.EPI_RELU | ilpm.EPI_MAXPOOL2
    full = ilpm.conv2d(xd, wd, bd, s, k // 2, plan=plan).cpu().numpy()
    got = ilpm.conv2d_epilogue(xd, wd, bd, s, k // 2, epi, plan=plan)
    got_packed = ilpm.conv2d_prepacked_epilogue(xd, packed, c_out, k, bd, s, k // 2, epi, plan=plan)
    torch.cuda.synchronize()
    ho, wo = full.shape[2] // 2 * 2, full.shape[3] // 2 * 2
    windows = [full[:, :, i:ho:2, j:wo:2] for i in (0, 1) for j in (0, 1)]
    want = windows[0]
    with np.errstate(invalid="ignore"):
        for q in windows[1:]:
            want = np.where(q > want, q, want)
        want = np.where(want < 0, np.float32(0), want)
    assert np.isnan(want).any() and np.isinf(want).any()
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    np.testing.assert_array_equal(got_packed.cpu().numpy(), want)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(64, 224, 224, 64, 3, 1, 1), (512, 60, 60, 256, 1, 1, 0), (96, 90, 90, 64, 5, 2, 2)], ids=str)
def test_values_that_are_not_finite_cost_no_more_than_a_few_calls(gpu, shape):
    """One NaN pixel, and NaN everywhere: the outputs they reach are computed
    again, in at most 20 times a finite call's time (measured 2 to 8; by single
    lanes it was more than 100)."""
    import torch
    c_in, h, w, c_out, k, s, pad = shape
    plan = ilpm.plan(*shape)
    assert plan.variant in SPLIT
    x, wt, b = gpu.random_case(9600, c_in, h, w, c_out, k)
    xd, wd, bd = gpu.dev(x), gpu.dev(wt), gpu.dev(b)
    one = xd.clone()
    one[0, 3, h // 2, w // 2] = float("nan")
    out = ilpm.conv2d(xd, wd, bd, s, pad)

    def us(t):
        times = []
        for _ in range(10):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            for _ in range(4):
                ilpm.conv2d(t, wd, bd, s, pad, out=out)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1) * 250.0)
        return sorted(times)[5]

    for _ in range(3):
        us(xd)
    finite, single, every = us(xd), us(one), us(torch.full_like(xd, float("nan")))
    gpu.note(f"[split not finite, time] {shape}: finite {finite:.1f} us, one NaN {single:.1f}, all NaN {every:.1f}")
    assert single < 20 * finite and every < 20 * finite


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(388, 15, 16, 399, 3, 1, 1), (208, 21, 23, 224, 1, 2, 0), (144, 61, 68, 32, 5, 1, 2),
                                   (44, 84, 84, 52, 5, 2, 2)], ids=str)
def test_unsplit_shapes_need_no_workspace(gpu, shape):
    """Shapes whose fp32 plan is unsplit: their default calls run beside a
    registered workspace that is too small for any partial sums, and under
    capture there, OIHW and packed, with the bits of the no-alloc call."""
    import torch
    c_in, h, w, c_out, k, s, pad = shape
    x, wt, b = gpu.random_case(9500, c_in, h, w, c_out, k)
    ref, sab = oracle.conv2d_f64(x, wt, b, s, pad)
    xd, wd, bd = gpu.dev(x), gpu.dev(wt), gpu.dev(b)
    plan = ilpm.plan_prepacked(*shape)
    packed = ilpm.prepack_weights(wd, plan)
    ho, wo = ilpm.out_size(h, k, s, pad), ilpm.out_size(w, k, s, pad)
    out, out_packed = (torch.empty((1, c_out, ho, wo), device="cuda") for _ in range(2))
    want = ilpm.conv2d_noalloc(xd, wd, bd, s, pad, out=out).cpu().numpy()
    gpu.assert_matches(want, ref, sab, c_in, k, f"noalloc {shape}")
    small = torch.empty(64, dtype=torch.float32, device="cuda")
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    ilpm.set_workspace(small)
    try:
        gpu.note(f"[split] {shape} with a small registered workspace")
        np.testing.assert_array_equal(gpu.run_conv(x, wt, b, s, pad), want)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            ilpm.conv2d(xd, wd, bd, s, pad, out=out)
            ilpm.conv2d_prepacked(xd, packed, c_out, k, bd, s, pad, out=out_packed, plan=plan)
        for i in range(3):
            out.fill_(float("nan"))
            out_packed.fill_(float("nan"))
            g.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(out.cpu().numpy(), want, err_msg=f"replay {i}")
            np.testing.assert_array_equal(out_packed.cpu().numpy(), want, err_msg=f"replay {i}, packed")
    finally:
        torch.cuda.synchronize()
        ilpm.set_workspace(None)
