"""The bf16-split variants (fp32 operands as three bf16 parts): what the tests
over all variants do not reach -- 1x1 filters with a stride, tile edges, values
that are not finite, and the workspace rules of their default plans.  Against
the oracle with its own tolerance; the split's products are exact to 2^-24 and
its sums rounded less often than an fp32 chain's, so no wider one is needed."""
import numpy as np
import pytest

import oracle
import paper_1909_02765_amd as ilpm
import workloads

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
def test_default_call_without_room_for_partial_sums(gpu):
    """640->640 at 20x20: the default plan splits the channels, the plan of the
    fp32 variants needs no workspace.  With a registered workspace that is too
    small, and under capture with none, the call still runs."""
    import torch
    shape = (640, 20, 20, 640, 3, 1, 1)
    p = ilpm.plan(*shape)
    assert p.variant in SPLIT and p.splits > 1
    x = workloads.uniform(9500, (1, 640, 20, 20), 0.0, 1.0)
    wt = workloads.normal(9501, (640, 640, 3, 3), 0.0, workloads.he_std(640, 3))
    ref, sab = oracle.conv2d_f64(x, wt, None, 1, 1)
    small = torch.empty(1024, dtype=torch.float32, device="cuda")
    ilpm.set_workspace(small)
    try:
        gpu.note("[split] default call with a small registered workspace")
        got = gpu.run_conv(x, wt, None, 1, 1)
        gpu.assert_matches(got, ref, sab, 640, 3, "small workspace")
    finally:
        torch.cuda.synchronize()
        ilpm.set_workspace(None)
    xd, wd = gpu.dev(x), gpu.dev(wt)
    out = torch.empty((1, 640, 20, 20), device="cuda")
    ilpm.conv2d_noalloc(xd, wd, None, 1, 1, out=out)
    torch.cuda.synchronize()
    gpu.assert_matches(out.cpu().numpy(), ref, sab, 640, 3, "noalloc")
