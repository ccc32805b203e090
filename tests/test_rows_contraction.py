"""The row kernels at contractions of 29 to 148 products: the edges of their
matrix-step counts, ragged rows and channel groups, and the rule that plans
them by default.  Against the oracle with its own tolerance (one fp32 chain
per output, as in the kernels that the tolerance was derived for)."""
import numpy as np
import pytest

import oracle
import paper_1909_02765_amd as ilpm

ROWS = [v for v in range(ilpm.num_variants(ilpm.PATH_DIRECT))
        if ilpm.variant_name(ilpm.PATH_DIRECT, v).startswith(("direct_rows_k76", "direct_rows_k148"))]


def _name(v):
    return ilpm.variant_name(ilpm.PATH_DIRECT, v)


@pytest.mark.parametrize("v", ROWS, ids=_name)
def test_contraction_limit(v):
    """A plan up to the variant's contraction, none past it."""
    fits, past = ((3, 5), (1, 9)) if "_k76_" in _name(v) else ((3, 7), (1, 13))
    for (c_in, k), ok in ((fits, True), (past, False)):
        if ok:
            assert ilpm.plan_variant(c_in, 20, 20, 16, k, 1, 0, ilpm.PATH_DIRECT, v, 1).variant == v
        else:
            with pytest.raises(ilpm.IlpmError):
                ilpm.plan_variant(c_in, 20, 20, 16, k, 1, 0, ilpm.PATH_DIRECT, v, 1)


@pytest.mark.parametrize("shape,rows", [
    ((3, 224, 224, 64, 7, 2, 3), True), ((1, 40, 300, 9, 11, 4, 0), True), ((3, 224, 224, 64, 5, 1, 2), True),
    ((1, 175, 121, 52, 5, 1, 2), True), ((3, 64, 64, 96, 5, 1, 2), False), ((3, 117, 103, 23, 5, 1, 2), False),
    ((3, 11, 10, 70, 5, 1, 2), False), ((3, 38, 38, 10, 5, 1, 2), False), ((3, 104, 104, 29, 5, 1, 2), False),
    ((3, 100, 100, 32, 3, 2, 1), True), ((4, 100, 100, 32, 3, 2, 1), False), ((4, 64, 64, 64, 7, 1, 3), False),
    ((5, 64, 64, 64, 3, 1, 1), False), ((16, 64, 64, 64, 5, 2, 2), False)])
def test_default_plan(shape, rows):
    """Rows where the contraction fits, the LDS-tiled kernel has no 4-channel
    stage and is not the faster one (5x5 3->23 at 117x103: 4.3 us tiled, 5.6 by
    rows); pooled and prepacked calls keep a plan that pools and packs."""
    p = ilpm.plan(*shape)
    assert ("_rows_" in ilpm.variant_name(p.path, p.variant)) == rows
    if p.path == ilpm.PATH_DIRECT and rows:
        assert p.workspace_bytes == 0 and p.splits == 1
    if shape[4] == 5 and shape[5] == 1:
        q = ilpm.plan_prepacked(*shape)
        assert q.path == ilpm.PATH_IGEMM


@pytest.mark.parametrize("log2", [12, 16, 20, 24, 26, 27, 28, 29, 30, 31])
def test_strides_longer_than_the_lds(log2):
    """Strides whose segments do not fit in LDS, also where their length passes
    2^31: no row variant plans them unless its segment fits, and every plan's
    LDS is what its rows need (host only)."""
    for stride in {2 ** log2 - 1, min(2 ** log2, 2 ** 31 - 1), 3 * 2 ** (log2 - 2)}:
        for c_in, h, w, k, pad in [(1, 3, 3, 3, 0), (3, 5, 5, 5, 2), (3, 224, 224, 7, 3)]:
            for p in [ilpm.plan(c_in, h, w, 64, k, stride, pad)] + _row_plans(c_in, h, w, 64, k, stride, pad):
                assert 0 <= p.lds_bytes <= 160 * 1024
                if p.path == ilpm.PATH_DIRECT and "_rows_" in _name(p.variant):
                    assert p.lds_bytes >= 4 * c_in * k * ((p.tile_w - 1) * stride + k)


def _row_plans(*shape):
    plans = []
    for v in range(ilpm.num_variants(ilpm.PATH_DIRECT)):
        if "_rows_" in _name(v):
            try:
                plans.append(ilpm.plan_variant(*shape, ilpm.PATH_DIRECT, v, 1))
            except ilpm.IlpmError:
                pass
    return plans


@pytest.fixture
def gpu():
    import gpu_common
    gpu_common.torch_cuda()
    oracle.set_threads(16)
    return gpu_common


@pytest.mark.gpu
@pytest.mark.parametrize("v", ROWS, ids=_name)
def test_edges_against_oracle(gpu, v):
    """Contractions of 29, the limit and short of it; one channel more and less
    than the group; one-pixel rows, rows one pixel past a segment; stride 3;
    padding wider than the filter; widths with and without 16-byte rows."""
    limit = int(_name(v).split("_k")[1].split("_")[0])
    info = ilpm.variant_info(ilpm.PATH_DIRECT, v)
    cot, seg = info["co_tile"], info["tile_w"]
    shapes = [(29, 5, seg + 1, cot + 1, 1, 1, 0), (limit // 4, 6, 20, cot - 1, 2, 3, 2), (limit // 4, 3, 7, 2 * cot, 2, 1, 0),
              (limit // 9, 4, 9, 2 * cot, 3, 1, 0),
              (3, 11, 4 * seg, cot, 5 if limit == 76 else 7, 2, 3), (limit // 9, 9, seg, cot + 3, 3, 1, 4),
              (1, 7, 7, 5, 7, 1, 0)]
    for i, (c_in, h, w, c_out, k, s, pad) in enumerate(shapes):
        try:
            plan = ilpm.plan_variant(c_in, h, w, c_out, k, s, pad, ilpm.PATH_DIRECT, v, 1)
        except ilpm.IlpmError:
            continue  # rows too long for LDS
        gpu.note(f"[rows] {_name(v)} {shapes[i]}")
        x, wt, b = gpu.random_case(9500 + i, c_in, h, w, c_out, k, bias=i % 2 == 0)
        ref, sab = oracle.conv2d_f64(x, wt, b, s, pad)
        gpu.assert_matches(gpu.run_conv(x, wt, b, s, pad, plan=plan), ref, sab, c_in, k, f"{_name(v)} {shapes[i]}")


@pytest.mark.gpu
def test_default_route_matches_the_direct_kernel(gpu):
    """First layers whose default plan is a row kernel, with inputs that start
    off a 16-byte boundary, infinities and NaN: not finite where the per-output
    direct kernel's results are, and within rounding of it elsewhere."""
    import torch
    for i, (c_in, h, w, c_out, k, s, pad) in enumerate(
            [(3, 50, 52, 33, 7, 2, 3), (1, 33, 47, 20, 9, 1, 4), (1, 30, 30, 70, 5, 1, 2), (3, 21, 40, 16, 3, 2, 1)]):
        plan = ilpm.plan(c_in, h, w, c_out, k, s, pad)
        assert "_rows_" in ilpm.variant_name(plan.path, plan.variant)
        x, wt, b = gpu.random_case(9600 + i, c_in, h, w, c_out, k)
        x[0, 0, 5, 6], x[0, c_in - 1, 9, 9] = np.inf, np.nan
        flat = torch.empty(x.size + 1, device="cuda")
        xd = flat[1:].view(x.shape)
        xd.copy_(torch.from_numpy(x))
        wd, bd = gpu.dev(wt), gpu.dev(b)
        gpu.note(f"[rows default] {(c_in, h, w, c_out, k, s, pad)}")
        got = ilpm.conv2d(xd, wd, bd, s, pad)
        ref = ilpm.conv2d(gpu.dev(x), wd, bd, s, pad, plan=ilpm.plan_variant(c_in, h, w, c_out, k, s, pad, ilpm.PATH_DIRECT, 1, 1))
        torch.cuda.synchronize()
        g, r = got.cpu().numpy(), ref.cpu().numpy()
        np.testing.assert_array_equal(np.isnan(g), np.isnan(r))
        np.testing.assert_array_equal(np.isinf(g), np.isinf(r))
        fin = np.isfinite(r)
        # Two fp32 chains of kt products each: at most 2*(kt + 2) roundings of 2^-24 of sum|a*b|.
        xa = np.where(np.isfinite(x), np.abs(x), 0).astype(np.float32)
        bound = oracle.conv2d_f64(xa, np.abs(wt), np.abs(b), s, pad)[0] * 2 * (c_in * k * k + 2) * 2.0 ** -24
        assert np.all(np.abs(g - r)[fin] <= bound.reshape(r.shape)[fin])
