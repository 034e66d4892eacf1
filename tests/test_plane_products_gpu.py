"""The split-bf16 products on pre-split operands: sizes at the edges of their
32-element blocks and of their 64, 128 and 256 tiles, odd strides (element-wise
float32 loads) and the layouts that keep float32 operands, against the oracle.

Tolerance: every product is accurate to 2^-16 of its operands' sizes and these
spectra (m >= 1.25 n Gaussian matrices, condition about 10 to 40) amplify a step's
error by at most their condition number: 40 * 2^-16 = 6e-4 in the worst case,
1e-5 to 4e-5 measured; 2e-4 is required.
"""
import numpy as np
import pytest

from _helpers import KIND_ISO, oracle_per_tensor, relF

TOL = 2e-4
STATIC_LIMIT = 128 << 20

EDGES = [(1, 1), (5, 1), (1, 7), (33, 26), (31, 64), (40, 32), (66, 33), (81, 64), (65, 130), (160, 127), (129, 260),
         (320, 255), (31, 300), (257, 700)]


def _step(iso, shapes, align, opts=None, seed=0, static=False, tiles=None):
    torch = pytest.importorskip("torch")
    from workload import custom_layout
    lay, n = custom_layout([(r, c, KIND_ISO) for r, c in shapes], align=align)
    dev = torch.device("cuda", 0)
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    # from theta = 0 with the single worker -Delta: Delta is exact in float32
    w = torch.randn(1, (n + 3) // 4 * 4, generator=g, device=dev).mul_(1e-3)[:, :n]
    theta = torch.zeros(n, device=dev)
    mom = torch.zeros(n, device=dev)
    plan = iso.IsoLoCoPlan(lay, n, 1, iso.ISOLOCO_F32, opts=opts, device=dev, workspace=not static)
    if tiles:
        p, cls = plan.products(), int(max(shapes[0]) >= 2 * min(shapes[0]))
        assert (p.gram_tile[cls], p.poly_tile[cls], p.update_tile[cls]) == tiles
    (plan.aggregate_static if static else plan.aggregate)(theta, w, mom, 1.0, 0.7, 0.9)
    torch.cuda.synchronize()
    st = plan.stats()
    plan.close()
    return lay, n, w.cpu().numpy()[0], theta.cpu().numpy(), mom.cpu().numpy(), st


def _check(lay, n, w, mom, st, select=None):
    zero = np.zeros(n, np.float32)
    ref = oracle_per_tensor(lay, zero, [w], zero, 1.0, 0.7, 0.9, select=select)
    for i, (_, b_r, sb_r) in ref.items():
        off, rows, cols, _ = lay[i]
        e = relF(mom[off:off + rows * cols], b_r)
        print("tensor %d (%d x %d): %.2e, sigma_bar %.2e, steps %d" %
              (i, rows, cols, e, abs(st[i].sigma_bar / sb_r - 1), st[i].steps), flush=True)
        assert e <= TOL, (rows, cols, e)
        assert abs(st[i].sigma_bar - sb_r) <= TOL * sb_r


@pytest.fixture(scope="module")
def iso():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_03011_amd as iso
    return iso


@pytest.mark.gpu
@pytest.mark.parametrize("align", [1, 4])
@pytest.mark.parametrize("precision", ["mixed", "bf16x3"])
def test_block_and_tile_edges(iso, align, precision):
    opts = {"precision": {"mixed": iso.ISOLOCO_PREC_MIXED, "bf16x3": iso.ISOLOCO_PREC_BF16X3}[precision]}
    lay, n, w, _, mom, st = _step(iso, EDGES, align, opts, seed=align)
    _check(lay, n, w, mom, st)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["mixed", "bf16x3"])
@pytest.mark.parametrize("name, shape, count, tiles", [
    # enough matrices for 128 x 128 and for 256 x 256 tiles, with and without
    # 16-byte aligned columns, tiles reaching past the matrix
    ("128", (252, 316), 100, (128, 128, 128)), ("128 odd", (249, 313), 100, (128, 128, 128)),
    ("256 symmetric", (500, 628), 60, (256, 256, 128)), ("256 symmetric odd", (499, 633), 60, (256, 256, 128)),
    ("256 update", (500, 760), 40, (128, 128, 256)), ("256 update odd", (499, 757), 40, (128, 128, 256)),
    # tall: factored steps, and a split Gram
    ("128 tall", (120, 509), 300, (128, 128, 128)), ("256 tall", (233, 997), 64, (64, 64, 256)),
    ("split", (4500, 250), 10, (64, 64, 256)), ("split 128", (4497, 250), 20, (128, 64, 128)),
    # thin, columns past n are not stored
    ("thin", (1500, 8), 40, (64, 64, 64)), ("thin wide", (33, 2050), 20, (64, 64, 64)),
    ("thin split", (4611, 17), 12, (64, 64, 64)),
])
def test_tile_shapes(iso, name, shape, count, tiles, precision):
    print("case: %s, %d matrices of %d x %d, %s" % (name, count, *shape, precision), flush=True)
    shapes = [shape] * count
    opts = {"precision": {"mixed": iso.ISOLOCO_PREC_MIXED, "bf16x3": iso.ISOLOCO_PREC_BF16X3}[precision]}
    lay, n, w, _, mom, st = _step(iso, shapes, 4, opts, seed=count, tiles=tiles)
    _check(lay, n, w, mom, st, select=[0, count - 1])
    # every matrix of the launch: an orthogonal factor
    assert all(0 <= s.orth_resid <= 1e-4 for s in st)


def test_small_matrices_keep_their_place_in_the_static_workspace():
    # padded to 32 x 32 blocks these would not fit the static workspace
    import paper_2607_03011_amd as iso
    from workload import custom_layout
    lay, n = custom_layout([(2, 2, KIND_ISO)] * 20000, align=4)
    h = iso.isoloco_plan(lay, n, 4)
    try:
        assert iso.isoloco_workspace_size(h) <= STATIC_LIMIT == iso.ISOLOCO_STATIC_WORKSPACE_BYTES
    finally:
        iso.isoloco_plan_destroy(h)


@pytest.mark.gpu
def test_small_matrices_static_step(iso):
    shapes = [(2, 2), (5, 4)] * 6000
    lay, n, w, _, mom, st = _step(iso, shapes, 4, seed=3, static=True)
    # (a 2 x 2 Gaussian matrix may be nearly singular: the 5 x 4 ones)
    _check(lay, n, w, mom, st, select=[1, 3, 11999])


@pytest.mark.gpu
def test_float32_operands_run_the_modes_products(iso):
    """A plan that keeps float32 operands (its factored steps would start at step
    1) runs the products of its mode: mixed, bf16x3 and bf16x6 all match the
    oracle, with different rounding."""
    moms = []
    for precision in (iso.ISOLOCO_PREC_MIXED, iso.ISOLOCO_PREC_BF16X3, iso.ISOLOCO_PREC_BF16X6):
        lay, n, w, _, mom, st = _step(iso, [(768, 256), (200, 600), (320, 256), (70, 50)], 4,
                                      dict(precision=precision, phase_tall=(0.1, -1.0, -1.0)), seed=4)
        _check(lay, n, w, mom, st)
        moms.append(mom)
    for i in range(3):
        for j in range(i):
            assert not np.array_equal(moms[i], moms[j]), (i, j)
