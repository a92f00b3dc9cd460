"""Host-side checks of the planner (no GPU): every plan it hands out must fit the
machine (LDS per workgroup, a non-empty grid, a workspace that covers the partial
results), for the benchmark layers and for a seeded sweep of other descriptors, and
the kernel families must be chosen where they apply."""
import re

import numpy as np
import pytest

from paper_1808_05567_amd import conv, inputs

LDS_PER_CU = 160 * 1024


def _plans(shape, dt):
    h = conv.conv_create(*shape, dt)
    out = {}
    try:
        info = conv.conv_query(h)
        for which in (conv.PASS_FWD, conv.PASS_BWD_DATA, conv.PASS_UPD):
            # (every pass has a plan: a tiled kernel, or the untiled direct one)
            out[which] = conv.conv_describe(h, which)
    finally:
        conv.conv_destroy(h)
    return info, out


def _field(text, name):
    m = re.search(r"\b%s=(\d+)" % name, text)
    assert m, (name, text)
    return int(m.group(1))


def _tiled(text):
    return not text.startswith("direct ")


def _check(info, plans):
    for which, text in plans.items():
        if _tiled(text):
            assert 0 < _field(text, "lds") <= LDS_PER_CU, text
        else:
            assert _field(text, "lds") <= 64 * 1024, text  # static LDS only
        assert 1 <= _field(text, "grid") < 2 ** 31, text
    assert info.upd_splits >= 1
    if _tiled(plans[conv.PASS_UPD]):
        # every partial copy of dW the update kernel writes fits the workspace
        assert info.workspace_bytes >= info.upd_splits * info.dwt_bytes
    else:
        assert info.upd_splits == 1  # the direct kernel writes dW itself
    if _tiled(plans[conv.PASS_BWD_DATA]):
        # the transformed weights of the backward pass live in the workspace
        assert info.workspace_bytes >= 16


@pytest.mark.parametrize("dt", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 256])
def test_inception_v3_plans_fit_the_machine(N, dt):
    """Every shape of the second workload has a tiled kernel in all three passes (rectangular filters, per-axis
    padding, unpadded stride 2, rows wider than an update band)."""
    assert len(inputs.INCEPTION_V3) == 43
    for l in inputs.INCEPTION_V3:
        info, plans = _plans((N, l.C, l.K, l.H, l.W, l.R, l.S, l.stride, l.pad), dt)
        _check(info, plans)
        assert all(_tiled(p) for p in plans.values()), (l.id, plans)
        assert (info.P, info.Q) == (l.P, l.Q)


def test_update_of_tall_filters_and_wide_rows(monkeypatch):
    def upd(shape, dt=conv.CONV_F32):
        return _plans(shape, dt)[1][conv.PASS_UPD]
    shapes = [(4, 64, 64, 17, 17, 7, 1, 1, (3, 0)), (4, 64, 64, 17, 17, 1, 7, 1, (0, 3)), (4, 48, 64, 35, 35, 5, 5, 1, 2),
              (2, 32, 64, 147, 147, 3, 3, 1, 1)]
    for s in shapes:
        for dt in (conv.CONV_F32, conv.CONV_BF16):
            assert upd(s, dt).startswith("upd_ring ") and "launches=1" in upd(s, dt)
    # without the ring kernel (images and minibatches beyond its indices)
    monkeypatch.setenv("CONVMI_UPD_RING", "0")
    # 7x1 and 1x7: one launch; 5x5: one launch per filter row
    assert "RS=7x1" in upd(shapes[0]) and "launches=1" in upd(shapes[0])
    assert "launches=1" in upd(shapes[1])
    assert "RS=1x5" in upd(shapes[2]) and "launches=5" in upd(shapes[2])
    # 147-wide rows: strips of output columns, one launch each
    assert "launches=3" in upd(shapes[3])
    assert "launches=2" in upd(shapes[3], conv.CONV_BF16)


@pytest.mark.parametrize("dt", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 2, 256])
def test_table1_plans_fit_the_machine(N, dt):
    for l in inputs.TABLE_I:
        info, plans = _plans((N, l.C, l.K, l.H, l.W, l.R, l.S, l.stride, l.pad), dt)
        _check(info, plans)
        assert all(_tiled(p) for p in plans.values()), (l.id, plans)


def test_seeded_descriptor_sweep_plans_fit_the_machine():
    rng = np.random.default_rng(180805567)
    planned = 0
    for _ in range(400):
        R = int(rng.choice([1, 1, 3, 3, 7]))
        stride = int(rng.choice([1, 1, 2, 3]))
        pad = int(rng.integers(0, R // 2 + 1))
        H = int(rng.integers(max(R, 1), 70))
        W = int(rng.integers(max(R, 1), 70))
        C = int(rng.choice([1, 3, 4, 8, 20, 64, 100, 128, 256, 264, 512, 1030]))
        K = int(rng.choice([1, 8, 12, 64, 72, 128, 256, 320, 1024, 2048]))
        N = int(rng.choice([1, 2, 3, 16, 64]))
        for dt in (conv.CONV_F32, conv.CONV_BF16):
            info, plans = _plans((N, C, K, H, W, R, R, stride, pad), dt)
            _check(info, plans)
            planned += sum(_tiled(p) for p in plans.values())
    assert planned > 1500  # most passes have a tiled kernel


def test_seeded_rectangular_sweep_plans_fit_the_machine():
    """Rectangular filters, padding per axis, images up to 300 wide (column strips)."""
    rng = np.random.default_rng(1808055670)
    planned = 0
    for _ in range(300):
        R, S = [(1, 7), (7, 1), (1, 3), (3, 1), (5, 5), (3, 3), (1, 5), (5, 1), (3, 7)][int(rng.integers(0, 9))]
        stride = int(rng.choice([1, 1, 1, 2]))
        ph, pw = int(rng.integers(0, R // 2 + 2)), int(rng.integers(0, S // 2 + 2))
        H = int(rng.integers(R, 40))
        W = int(rng.integers(S, 300 if rng.integers(0, 4) == 0 else 40))
        C = int(rng.choice([3, 8, 32, 48, 160, 192, 384]))
        K = int(rng.choice([8, 32, 64, 96, 160, 192, 448]))
        N = int(rng.choice([1, 2, 32]))
        for dt in (conv.CONV_F32, conv.CONV_BF16):
            info, plans = _plans((N, C, K, H, W, R, S, stride, (ph, pw)), dt)
            _check(info, plans)
            assert (info.P, info.Q) == ((H + 2 * ph - R) // stride + 1, (W + 2 * pw - S) // stride + 1)
            planned += sum(_tiled(p) for p in plans.values())
    assert planned > 1000  # (tiled kernels; the rest run on the direct ones)


def test_update_families_without_the_ring_kernel(monkeypatch):
    monkeypatch.setenv("CONVMI_UPD_RING", "0")
    # fp32 1x1 with 256 channels on one side: eight-wave kernel on the flat pixel list
    _, p = _plans((256, 256, 1024, 14, 14, 1, 1, 1, 0), conv.CONV_F32)
    assert p[conv.PASS_UPD].startswith("upd_1x1 dt=0") and "in x out" in p[conv.PASS_UPD]
    _, p = _plans((256, 64, 256, 56, 56, 1, 1, 1, 0), conv.CONV_F32)
    assert p[conv.PASS_UPD].startswith("upd_1x1 dt=0") and "out x in" in p[conv.PASS_UPD]
    # ... below that, the four-wave kernel
    _, p = _plans((256, 64, 64, 56, 56, 1, 1, 1, 0), conv.CONV_F32)
    assert p[conv.PASS_UPD].startswith("upd dt=0")
    # bf16 1x1: flat pixel list at every width
    for C, K in ((64, 64), (64, 256), (1024, 2048)):
        _, p = _plans((256, C, K, 14, 14, 1, 1, 1, 0), conv.CONV_BF16)
        assert p[conv.PASS_UPD].startswith("upd_1x1 dt=1")
    # 3x3 stride 1: band kernel (fp32), row kernel (bf16)
    _, p = _plans((256, 256, 256, 14, 14, 3, 3, 1, 1), conv.CONV_F32)
    assert p[conv.PASS_UPD].startswith("upd_bands")
    _, p = _plans((256, 256, 256, 14, 14, 3, 3, 1, 1), conv.CONV_BF16)
    assert p[conv.PASS_UPD].startswith("upd_rows")


# N, C, K, H, R, stride, pad, type: update kernel, on either side of the ring kernel's lines
RING_LINES = [
    (128, 512, 1024, 28, 1, 2, 0, conv.CONV_F32, "upd_ring dt=0"), (192, 512, 1024, 28, 1, 2, 0, conv.CONV_F32, "upd_1x1 dt=0"),
    (256, 760, 760, 9, 1, 1, 0, conv.CONV_F32, "upd_ring dt=0"), (256, 256, 512, 56, 1, 2, 0, conv.CONV_F32, "upd_1x1 dt=0"),
    (256, 64, 64, 56, 1, 1, 0, conv.CONV_F32, "upd_ring dt=0"), (256, 256, 256, 14, 3, 1, 1, conv.CONV_F32, "upd_ring dt=0"),
    (64, 64, 256, 56, 1, 1, 0, conv.CONV_BF16, "upd_ring dt=1"), (128, 64, 256, 56, 1, 1, 0, conv.CONV_BF16, "upd_1x1 dt=1"),
    (128, 64, 64, 56, 1, 1, 0, conv.CONV_BF16, "upd_ring dt=1"), (256, 64, 64, 56, 1, 1, 0, conv.CONV_BF16, "upd_1x1 dt=1"),
    (160, 512, 256, 28, 1, 2, 0, conv.CONV_BF16, "upd_ring dt=1"), (192, 512, 256, 28, 1, 2, 0, conv.CONV_BF16, "upd_1x1 dt=1"),
    (160, 288, 64, 35, 1, 1, 0, conv.CONV_BF16, "upd_ring dt=1"), (160, 768, 192, 17, 1, 1, 0, conv.CONV_BF16, "upd_1x1 dt=1"),
    (96, 1024, 2048, 14, 1, 2, 0, conv.CONV_BF16, "upd_ring dt=1"), (128, 1024, 2048, 14, 1, 2, 0, conv.CONV_BF16, "upd_1x1 dt=1"),
    (64, 288, 384, 35, 3, 2, 0, conv.CONV_BF16, "upd_ring dt=1"), (96, 288, 384, 35, 3, 2, 0, conv.CONV_BF16, "upd_rows dt=1"),
    (256, 256, 256, 14, 3, 1, 1, conv.CONV_BF16, "upd_ring dt=1"),
]


@pytest.mark.parametrize("case", RING_LINES, ids=lambda c: "x".join(map(str, c[:7])) + ("-bf16" if c[7] else "-f32"))
def test_update_on_either_side_of_the_ring_kernels_lines(case):
    N, C, K, H, R, stride, pad, dt, want = case
    assert _plans((N, C, K, H, H, R, R, stride, pad), dt)[1][conv.PASS_UPD].startswith(want)


def test_kernel_families_are_chosen_where_they_apply():
    # one input channel block, fp32: filter-row kernel; backward: all classes in one launch
    _, p = _plans((256, 3, 64, 224, 224, 7, 7, 2, 3), conv.CONV_F32)
    assert p[conv.PASS_UPD].startswith("upd_c4")
    assert "launches=1" in p[conv.PASS_BWD_DATA]
    # 3x3 stride 2 backward: the residue classes in one launch, fp32 one launch each where a long reduction over
    # few tiles would be one chain
    for C, dt, launches in ((64, conv.CONV_F32, 1), (256, conv.CONV_F32, 4), (256, conv.CONV_BF16, 1)):
        _, p = _plans((4, C, C, 14, 14, 3, 3, 2, 1), dt)
        assert "launches=%d" % launches in p[conv.PASS_BWD_DATA]
    # a filter without a staged kernel: the register-operand kernel, whatever the size
    _, p = _plans((1, 8, 8, 9, 9, 1, 5, 1, (0, 2)), conv.CONV_F32)
    assert p[conv.PASS_FWD].startswith("igemm_reg ") and p[conv.PASS_BWD_DATA].startswith("igemm_reg ")
    # small minibatch, long reduction: the forward reduction is split
    _, p = _plans((1, 512, 512, 7, 7, 3, 3, 1, 1), conv.CONV_F32)
    assert _field(p[conv.PASS_FWD], "ksplit") > 1


def _describe_all(h):
    return [conv.conv_describe(h, w) for w in (conv.PASS_FWD, conv.PASS_BWD_DATA, conv.PASS_UPD)]


def test_minibatch_chunks_on_request():
    shape = (10, 64, 64, 14, 14, 3, 3, 1, 1)
    h = conv.conv_create_chunked(*shape, 4)
    try:
        info = conv.conv_query(h)
        assert all(t.startswith("chunks=3 images=4: ") for t in _describe_all(h))
        # one dW per chunk behind the chunks' own workspace
        assert info.upd_splits == 3 and info.workspace_bytes >= 3 * info.dwt_bytes
    finally:
        conv.conv_destroy(h)
    # a bound the minibatch already meets changes nothing
    h, g = conv.conv_create_chunked(*shape, 10), conv.conv_create(*shape)
    try:
        assert _describe_all(h) == _describe_all(g)
    finally:
        conv.conv_destroy(h)
        conv.conv_destroy(g)
    with pytest.raises(conv.ConvError) as e:
        conv.conv_create_chunked(*shape, 0)
    assert e.value.status == conv.CONV_EINVAL


@pytest.mark.parametrize("dt", [conv.CONV_F32, conv.CONV_BF16], ids=["f32", "bf16"])
def test_tensors_beyond_32bit_offsets_run_in_chunks_on_tiled_kernels(dt):
    """4 GB and more in one tensor, or more linear rows than the kernels' exact divisions
    reach: the planner splits the minibatch so that every pass keeps its tiled kernel."""
    for shape in ((1024 if dt == conv.CONV_BF16 else 512, 64, 64, 224, 224, 3, 3, 1, 1),
                  (8192 if dt == conv.CONV_BF16 else 4096, 64, 256, 56, 56, 1, 1, 1, 0),
                  (300000, 8, 8, 14, 14, 3, 3, 1, 1)):
        info, plans = _plans(shape, dt)
        _check(info, plans)
        assert all(_tiled(p) for p in plans.values()), (shape, plans)
        assert plans[conv.PASS_FWD].startswith("chunks=") and plans[conv.PASS_BWD_DATA].startswith("chunks=")
    # the benchmark's own sizes are never chunked
    for l in inputs.TABLE_I:
        _, plans = _plans((256, l.C, l.K, l.H, l.W, l.R, l.S, l.stride, l.pad), dt)
        assert not any(p.startswith("chunks=") for p in plans.values())


def test_extreme_descriptors_plan_quickly_and_within_bounds():
    """Very tall images, millions of images, thousands of channels under a large filter:
    planning time must not grow with N*P, and the update's partial copies must not dwarf
    the tensors (such plans are left to the direct kernel, which needs no workspace)."""
    import time
    for shape, dt in (((77948, 3, 4, 16060, 9, 7, 7, 3, (2, 5)), conv.CONV_F32),
                      ((2000000, 8, 8, 9, 9, 3, 3, 1, 1), conv.CONV_BF16),
                      ((2, 5585, 5431, 330, 2214, 7, 7, 3, (6, 1)), conv.CONV_F32),
                      ((19, 5746, 6495, 325, 972, 7, 1, 1, (6, 0)), conv.CONV_F32)):
        t0 = time.time()
        info, plans = _plans(shape, dt)
        assert time.time() - t0 < 20.0, shape
        _check(info, plans)
        assert info.workspace_bytes <= max(2 * (info.in_bytes + info.out_bytes), 8e9) + 64 * info.dwt_bytes


@pytest.mark.parametrize("bad", [dict(C=2 ** 31 - 1), dict(K=2 ** 31 - 1), dict(W=2 ** 31 - 1),
                                 dict(H=2 ** 31 - 1), dict(N=2 ** 31 - 1), dict(stride=2 ** 31 - 1),
                                 dict(R=2 ** 20, H=2 ** 21), dict(pad=2 ** 30),
                                 dict(N=2 ** 24, C=2 ** 12, H=2 ** 12, W=2 ** 12)],
                         ids=lambda b: ",".join("%s=%d" % kv for kv in b.items()))
def test_extents_beyond_the_size_limits_are_refused_not_miscomputed(bad):
    """Extents near INT32_MAX once left the planner's int arithmetic (a garbage plan, a division
    by zero, half a minute inside conv_create): they are bounded in 64-bit before any planning."""
    import time
    d = dict(N=2, C=8, K=8, H=8, W=8, R=3, S=3, stride=1, pad=1, dtype=0)
    d.update(bad)
    t0 = time.time()
    with pytest.raises(conv.ConvError) as e:
        conv.conv_create(**d)
    assert e.value.status == conv.CONV_EUNSUPPORTED
    assert time.time() - t0 < 1.0


def test_large_but_legal_extents_plan_within_bounds():
    """Just inside the limits: a plan comes back at once, every figure positive."""
    import time
    for shape in ((1, 2 ** 20, 8, 1, 1, 1, 1, 1, 0), (2 ** 24, 4, 4, 1, 1, 1, 1, 1, 0),
                  (1, 4, 4, 2 ** 18, 2 ** 18, 3, 3, 1, 1), (1, 8, 8, 70000, 9, 5, 3, 60000, (0, 1)),
                  (3, 8, 8, 9, 40000, 3, 3, 1, 1)):
        t0 = time.time()
        info, plans = _plans(shape, conv.CONV_F32)
        assert time.time() - t0 < 5.0, shape
        _check(info, plans)
        assert info.P >= 1 and info.Q >= 1 and info.in_bytes > 0 and info.out_bytes > 0


def test_checked_workspace_entry_points_refuse_a_short_buffer():
    """conv_*_ws return CONV_EWORKSPACE before anything is launched (host only here: the
    pointers are never dereferenced because the size check comes first)."""
    lib = conv.load()
    h = conv.conv_create(4, 64, 64, 14, 14, 3, 3, 1, 1, 0)
    try:
        need = conv.conv_query(h).workspace_bytes
        assert need > 0
        assert lib.conv_bwd_data_ws(h, 16, 16, 16, 16, 0, None) == conv.CONV_EWORKSPACE
        assert lib.conv_upd_ws(h, 16, 16, 16, 16, need // 2, None) == conv.CONV_EWORKSPACE
        assert lib.conv_upd_ws(None, 16, 16, 16, 16, need, None) == conv.CONV_EINVAL
    finally:
        conv.conv_destroy(h)


def test_large_tiles_where_small_ones_are_slower():
    # bf16 in small tiles: 5x5 from where the large tiles fill the chip (N = 96: 1.18 of their time), and one channel
    # tile from 130 MB of tensors on (N = 160: 1.24)
    for N, rest, small in ((16, (48, 64, 35, 35, 5, 5, 1, 2), True), (96, (48, 64, 35, 35, 5, 5, 1, 2), False),
                           (96, (512, 128, 28, 28, 1, 1, 1, 0), True), (160, (512, 128, 28, 28, 1, 1, 1, 0), False)):
        _, p = _plans((N,) + rest, conv.CONV_BF16)
        assert p[conv.PASS_FWD].startswith("igemm dt=1 waves=2x2 frags=1x2" if small and rest[4] == 5 else
                                           "igemm dt=1 waves=2x2 frags=2x2" if small else "igemm dt=1 waves=1x4 frags=2x4")


def test_fp32_small_tiles_in_registers_only_for_few_of_them():
    # 288 -> 64 backward at 35x35: beyond a dozen workgroups to a CU (N = 112: 96 us, 73 staged) not in registers
    for N, name in ((24, "igemm_reg "), (112, "igemm ")):
        assert _plans((N, 288, 64, 35, 35, 1, 1, 1, 0), conv.CONV_F32)[1][conv.PASS_BWD_DATA].startswith(name)


def test_shares_of_the_xcds():
    # one channel group: whole pixel tiles (21 of 8 tiles: 24 to an XCD) for bf16 1x1 where they cost no CU a tile more, else
    # equal shares
    for shape, dt, tiles, grid in (((24, 512, 1024, 28, 28, 1, 1, 2, 0), conv.CONV_BF16, 168, 192),
                                   ((112, 256, 256, 14, 14, 3, 3, 1, 1), conv.CONV_BF16, 176, 176)):
        p = _plans(shape, dt)[1][conv.PASS_FWD]
        assert (_field(p, "tiles"), _field(p, "xcd_kgroups"), _field(p, "grid")) == (tiles, 1, grid)


def test_fp32_1x1_takes_small_tiles_where_large_ones_leave_a_round_part_empty():
    """Either side of the lines: 896 and 448 large tiles (of 512 that run at once) behind 32 steps and 64-row tiles
    in one to two rounds on the small tile, 1 792 and 224 large tiles and four rounds on the large one."""
    def tile(shape, which):
        L = conv.conv_create(*shape[:7], shape[7], (0, 0), conv.CONV_F32)
        try:
            return "frags=1x2" in conv.conv_describe(L, which)
        finally:
            conv.conv_destroy(L)
    assert tile((256, 512, 2048, 7, 7, 1, 1, 1), conv.PASS_FWD)
    assert tile((256, 512, 256, 28, 28, 1, 1, 2), conv.PASS_FWD)
    assert tile((96, 64, 64, 56, 56, 1, 1, 1), conv.PASS_FWD)
    assert not tile((256, 512, 1024, 28, 28, 1, 1, 2), conv.PASS_FWD)
    assert not tile((256, 2048, 512, 7, 7, 1, 1, 1), conv.PASS_FWD)
    assert not tile((256, 192, 64, 35, 35, 1, 1, 1), conv.PASS_BWD_DATA)


def test_large_images_under_long_filters_plan_quickly():
    """The longest run of input positions under a tile is found without a walk over every tile of the result (4e6 pixels,
    in the order of 1e5 tiles for each of nine variants: 6 ms and more; 0.3 without): best of five."""
    import time
    for shape in ((33, 16, 16, 347, 345, 1, 7, 1, (0, 3)), (33, 16, 16, 347, 347, 1, 7, 1, (0, 0)),
                  (100, 16, 16, 667, 59, 3, 3, 1, (1, 1))):
        best = 1.0
        for _ in range(5):
            t0 = time.perf_counter()
            h = conv.conv_create(*shape, conv.CONV_BF16)
            best = min(best, time.perf_counter() - t0)
            conv.conv_destroy(h)
        assert best < 2e-3, (shape, best)


def test_longest_patch_of_the_pixels_in_lds(monkeypatch):
    """LDS of the kernel that keeps a tile's pixels there (eight waves, two buffers of two channel blocks and a chunk each)
    against the longest run of input positions under any tile, by enumeration: images smaller than a tile, rows and
    images that no tile start falls together with, no padding, strides, a last tile that is not whole."""
    monkeypatch.setenv("CONVMI_IGEMM_PATCH", "1,2,8")
    rng = np.random.default_rng(7)
    ran = 0
    for i in range(200):
        R, S, st = [(3, 3, 1), (3, 3, 2), (1, 7, 1), (7, 1, 1)][i % 4]
        N, H, W = int(rng.integers(1, 7)), int(rng.integers(R, 22)), int(rng.integers(S, 40))
        ph, pw = (int(rng.integers(0, x // 2 + 1)) for x in (R, S))
        text = _plans((N, 16, 16, H, W, R, S, st, (ph, pw)), conv.CONV_BF16)[1][conv.PASS_FWD]
        if not text.startswith("igemm_patch "):
            continue
        P, Q = (H + 2 * ph - R) // st + 1, (W + 2 * pw - S) // st + 1
        at = [(m // (P * Q)) * H * W + m % (P * Q) // Q * st * W + m % Q * st for m in range(N * P * Q)]
        run = max(at[min(len(at), m + 64) - 1] - at[m] for m in range(0, len(at), 64))
        pls = -(-(run + (R - 1) * W + S) // 64) * 64
        assert _field(text, "lds") == max(8 * 2 * (2 * pls * 16 + 16), 2 * 8 * 4096), (N, H, W, R, S, st, ph, pw, text)
        ran += 1
    assert ran > 100, ran


def test_bf16_backward_on_transformed_weights_where_the_kernels_on_the_forward_ones_are_slower():
    """The register-operand kernel behind a transform: channel blocks that only the one-block tile takes else, and many
    tiles; of two tiles that memory bounds alike, the larger."""
    for shape in ((8, 256, 48, 35, 35, 1, 1, 1, 0), (98, 344, 216, 19, 21, 1, 1, 1, 0), (12, 360, 360, 46, 47, 7, 1, 1, (3, 0)),
                  (81, 324, 456, 55, 55, 1, 1, 2, 0), (190, 204, 296, 23, 26, 1, 1, 2, 0)):
        p = _plans(shape, conv.CONV_BF16)[1][conv.PASS_BWD_DATA]
        assert p.startswith("igemm_reg ") and "frags=2x2" in p and "forward_weights=1" not in p, p
    p = _plans((8, 1024, 256, 14, 14, 1, 1, 1, 0), conv.CONV_BF16)[1][conv.PASS_BWD_DATA]
    assert "forward_weights=1" in p, p
    # scattering and bound by memory: 31 us where the staged tile of one channel block takes 24
    p = _plans((196, 168, 52, 32, 35, 1, 1, 2, 0), conv.CONV_BF16)[1][conv.PASS_BWD_DATA]
    assert p.startswith("igemm ") and "npl=1" in p, p


def test_bf16_strided_1x1_backward_of_few_tiles_is_not_staged():
    # (8.3 and 8.6 us in the staged tile, 7.3 and 7.4 in registers)
    for shape in ((53, 248, 256, 15, 16, 1, 1, 2, 0), (9, 512, 256, 28, 28, 1, 1, 2, 0)):
        p = _plans(shape, conv.CONV_BF16)[1][conv.PASS_BWD_DATA]
        assert p.startswith("igemm_reg ") and "forward_weights=1" in p, p


def test_fp32_1x1_keeps_large_tiles_where_small_ones_are_slower():
    """Beside the lines of the test above (time of the small tile / the large one): 464 and 462 large tiles 1.05,
    744 tiles 1.06, 940 tiles 1.04, a short strided reduction over 442 tiles 1.05, half-empty tiles in one round 1.04."""
    def small(shape, which):
        return "frags=1x2" in _plans(shape, conv.CONV_F32)[1][which]
    assert not small((33, 128, 512, 28, 28, 1, 1, 1, 0), conv.PASS_FWD)
    assert not small((132, 512, 128, 28, 28, 1, 1, 1, 0), conv.PASS_FWD)
    assert not small((53, 128, 512, 28, 28, 1, 1, 1, 0), conv.PASS_FWD)
    assert not small((67, 128, 512, 28, 28, 1, 1, 1, 0), conv.PASS_FWD)
    assert not small((63, 256, 128, 56, 56, 1, 1, 2, 0), conv.PASS_BWD_DATA)
    assert not small((160, 192, 32, 35, 35, 1, 1, 1, 0), conv.PASS_FWD)
    # within them: 0.90, 0.91, 0.85
    assert small((61, 128, 256, 28, 28, 1, 1, 1, 0), conv.PASS_FWD)
    assert small((94, 320, 640, 20, 20, 1, 1, 1, 0), conv.PASS_FWD)
    assert small((211, 192, 32, 35, 35, 1, 1, 1, 0), conv.PASS_FWD)


def test_window_update_from_where_it_is_faster():
    """Time of the window kernel / the ring kernel beside each; both print as upd_ring."""
    for (N, C, K, H, W, pad), want in (((30, 400, 400, 20, 20, 1), False),      # 0.90, below 1e10 operations
                                       ((35, 400, 400, 20, 20, 1), True),       # 0.85
                                       ((37, 288, 384, 35, 35, 0), True),       # 0.93
                                       ((78, 128, 128, 56, 56, 1), True),       # 0.97
                                       ((87, 128, 256, 56, 56, 1), True),       # 0.89
                                       ((5, 512, 320, 55, 54, 1), False),       # 1.43: 240 half blocks, or 120
                                       ((21, 740, 180, 30, 31, 1), False),      # 1.18: 216, or two splits of 108
                                       ((20, 672, 232, 39, 38, 0), False),      # 1.53: 252, or three splits of 132
                                       ((21, 716, 240, 36, 36, 0), True),       # 0.83: 276, or three splits of 144
                                       ((25, 732, 128, 30, 33, 1), True),       # 0.85: 138, or three splits of 72
                                       ((172, 440, 256, 13, 14, 1), True)):     # 0.67: 168, or three splits of 84
        p = _plans((N, C, K, H, W, 3, 3, 2, pad), conv.CONV_BF16)[1][conv.PASS_UPD]
        assert p.startswith("upd_ring ") and (_field(p, "window") > 0) == want, (N, C, K, p)


def test_group_is_what_the_kernel_sums(monkeypatch):
    """The staged kernel on the forward pass's weights sums in one chain; the plan must not say otherwise."""
    monkeypatch.setenv("CONVMI_IGEMM_REG", "0")
    monkeypatch.setenv("CONVMI_IGEMM_CAND", "2,2,1,2,2,4")
    monkeypatch.setenv("CONVMI_IGEMM_GROUP", "2")
    p = _plans((4, 128, 128, 28, 28, 1, 1, 1, 0), conv.CONV_F32)[1]
    assert p[conv.PASS_FWD].startswith("igemm ") and _field(p[conv.PASS_FWD], "group") == 2
    assert "forward_weights=1" in p[conv.PASS_BWD_DATA] and _field(p[conv.PASS_BWD_DATA], "group") == 0


def test_lds_of_the_register_operand_kernel_counts_its_ring_of_weights(monkeypatch):
    """Four steps of 1 KiB a wave and channel fragment, where that is more than the exchange of the sums."""
    for variant, fwd, bwd in (("2,2,4", 16384, 32768), ("1,1,8", 32768, 32768), ("2,1,8", 65536, 65536)):
        monkeypatch.setenv("CONVMI_IGEMM_REG", variant)
        p = _plans((4, 128, 128, 28, 28, 1, 1, 1, 0), conv.CONV_BF16)[1]
        assert "forward_weights=1" in p[conv.PASS_BWD_DATA]
        assert (_field(p[conv.PASS_FWD], "lds"), _field(p[conv.PASS_BWD_DATA], "lds")) == (fwd, bwd), (variant, p)


def test_every_tile_on_forward_weights_is_reached_by_the_test_that_runs_them(monkeypatch):
    """The instantiations of the staged kernel that read the forward pass's weights, against what the shapes, tiles and
    input policies of test_gpu_forward_weights.py plan."""
    from test_gpu_forward_weights import SHAPES, staged_variant, tiles
    want = set()

    def built(dtype, waves, frags, npl, rs, ppt, nb=2, policies=(0,)):
        want.update((dtype, waves, frags, npl, rs, ppt, nb, nt) for nt in policies)
    F32, BF16 = conv.CONV_F32, conv.CONV_BF16
    for dtype in (F32, BF16):
        for frags in ("1x2", "2x2"):
            for npl, rs, ppt in ((4, "1x1", 0), (8, "1x1", 0), (2, "3x3", 1), (2, "3x3", 2), (2, "3x3", 3), (2, "1x7", 1),
                                 (2, "7x1", 1), (2, "7x1", 2)):
                built(dtype, "2x2", frags, npl, rs, ppt)
    for nb in (2, 3):
        built(BF16, "4x1", "1x7", 4, "1x1", 1, nb, (0, 1))
        built(BF16, "2x2", "1x7", 4, "1x1", 2, nb, (0, 1))
    built(BF16, "4x2", "2x4", 8, "1x1", 1, 2, (0, 1))
    built(BF16, "2x2", "2x4", 4, "1x1", 1)
    built(BF16, "4x1", "1x7", 8, "1x1", 1)
    built(F32, "4x1", "1x7", 4, "1x1", 1, 2, (0, 1))
    built(F32, "2x2", "1x7", 4, "1x1", 2, 2, (0, 1))
    for waves in ("1x4", "2x4"):
        for ppt in (3, 4):
            built(BF16, waves, "2x4", 2, "3x3", ppt)
    built(BF16, "1x4", "2x4", 2, "1x7", 3)
    built(BF16, "1x4", "2x4", 2, "7x1", 3)
    built(F32, "4x1", "1x7", 2, "3x3", 2)
    built(F32, "2x2", "1x7", 2, "3x3", 3)
    for ppt in (5, 6):
        built(F32, "1x4", "1x7", 2, "3x3", ppt)
    assert len(want) == 58
    monkeypatch.setenv("CONVMI_IGEMM_REG", "0")
    got = set()
    for shape in SHAPES:
        for dtype in (F32, BF16):
            for tile in tiles(shape, dtype):
                for nt in ("0", "1"):
                    monkeypatch.setenv("CONVMI_IGEMM_CAND", tile)
                    monkeypatch.setenv("CONVMI_IGEMM_NT", nt)
                    got.add(staged_variant(tile, _plans(shape, dtype)[1][conv.PASS_BWD_DATA]))
    assert got - {None} == want


def test_fp32_backward_transforms_the_weights_where_the_launch_is_long():
    """Time on the forward pass's weights / with the transform beside each."""
    for shape, forward in (((28, 84, 736, 59, 57, 3, 3, 2, 1), False),       # 1.03
                           ((64, 64, 64, 56, 56, 3, 3, 2, 1), True),         # 0.97
                           ((64, 64, 640, 30, 30, 7, 1, 1, (3, 0)), False),  # 1.03
                           ((256, 512, 2048, 7, 7, 1, 1, 1, 0), False),      # 1.04
                           ((256, 512, 1024, 28, 28, 1, 1, 2, 0), True),     # 0.99: two pixel fragments
                           ((8, 1024, 256, 14, 14, 1, 1, 1, 0), True)):
        p = _plans(shape, conv.CONV_F32)[1][conv.PASS_BWD_DATA]
        assert ("forward_weights=1" in p) == forward, (shape, p)


def test_planning_what_runs_on_the_bf16_instructions_costs_less_than_the_rest_of_it(monkeypatch):
    """conv_create in fp32 looks at some 300 more variants: with them it takes 1.5 - 1.6 times what it takes without (2.1 with every
    variant planned in full).  The smallest of 40 times of each layer, both in turn, since other work on the machine only adds."""
    import ctypes
    import time
    lib = conv.load()
    h = ctypes.c_void_p()
    layers = [(N, l) for N in (1, 28, 256) for l in inputs.TABLE_I + inputs.INCEPTION_V3]
    least = {k: [1e9] * len(layers) for k in ("with", "without")}
    for _ in range(40):
        for k in least:
            for name in ("CONVMI_IGEMM_SPLIT", "CONVMI_UPD_SPLIT"):
                monkeypatch.delenv(name, raising=False)
                if k == "without":
                    monkeypatch.setenv(name, "0")
            for i, (N, l) in enumerate(layers):
                d = conv.ConvDesc(N, l.C, l.K, l.H, l.W, l.R, l.S, l.stride, 0, conv.CONV_F32)
                t0 = time.perf_counter()
                assert lib.conv_create_rect(ctypes.byref(d), l.pads[0], l.pads[1], ctypes.byref(h)) == 0
                least[k][i] = min(least[k][i], time.perf_counter() - t0)
                lib.conv_destroy(h)
    assert sum(least["with"]) < 1.8 * sum(least["without"]), {k: sum(v) / len(layers) for k, v in least.items()}


# fp32, pass, layer: whether it runs on the bf16 instructions.  Beside each the time there and on the fp32 instructions, us.
@pytest.mark.parametrize("which,shape,on", [
    (0, (45, 192, 32, 35, 35, 1, 1, 1), False),   # 16.6, 11.9
    (0, (23, 192, 32, 35, 35, 1, 1, 1), False),   # 10.8, 8.5
    (1, (90, 32, 316, 51, 53, 1, 1, 1), False),   # 113, 77
    (0, (166, 164, 32, 48, 51, 1, 1, 1), True),   # 84, 151
    (0, (2, 64, 64, 56, 56, 3, 3, 1), False),     # 9.6, 8.6
    (0, (1, 296, 276, 18, 18, 3, 3, 1), False),   # 13.1, 12.9
    (0, (8, 512, 512, 7, 7, 3, 3, 1), True),
    (0, (28, 128, 128, 28, 28, 3, 3, 1), True)], ids=str)  # 47, 73
def test_fp32_layers_stay_on_the_fp32_instructions_where_those_are_faster(which, shape, on):
    h = conv.conv_create(*shape, (shape[5] - 1) // 2, dtype=conv.CONV_F32)
    try:
        assert (" on_bf16x3=" in conv.conv_describe(h, which)) == on
    finally:
        conv.conv_destroy(h)


# bf16 updates of seven rows: whether both operands are staged for all waves.  Beside each the time with and without, us.
@pytest.mark.parametrize("shape,on", [
    ((139, 140, 48, 46, 48), False),   # 136, 90
    ((87, 624, 52, 58, 56), False),    # 385, 277
    ((218, 308, 264, 28, 31), False),  # 413, 345
    ((32, 84, 264, 47, 48), False),    # 63, 55
    ((84, 708, 140, 25, 27), True),    # 122, 295
    ((80, 200, 460, 33, 34), True),    # 139, 284
    ((18, 632, 40, 59, 60), True)], ids=str)  # 89, 113
def test_updates_of_seven_rows_are_staged_for_all_waves_where_that_is_faster(shape, on):
    h = conv.conv_create(*shape, 7, 1, 1, (3, 0), dtype=conv.CONV_BF16)
    try:
        assert (" instead=upd_shared," in conv.conv_describe(h, conv.PASS_UPD)) == on
    finally:
        conv.conv_destroy(h)


@pytest.mark.parametrize("shape,on", [
    ((166, 332, 52, 60, 63), False),   # 182, 151
    ((163, 728, 40, 44, 47), False),   # 199, 172
    ((248, 64, 204, 33, 33), False),   # 38, 33
    ((99, 636, 592, 12, 12), True),    # 38, 58
    ((224, 96, 88, 49, 48), True)], ids=str)  # 52, 74
def test_strided_updates_of_few_channels_keep_the_ring_kernel(shape, on):
    lines = []
    for pad in (0, 1):
        h = conv.conv_create(*shape, 3, 3, 2, pad, dtype=conv.CONV_BF16)
        try:
            lines.append(" instead=upd_shared," in conv.conv_describe(h, conv.PASS_UPD))
        finally:
            conv.conv_destroy(h)
    assert lines == [on, on] if not on else any(lines), lines
