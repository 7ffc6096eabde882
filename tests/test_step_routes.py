"""Which kernels a step goes out as, by storage, sizes and statistics: both sides of every rule, on a
host double of the HIP runtime (no GPU).  The rules are choices of speed between kernels of equal
results; the figures behind them stand at their constants."""
import pytest

from host_double import double

CODE = """
R = Runtime()
A, L = R.A, R.L
shape, kw, planes, reference, steps = %r
h = R.channel(*shape, **kw)
if planes:
    arr = (C.c_int32 * len(planes))(*planes)
    assert L.lbm_stats(h, A.STATS_ATTACH, arr, len(planes), None, None) == A.LBM_OK
if reference:
    assert L.lbm_set_reference(h, R.plane(9)) == A.LBM_OK
R.launches.clear()
assert L.lbm_step(h, None, steps) == A.LBM_OK
emit([l for l in R.launches if l[0].startswith("collide_")])
"""


def step(tmp_path, shape, planes=(), reference=False, steps=1, **kw):
    return double(CODE % ((shape, kw, list(planes), reference, steps),), tmp_path)


@pytest.mark.parametrize("shape,ranges", [((1536, 128, 384), 5), ((1536, 256, 384), 10), ((1040, 128, 128), 1)])
def test_fp16_bulk_ranges_without_reference_offsets_only(shape, ranges, tmp_path):
    names = [k for k, *_ in step(tmp_path, shape, storage=1)]
    assert names == ["collide_bulk_kernel"] * ranges
    whole = step(tmp_path, shape, storage=1, reference=True)
    assert [k for k, *_ in whole] == ["collide_bulk_kernel"]
    # every block of the lattice once, and at most what evens the eight XCDs' lists out
    blocks = shape[0] * shape[1] // 4 * (shape[2] // 64)
    assert blocks <= whole[0][1][0] <= blocks + 8 * 64 * ranges


def lattice(nz, mb, storage, ny=90):
    """The lattice of ny x nz whose nodes touch closest to mb million bytes of 128-byte lines."""
    el = 4 if storage == 0 else 2
    line = 2 * 19 * (-(-el * nz // 128) * 128) * ny
    return round(mb * 1e6 / line), ny, nz


@pytest.mark.parametrize("nz,mb,lanes", [(16, 60, 16), (16, 300, 16), (16, 305, 64), (9, 500, 64), (1, 290, 16),
                                         (17, 300, 32), (32, 330, 32), (32, 340, 64), (24, 800, 64), (33, 60, 64)])
def test_short_rows_within_the_caches_only(nz, mb, lanes, tmp_path):
    for ref in (False, True):
        (name, grid, threads, targs), = step(tmp_path, lattice(nz, mb, 1), reference=ref, storage=1)
        assert name == "collide_fused_kernel" and threads == 4 * lanes and targs[3] == lanes


@pytest.mark.parametrize("nz,mb,rows", [(16, 300, 1), (16, 305, 0), (32, 300, 1), (24, 300, 1), (17, 275, 1),
                                        (17, 280, 0), (3, 300, 0), (28, 230, 1), (28, 240, 0), (33, 60, 0)])
def test_row_kernel_within_the_infinity_cache_only(nz, mb, rows, tmp_path):
    (name, *_), = step(tmp_path, lattice(nz, mb, 0, ny=60))
    assert name == ("collide_rows_kernel" if rows else "collide_general_kernel")


@pytest.mark.parametrize("storage,nz,mb,nt", [
    # FP32: 288 MiB (302 MB) with whole lines, 268 MiB (281 MB) with a part of one
    (0, 64, 300, 0), (0, 64, 305, 1), (0, 96, 300, 0), (0, 112, 278, 0), (0, 112, 284, 1), (0, 100, 284, 1),
    (0, 33, 284, 1), (0, 33, 270, 0),
    # FP16 with 64-lane rows: 236 MiB (247 MB) where at most half of the last line is used
    (1, 64, 300, 0), (1, 64, 305, 1), (1, 100, 300, 0), (1, 48, 300, 0), (1, 96, 250, 1), (1, 80, 250, 1),
    (1, 70, 245, 0), (1, 200, 250, 1), (1, 200, 244, 0), (1, 97, 300, 0)])
def test_cached_stores_within_the_infinity_cache_only(storage, nz, mb, nt, tmp_path):
    """The first of two steps (a call's last one stores non-temporally on large lattices)."""
    first, last = step(tmp_path, lattice(nz, mb, storage, ny=80), steps=2, storage=storage)
    assert first[0] == ("collide_fused_kernel" if storage else "collide_general_kernel")
    template = 2 if storage else 1
    assert first[3][template] == nt and last[3][template] == 1


@pytest.mark.parametrize("shape,kw,rows", [
    ((40, 24, 6), dict(wall_model=1), 0), ((24, 60, 8), dict(wall_model=1), 1), ((13, 60, 32), dict(wall_model=1), 0),
    ((40, 24, 6), dict(), 1), ((13, 60, 2), dict(), 0), ((40, 60, 1), dict(), 0), ((60, 60, 1), dict(), 1),
    ((40, 24, 6), dict(wall_model=1, xbc=1), 1), ((13, 60, 2), dict(xbc=1), 1), ((5, 9, 16), dict(xbc=1), 1)])
def test_small_closed_channels_keep_the_general_kernel(shape, kw, rows, tmp_path):
    assert [k for k, *_ in step(tmp_path, shape, **kw)] == ["collide_rows_kernel" if rows else "collide_general_kernel"]


@pytest.mark.parametrize("shape,sampled", [
    ((41, 60, 2), "general"), ((240, 60, 2), "general"), ((308, 60, 2), "rows"), ((41, 20, 1), "general"),
    ((41, 20, 4), "general"), ((120, 60, 4), "rows"), ((41, 60, 24), "general"), ((103, 60, 24), "rows"),
    ((41, 50, 12), "general"), ((168, 16, 5), "general"), ((70, 50, 8), "rows"), ((70, 50, 6), "general"),
    ((89, 64, 3), "general"), ((120, 50, 6), "rows"), ((16, 20, 16), "rows"), ((16, 20, 28), "rows"),
    ((16, 20, 32), "rows"), ((200, 20, 16), "rows")])
def test_sampled_steps_leave_the_row_kernel_where_its_sums_take_longer(shape, sampled, tmp_path):
    assert [k for k, *_ in step(tmp_path, shape, xbc=1)] == ["collide_rows_kernel"]
    assert [k for k, *_ in step(tmp_path, shape, planes=[1, 3], xbc=1)] == ["collide_%s_kernel" % sampled]


@pytest.mark.parametrize("nz,mb,reference,late", [(64, 40, True, 0), (64, 200, True, 0), (64, 305, True, 1),
                                                  (64, 305, False, 0), (80, 260, True, 1), (20, 330, True, 0),
                                                  (20, 340, True, 1)])
def test_storage_offsets_ahead_of_the_stores_within_the_caches(nz, mb, reference, late, tmp_path):
    for _, _, _, targs in step(tmp_path, lattice(nz, mb, 1), reference=reference, steps=2, storage=1):
        assert targs[4] == late


ADJOINT = """
R = Runtime()
A, L = R.A, R.L
shape, storage, reference = %r
h = R.channel(*shape, storage=storage)
if reference:
    assert L.lbm_set_reference(h, R.plane(9)) == A.LBM_OK
R.launches.clear()
p = R.plane
assert L.lbm_adjoint_step(h, None, p(10), None, 1.0, p(11), None, p(12), *[None] * 6) == A.LBM_OK
emit([l for l in R.launches if l[0] == "adjoint_kernel"])
"""


@pytest.mark.parametrize("storage,nz,mb,nt", [
    (0, 64, 120, 0), (0, 64, 128, 1), (0, 64, 330, 1), (0, 64, 340, 0), (0, 128, 128, 1), (0, 160, 200, 0),
    (0, 101, 194, 0), (0, 101, 205, 1), (0, 40, 205, 1), (0, 70, 130, 0),
    (1, 64, 230, 0), (1, 64, 240, 1), (1, 101, 230, 0), (1, 101, 240, 1), (1, 64, 340, 0)])
def test_adjoint_pulls_the_state_non_temporally_where_sweeps_gain(storage, nz, mb, nt, tmp_path):
    shape = lattice(nz, mb, 0)  # lambda is FP32
    for ref in (False, True)[:1 + storage]:
        (_, _, _, targs), = double(ADJOINT % ((shape, storage, ref),), tmp_path)
        assert targs == [storage, int(ref), nt]


DISPATCHES = """
R = Runtime()
A, L = R.A, R.L
shape, kw, reference = %r
h = R.channel(*shape, **kw)
if reference:
    assert L.lbm_set_reference(h, R.plane(9)) == A.LBM_OK
R.launches.clear()
d, p = C.c_int32(-1), C.c_int32(-1)
assert L.lbm_timed_dispatches(None, C.byref(d), C.byref(p)) == A.LBM_ERR_ARG and d.value == p.value == -1
assert L.lbm_timed_dispatches(h, C.byref(d), None) == L.lbm_timed_dispatches(h, None, C.byref(p)) == A.LBM_OK
assert L.lbm_step(h, None, 1) == A.LBM_OK
emit([[d.value, p.value], len([k for k, *_ in R.launches if k in ("collide_bulk_kernel", "collide_fused_kernel")]),
      len([k for k, *_ in R.launches if k in ("collide_general_kernel", "collide_rows_kernel")])])
"""


@pytest.mark.parametrize("shape,storage,reference,dispatches", [
    ((1536, 128, 384), 0, False, (10, 154)), ((64, 32, 32), 0, False, (1, 64)),
    ((1536, 128, 384), 1, False, (5, 308)), ((1536, 256, 384), 1, False, (10, 154)),
    ((1536, 128, 384), 1, True, (1, 1536)), ((768, 64, 192), 1, False, (1, 768)), ((64, 32, 32), 1, True, (1, 64))])
def test_reported_dispatches_are_those_of_a_step(shape, storage, reference, dispatches, tmp_path):
    got, bulk, other = double(DISPATCHES % ((shape, dict(storage=storage), reference),), tmp_path)
    assert tuple(got) == dispatches and (bulk if storage else other) == dispatches[0]


ORDER = """
R = Runtime()
A, L = R.A, R.L
shape, planes = %r
h = R.channel(*shape)
arr = (C.c_int32 * len(planes))(*planes)
assert L.lbm_stats(h, A.STATS_ATTACH, arr, len(planes), None, None) == A.LBM_OK
lists = []
R.on_launch = lambda kernel, args: lists.append(C.cast(args[1], C.POINTER(C.c_void_p))[0])
assert L.lbm_step(h, None, 1) == A.LBM_OK
n = R.launches[0][1][0]
per_plane = -(-shape[1] // 4) * -(-shape[2] // 64)
xs = [e // per_plane for e in (C.c_int32 * n).from_address(lists[0]) if e >= 0]
emit([R.launches[0][0], xs])
"""


@pytest.mark.parametrize("shape,first", [((41, 64, 64), 1), ((20, 30, 128), 1), ((41, 22, 64), 0), ((30, 22, 100), 0),
                                         ((55, 22, 100), 1), ((100, 22, 64), 0), ((220, 40, 64), 0)])
def test_sampled_planes_first_where_they_would_be_the_tail(shape, first, tmp_path):
    planes = [7, 12]
    kernel, xs = double(ORDER % ((shape, planes),), tmp_path)
    blocks = -(-shape[1] // 4) * -(-shape[2] // 64)
    assert kernel == "collide_general_kernel"
    assert sorted(xs) == sorted(list(range(shape[0])) * blocks)
    assert (set(xs[:8]) <= set(planes)) == bool(first)  # one of each XCD
