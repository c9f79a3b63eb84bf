"""The matrix-core kernel divides the rows of a batch evenly over its waves, across the borders of contexts: every way
a share can begin, end and be merged, against the fp32 oracle (max-abs 2e-3 / relative L2 1e-3, as everywhere); and few
contexts into chunks, by one wave or four."""
import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3
from tests.harness import assert_close

torch = pytest.importorskip("torch")
FAMS = [
    ("d64 group 3", 24, 8, 64, s3.S3_BF16, s3.S3_BF16, 1),
    ("d128 group 4", 32, 8, 128, s3.S3_BF16, s3.S3_BF16, 2),
    ("d128 group 24", 24, 1, 128, s3.S3_F16, s3.S3_F16, 2),
    ("d256 group 16", 16, 1, 256, s3.S3_F16, s3.S3_F16, 2),
    ("d64 e4m3 group 8", 8, 1, 64, s3.S3_E4M3, s3.S3_F16, 4),
    ("d128 e4m3 group 2", 16, 8, 128, s3.S3_E4M3, s3.S3_BF16, 4),
    ("d256 e4m3 group 2", 6, 3, 256, s3.S3_E4M3, s3.S3_F16, 4),
]


def batches():
    rng = np.random.default_rng(5)
    return [
        ("one row", [1]),
        ("one long context cut by every share", [2047]),
        ("tile edges, empty first and last", [0, 15, 16, 17, 0, 31, 32, 33, 1, 63, 64, 65, 0]),
        ("a long one between short ones", [3, 1900, 1, 1, 40]),
        ("hundreds", [int(x) for x in rng.integers(0, 400, size=300)]),
        ("more than fit a team's LDS", [int(x) for x in rng.integers(1, 12, size=1100)]),
    ]


@pytest.mark.gpu
@pytest.mark.parametrize("fam", FAMS, ids=[f[0] for f in FAMS])
def test_even_division_over_batches(fam):
    from tests.test_gpu_numeric_edges import EdgeRig

    name, H, Hkv, D, kvt, act, kind = fam
    for what, lens in batches():
        rng = np.random.default_rng(len(lens) + D)
        rig = EdgeRig(fam, lens, M=2048)
        rig.put([rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens],
                [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens])
        if kind == 1:  # fewer than four query heads per cached head: the matrix-core kernel on request
            assert s3.s3_kv_set_param(rig.a, "variant", s3.s3_kv_get_param(rig.a, "n_variants")[1] - 1) == 0
        n = len(lens)
        q = rng.standard_normal((n, H, D), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{name} / {what}")
        # the division does not depend on the grid, nor do the bits (no more contexts and columns than compute units: eight waves a
        # workgroup, on a grid of their own)
        for grid in (1, 7) if n * Hkv * -(-(H // Hkv) // 16) > 256 else ():
            assert s3.s3_kv_set_param(rig.a, "grid_blocks", grid) == 0
            assert np.array_equal(rig.attend(q)[1], att), (name, what, grid)
        assert s3.s3_kv_set_param(rig.a, "grid_blocks", 0) == 0
        longer = [L + 1 for L in lens]
        qb, step = rig.step(q, rng.standard_normal((n, Hkv, D), dtype=np.float32), rng.standard_normal((n, Hkv, D), dtype=np.float32))
        assert_close(step, rig.want(qb, longer), f"{name} / {what} / step")
        assert np.array_equal(rig.attend(q, lens=longer)[1], step), (name, what)
        rig.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [300, 600, 1007, 1100, 1999, 2008, 2009])
def test_short_contexts_around_the_fixed_buffers_size(n):
    """At most 256 rows a context, 32 query on 8 cached heads of 128: 2008 contexts fit the fixed buffer of
    s3_decode_step_static whole, from 1005 on with fewer slots left than contexts.  Attention, the step and the static
    step (refused beyond) agree bit for bit."""
    from tests.test_gpu_numeric_edges import TDT, EdgeRig, device_bits, wl

    H, Hkv, D, kvt = 32, 8, 128, s3.S3_BF16
    rng = np.random.default_rng(n)
    lens = [int(x) for x in rng.integers(0, 30, size=n)]
    for b, L in ((0, 250), (n // 2, 16), (n - 2, 255), (n - 1, 0)):
        lens[b] = L
    rig = EdgeRig(("short", H, Hkv, D, kvt, kvt, 2), lens, M=256)
    rows = rng.standard_normal((256, Hkv, D), dtype=np.float32)
    rig.put([np.roll(rows, b, axis=0)[:L] for b, L in enumerate(lens)], [np.roll(rows, 2 * b, axis=0)[:L] for b, L in enumerate(lens)])
    q = rng.standard_normal((n, H, D), dtype=np.float32)
    qb, att = rig.attend(q)
    assert_close(att, rig.want(qb), "attention")
    k_new, v_new = (rng.standard_normal((n, Hkv, D), dtype=np.float32) for _ in range(2))
    qb, step = rig.step(q, k_new, v_new)
    longer = [L + 1 for L in lens]
    assert_close(step, rig.want(qb, longer), "step")
    assert np.array_equal(rig.attend(q, lens=longer)[1], step)
    out = torch.full((n, H, D), float("nan"), dtype=torch.float32, device="cuda:0")
    args = [device_bits(wl.to_bits(x, kvt), TDT[kvt], "cuda:0") for x in (q, k_new, v_new)]
    st = s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, torch.tensor(lens, dtype=torch.int32, device="cuda:0"), *args, out, s3.S3_F32, 0.0,
                                  None, rig.stream)
    torch.cuda.synchronize()
    assert st == (s3.S3_ERR_SCRATCH if n > 2008 else 0)
    assert n > 2008 or np.array_equal(out.cpu().numpy(), step)
    rig.close()


# (tiles of 16 rows, of 32 where a cached row of one head has at most 128 bytes; columns decide how many chunks run at once)
FEW = [
    ("a wave each, a row to a tile", [1, 15, 16, 17, 31, 32, 33]),
    ("quarters: one to five tiles", [64, 65, 79, 80, 128, 129, 160, 161, 0]),
    ("the longest whole one", [224, 223, 100, 448, 7]),
    ("one beyond it", [225, 449, 100, 7]),
    ("two long among short", [5, 2047, 40, 1700, 0, 1]),
    ("64", [130 + 9 * (b % 7) for b in range(64)]),
    ("65", [130 + 9 * (b % 7) for b in range(64)] + [1500]),
    ("256", [(37 * b) % 160 for b in range(255)] + [900]),
    ("257", [(37 * b) % 160 for b in range(256)] + [900]),
    ("as many as run at once", [300] * 63 + [17]),
    ("contexts that divide badly", [257] * 40 + [300] * 8),
]


@pytest.mark.gpu
@pytest.mark.parametrize("fam", FAMS, ids=[f[0] for f in FAMS])
def test_few_contexts_by_waves_and_teams(fam):
    """Chunks of single contexts, each by one wave or by the four waves of a workgroup: tile and quarter edges, the
    borders of the rule (contexts taken whole, one view entry or four per lane, the largest batch it takes), few and
    many chunks, in both orderings of the merge, launch after launch; on grids that make a workgroup take many, where the launch
    has a grid of the caller's (more contexts and columns than compute units; fewer go to workgroups of eight waves, one chunk each), and for
    chunks of the caller's size in every batch."""
    from tests.test_gpu_numeric_edges import EdgeRig

    name, H, Hkv, D, kvt, act, kind = fam
    for what, lens in FEW:
        rng = np.random.default_rng(len(lens) + D)
        rig = EdgeRig(fam, lens, M=2048)
        rig.put([rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens],
                [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens])
        if kind == 1:
            assert s3.s3_kv_set_param(rig.a, "variant", s3.s3_kv_get_param(rig.a, "n_variants")[1] - 1) == 0
        q = rng.standard_normal((len(lens), H, D), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{name} / {what}")
        columns = Hkv * -(-(H // Hkv) // 16)
        for grid, sync in ((1, 0), (5, 1), (0, 1), (0, 0)) if len(lens) * columns > 256 else ((0, 1), (0, 0)):
            assert s3.s3_kv_set_param(rig.a, "grid_blocks", grid) == 0 and s3.s3_kv_set_param(rig.a, "merge_sync", sync) == 0
            assert np.array_equal(rig.attend(q)[1], att), (name, what, grid, sync)
        longer = [L + 1 for L in lens]
        qb, step = rig.step(q, rng.standard_normal((len(lens), Hkv, D), dtype=np.float32), rng.standard_normal((len(lens), Hkv, D), dtype=np.float32))
        assert_close(step, rig.want(qb, longer), f"{name} / {what} / step")
        assert np.array_equal(rig.attend(q, lens=longer)[1], step), (name, what)
        for chunk in (32, 96):
            assert s3.s3_kv_set_param(rig.a, "chunk", chunk) == 0
            got = rig.attend(q, lens=longer)[1]
            assert_close(got, rig.want(qb, longer), f"{name} / {what} / chunk {chunk}")
            for grid, sync in ((1, 0), (5, 1), (0, 0)):
                assert s3.s3_kv_set_param(rig.a, "grid_blocks", grid) == 0 and s3.s3_kv_set_param(rig.a, "merge_sync", sync) == 0
                assert np.array_equal(rig.attend(q, lens=longer)[1], got), (name, what, chunk, grid, sync)
        rig.close()


@pytest.mark.gpu
@pytest.mark.parametrize("sync,launches", [(0, 150), (1, 20)])
def test_soak_of_the_matrix_core_merge(sync, launches):
    """Many pieces that meet through counters and write-through partials on every compute unit, in shares across contexts
    and in chunks: the same bits launch after launch, those of the oracle's tolerance."""
    from tests.test_gpu_numeric_edges import EdgeRig

    for H, Hkv, D, kvt, lens in ((32, 8, 128, s3.S3_BF16, [int(x) for x in np.random.default_rng(8).integers(200, 1000, size=300)]),
                                 (32, 8, 128, s3.S3_BF16, [2040, 1500, 700]), (16, 1, 256, s3.S3_F16, [1024 - 3 * b for b in range(60)])):
        rng = np.random.default_rng(len(lens))
        rig = EdgeRig(("soak", H, Hkv, D, kvt, kvt, 2), lens, M=2048)
        rows = rng.standard_normal((2048 + 300, Hkv, D), dtype=np.float32)
        rig.put([rows[b:b + L] for b, L in enumerate(lens)], [rows[300 - b:300 - b + L] for b, L in enumerate(lens)])
        q = rng.standard_normal((len(lens), H, D), dtype=np.float32)
        assert s3.s3_kv_set_param(rig.a, "merge_sync", sync) == 0
        qb, first = rig.attend(q)
        assert_close(first, rig.want(qb), f"{len(lens)} contexts")
        for i in range(launches):
            assert np.array_equal(rig.attend(q)[1], first), (len(lens), i)
        rig.close()


@pytest.mark.gpu
@pytest.mark.parametrize("fam", FAMS, ids=[f[0] for f in FAMS])
def test_eight_waves_a_workgroup_and_the_borders_of_their_rule(fam):
    """Workgroups of eight waves take the launches of no more (context, column) pairs than compute units: the last batch of
    the rule and the first beyond it, the longest whole context (22 tiles) and one row more, fewer tiles than waves, one
    tile more than a wave each, a context cut as finely as it gets, and a long one where no unit is left to cut it for."""
    from tests.test_gpu_numeric_edges import EdgeRig

    name, H, Hkv, D, kvt, act, kind = fam
    tile = 32 if D * (1 if kind == 4 else 2) <= 128 else 16
    columns = Hkv * -(-(H // Hkv) // 16)
    full = 256 // columns
    for what, lens in (("a wave each, and one more", [8 * tile, 8 * tile + 1, 7 * tile - 1, 1, 0]), ("whole", [22 * tile, 5]),
                       ("cut", [22 * tile + 1, 9]), ("finest", [2047]), ("a unit each", [(37 * b) % 150 for b in range(full - 1)] + [1300]),
                       ("one more", [(37 * b) % 150 for b in range(full)] + [1300])):
        rng = np.random.default_rng(len(lens) + D)
        rig = EdgeRig(fam, lens, M=2048)
        rig.put([rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens],
                [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens])
        if kind == 1:
            assert s3.s3_kv_set_param(rig.a, "variant", s3.s3_kv_get_param(rig.a, "n_variants")[1] - 1) == 0
        q = rng.standard_normal((len(lens), H, D), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{name} / {what}")
        # the bits depend on neither (eight waves: a grid of their own, whatever the caller's)
        for grid, sync in ((3, 0), (0, 1), (0, 0)) if what == "one more" else ((0, 1), (0, 0)):
            assert s3.s3_kv_set_param(rig.a, "grid_blocks", grid) == 0 and s3.s3_kv_set_param(rig.a, "merge_sync", sync) == 0
            assert np.array_equal(rig.attend(q)[1], att), (name, what, grid, sync)
        longer = [L + 1 for L in lens]
        qb, step = rig.step(q, rng.standard_normal((len(lens), Hkv, D), dtype=np.float32), rng.standard_normal((len(lens), Hkv, D), dtype=np.float32))
        assert_close(step, rig.want(qb, longer), f"{name} / {what} / step")
        assert np.array_equal(rig.attend(q, lens=longer)[1], step), (name, what)
        rig.close()


@pytest.mark.gpu
@pytest.mark.parametrize("H", [7, 8, 9, 16, 20])
@pytest.mark.parametrize("kvt,kind", [(s3.S3_F16, 2), (s3.S3_E4M3, 4)], ids=["f16", "e4m3"])
def test_eight_waves_combine_one_or_two_quads_a_thread(H, kvt, kind):
    """Eight waves' parts of a chunk, rows of 256: one quad of elements a thread up to eight query heads, two of one head
    beyond (20: a column of sixteen and one of four); contexts of one chunk, that are stored, and of several, that merge."""
    from tests.test_gpu_numeric_edges import EdgeRig

    for lens in ([17, 130, 1, 0, 350], [2000, 40]):
        rng = np.random.default_rng(len(lens) + H)
        rig = EdgeRig(("quads", H, 1, 256, kvt, s3.S3_F16, kind), lens, M=2048)
        rig.put([rng.standard_normal((L, 1, 256), dtype=np.float32) for L in lens],
                [rng.standard_normal((L, 1, 256), dtype=np.float32) for L in lens])
        q = rng.standard_normal((len(lens), H, 256), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{H} heads, {lens}")
        longer = [L + 1 for L in lens]
        qb, step = rig.step(q, *(rng.standard_normal((len(lens), 1, 256), dtype=np.float32) for _ in range(2)))
        assert_close(step, rig.want(qb, longer), f"{H} heads, {lens} / step")
        assert np.array_equal(rig.attend(q, lens=longer)[1], step)
        rig.close()


@pytest.mark.gpu
@pytest.mark.parametrize("H,Hkv,D,kvt,act,kind", [(1028, 257, 256, s3.S3_F16, s3.S3_F16, 2), (1280, 320, 256, s3.S3_BF16, s3.S3_BF16, 2), (960, 320, 256, s3.S3_F16, s3.S3_F16, 1),
                                                  (1200, 300, 256, s3.S3_E4M3, s3.S3_BF16, 4), (2400, 600, 128, s3.S3_BF16, s3.S3_BF16, 2)])
def test_more_columns_than_workgroups_run_at_once(H, Hkv, D, kvt, act, kind):
    """A context that a team of four waves takes in each of more columns than there are workgroups: every head's output and every
    head's new row."""
    from tests.test_gpu_numeric_edges import EdgeRig

    for lens in ([600], [600, 7, 0, 90]):
        n = len(lens)
        rng = np.random.default_rng(Hkv + n)
        rows = rng.standard_normal((640, Hkv, D), dtype=np.float32)
        rig = EdgeRig(("columns", H, Hkv, D, kvt, act, kind), lens, M=640)
        rig.put([rows[b:b + L] for b, L in enumerate(lens)], [rows[n - b:n - b + L] for b, L in enumerate(lens)])
        q = rng.standard_normal((n, H, D), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{H}/{Hkv} x {D}, {lens}")
        longer = [L + 1 for L in lens]
        qb, step = rig.step(q, *(rng.standard_normal((n, Hkv, D), dtype=np.float32) for _ in range(2)))
        assert_close(step, rig.want(qb, longer), f"{H}/{Hkv} x {D}, {lens} / step")
        assert np.array_equal(rig.attend(q, lens=longer)[1], step)
        rig.close()
