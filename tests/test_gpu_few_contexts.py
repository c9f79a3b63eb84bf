"""Batches of few contexts are cut into chunks by a rule on their total and longest rows that runs on the device, one rule in
the kernel of one item a workgroup, which serves up to 64 contexts, and another in the streaming kernels: both sides of their
bounds (the smallest chunk, the longest, the number of contexts at which they end) against the fp32 oracle, and the decode step
against append + attention, bit for bit."""
import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3
from paper_2306_06000_amd import workloads as wl
from tests.harness import assert_close, device_bits
from tests.test_gpu_numeric_edges import TDT, EdgeRig

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FAMS = [
    ("16 x 256", 16, 16, 256, s3.S3_F16, s3.S3_F16, 0),
    ("12 x 128", 12, 12, 128, s3.S3_BF16, s3.S3_BF16, 0),
    ("5 x 96", 5, 5, 96, s3.S3_BF16, s3.S3_BF16, 0),
    ("3 x 64", 3, 3, 64, s3.S3_F16, s3.S3_F16, 0),
    ("16 x 256 e4m3", 16, 16, 256, s3.S3_E4M3, s3.S3_F16, 3),
    ("3 x 128 e4m3", 3, 3, 128, s3.S3_E4M3, s3.S3_BF16, 3),
]


def streaming(rig, kind):
    """The rig's arena on its streaming kernel: a `variant` of the caller's keeps batches off the kernel of one item a workgroup,
    whose grid is its own, and leaves the division of few contexts as it is."""
    variant = s3.s3_kv_get_param(rig.a, "default_variant")[1] if kind == 0 else 2
    assert s3.s3_kv_set_param(rig.a, "variant", variant) == 0


@pytest.mark.parametrize("fam", FAMS, ids=[f[0] for f in FAMS])
def test_few_contexts_are_cut_by_their_rows(fam):
    """By the default kernel (one item a workgroup up to 64 contexts, streaming beyond), and by the streaming kernel for every
    batch, on its own grid and on one of seven workgroups."""
    name, H, Hkv, D, kvt, act, kind = fam
    rng = np.random.default_rng(D + H)
    per_load = 1024 // D if kind == 3 else 4 if D == 96 else 512 // D
    last = 192 // -(-H // per_load)  # the largest batch the rule takes
    for what, lens in (("one row", [1]), ("one piece", [31]), ("two pieces", [33]), ("one long", [2047]),
                       ("mixed, empty ones", [0, 700, 1, 16, 17, 1500, 0]), ("the rule's last batch", [40] * (last - 1) + [1030]),
                       ("the first beyond it", [40] * last + [1030])):
        n = len(lens)
        rig = EdgeRig(fam, lens, M=2048)
        rig.put([rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens],
                [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens])
        q = rng.standard_normal((n, H, D), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{name} / {what}")
        assert np.array_equal(rig.attend(q)[1], att)
        longer = [L + 1 for L in lens]
        k_new, v_new = (rng.standard_normal((n, Hkv, D), dtype=np.float32) for _ in range(2))
        qb, step = rig.step(q, k_new, v_new)
        assert_close(step, rig.want(qb, longer), f"{name} / {what} / step")
        if kind == 0:  # (8-bit rows: the step takes the new row in its last wave, in another order of sums)
            assert np.array_equal(rig.attend(q, lens=longer)[1], step), (name, what)
        streaming(rig, kind)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{name} / {what} / streaming")
        qb, step = rig.step(q, k_new, v_new)
        assert_close(step, rig.want(qb, longer), f"{name} / {what} / streaming step")
        assert s3.s3_kv_set_param(rig.a, "grid_blocks", 7) == 0
        assert np.array_equal(rig.attend(q)[1], att), (name, what)
        assert np.array_equal(rig.step(q, k_new, v_new)[1], step), (name, what)
        if kind == 0:
            assert np.array_equal(rig.attend(q, lens=longer)[1], step), (name, what)
        rig.close()


@pytest.mark.parametrize("fam,batches", [(FAMS[4], (52, 89, 90)), (FAMS[5], (193, 358, 359))], ids=["16 x 256 e4m3", "3 x 128 e4m3"])
def test_eight_bit_rows_fill_the_workgroups_that_run_at_once(fam, batches):
    """Beyond the batches above, 8-bit rows are cut until their chunks fill two workgroups a compute unit, by a count on the
    device: the first batch of that rule, the last and the first beyond it, with lengths that divide well and badly."""
    name, H, Hkv, D, kvt, act, kind = fam
    for n in batches:
        for what, lens in (("even", [240] * n), ("badly", [129 + 3 * (b % 5) for b in range(n)]), ("short", [b % 40 for b in range(n)]),
                           ("a long one", [1500] + [20 + b % 90 for b in range(n - 1)])):
            rng = np.random.default_rng(n + D)
            rig = EdgeRig(fam, lens, M=2048)
            rows = rng.standard_normal((2048, Hkv, D), dtype=np.float32)
            rig.put([np.roll(rows, b, axis=0)[:L] for b, L in enumerate(lens)], [np.roll(rows, 2 * b, axis=0)[:L] for b, L in enumerate(lens)])
            q = rng.standard_normal((n, H, D), dtype=np.float32)
            qb, att = rig.attend(q)
            assert_close(att, rig.want(qb), f"{name} / {n} / {what}")
            for grid in (7, 0):
                assert s3.s3_kv_set_param(rig.a, "grid_blocks", grid) == 0
                assert np.array_equal(rig.attend(q)[1], att), (n, what, grid)
            qb, step = rig.step(q, rng.standard_normal((n, Hkv, D), dtype=np.float32), rng.standard_normal((n, Hkv, D), dtype=np.float32))
            assert_close(step, rig.want(qb, [L + 1 for L in lens]), f"{name} / {n} / {what} / step")
            rig.close()


def test_eight_bit_rows_in_the_longest_chunks():
    """The chunks of the rule above grow to the 1024 rows that a chunk may have: contexts on either side of one and of two
    such chunks, and more chunks than run at once, through every entry point."""
    fam = ("2 x 64 e4m3", 2, 2, 64, s3.S3_E4M3, s3.S3_BF16, 3)
    name, H, Hkv, D, kvt, act, kind = fam
    n = 358
    rng = np.random.default_rng(5)
    rows = rng.standard_normal((4096 + n, Hkv, D), dtype=np.float32)
    for what, lens in (("one chunk each", [1022 + b % 3 for b in range(n)]), ("two", [2047 + b % 3 for b in range(n)]),
                       ("a few long ones", [4000, 2049, 3000] + [1030] * (n - 3))):
        rig = EdgeRig(fam, lens, M=4096)
        rig.put([rows[b:b + L] for b, L in enumerate(lens)], [rows[n - b:n - b + L] for b, L in enumerate(lens)])
        q = rng.standard_normal((n, H, D), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), what)
        k_new, v_new = (rng.standard_normal((n, Hkv, D), dtype=np.float32) for _ in range(2))
        qb, step = rig.step(q, k_new, v_new)
        assert_close(step, rig.want(qb, [L + 1 for L in lens]), what + " / step")
        assert np.array_equal(static_step(rig, q, k_new, v_new), step), what
        rig.close()


@pytest.mark.parametrize("fam,batches", [(FAMS[0], (17, 18, 24, 25, 32, 33, 42, 43, 56, 57)), (FAMS[1], (47, 48, 64, 65, 85, 86, 114, 128)), (FAMS[2], (72, 96, 97, 128)),
                                         (("16 x 64", 16, 16, 64, s3.S3_F16, s3.S3_F16, 0), (72, 97))], ids=["16 x 256", "12 x 128", "5 x 96", "16 x 64"])
def test_sixteen_bit_rows_fill_the_workgroups_that_run_at_once(fam, batches):
    """16-bit rows, 9/16 of an item to one and 4/3 to 7/4 items a compute unit: the first and the last batch of the host's
    part of the rule (up to 64 contexts and 3/4 of an item it is asked no more: these batches are attn_few_kernel's, and are run on the
    streaming kernel too, whose division of them has no such rule), and those beside them, with lengths on either side of the device's part: few contexts whose chunks are
    more than the units, by a little and by an eighth; a long tail, and lengths without one; contexts whole that would be cut
    at 1024 rows; one longer than any chunk; empty ones between.  Attention against the
    oracle; the step against both it and attention over the appended rows, through both of its entry points, bit for bit."""
    name, H, Hkv, D, kvt, act, kind = fam
    top = 4096
    rng = np.random.default_rng(D)
    rows = rng.standard_normal((top + 130, Hkv, D), dtype=np.float32)
    for n in batches:
        for what, lens in (("level", [700 + 9 * (b % 7) for b in range(n)]), ("above a thousand", [1010 + 9 * (b % 3) for b in range(n)]),
                           ("below", [390] * n), ("a tail", [40 + 7 * (b % 30) for b in range(n - 2)] + [900, 1100]),
                           ("a long tail", [60 + 5 * (b % 50) for b in range(n - 1)] + [3500]),
                           ("up to 1500", [64 + (b * 131) % 1430 for b in range(n)]),
                           ("with empty ones", [0 if b % 3 else 1300 for b in range(n)])):
            if n not in batches[::2] and what not in ("above a thousand", "a tail", "up to 1500"):
                continue
            rig = EdgeRig(fam, lens, M=top)
            rig.put([rows[b:b + L] for b, L in enumerate(lens)], [rows[n - b:n - b + L] for b, L in enumerate(lens)])
            q = rng.standard_normal((n, H, D), dtype=np.float32)
            qb, att = rig.attend(q)
            assert_close(att, rig.want(qb), f"{name} / {n} / {what}")
            if n <= 64 and n * -(-H // (4 if D == 96 else 512 // D)) <= 192:
                streaming(rig, kind)
                qb, other = rig.attend(q)
                assert_close(other, rig.want(qb), f"{name} / {n} / {what} / streaming")
            else:
                other = att
            assert s3.s3_kv_set_param(rig.a, "grid_blocks", 7) == 0
            assert np.array_equal(rig.attend(q)[1], other), (n, what)
            assert s3.s3_kv_set_param(rig.a, "grid_blocks", 0) == 0 and s3.s3_kv_set_param(rig.a, "variant", -1) == 0
            k_new, v_new = (rng.standard_normal((n, Hkv, D), dtype=np.float32) for _ in range(2))
            qb, step = rig.step(q, k_new, v_new)
            longer = [L + 1 for L in lens]
            assert_close(step, rig.want(qb, longer), f"{name} / {n} / {what} / step")
            assert np.array_equal(rig.attend(q, lens=longer)[1], step), (n, what)
            assert np.array_equal(static_step(rig, q, k_new, v_new), step), (n, what)
            rig.close()


def static_step(rig, q, k_new, v_new):
    """s3_decode_step_static at pos = lens (again: the rows are there already)."""
    n = len(rig.lens)
    out = torch.full((n, rig.H, rig.D), float("nan"), dtype=torch.float32, device="cuda:0")
    pos = torch.tensor(rig.lens, dtype=torch.int32, device="cuda:0")
    args = [device_bits(wl.to_bits(x, rig.act), TDT[rig.act], "cuda:0") for x in (q, k_new, v_new)]
    assert s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, pos, *args, out, s3.S3_F32, 0.0, None, rig.stream) == 0
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("H,D,kvt,n", [(12, 128, s3.S3_BF16, 128), (16, 256, s3.S3_F16, 48), (64, 96, s3.S3_BF16, 24), (32, 64, s3.S3_F16, 96)])
def test_longer_chunks_sum_no_longer_runs(H, D, kvt, n):
    """16-bit rows, whole contexts that would be cut at 1024 rows: against 64 bits the outputs are as exact as in such chunks."""
    rng = np.random.default_rng(D)
    lens = [int(x) for x in rng.integers(1000, 1790, size=n)]
    rig = EdgeRig(("runs", H, H, D, kvt, kvt, 0), lens, M=2048)
    K, V = [], []
    for L in lens:
        K.append(rng.standard_normal((L, H, D), dtype=np.float32))
        V.append(rng.standard_normal((L, H, D), dtype=np.float32))
    rig.put(K, V)
    dt = {s3.S3_F16: torch.float16, s3.S3_BF16: torch.bfloat16}[kvt]

    def stored(x):  # [rows][H][D] -> [H][rows][D] in 64 bits, as the cache holds it
        return torch.from_numpy(x).to("cuda:0").to(dt).double().permute(1, 0, 2).contiguous()

    q = rng.standard_normal((n, H, D), dtype=np.float32)
    want = np.empty((n, H, D))
    for b in range(n):
        s = torch.matmul(stored(K[b]), stored(q[b][None]).permute(0, 2, 1).contiguous()).squeeze(2) / D**0.5
        p = torch.softmax(s, dim=1)
        want[b] = torch.matmul(p.unsqueeze(1), stored(V[b])).squeeze(1).cpu().numpy()
    off = []
    for chunk in (0, 1024):
        assert s3.s3_kv_set_param(rig.a, "chunk", chunk) == 0
        off.append(np.linalg.norm(rig.attend(q)[1] - want) / np.linalg.norm(want))
    rig.close()
    assert off[0] <= 1.03 * off[1], off  # (the division of the rows differs, and with it every rounding: 1 % either way)


FEW = [FAMS[0], FAMS[1], FAMS[2], ("3 x 128", 3, 3, 128, s3.S3_BF16, s3.S3_BF16, 0), ("16 x 64", 16, 16, 64, s3.S3_F16, s3.S3_F16, 0),
       FAMS[4], FAMS[5], ("17 x 64 e4m3", 17, 17, 64, s3.S3_E4M3, s3.S3_BF16, 3), ("4 x 128 e4m3", 4, 4, 128, s3.S3_E4M3, s3.S3_F16, 3)]


@pytest.mark.parametrize("fam", FEW, ids=[f[0] for f in FEW])
def test_few_contexts_shares_and_pieces(fam):
    """The kernel of few contexts at the edges of what a wave takes (a row, fours of them, twelve, thirteen, runs of 128; 8-bit
    rows: threes, six, seven) and of what a merge takes (16 pieces a round trip, 32, more), with the new row first, inside and last in a
    four; the largest batches of it and the first beyond; empty contexts between; head groups that are not full, and rows that go several to a
    load (the streaming kernel's).  Attention and step against the oracle; the step bit for bit the same through both of its entry points and
    with both orderings of the merge, and, 16-bit rows, as attention over the appended rows (8-bit rows take the new row last)."""
    name, H, Hkv, D, kvt, act, kind = fam
    n_hg = -(-H // (1024 // D if kind == 3 else 4 if D == 96 else 512 // D))
    last = min(64, (204 if kind == 3 else 192) // n_hg)
    rng = np.random.default_rng(7 * D + H)
    top = 8192
    rows = rng.standard_normal((top + 130, Hkv, D), dtype=np.float32)
    cases = [[1], [7], [8], [9], [31], [32], [33], [63], [64], [65], [96], [97], [104], [128], [129], [256], [519], [2048], [4100], [8000],
             [64] * 2, [65, 2], [0, 130], [3000, 40, 0, 700], [1500] * min(4, last), [100] * last, [40 + 37 * b for b in range(last)],
             [700] * (last - 1) + [2100]] + ([[90] * (last + 1)] if last < 64 else [])
    for lens in cases:
        n = len(lens)
        rig = EdgeRig(fam, lens, M=top)
        rig.put([rows[b:b + L] for b, L in enumerate(lens)], [rows[n - b:n - b + L] for b, L in enumerate(lens)])
        q = rng.standard_normal((n, H, D), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{name} / {lens[:4]} x {n}")
        k_new, v_new = (rng.standard_normal((n, Hkv, D), dtype=np.float32) for _ in range(2))
        qb, step = rig.step(q, k_new, v_new)
        longer = [L + 1 for L in lens]
        assert_close(step, rig.want(qb, longer), f"{name} / {lens[:4]} x {n} / step")
        again = rig.attend(q, lens=longer)[1]
        if kind == 0:
            assert np.array_equal(again, step), lens
        assert_close(again, rig.want(qb, longer), f"{name} / {lens[:4]} x {n} / appended")
        assert np.array_equal(static_step(rig, q, k_new, v_new), step), lens
        assert s3.s3_kv_set_param(rig.a, "merge_sync", 1) == 0
        assert np.array_equal(rig.attend(q, lens=longer)[1], again), lens
        rig.close()


TURNS = [FAMS[1], ("64 x 96", 64, 64, 96, s3.S3_BF16, s3.S3_BF16, 0), ("16 x 64", 16, 16, 64, s3.S3_F16, s3.S3_F16, 0), FAMS[0]]


@pytest.mark.parametrize("fam", TURNS, ids=[f[0] for f in TURNS])
def test_shares_of_thirteen_to_sixteen_rows(fam):
    """Whole contexts of 96 to 128 rows, twelve to sixteen a wave: beyond twelve rows a second turn of four (heads of 256: the
    loop), with the new row at every place of it."""
    name, H, Hkv, D, kvt, act, kind = fam
    last = min(64, 192 // -(-H // (4 if D == 96 else 512 // D)))
    rng = np.random.default_rng(D)
    rows = rng.standard_normal((200, Hkv, D), dtype=np.float32)
    for first in range(0, 32, last):
        lens = [96 + (first + b) % 32 for b in range(last)]
        rig = EdgeRig(fam, lens, M=256)
        rig.put([rows[b:b + L] for b, L in enumerate(lens)], [rows[last - b:last - b + L] for b, L in enumerate(lens)])
        q, k_new, v_new = (rng.standard_normal((last, h, D), dtype=np.float32) for h in (H, Hkv, Hkv))
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{name} / from {lens[0]}")
        longer = [L + 1 for L in lens]
        qb, step = rig.step(q, k_new, v_new)
        assert_close(step, rig.want(qb, longer), f"{name} / from {lens[0]} / step")
        assert np.array_equal(rig.attend(q, lens=longer)[1], step)
        rig.close()
