"""s3_decode_step_static (the decode step for callers that cannot allocate device memory) against
s3_decode_step: same outputs and same appended rows, bit for bit, and within the attention tolerance of the
oracle; two calls in a row, the second on a smaller batch; across kernel families that lay the fixed scratch
out differently; refusal of a call that does not fit; no device allocation."""
import os

import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3
from paper_2306_06000_amd import workloads as wl
from tests.harness import assert_close, device_bits
from tests.test_gpu_numeric_edges import FAMILIES, TDT, EdgeRig

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def need_gpu_and_lib():
    assert torch.cuda.is_available(), "these tests need the GPU box"
    assert os.path.exists(s3.LIB_PATH), "libs3kv.so must be built before the GPU tests run"
    s3.lib()


def one_call(fam, lens, chunk, seed, entry):
    """Fill a fresh arena with seeded rows, run one decode step through `entry`, return what it produced."""
    name, H, Hkv, D, kvt, act, kind = fam
    rng = np.random.default_rng(seed)
    rig = EdgeRig(fam, lens, M=2048)
    rig.put([rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens],
            [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens])
    assert s3.s3_kv_set_param(rig.a, "chunk", chunk) == 0
    n = len(lens)
    qb = wl.normal_bits(rng, (n, H, D), act)
    kb = wl.normal_bits(rng, (n, Hkv, D), act)
    vb = wl.normal_bits(rng, (n, Hkv, D), act)
    q, k_new, v_new = (device_bits(x, TDT[act], DEV) for x in (qb, kb, vb))
    pos_d = torch.tensor(lens, dtype=torch.int32, device=DEV)
    out = torch.full((n, H, D), float("nan"), dtype=torch.float32, device=DEV)
    len_out = torch.zeros(n, dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    free_before = torch.cuda.mem_get_info()[0]
    st = entry(rig.a, 0, n, rig.off_d, pos_d, q, k_new, v_new, out, s3.S3_F32, 0.0, len_out, rig.stream,
               slot_id=rig.ids, pos_host=lens)
    torch.cuda.synchronize()
    free_after = torch.cuda.mem_get_info()[0]
    assert st == 0, (name, st)
    for b, sid in enumerate(rig.ids.tolist()):
        assert rig.o.append(sid, 0, lens[b], kb[b], vb[b]) == 0
    want = rig.want(qb, [L + 1 for L in lens])
    res = dict(out=out.clone(), mem=rig.mem.clone(), len_out=len_out.cpu().tolist(), want=want,
               scratch=s3.s3_kv_get_param(rig.a, "scratch_bytes")[1], freed=free_before - free_after)
    rig.close()
    return res


def compare(fam, lens, chunk, seed):
    ref = one_call(fam, lens, chunk, seed, s3.s3_decode_step)
    got = one_call(fam, lens, chunk, seed, s3.s3_decode_step_static)
    what = f"{fam[0]} n={len(lens)} chunk={chunk}"
    assert got["len_out"] == ref["len_out"] == [L + 1 for L in lens], what
    assert torch.equal(got["out"], ref["out"]), what          # same kernels, same arithmetic: same bits
    assert torch.equal(got["mem"], ref["mem"]), what          # the appended rows, and nothing else, changed
    assert_close(got["out"].cpu().numpy(), got["want"], what)  # and both are right
    assert got["scratch"] == 0, what   # the arena's own scratch was never allocated on this path
    assert got["freed"] == 0, what     # free device memory is the same before and after the call
    assert ref["scratch"] > 0, what    # (the existing entry point did allocate its scratch)


def test_static_scratch_step_equals_the_allocating_step_two_calls_in_a_row():
    rng = np.random.default_rng(77)
    big = [int(x) for x in rng.integers(1, 1500, size=48)] + [0, 1, 2047]
    small = [700, 3, 64, 129, 0, 1999, 65]
    mha = FAMILIES[0]
    # many chunks per context (the partials and the arrival counters live in the fixed buffer), then a smaller
    # batch right after it: stale partials and counters of the first call must not leak into the second
    compare(mha, big, 64, seed=1)
    compare(mha, small, 64, seed=2)
    compare(mha, small, 0, seed=3)
    # other families lay the buffer out differently (no counters; counters for other head-group counts): the
    # layout changes back and forth between calls
    for fam, chunk in ((FAMILIES[4], 32), (FAMILIES[6], 64), (FAMILIES[3], 64), (FAMILIES[7], 32), (FAMILIES[2], 64),
                       (mha, 64)):
        compare(fam, small, chunk, seed=4)
        compare(fam, big[:20], chunk, seed=5)


def test_static_scratch_step_refuses_what_does_not_fit_and_launches_nothing():
    fam = FAMILIES[0]
    name, H, Hkv, D, kvt, act, kind = fam
    n = 600
    lens = [10] * n
    rig = EdgeRig(fam, lens, M=2048)
    assert s3.s3_kv_set_param(rig.a, "chunk", 32) == 0  # 64 chunk slots x 600 sequences x 16 heads x 1032 B > 32 MiB
    need = n * 64 * H * (4 * D + 8)
    assert need > s3.S3_STATIC_SCRATCH_BYTES
    z = torch.zeros((n, H, D), dtype=TDT[act], device=DEV)
    pos_d = torch.tensor(lens, dtype=torch.int32, device=DEV)
    out = torch.full((n, H, D), float("nan"), dtype=torch.float32, device=DEV)
    snap = rig.mem.clone()
    st = s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, pos_d, z, z, z, out, s3.S3_F32, 0.0, None, rig.stream)
    torch.cuda.synchronize()
    assert st == s3.S3_ERR_SCRATCH
    assert s3.lib().s3_status_str(st) == b"S3_ERR_SCRATCH"
    assert torch.isnan(out).all() and torch.equal(snap, rig.mem)
    # the same call fits at the default chunk (two chunk slots per sequence)
    assert s3.s3_kv_set_param(rig.a, "chunk", 0) == 0
    assert s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, pos_d, z, z, z, out, s3.S3_F32, 0.0, None, rig.stream) == 0
    torch.cuda.synchronize()
    assert torch.isfinite(out).all()
    rig.close()


def test_static_scratch_step_recorded_in_a_graph_replays_exactly_with_the_dynamic_work_list():
    """What the entry point is for: the step is recorded into a HIP graph (nothing in it allocates) and replayed,
    with eager work on the same arena in between.  The kernel shape with the dynamic work list on a grid much
    smaller than the list: the list's counters and the arrival counters of the chunk merge, which live in the fixed
    buffer, must be back at zero after every launch, replayed or not."""
    fam = FAMILIES[0]
    name, H, Hkv, D, kvt, act, kind = fam
    rng = np.random.default_rng(91)
    lens = [0, 1, 63, 200, 511, 700, 64, 5, 999, 130]
    rig = EdgeRig(fam, lens, M=2048)
    rig.put([rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens],
            [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens])
    assert s3.s3_kv_set_param(rig.a, "chunk", 64) == 0
    assert s3.s3_kv_set_param(rig.a, "variant", 13) == 0
    assert s3.s3_kv_set_param(rig.a, "grid_blocks", 16) == 0
    n = len(lens)
    q, k, v = (device_bits(wl.normal_bits(rng, (n, H, D), act), TDT[act], DEV) for _ in range(3))
    pos_d = torch.tensor(lens, dtype=torch.int32, device=DEV)
    len_out = torch.zeros(n, dtype=torch.int32, device=DEV)
    want = torch.full((n, H, D), float("nan"), dtype=torch.float32, device=DEV)
    assert s3.s3_decode_step(rig.a, 0, n, rig.off_d, pos_d, q, k, v, want, s3.S3_F32, 0.0, len_out, rig.stream) == 0
    first = torch.full_like(want, float("nan"))
    assert s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, pos_d, q, k, v, first, s3.S3_F32, 0.0, len_out, rig.stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(first, want)
    out = torch.full_like(want, float("nan"))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        st = s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, pos_d, q, k, v, out, s3.S3_F32, 0.0, len_out,
                                      torch.cuda.current_stream().cuda_stream)
    assert st == 0
    for rep in range(4):
        out.fill_(float("nan"))
        len_out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {rep}"
        assert len_out.cpu().tolist() == [L + 1 for L in lens]
        again = torch.full_like(want, float("nan"))
        assert s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, pos_d, q, k, v, again, s3.S3_F32, 0.0, len_out,
                                        rig.stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(again, want)
    assert s3.s3_kv_get_param(rig.a, "scratch_bytes")[1] > 0  # (from the allocating reference call only)
    rig.close()


def test_recorded_steps_of_different_kernels_and_arenas_replay_in_any_order():
    """One recorded step per batch size and arena is what the entry point is for.  An arena of two query heads per cached
    head changes its kernel with the batch, and the kernels and arenas lay their scratch out differently: whatever was
    replayed or called before, every step finds its arrival counters at zero.  All of them have contexts in several
    pieces, and their partials are large enough to cover every other step's counters."""
    small_groups = ("two heads a cached head", 16, 8, 128, s3.S3_BF16, s3.S3_BF16, 1)
    steps = []
    for fam, n in ((small_groups, 20), (small_groups, 64), (small_groups, 65), (small_groups, 200), (FAMILIES[0], 12), (FAMILIES[5], 40),
                   (FAMILIES[6], 30)):
        name, H, Hkv, D, kvt, act, kind = fam
        rng = np.random.default_rng(n + D)
        lens = [1500 - 11 * b if b < 40 else 3 + b % 20 for b in range(n)]
        rig = EdgeRig(fam, lens, M=2048)
        rows = rng.standard_normal((2048, Hkv, D), dtype=np.float32)
        rig.put([np.roll(rows, b, axis=0)[:L] for b, L in enumerate(lens)], [np.roll(rows, 3 * b, axis=0)[:L] for b, L in enumerate(lens)])
        q, k, v = (device_bits(wl.normal_bits(rng, (n, h, D), act), TDT[act], DEV) for h in (H, Hkv, Hkv))
        pos_d = torch.tensor(lens, dtype=torch.int32, device=DEV)
        want = torch.full((n, H, D), float("nan"), dtype=torch.float32, device=DEV)
        assert s3.s3_decode_step(rig.a, 0, n, rig.off_d, pos_d, q, k, v, want, s3.S3_F32, 0.0, None, rig.stream) == 0
        out = torch.empty_like(want)

        def call(rig=rig, n=n, pos_d=pos_d, args=(q, k, v, out)):
            return s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, pos_d, *args, s3.S3_F32, 0.0, None,
                                            torch.cuda.current_stream().cuda_stream)

        def check(what, out=out, want=want, name=f"{name}, {n} contexts"):
            torch.cuda.synchronize()
            assert torch.equal(out, want), (name, what)

        out.fill_(float("nan"))
        assert call() == 0  # (an eager call, then the recording: the host saw the same layout twice)
        check("eager")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            assert call() == 0
        steps.append((rig, graph, call, check, out))
    order = [0, 3, 0, 2, 1, 3, 1, 4, 0, 5, 2, 0, 6, 1, 2, 5, 3, 4, 6, 3, 5, 0]
    for eager_between in (False, True):
        for i, k in enumerate(order):
            rig, graph, call, check, out = steps[k]
            out.fill_(float("nan"))
            graph.replay()
            check(f"replay {i}")
            if eager_between:
                rig, graph, call, check, out = steps[order[-1 - i]]
                out.fill_(float("nan"))
                assert call() == 0
                check(f"call after replay {i}")
    for rig, *_ in steps:
        rig.close()
