"""The arena's scratch (arrival counters, then chunk partials) over calls that lay it out differently: every call must
find its counters at zero whatever ran before it on the arena."""
import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3
from tests.harness import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,D,kvt", [(32, 8, 128, s3.S3_BF16), (16, 1, 256, s3.S3_F16), (8, 2, 64, s3.S3_F16)])
def test_both_kernels_of_a_shared_head_arena_in_turn(H, Hkv, D, kvt):
    """Matrix cores, vector ALU with sequence 0 in many chunks (its partials come first in the scratch), matrix cores
    again: all three against the oracle, and the third bit for bit the first."""
    from tests.test_gpu_numeric_edges import EdgeRig

    lens = [1000, 300, 0, 17, 1900]
    rng = np.random.default_rng(60 + D)
    rig = EdgeRig(("switch", H, Hkv, D, kvt, kvt, 2), lens, M=2048)
    rig.put([rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens],
            [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens])
    q = rng.standard_normal((len(lens), H, D), dtype=np.float32)
    qb, first = rig.attend(q)
    want = rig.want(qb)
    assert_close(first, want, "matrix cores")
    for chunk in (0, 32):
        assert s3.s3_kv_set_param(rig.a, "variant", 0) == 0 and s3.s3_kv_get_param(rig.a, "kernel_kind") == (0, 1)
        assert s3.s3_kv_set_param(rig.a, "chunk", chunk) == 0
        assert_close(rig.attend(q)[1], want, f"vector ALU, chunk {chunk}")
        assert s3.s3_kv_set_param(rig.a, "variant", -1) == 0 and s3.s3_kv_set_param(rig.a, "chunk", 0) == 0
        assert np.array_equal(rig.attend(q)[1], first), f"matrix cores after the vector ALU, chunk {chunk}"
    rig.close()


@pytest.mark.parametrize("H,Hkv,D,kvt,act,kind,n,M", [(16, 16, 256, s3.S3_F16, s3.S3_F16, 0, 30, 1024), (12, 12, 128, s3.S3_BF16, s3.S3_BF16, 0, 90, 256),
                                                      (16, 16, 256, s3.S3_E4M3, s3.S3_F16, 3, 60, 1024), (32, 8, 128, s3.S3_BF16, s3.S3_BF16, 2, 300, 256),
                                                      (16, 8, 128, s3.S3_F16, s3.S3_F16, 1, 300, 2048)])
def test_a_smaller_batch_never_moves_the_scratch(H, Hkv, D, kvt, act, kind, n, M):
    """The scratch grows for a larger batch only: its address is in recorded graphs.  (Few contexts are cut finer and
    may need more room than many.)  A smaller "chunk" may move it."""
    from tests.test_gpu_numeric_edges import EdgeRig

    rig = EdgeRig(("grow", H, Hkv, D, kvt, act, kind), [1] * n, M=M)
    rng = np.random.default_rng(n)
    rig.put([rng.standard_normal((1, Hkv, D), dtype=np.float32)] * n, [rng.standard_normal((1, Hkv, D), dtype=np.float32)] * n)
    q = rng.standard_normal((n, H, D), dtype=np.float32)
    rig.attend(q)
    held = s3.s3_kv_get_param(rig.a, "scratch_bytes")[1]
    for k in [k for k in range(1, n) if k < 40 or k % 16 in (0, 1)]:
        rig.attend(q[:k], lens=[1] * k)
        assert s3.s3_kv_get_param(rig.a, "scratch_bytes")[1] == held, k
    assert s3.s3_kv_reserve_scratch(rig.a, n) == 0 and s3.s3_kv_get_param(rig.a, "scratch_bytes")[1] == held
    assert s3.s3_kv_set_param(rig.a, "chunk", 32) == 0
    qb, got = rig.attend(q)
    assert_close(got, rig.want(qb), "chunk 32")
    rig.close()


def test_the_first_call_of_an_arena_on_a_stream_of_its_own():
    """Every call starts with no scratch: the counters are zero before a kernel on a stream that does not wait for the
    default stream looks at them."""
    import torch

    from tests.test_gpu_numeric_edges import EdgeRig

    lens = [1900, 3, 2000]
    rng = np.random.default_rng(77)
    rows = [rng.standard_normal((L, 8, 128), dtype=np.float32) for L in lens]
    q = rng.standard_normal((3, 32, 128), dtype=np.float32)
    side = torch.cuda.Stream()
    for i in range(4):
        rig = EdgeRig(("first", 32, 8, 128, s3.S3_BF16, s3.S3_BF16, 2), lens, M=2048)
        rig.put(rows, rows)
        torch.cuda.synchronize()
        rig.stream = side.cuda_stream
        with torch.cuda.stream(side):
            qb, got = rig.attend(q)
        assert_close(got, rig.want(qb), f"arena {i}")
        rig.close()
