"""Batches on the dynamic work list: the classes of its order, and whether positions are claimed, are decided on the device
by the mean rows of a context.  Both sides of both bounds, in every build of the batch view (one wave up to 512 contexts,
the workgroup beyond, in several passes from 2305 on), against the fp32 oracle, and the step against append + attention."""
import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3
from tests.harness import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mean", [1, 23, 24, 127, 128, 200])
@pytest.mark.parametrize("n", [129, 512, 513, 700, 2304, 2305, 4095])
def test_work_order_by_mean_rows(n, mean):
    from tests.test_gpu_numeric_edges import EdgeRig

    if n > 2000 and mean > 128:
        mean = 129
    H, D = 3, 64
    rng = np.random.default_rng(n + mean)
    lens = rng.integers(0, 2 * mean + 1, size=n)
    lens[[0, n // 2, n - 1]] = 0, 1, 2 * mean
    spare = mean * n - int(lens.sum())  # exactly the mean, in attention; one more row each in the step
    for b in range(1, n - 1):
        take = max(-int(lens[b]), min(spare, 2040 - int(lens[b]) if b % 97 == 1 else 2 * mean - int(lens[b])))
        lens[b] += take
        spare -= take
    assert spare == 0 or abs(spare) < n
    lens = [int(x) for x in lens]
    rig = EdgeRig(("mean", H, H, D, s3.S3_F16, s3.S3_F16, 0), lens, M=2048)
    K, V = (rng.standard_normal((4096, H, D), dtype=np.float32) for _ in range(2))
    starts = rng.integers(0, 2048, size=n)
    rig.put([K[x:x + L] for x, L in zip(starts, lens)], [V[x:x + L] for x, L in zip(starts, lens)])
    q = rng.standard_normal((n, H, D), dtype=np.float32)
    qb, att = rig.attend(q)
    assert_close(att, rig.want(qb), f"n {n} mean {mean}")
    assert s3.s3_kv_set_param(rig.a, "classes", 4) == 0
    assert np.array_equal(rig.attend(q)[1], att)  # the order of the items changes no bit
    assert s3.s3_kv_set_param(rig.a, "classes", 0) == 0
    qb, step = rig.step(q, *(rng.standard_normal((n, H, D), dtype=np.float32) for _ in range(2)))
    longer = [L + 1 for L in lens]
    assert_close(step, rig.want(qb, longer), f"n {n} mean {mean} step")
    for rep in range(3):  # the claim counters come back to zero
        assert np.array_equal(rig.attend(q, lens=longer)[1], step), rep
    rig.close()
