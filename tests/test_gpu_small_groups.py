"""Two or three query heads per cached head: by default the matrix-core kernel where it is faster, with the weights in three
16-bit parts, else the vector-ALU kernel.  Around the borders of that rule: against the fp32 oracle, against the vector-ALU
kernel to the accuracy of fp32 sums, and all entry points to the same bits."""
import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3
from tests.harness import assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,D,kvt,last", [(16, 8, 128, s3.S3_BF16, 64), (16, 8, 64, s3.S3_F16, 64), (6, 3, 256, s3.S3_F16, 85),
                                              (24, 8, 64, s3.S3_BF16, 32), (9, 3, 256, s3.S3_BF16, 85), (3, 1, 128, s3.S3_F16, 256)])
def test_both_kernels_of_small_groups_agree(H, Hkv, D, kvt, last):
    from tests.test_gpu_numeric_edges import TDT, EdgeRig, device_bits, wl

    for n in (1, last, last + 1):
        rng = np.random.default_rng(n + D)
        lens = [int(x) for x in rng.integers(0, 90, size=n)]
        lens[0], lens[-1] = 900, lens[-1] + 1
        rig = EdgeRig(("small groups", H, Hkv, D, kvt, kvt, 1), lens, M=1024)
        rig.put([rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens],
                [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens])
        q = rng.standard_normal((n, H, D), dtype=np.float32)
        qb, att = rig.attend(q)
        assert_close(att, rig.want(qb), f"{n} contexts")
        assert s3.s3_kv_set_param(rig.a, "variant", 0) == 0
        vector = rig.attend(q)[1]
        assert s3.s3_kv_set_param(rig.a, "variant", -1) == 0
        # each is within 3e-7 of 64 bits (fp32 sums over rows and elements): twice their sum
        assert np.linalg.norm(att - vector) <= 1.2e-6 * np.linalg.norm(vector), n
        k_new, v_new = (rng.standard_normal((n, Hkv, D), dtype=np.float32) for _ in range(2))
        longer = [L + 1 for L in lens]
        qb, step = rig.step(q, k_new, v_new)
        assert_close(step, rig.want(qb, longer), f"{n} contexts / step")
        assert np.array_equal(rig.attend(q, lens=longer)[1], step), n
        out = torch.full((n, H, D), float("nan"), dtype=torch.float32, device="cuda:0")
        args = [device_bits(wl.to_bits(x, kvt), TDT[kvt], "cuda:0") for x in (q, k_new, v_new)]
        assert s3.s3_decode_step_static(rig.a, 0, n, rig.off_d, torch.tensor(lens, dtype=torch.int32, device="cuda:0"), *args, out, s3.S3_F32,
                                        0.0, None, rig.stream) == 0
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), step), n
        rig.close()
