"""Two or three query heads per cached head: by default the kernel with the scores on the matrix cores where it is faster, else
the vector-ALU kernel.  Around the borders of that rule: against the fp32 oracle, against the vector-ALU kernel to the accuracy
of fp32 sums, all entry points to the same bits, and both kernels alike for infinite values, for values near the type's largest
and for weights that are small."""
import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3
from tests.harness import assert_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


SHAPES = [(16, 8, 128, s3.S3_BF16, 64), (16, 8, 64, s3.S3_F16, 64), (6, 3, 256, s3.S3_F16, 85), (24, 8, 64, s3.S3_BF16, 32),
          (9, 3, 256, s3.S3_BF16, 85), (3, 1, 128, s3.S3_F16, 256)]


@pytest.mark.parametrize("H,Hkv,D,kvt,last", SHAPES)
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


def in_64_bits(q, K, V, scale):
    """q [H][D], K and V [rows][Hkv][D] -> [H][D]."""
    H, Hkv = q.shape[0], K.shape[1]
    out = np.empty(q.shape)
    for h in range(H):
        s = K[:, h * Hkv // H].astype(np.float64) @ q[h].astype(np.float64) * scale
        p = np.exp(s - s.max())
        p /= p.sum()
        v = V[:, h * Hkv // H].astype(np.float64)
        with np.errstate(invalid="ignore"):
            out[h] = (p[:, None] * v).sum(axis=0)
    return out


@pytest.mark.parametrize("H,Hkv,D,kvt,last", SHAPES)
def test_infinite_large_and_lightly_weighted_values(H, Hkv, D, kvt, last):
    """Weights are held in fp32 and are at most 1, whichever kernel serves the batch.  Even head dimensions: infinities in one
    row, which give infinite elements and leave all others alone.  Others: values near the type's largest, far above the other
    rows' weights; and a large value under a weight of e^-14, which with weights of fewer bits is off by 1e-5."""
    from tests.test_gpu_numeric_edges import EdgeRig

    large = 6e4 if kvt == s3.S3_F16 else 1e37
    for n in (1, 3, last, last + 1):
        lens = [1040 + 64 * (b % 3) if b < 40 else 130 for b in range(n)]
        rig = EdgeRig(("small groups", H, Hkv, D, kvt, kvt, 1), lens, M=2048)
        K = [np.zeros((L, Hkv, D), np.float32) for L in lens]
        V = [np.zeros((L, Hkv, D), np.float32) for L in lens]
        for b, L in enumerate(lens):
            V[b][:] = ((np.arange(L) % 7) - 3.0)[:, None, None]
            V[b][0, :, 0], V[b][64, :, 2] = np.inf, -np.inf          # two infinite elements
            # every 64th row weighs 2^6 times as much as the others (scores: q[0] = 1, scale 1), and holds the largest values
            K[b][40::64, :, 0] = 6 * 0.6931
            V[b][40::64, :, 4] = large
            # q[1] = 1 for the odd heads: the last row weighs e^-14 of any other
            K[b][:-1, :, 1] = 14.0
            V[b][:, :, 6] = 0.0
            V[b][-1, :, 6] = 6e4
        rig.put(K, V)
        K, V = ([from_bits(rig, x) for x in xs] for xs in (K, V))
        q = np.zeros((n, H, D), np.float32)
        q[:, 0::2, 0] = 1.0
        q[:, 1::2, 1] = 1.0
        wants = [in_64_bits(q[b], K[b], V[b], 1.0) for b in range(n)]
        for variant in (-1, 0, s3.s3_kv_get_param(rig.a, "n_variants")[1] - 1):
            assert s3.s3_kv_set_param(rig.a, "variant", variant) == 0
            got = attend_with_scale_1(rig, q)
            for b, want in enumerate(wants):
                what = (n, variant, b)
                assert np.array_equal(np.isposinf(got[b]), np.isposinf(want)), what
                assert np.array_equal(np.isneginf(got[b]), np.isneginf(want)), what
                assert not np.isnan(got[b]).any(), what
                # Scores of up to 14 * log2(e) = 20.2 rounded to fp32 (2^-20 at most, twice: the scale, the product) and their
                # exponential (2^-23): 2 * 0.7 * 2^-20 + 2^-23 = 1.4e-6; sums of 1200 rows below 2e-7.
                for d in (4, 6):
                    assert (np.abs(got[b][:, d] - want[:, d]) <= 2e-6 * np.abs(want[:, d])).all(), what + (d,)
        rig.close()


def from_bits(rig, x):
    from tests.test_gpu_numeric_edges import wl

    bits = wl.to_bits(x, rig.kvt)
    return bits.view(np.float16).astype(np.float32) if rig.kvt == s3.S3_F16 else (bits.astype(np.uint32) << 16).view(np.float32)


def attend_with_scale_1(rig, q):
    from tests.test_gpu_numeric_edges import TDT, device_bits, wl

    n = q.shape[0]
    out = torch.full((n, rig.H, rig.D), float("nan"), dtype=torch.float32, device="cuda:0")
    lens = torch.tensor(rig.lens, dtype=torch.int32, device="cuda:0")
    assert s3.s3_decode_attention(rig.a, 0, n, device_bits(wl.to_bits(q, rig.act), TDT[rig.act], "cuda:0"), rig.off_d, lens, out, s3.S3_F32, 1.0,
                                  rig.stream) == 0
    torch.cuda.synchronize()
    return out.cpu().numpy()
