"""Scores that overflow to -inf (finite queries and keys) in the first rows of a context, ordinary scores behind them:
the overflowing rows weigh nothing, wherever chunks, shares and pieces of the context begin and end, also where a
whole piece holds nothing else."""
import numpy as np
import pytest

from paper_2306_06000_amd import binding as s3
from tests.harness import assert_close

pytestmark = pytest.mark.gpu

FAMS = [
    ("matrix cores d128", 32, 8, 128, s3.S3_BF16, s3.S3_BF16, 2),
    ("matrix cores d256 group 16", 16, 1, 256, s3.S3_BF16, s3.S3_BF16, 2),
    ("matrix cores d64 e4m3", 8, 1, 64, s3.S3_E4M3, s3.S3_BF16, 4),
    ("8-bit rows d128", 4, 4, 128, s3.S3_E4M3, s3.S3_BF16, 3),
    ("two heads a cached head d128", 16, 8, 128, s3.S3_BF16, s3.S3_BF16, 1),
    ("three heads a cached head d64", 24, 8, 64, s3.S3_BF16, s3.S3_BF16, 1),
    ("three heads a cached head d256", 6, 2, 256, s3.S3_BF16, s3.S3_BF16, 1),
]


@pytest.mark.parametrize("fam", FAMS, ids=[f[0] for f in FAMS])
def test_rows_of_minus_infinity_weigh_nothing(fam):
    from tests.test_gpu_numeric_edges import EdgeRig

    name, H, Hkv, D, kvt, act, kind = fam
    rng = np.random.default_rng(D + kind)
    for what, lens, lost in (("one", [2000], [1900]), ("few", [700, 40, 1000, 900], [300, 39, 0, 890]),
                             ("many", [300] * 270 + [40] * 30, [256] * 270 + [39] * 30)):
        rig = EdgeRig(fam, lens, M=2048)
        K = [np.zeros((L, Hkv, D), np.float32) for L in lens]
        for k, x in zip(K, lost):
            k[:x] = -400.0
        V = [rng.standard_normal((L, Hkv, D), dtype=np.float32) for L in lens]
        rig.put(K, V)
        q = np.full((len(lens), H, D), 2e36, np.float32)  # q . K: -400 * 2e36 * D < -3.4e38, times a scale below 1; or 0
        for chunk in (0, 32, 160):
            assert s3.s3_kv_set_param(rig.a, "chunk", chunk) == 0
            qb, got = rig.attend(q)
            assert_close(got, rig.want(qb), f"{name} / {what} / chunk {chunk}")
        rig.close()
