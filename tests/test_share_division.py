"""How many shares (waves) per column the matrix-core kernel divides a batch into when its pieces have to fit the fixed
buffer of s3_decode_step_static: never far fewer than the chunks of the documented rule, so that the chip has work (0:
every context whole, by a wave of its own).  Host integers on metadata-only arenas."""
import ctypes

import pytest

from paper_2306_06000_amd import binding as s3

STATIC = 32 << 20


@pytest.mark.parametrize("H,Hkv,D,kvt,max_len", [(32, 8, 128, s3.S3_BF16, 256), (64, 8, 128, s3.S3_BF16, 256), (64, 8, 128, s3.S3_E4M3, 128),
                                                 (16, 1, 256, s3.S3_F16, 128), (16, 1, 256, s3.S3_F16, 2048), (128, 8, 256, s3.S3_F16, 512),
                                                 (128, 8, 256, s3.S3_F16, 128), (24, 8, 64, s3.S3_BF16, 2048), (256, 1, 256, s3.S3_BF16, 64)])
def test_the_fixed_buffer_never_starves_the_division(H, Hkv, D, kvt, max_len):
    shares_of = s3.lib().s3i_gqa_max_shares
    shares_of.restype, shares_of.argtypes = ctypes.c_int64, [ctypes.c_void_p, ctypes.c_int32]
    cfg = s3.make_config(1, H, D, kvt, 64, max_len, Hkv, s3.S3_BF16)
    st, a = s3.s3_kv_arena_init(cfg, None, 1 << 30)
    assert st == 0
    columns = Hkv * -(-(H // Hkv) // 16)
    counters = -(-4096 * columns * 4 // 256) * 256 + 256
    slots = (STATIC - counters) // (H * (4 * D + 8))
    waves = -(-256 * 8 // columns)
    for n in range(1, 4096):
        shares = shares_of(a, n)
        chunks = n * -(-max_len // (256 if n * columns >= 4096 else 128))
        if chunks <= slots and shares + n > slots:
            assert shares == 0, (n, shares)  # no piece leaves its wave
        assert 0 <= shares <= waves, (n, shares)
        assert 2 * (shares or n) >= min(waves, chunks), (n, shares, chunks)
        assert shares or max_len <= (256 if n * columns >= 4096 else 128), n  # contexts of one chunk only
    s3.s3_kv_arena_destroy(a)
