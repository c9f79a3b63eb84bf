"""How many shares (waves) per column the matrix-core kernel divides a batch into when its pieces have to fit the fixed
buffer of s3_decode_step_static: never far fewer than the chunks of the documented rule, so that the chip has work (0:
every context whole, by a wave of its own); and that the instance without a loop over units is taken only where every unit
has a wave, or a workgroup, of its own.  Host integers on metadata-only arenas."""
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


@pytest.mark.parametrize("group,D,kvt", [(4, 256, s3.S3_F16), (4, 128, s3.S3_BF16), (3, 256, s3.S3_BF16), (4, 256, s3.S3_E4M3), (20, 64, s3.S3_F16)])
@pytest.mark.parametrize("per_cu", [1, 2])
def test_no_more_units_than_run_at_once_without_the_loop(group, D, kvt, per_cu):
    """A column is divided into at most wave_shares units, a wave each, or team_shares, a workgroup each (at least one, however many
    the columns are)."""
    units_of = s3.lib().s3i_gqa_units
    units_of.restype, units_of.argtypes = ctypes.c_int32, [ctypes.c_void_p, ctypes.c_int32] + [ctypes.POINTER(ctypes.c_int32)] * 2
    workgroups = 256 * per_cu
    for Hkv in (1, 3, 8, 100, 128, 129, 200, 255, 256, 257, 300, 320, 511, 512, 513, 600, 1023, 1024, 1025, 2048, 2049, 3000):
        cfg = s3.make_config(1, group * Hkv, D, kvt, 64, 2048, Hkv, s3.S3_BF16)
        st, a = s3.s3_kv_arena_init(cfg, None, 1 << 30)
        assert st == 0
        columns = Hkv * -(-group // 16)
        waves, teams = ctypes.c_int32(), ctypes.c_int32()
        loop = units_of(a, per_cu, waves, teams)
        assert waves.value == max(1, 4 * workgroups // columns) and teams.value == max(1, workgroups // columns)
        if not loop:
            assert waves.value * columns <= 4 * workgroups and teams.value * columns <= workgroups, (Hkv, per_cu)
        assert loop == (columns > workgroups)
        for param in ("chunk", "grid_blocks"):  # the caller's division, the caller's grid
            assert s3.s3_kv_set_param(a, param, 64) == 0 and units_of(a, per_cu, waves, teams)
            assert s3.s3_kv_set_param(a, param, 0) == 0
        s3.s3_kv_arena_destroy(a)
