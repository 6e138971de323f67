"""How the first launch of a step is laid out for a shape (worked out on the host, no GPU)."""
import paper_1804_06609_amd as dba

UNITS, UNIT_LDS, LAUNCH_LDS = 256, 160 * 1024, 64 * 1024


def shapes():
    """Every number of rows per compute unit up to 40 and some beyond, short rows to long ones."""
    for share in list(range(1, 41)) + [100, 1000, 10000]:
        for V in (64, 1000, 8191, 16384, 32003, 50000, 131072, 524288):
            for rows in {256 * share, 256 * share - 129}:
                for k in (1, 7, 64):
                    if rows // k <= 65535:
                        yield max(1, rows // k), k, V


def test_unused_lds_lets_no_more_rows_on_a_compute_unit_than_meant():
    """A workgroup's LDS is within what a launch may ask for, leaves a tenth of the unit free where rows are
    held back, and never holds them below the unit's even share where all of them would fit at once."""
    for B, k, V in shapes():
        for fmt in (dba.DBA_LOGP_F32, dba.DBA_LOGP_F16, dba.DBA_LOGP_BF16):
            waves, tiles, lds, _ = dba.dba_debug_stream_plan(B, k, V, fmt)
            own = {4: 17440, 8: 34880}[waves]
            share, fit = -(-B * k // UNITS), UNIT_LDS // lds
            assert (waves, tiles) in ((4, 2), (8, 2), (8, 4)) and own <= lds <= LAUNCH_LDS, (B, k, V, waves, tiles, lds)
            if share <= 32 // waves:
                assert fit >= share, (B, k, V, fit)
            if lds > own:
                assert share > 32 // waves or fit == share, (B, k, V, fit)
                assert UNIT_LDS - fit * lds >= UNIT_LDS // 10, (B, k, V, fit, lds)


def test_bad_arguments_are_refused():
    for bad in ((0, 1, 100, 0), (1, 65, 100, 0), (1, 5, 4, 0), (1, 5, 100, 3), (1, 5, 100, -1)):
        try:
            dba.dba_debug_stream_plan(*bad)
        except dba.DbaError:
            continue
        raise AssertionError(bad)


def test_sentences_are_numbered_eight_abreast_only_where_rows_are_short():
    """Many long rows a power of two apart share a part of a die's L2 if the die streams neighbouring rows."""
    for B, k, V, fmt, abreast in ((64, 20, 32000, dba.DBA_LOGP_F32, 1280), (67, 20, 32000, dba.DBA_LOGP_F32, 1280),
                                  (7, 20, 32000, dba.DBA_LOGP_F32, 0), (128, 64, 127999, dba.DBA_LOGP_F32, 8192),
                                  (128, 64, 128000, dba.DBA_LOGP_F32, 0), (128, 64, 128000, dba.DBA_LOGP_F16, 8192),
                                  (16, 64, 262144, dba.DBA_LOGP_BF16, 0), (16, 64, 262144, dba.DBA_LOGP_F32, 0),
                                  (8, 64, 131072, dba.DBA_LOGP_F32, 0), (8, 63, 131072, dba.DBA_LOGP_F32, 504),
                                  (34, 8, 159134, dba.DBA_LOGP_F32, 256)):
        assert dba.dba_debug_stream_plan(B, k, V, fmt)[3] == abreast, (B, k, V, fmt)


def test_only_long_rows_that_follow_one_another_are_held_to_six_waves_a_simd():
    """Short rows are latency, and more of them at a time hide more of it."""
    for B, k, V, fmt, held in ((110, 20, 8000, dba.DBA_LOGP_F32, False), (400, 20, 1000, dba.DBA_LOGP_F32, False),
                               (128, 64, 16000, dba.DBA_LOGP_BF16, False), (128, 64, 12287, dba.DBA_LOGP_F32, False),
                               (128, 64, 12288, dba.DBA_LOGP_F32, True), (128, 64, 32000, dba.DBA_LOGP_BF16, True),
                               (110, 20, 32000, dba.DBA_LOGP_F32, True), (64, 32, 32000, dba.DBA_LOGP_F32, False)):
        waves, _, lds, _ = dba.dba_debug_stream_plan(B, k, V, fmt)
        assert waves == 4 and UNIT_LDS // lds == (6 if held else 9), (B, k, V, fmt, lds)


def test_tiles_in_flight_beyond_a_row_per_compute_unit():
    """One launch keeps two tiles there too, and four only for rows of seven tiles a wave (six with 16-bit elements);
    two launches (k > 32 here) always two."""
    f32, bf16 = dba.DBA_LOGP_F32, dba.DBA_LOGP_BF16
    for B, k, V, fmt, tiles in ((16, 16, 32000, f32, 4), (257, 1, 32000, f32, 2), (26, 10, 32000, f32, 2), (16, 30, 50000, f32, 2),
                                (26, 10, 57343, f32, 2), (26, 10, 57344, f32, 4), (16, 32, 100000, f32, 4), (30, 16, 65000, bf16, 2),
                                (26, 10, 98303, bf16, 2), (26, 10, 98304, bf16, 4), (8, 33, 100000, f32, 2), (52, 10, 100000, f32, 2),
                                (4, 33, 100000, f32, 4)):
        waves, got = dba.dba_debug_stream_plan(B, k, V, fmt)[:2]
        assert (waves, got) == (8, tiles), (B, k, V, fmt, got)


def test_a_step_takes_one_launch_where_its_rows_have_the_waves_to_merge_with():
    """Up to 512 rows: always to k = 16, from there to k = 32 with eight waves a row, which rows of 32 KB and more have."""
    f32, f16 = dba.DBA_LOGP_F32, dba.DBA_LOGP_F16
    for B, k, V, fmt, launches in ((1, 1, 1, f32, 1), (512, 1, 100, f32, 1), (513, 1, 100, f32, 2), (32, 16, 100, f16, 1), (33, 16, 100, f32, 2),
                                   (1, 17, 8191, f32, 2), (1, 17, 8192, f32, 1), (30, 17, 16383, f16, 2), (30, 17, 16384, f16, 1),
                                   (16, 32, 2000, f32, 2), (16, 32, 32000, f32, 1), (17, 32, 32000, f32, 2), (1, 33, 32000, f32, 2)):
        assert dba.dba_debug_launches(B, k, V, fmt) == launches, (B, k, V, fmt)
    for bad in ((0, 1, 100, 0), (1, 65, 100, 0), (1, 5, 100, 3)):
        try:
            dba.dba_debug_launches(*bad)
        except dba.DbaError:
            continue
        raise AssertionError(bad)
