"""Which steps take one launch, at the edges of the rule (worked out on the host, no GPU)."""
import paper_1804_06609_amd as dba


def test_steps_beyond_two_rows_a_compute_unit():
    """k <= 16, up to 1408 rows of four waves or 704 of eight; not for vocabularies below 512."""
    f32, bf16 = dba.DBA_LOGP_F32, dba.DBA_LOGP_BF16
    for B, k, V, fmt, launches in ((88, 16, 512, f32, 1), (88, 16, 511, f32, 2), (89, 16, 512, f32, 2), (1408, 1, 32000, bf16, 1), (1409, 1, 32000, bf16, 2),
                                   (31, 17, 32000, f32, 2), (64, 11, 40959, f32, 1), (64, 11, 40960, f32, 1), (65, 11, 40960, f32, 2),
                                   (65, 11, 40960, bf16, 1), (513, 1, 100000, f32, 1), (705, 1, 100000, f32, 2)):
        assert dba.dba_debug_launches(B, k, V, fmt) == launches, (B, k, V, fmt)


def test_short_rows_of_beams_of_17_to_28():
    f32, f16 = dba.DBA_LOGP_F32, dba.DBA_LOGP_F16
    for B, k, V, fmt, launches, waves in ((1, 17, 17, f32, 1, 8), (18, 28, 7168, f32, 1, 8), (18, 28, 7169, f32, 2, 4), (18, 29, 2000, f32, 2, 4), (19, 28, 2000, f32, 2, 4),
                                          (18, 28, 2000, f16, 2, 4), (32, 16, 2000, f32, 1, 4)):
        assert dba.dba_debug_launches(B, k, V, fmt) == launches, (B, k, V, fmt)
        assert dba.dba_debug_stream_plan(B, k, V, fmt)[0] == waves, (B, k, V, fmt)


def test_wide_beams_with_16_bit_rows_beyond_two_rows_a_compute_unit():
    f32, f16, bf16 = dba.DBA_LOGP_F32, dba.DBA_LOGP_F16, dba.DBA_LOGP_BF16
    for B, k, V, fmt, launches in ((50, 28, 4096, f16, 1), (50, 28, 4096, f32, 2), (50, 28, 4095, f16, 2), (50, 29, 4096, f16, 2), (51, 28, 4096, bf16, 2),
                                   (31, 17, 81919, bf16, 1), (31, 17, 81920, bf16, 2), (88, 16, 4096, bf16, 1)):
        assert dba.dba_debug_launches(B, k, V, fmt) == launches, (B, k, V, fmt)


def test_a_workgroup_per_sentence_for_short_rows_and_narrow_beams():
    """Eight tiles of 4 KB in all, four a row, 768 sentences."""
    f32, f16, bf16 = dba.DBA_LOGP_F32, dba.DBA_LOGP_F16, dba.DBA_LOGP_BF16
    for B, k, V, fmt, per_sentence in ((1, 5, 1000, f32, 1), (3, 8, 1024, f32, 1), (3, 8, 1025, f32, 0), (3, 8, 2048, bf16, 1), (3, 8, 2049, bf16, 0), (3, 9, 60, f32, 0),
                                       (3, 4, 2048, f16, 1), (3, 4, 2048, f32, 1), (3, 4, 2049, f32, 0), (3, 5, 1025, f32, 0), (3, 3, 2730, f32, 0), (3, 3, 2048, f32, 1),
                                       (2, 2, 4096, f32, 1), (2, 2, 4097, f32, 0), (2, 1, 4096, f32, 1), (2, 1, 4097, f32, 0), (2, 1, 8192, bf16, 1), (2, 1, 8193, bf16, 0),
                                       (768, 1, 600, f32, 1), (769, 1, 600, f32, 0), (176, 8, 600, f32, 1), (177, 8, 600, f32, 0), (512, 1, 300, f32, 1), (513, 1, 300, f32, 0)):
        assert dba.dba_debug_per_sentence(B, k, V, fmt) == bool(per_sentence), (B, k, V, fmt)
        assert not per_sentence or dba.dba_debug_launches(B, k, V, fmt) == 1


def test_no_lds_is_left_unused_beside_a_row_of_a_single_launch():
    for B, k, V, fmt in ((96, 12, 32003, dba.DBA_LOGP_BF16), (64, 20, 32000, dba.DBA_LOGP_F16), (1408, 1, 32000, dba.DBA_LOGP_F32), (80, 16, 32000, dba.DBA_LOGP_F32)):
        assert dba.dba_debug_launches(B, k, V, fmt) == 1
        assert dba.dba_debug_stream_plan(B, k, V, fmt)[2] == dba.dba_debug_stream_plan(1, 10, 1000, fmt)[2], (B, k, V, fmt)
    assert dba.dba_debug_stream_plan(64, 20, 32000, dba.DBA_LOGP_F32)[2] > dba.dba_debug_stream_plan(1, 10, 1000)[2]


def test_a_workspace_for_the_largest_job_serves_every_smaller_one():
    """Steps of one launch have places of their own, 1024 bytes a row, in the workspace of every shape up to 1408 rows, and
    larger ones have no less: the size grows with the batch, the beam and the steps and goes by nothing else."""
    def size(B, k, N=100, V=32000):
        return dba.dba_workspace_bytes(B, k, V, N, 0)
    for larger, smaller in (((72, 20), (70, 20)), ((89, 16), (88, 16)), ((50, 29), (50, 28)), ((105, 20), (71, 20))):
        assert size(*larger) > size(*smaller), (larger, smaller)
    for k in list(range(1, 65)):
        for B in (1, 8, 15, 16, 17, 22, 25, 44, 64, 88, 89, 511, 512, 513, 703, 704, 1407, 1408, 1409, 2000, 65534):
            here = size(B, k)
            assert size(B + 1, k) >= here and size(B, k, 101) >= here and (k == 64 or size(B, k + 1) >= here), (B, k)
            assert len({size(B, k, V=V) for V in (64, 511, 512, 4095, 4096, 32000, 1 << 20)}) == 1, (B, k)
    for B, k, rows in ((1, 1, 1), (88, 16, 1408), (89, 16, 1408), (1000, 64, 1408)):
        without = 2 * 32 * B * k + 2112 * B + 1024 * B * k   # the two beams, the constraints, the lists and keys of two launches
        assert 1024 * rows <= size(B, k, 1) - without <= 1024 * rows + 8 * B * k + (4 * 4 + 33) * B + 20 * 256, (B, k)
