"""-m gpu: steps of one launch at the edges of the rule that chooses it, against two launches and the oracle."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


def _session(wl, waves, first=0):
    import torch
    import paper_1804_06609_amd as dba
    from paper_1804_06609_amd.session import Session
    ses = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, *wl.csr(), stream=torch.cuda.current_stream(),
                  options={dba.DBA_OPT_MERGE_WAVES: waves})
    return ses, dba.dba_debug_sentences_first(ses.ctx, first)


def _bytes(ses):
    return [a.tobytes() for a in ses.outputs()] + [a.tobytes() for a in ses.state().values()]


@pytest.mark.parametrize("B,k,V,fmts,one", [
    (88, 16, 512, ("f32",), True), (89, 16, 512, ("f32",), False), (88, 16, 511, ("f32",), False), (1408, 1, 700, ("f16",), True),
    (176, 8, 1031, ("bf16", "f32"), True), (127, 11, 2049, ("f32", "f16"), True), (93, 15, 3001, ("f32",), True), (64, 11, 41001, ("f32", "bf16"), True),
    (65, 11, 41001, ("f32", "bf16"), True), (89, 8, 41001, ("bf16", "f32"), True), (46, 16, 41001, ("f16", "f32"), True),
    (18, 28, 7168, ("f32", "f16"), True), (18, 28, 7169, ("f32",), None), (30, 17, 1000, ("f32",), True), (1, 17, 17, ("f32",), True), (5, 24, 1024, ("f32", "bf16"), True),
    (50, 28, 4096, ("f16", "f32"), True), (31, 17, 9001, ("bf16", "f32"), True), (50, 28, 4095, ("f16",), False), (25, 24, 16387, ("f32", "f16", "bf16"), True),
    (3, 8, 1024, ("f32", "bf16"), True), (3, 8, 1023, ("f32", "f16"), True), (41, 4, 2047, ("f32", "bf16"), True), (5, 2, 4093, ("f32",), True), (2, 1, 8190, ("bf16", "f32"), True),
    (7, 5, 700, ("f16",), True), (768, 1, 600, ("f32",), True), (769, 1, 600, ("f32",), True), (6, 8, 60, ("f32", "bf16"), True), (2, 7, 9, ("f32",), True)])
def test_one_launch_and_two(B, k, V, fmts, one):
    """Every step against the two launches, with the element types by turns (where they decide how many launches a step takes,
    the places that rows hand their keys over in are left empty by both), the step with its own scratch among them, and with the
    sentences' workgroups giving up at once.  one: whether steps of these element types take one launch (None: of such a ctx some
    might, these take two)."""
    import torch
    import paper_1804_06609_amd as dba
    tdt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
    code = {"f32": dba.DBA_LOGP_F32, "f16": dba.DBA_LOGP_F16, "bf16": dba.DBA_LOGP_BF16}
    wl = si.make_small(9700 + V + k, B, k, V, 6, max_phrases=4, max_len=3, dup_prob=0.3)
    wl.eos_switch = 4
    dev = [torch.from_numpy(wl.logp(t)).cuda().to(tdt[fmts[t // 2 % len(fmts)]]) for t in range(wl.T)]
    two, is_one = _session(wl, 8)
    assert not is_one
    others = [_session(wl, 0, first) for first in (0, 1, 2)]
    assert all(o[1] == (one is not False) for o in others)
    assert any(dba.dba_debug_launches(B, k, V, code[f]) == 1 for f in fmts) == (one is True)
    for t in range(wl.T):
        two.step(dev[t])
        want = _bytes(two)
        for i, (ses, _) in enumerate(others):
            ses.step(dev[t], noalloc=(t + i) % 3 == 2)
            assert _bytes(ses) == want, (t, i)
    want = [np.asarray(a).tobytes() for a in two.finalize()]
    for ses, _ in others:
        assert [np.asarray(a).tobytes() for a in ses.finalize()] == want
        ses.close()
    two.close()


@pytest.mark.parametrize("k,fmt", [(13, None), (16, None), (17, None), (24, None), (28, None), (32, None), (36, None), (48, None), (64, "bf16"), (20, "f16")])
def test_floors_of_rows_of_one_tile_to_six(k, fmt):
    """The floor of a row comes from as many lists as it has tiles: sorted pools of their best, or all of them merged."""
    import harness
    tile = 1024 if fmt is None else 2048
    for tiles in (1, 2, 3, 4, 6):
        wl = si.make_small(9800 + tiles, 2, k, tiles * tile - 3, 3, max_phrases=2, max_len=2, dup_prob=0.3)
        wl.eos_switch = 2
        harness.run_parity(wl, logp_format=fmt)


@pytest.mark.parametrize("B,k,V,fmt", [(3, 8, 1024, None), (2, 8, 1021, "f16"), (4, 5, 1000, None), (3, 4, 4096, "bf16"), (3, 2, 4095, None), (2, 1, 4001, None), (5, 3, 40, "bf16"), (3, 8, 11, None)])
@pytest.mark.parametrize("shape", ["zipf", "rising", "equal"])
def test_a_sentence_in_one_workgroup(B, k, V, fmt, shape):
    """Rows of up to four tiles, one wave each, against the oracle: rising rows and equal elements fill a wave's room for groups and for keys."""
    import harness
    import paper_1804_06609_amd as dba
    assert dba.dba_debug_per_sentence(B, k, V, {None: dba.DBA_LOGP_F32, "f16": dba.DBA_LOGP_F16, "bf16": dba.DBA_LOGP_BF16}[fmt])
    base = si.make_small(9850 + V, B, k, V, 8, max_phrases=4, max_len=3, dup_prob=0.3)
    if shape == "zipf":
        wl = base
    else:
        class Shaped(si.Workload):
            def logp(self, t, out=None):
                lp = super().logp(t, out=out)
                if shape == "rising":
                    lp.sort(axis=-1)
                else:
                    lp.fill(np.float32(-3.0))
                return lp
        wl = Shaped(B=B, k=k, V=V, T=8, seed=base.seed, constraints=base.constraints)
    wl.eos_switch = 5
    harness.run_parity(wl, logp_format=fmt)
    harness.run_parity(wl, logp_format=fmt, normalize=True, prune=20.0, track=True)
