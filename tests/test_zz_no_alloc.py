"""-m gpu: dba_step_noalloc (the step with the library's own scratch, for callers that cannot allocate)
against dba_step_fmt, through the C ABI: same outputs, same state, same end of decoding, bit for bit.
Steps of two launches share the GPU's scratch array: decodes in a row, each smaller than the one before, so that it runs
over what that left behind, with 16-bit log-probs and with steps through the workspace in between.  Steps of one launch
hand over through the workspace in both forms.  Sizes beyond the array are refused."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


def _decode_both_ways(torch, wl, fmt=None, mix=False):
    from paper_1804_06609_amd.session import Session
    toks, poff, soff = wl.csr()
    plain = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, toks, poff, soff)
    own = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, toks, poff, soff)
    tdt = {None: torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[fmt]
    for t in range(wl.T):
        lp = wl.logp(t)
        if fmt is None:
            dev = torch.from_numpy(lp).cuda()
        else:
            dev = torch.from_numpy(si.narrow16(lp, fmt).view(np.int16)).cuda().view(tdt)
        plain.step(dev)
        own.step(dev, noalloc=not (mix and t % 3 == 1))      # mix: every third step through the workspace
        for a, b, name in zip(plain.outputs(), own.outputs(), ("token", "backptr", "score", "flags")):
            assert a.tobytes() == b.tobytes(), (name, t)
        sa, sb = plain.state(), own.state()
        for name in sa:
            assert sa[name].tobytes() == sb[name].tobytes(), (name, t)
        assert plain.finished().tobytes() == own.finished().tobytes(), t
    for a, b in zip(plain.finalize(), own.finalize()):
        assert a.tobytes() == b.tobytes()
    plain.close()
    own.close()


def test_noalloc_step_matches_the_step_with_workspace_scratch():
    import torch
    assert torch.cuda.is_available()
    first = si.make_small(9801, 6, 33, 4099, 12, max_phrases=5, max_len=3, dup_prob=0.3)
    first.eos_switch = 6
    _decode_both_ways(torch, first)
    second = si.make_small(9802, 2, 5, 257, 9, max_phrases=3, max_len=2, dup_prob=0.3)   # smaller, right after
    second.eos_switch = 4
    _decode_both_ways(torch, second)
    third = si.make_small(9803, 3, 13, 1023, 8, max_phrases=4, max_len=3, dup_prob=0.3)
    third.eos_switch = 4
    _decode_both_ways(torch, third, fmt="bf16", mix=True)


def test_noalloc_steps_of_two_launches_over_what_others_left_behind():
    import torch
    import paper_1804_06609_amd as dba
    for seed, B, k, V, T, fmt, mix in ((9805, 9, 64, 3001, 9, None, False), (9806, 2, 33, 257, 9, None, False), (9807, 3, 40, 1023, 8, "bf16", True),
                                       (9808, 2, 20, 2000, 8, "f16", True), (9809, 1, 36, 999, 8, "f16", False)):
        assert dba.dba_debug_launches(B, k, V, {None: dba.DBA_LOGP_F32, "f16": dba.DBA_LOGP_F16, "bf16": dba.DBA_LOGP_BF16}[fmt]) == 2
        wl = si.make_small(seed, B, k, V, T, max_phrases=5, max_len=3, dup_prob=0.3)
        wl.eos_switch = T // 2
        _decode_both_ways(torch, wl, fmt=fmt, mix=mix)


def test_a_graph_of_noalloc_steps_of_two_launches():
    """Two kernels a step, through the library's scratch, recorded once and replayed with other decodes in between."""
    import torch
    from paper_1804_06609_amd.session import Session
    wl = si.make_small(9810, 5, 34, 1500, 6, max_phrases=4, max_len=3, dup_prob=0.3)
    wl.eos_switch = 3
    dev = [torch.from_numpy(wl.logp(t)).cuda() for t in range(wl.T)]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        eager, ses = (Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, *wl.csr(), stream=stream) for _ in range(2))
        for s, noalloc in ((eager, False), (ses, True)):
            s.step(dev[0], noalloc=noalloc)
        start = ses.workspace.clone()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        graph.capture_begin()
        for t in range(1, wl.T):
            ses.step(dev[t], noalloc=True)
        graph.capture_end()
        for t in range(1, wl.T):
            eager.step(dev[t])
        want = [a.tobytes() for a in eager.outputs()] + [np.asarray(a).tobytes() for a in eager.finalize()]
        for _ in range(3):
            ses.workspace.copy_(start)
            graph.replay()
            assert [a.tobytes() for a in ses.outputs()] + [np.asarray(a).tobytes() for a in ses.finalize()] == want
            other = Session(wl.B, wl.k, wl.V, 2, wl.eos_id, wl.pad_id, *wl.csr(), stream=stream)
            other.step(dev[3], noalloc=True)
            other.close()
        ses.close()
        eager.close()


def test_noalloc_step_at_the_headline_shape():
    import torch
    wl = si.make_config(4, T=6)
    _decode_both_ways(torch, wl)


def test_noalloc_step_refuses_more_rows_than_its_scratch_holds():
    import torch
    import paper_1804_06609_amd as dba
    from paper_1804_06609_amd.session import Session
    B, k, V = 129, 64, 64                                   # 8256 beam rows > DBA_NOALLOC_MAX_ROWS
    assert B * k > dba.DBA_NOALLOC_MAX_ROWS
    wl = si.make_small(9804, B, k, V, 2, max_phrases=1, max_len=1)
    toks, poff, soff = wl.csr()
    ses = Session(B, k, V, 2, wl.eos_id, wl.pad_id, toks, poff, soff)
    dev = torch.from_numpy(wl.logp(0)).cuda()
    with pytest.raises(dba.DbaError, match="DBA_NOALLOC_MAX_ROWS") as ei:
        ses.step(dev, noalloc=True)
    assert ei.value.code == dba.DBA_EINVAL and dba.dba_steps_done(ses.ctx) == 0
    ses.step(dev)                                           # the ordinary step still works
    assert dba.dba_steps_done(ses.ctx) == 1
    ses.close()


def test_noalloc_step_writes_only_inside_its_buffers():
    """The guard-band check of tests/test_gpu_robustness.py with every step taken through dba_step_noalloc."""
    from test_gpu_robustness import guarded_decode
    guarded_decode("noalloc")
    guarded_decode("noalloc_two_launches")
