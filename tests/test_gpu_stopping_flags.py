"""-m gpu: the stopping flags that steps write to host memory themselves, once they have been asked for."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


def _decode(B, k, V, T, seed):
    import torch
    import paper_1804_06609_amd as dba
    from paper_1804_06609_amd.session import Session
    wl = si.make_small(seed, B, k, V, T, max_phrases=2, max_len=2, dup_prob=0.3)
    wl.eos_switch = T // 3
    lp = [torch.from_numpy(wl.logp(t)).cuda() for t in range(T)]

    def session(stream=None):
        return Session(B, k, V, T, wl.eos_id, wl.pad_id, *wl.csr(), stream=stream,
                       options={dba.DBA_OPT_NORMALIZE_FINISHED: 1, dba.DBA_OPT_PRUNE_THRESHOLD: 8.0})
    return lp, session


def _from_state(ses):
    """The flags by their definition: all live hypotheses completed, some completed."""
    import paper_1804_06609_amd as dba
    flags = ses.state()["flags"]
    live, done = (flags & dba.DBA_FLAG_DEAD) == 0, (flags & dba.DBA_FLAG_FINISHED) != 0
    stop_all = live.any(axis=1) & (done | ~live).all(axis=1)
    return (stop_all * dba.DBA_STOP_ALL | (live & done).any(axis=1) * dba.DBA_STOP_ANY).astype(np.uint8)


@pytest.mark.parametrize("B,k,V", [(1, 5, 300), (7, 4, 1000), (67, 6, 700), (9, 10, 9000), (3, 20, 5000), (5, 40, 2000), (260, 9, 600)])
def test_flags_after_every_step_and_now_and_then(B, k, V):
    T = 18
    lp, session = _decode(B, k, V, T, 9900 + V)
    always, sometimes, never = session(), session(), session()
    assert not always.finished().any()
    seen = 0
    for t in range(T):
        for ses in (always, sometimes, never):
            ses.step(lp[t])
        want = _from_state(never)
        seen |= int(np.bitwise_or.reduce(want))
        assert (always.finished() == want).all(), t
        assert (always.finished() == want).all(), t        # (asked twice)
        if t % 5 in (1, 2):
            assert (sometimes.finished() == want).all(), t
    assert seen == 3
    ends = [[np.asarray(a).tobytes() for a in ses.finalize()] for ses in (always, sometimes, never)]
    assert ends[0] == ends[1] == ends[2]
    for ses in (always, sometimes, never):
        ses.close()


def test_flags_with_steps_in_a_graph():
    """Steps recorded into a graph do not write to the host; the flags are those of what ran last, step or replay."""
    import torch
    T = 18
    lp, session = _decode(9, 6, 900, T, 9950)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ses, ref = session(stream), session(stream)
        for t in range(4):
            ses.step(lp[t])
            ref.step(lp[t])
            assert (ses.finished() == _from_state(ref)).all()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for t in range(4, 12):
                ses.step(lp[t])
        graph.replay()
        for t in range(4, 12):
            ref.step(lp[t])
        want = _from_state(ref)
        assert want.any() and (ses.finished() == want).all()
        for t in range(12, T):
            ses.step(lp[t])
            ref.step(lp[t])
            assert (ses.finished() == _from_state(ref)).all(), t
        ses.close()
        ref.close()


def test_a_ctx_that_goes_with_steps_under_way_leaves_its_block_alone():
    """A decode that is destroyed with steps under way on its stream, whose flags were asked for before, and another one on
    a stream of its own right behind it: between the other's step and its question the first one's steps write their words, which
    are not the other's to read.  (Were the block of host memory handed on with the ctx, the flags would be the first one's.)"""
    import torch
    import paper_1804_06609_amd as dba
    T = 12
    lp, session = _decode(40, 10, 9000, T, 9960)
    lp2, small = _decode(67, 3, 200, T, 9970)              # (as many sentences and more: its words would lie where the first one's are)
    ref = session()
    for t in range(T):
        ref.step(lp[t])
    theirs = ref.finished()
    ref.close()
    ref, want = small(), []
    for t in range(T):
        ref.step(lp2[t])
        want.append(ref.finished())
    ref.close()
    t0 = 2
    assert (theirs != want[t0][:40]).any()
    a = torch.randn(4096, 4096, device="cuda")
    a @ a
    torch.cuda.synchronize()
    side_by_side = 0
    for _ in range(6):
        first, second = torch.cuda.Stream(), torch.cuda.Stream()
        with torch.cuda.stream(second):
            small(second).close()                          # (no allocation below has to ask the driver, which may wait for the GPU)
        with torch.cuda.stream(first):
            ses = session(first)
            ses.finished()
        held = [small() for _ in range(32)]                # every block that is kept: the next one is the first decode's, if it comes back
        with torch.cuda.stream(first):
            for _ in range(20):                            # some milliseconds of work ahead of its steps
                a @ a
            for t in range(T):
                ses.step(lp[t])
        dba.dba_destroy(ses.ctx)
        ses.ctx = None                                     # (its buffers stay until its stream is through)
        assert not first.query()                           # nothing has waited for it
        with torch.cuda.stream(second):
            nxt = small(second)
            nxt.finished()
            for t in range(T):
                nxt.step(lp2[t])
                if t == t0:
                    second.synchronize()
                    side_by_side += not first.query()      # (not where the two streams share a hardware queue)
                    first.synchronize()
                assert (nxt.finished() == want[t]).all(), t
            nxt.close()
        for other in held:
            other.close()
    if not side_by_side:
        pytest.skip("the two streams never ran side by side")
