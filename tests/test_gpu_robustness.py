"""-m gpu: checks of the device side that compare the HIP path with itself or with guard patterns
rather than with the oracle: the same decode twice gives the same bytes, and a decode writes nowhere
outside the buffers it was given."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu


def _decode(torch, wl, options=None, fmt=None):
    """All bytes a decode leaves behind: every step's outputs, state and stopping bits, and the
    end of decoding (which walks the recorded history)."""
    from paper_1804_06609_amd.session import Session
    toks, poff, soff = wl.csr()
    ses = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, toks, poff, soff, options=options)
    trace = []
    for t in range(wl.T):
        lp = wl.logp(t)
        if fmt is None:
            dev = torch.from_numpy(lp).cuda()
        else:
            dev = torch.from_numpy(si.narrow16(lp, fmt).view(np.int16)).cuda().view(torch.bfloat16)
        ses.step(dev)
        trace.extend(a.tobytes() for a in ses.outputs())
        st = ses.state()
        trace.extend(st[name].tobytes() for name in sorted(st))
        trace.append(ses.finished().tobytes())
    trace.extend(np.asarray(a).tobytes() for a in ses.finalize())
    ses.close()
    return trace


@pytest.mark.parametrize("paper_setup", [False, True])
def test_the_same_decode_twice_gives_the_same_bytes(paper_setup):
    """Config-3 shapes (16 sentences, k = 10, V = 32000; boosted constraint tokens, so phrases start
    and break), 40 steps with end-of-sentence from step 25, bare and with the options of Sec. 4 on."""
    import torch
    from paper_1804_06609_amd import DBA_OPT_NORMALIZE_FINISHED, DBA_OPT_PRUNE_THRESHOLD, DBA_OPT_TRACK_COMPLETED
    wl = si.make_config(3, T=40)
    wl.eos_switch = 25
    opts = {DBA_OPT_NORMALIZE_FINISHED: 1, DBA_OPT_PRUNE_THRESHOLD: 20.0, DBA_OPT_TRACK_COMPLETED: 1} if paper_setup else None
    first = _decode(torch, wl, opts)
    second = _decode(torch, wl, opts)
    assert first == second


def test_the_same_bf16_decode_twice_gives_the_same_bytes():
    import torch
    wl = si.make_small(9951, 5, 20, 12345, 14, max_phrases=5, max_len=3, dup_prob=0.3)
    wl.eos_switch = 7
    assert _decode(torch, wl, fmt="bf16") == _decode(torch, wl, fmt="bf16")


GUARD = 1 << 16           # bytes of guard band on each side
PATTERN = 0xA5


class _Guarded:
    """A device buffer of `nbytes` with a guard band before and after it, filled with a pattern."""

    def __init__(self, torch, nbytes, align=256):
        self.torch = torch
        self.raw = torch.full((nbytes + 2 * GUARD + align,), PATTERN, dtype=torch.uint8, device="cuda")
        start = (self.raw.data_ptr() + GUARD + align - 1) // align * align
        self.off = start - self.raw.data_ptr()
        self.ptr, self.nbytes = start, nbytes

    def body(self):
        return self.raw[self.off:self.off + self.nbytes]

    def guards_intact(self):
        lo = self.raw[:self.off]
        hi = self.raw[self.off + self.nbytes:]
        return bool((lo == PATTERN).all().item()) and bool((hi == PATTERN).all().item())


@pytest.mark.parametrize("case", ["k64_c64", "odd_v", "bf16_odd_v"])
def test_a_decode_writes_only_inside_its_buffers(case):
    guarded_decode(case)


def guarded_decode(case):
    """Workspace and the four output arrays sit between guard bands; after decodes with the widest beam
    and the most constraint tokens (k = 64, 64 tokens), with rows of odd length (unaligned rows, ragged
    tiles) in fp32 and bf16, bare and with the options of Sec. 4 on, every guard byte is
    as it was, and the outputs agree with an unguarded run."""
    import torch
    import paper_1804_06609_amd as dba
    if case == "k64_c64":
        B, k, V, T = 3, 64, 5003, 8
        cons = si.fixed_total_constraints(61, B, V, 64, max_len=4)
        wl = si.Workload(B=B, k=k, V=V, T=T, seed=61, constraints=cons,
                         boost_tokens=[[w for p in s for w in p] for s in cons], boost_prob=0.3, boost_value=6.0)
    elif case == "noalloc_two_launches":                   # (the library's own scratch passes the keys on)
        wl = si.make_small(9962, 4, 35, 4099, 10, max_phrases=5, max_len=3, dup_prob=0.3)
        assert dba.dba_debug_launches(wl.B, wl.k, wl.V) == 2
    else:
        wl = si.make_small(9961, 4, 13, 4099, 10, max_phrases=5, max_len=3, dup_prob=0.3)
    wl.eos_switch = wl.T // 2
    fmt = "bf16" if case == "bf16_odd_v" else None
    want = _decode(torch, wl, fmt=fmt)
    toks, poff, soff = wl.csr()
    B, k, V, T = wl.B, wl.k, wl.V, wl.T
    stream = torch.cuda.current_stream()
    for options in ({}, {dba.DBA_OPT_NORMALIZE_FINISHED: 1, dba.DBA_OPT_PRUNE_THRESHOLD: 20.0,
                         dba.DBA_OPT_TRACK_COMPLETED: 1}):
        ws = _Guarded(torch, dba.dba_workspace_bytes(B, k, V, T, dba.DBA_MAX_CONS_TOKENS))
        o_tok, o_bp, o_sc = (_Guarded(torch, B * k * 4, align=4) for _ in range(3))
        o_fl = _Guarded(torch, B * k, align=1)
        ctx = dba.dba_init(B, k, V, T, wl.eos_id, wl.pad_id, toks, poff, soff, ws.ptr, ws.nbytes, stream.cuda_stream)
        for opt, val in options.items():
            dba.dba_set_option(ctx, opt, val)
        got = []
        for t in range(T):
            lp = wl.logp(t)
            if fmt is None:
                dev = torch.from_numpy(lp).cuda()
                code = dba.DBA_LOGP_F32
            else:
                dev = torch.from_numpy(si.narrow16(lp, fmt).view(np.int16)).cuda().view(torch.bfloat16)
                code = dba.DBA_LOGP_BF16
            step = dba.dba_step_noalloc if case.startswith("noalloc") else dba.dba_step_fmt
            step(ctx, dev.data_ptr(), code, o_tok.ptr, o_bp.ptr, o_sc.ptr, o_fl.ptr)
            torch.cuda.synchronize()
            got.append(o_tok.body().cpu().numpy().tobytes())
            got.append(o_bp.body().cpu().numpy().tobytes())
            got.append(o_sc.body().cpu().numpy().tobytes())
            got.append(o_fl.body().cpu().numpy().tobytes())
        fin = (np.empty((B, T), np.int32), np.empty(B, np.int32), np.empty(B, np.float32), np.empty(B, np.int32))
        dba.dba_finalize(ctx, *fin)
        dba.dba_destroy(ctx)
        for g in (ws, o_tok, o_bp, o_sc, o_fl):
            assert g.guards_intact(), (case, options)
        if not options:
            # the unguarded run's trace holds, per step, the four outputs first
            per_step = len(want[:-4]) // T
            for t in range(T):
                assert got[4 * t:4 * t + 4] == want[per_step * t:per_step * t + 4], (case, t)
            assert [a.tobytes() for a in fin] == want[-4:]


@pytest.mark.parametrize("N", [40, 1000, 1092, 1093, 1400])
def test_the_end_of_a_decode_is_the_same_however_long_its_token_rows_are(N):
    """dba_finalize brings small results over in one copy and long token rows on their own (from 512 KB on: 120
    sentences of 1093 tokens): the same decode with room for 9 tokens and for N, into ordinary and into pinned
    memory, with nothing written beside the four arrays."""
    import torch
    import paper_1804_06609_amd as dba
    B, k, V, T = 120, 4, 60, 9
    wl = si.make_small(8800, B, k, V, T, max_phrases=2, max_len=2)
    wl.eos_switch = 4
    toks, poff, soff = wl.csr()
    stream = torch.cuda.current_stream().cuda_stream

    def decode(n, pinned):
        ws = torch.empty(dba.dba_workspace_bytes(B, k, V, n, 64) + 256, dtype=torch.uint8, device="cuda")
        base = (ws.data_ptr() + 255) // 256 * 256
        ctx = dba.dba_init(B, k, V, n, wl.eos_id, wl.pad_id, toks, poff, soff, base, ws.numel() - 256, stream)
        keep = []
        for t in range(T):
            keep.append(torch.from_numpy(wl.logp(t)).cuda())
            dba.dba_step(ctx, keep[-1].data_ptr())
        whole = [torch.full((64 + m + 64,), -77, dtype=torch.int32, pin_memory=pinned).numpy() for m in (B * n, B, B, B)]
        tokens, length, score, status = (w[64:-64] for w in whole)
        dba.dba_finalize(ctx, tokens, length, score.view(np.float32), status)
        dba.dba_destroy(ctx)
        assert all((w[:64] == -77).all() and (w[-64:] == -77).all() for w in whole), (n, pinned)
        return tokens.reshape(B, n), length.tobytes() + score.tobytes() + status.tobytes()

    want = decode(T, False)
    for pinned in (False, True):
        got = decode(N, pinned)
        assert (got[0][:, :T] == want[0]).all() and (got[0][:, T:] == wl.pad_id).all() and got[1] == want[1], (N, pinned)


def test_a_decode_replayed_from_a_hip_graph_matches_eager_launches():
    """A step enqueues one kernel (here) or two and nothing else (no allocation, no memset, no copy), so a decode can
    be recorded into a HIP graph by a caller who wants to.  Steps 1..T-1 of a decode are recorded once and replayed three times, each
    time from the device state after step 0 (the workspace is copied back, with eager work and
    synchronisations in between); every replay must leave the beam, the state and the end of
    decoding of the eager decode."""
    import torch
    from paper_1804_06609_amd.session import Session
    wl = si.make_config(3, T=24)
    wl.eos_switch = 14
    toks, poff, soff = wl.csr()
    dev = [torch.from_numpy(wl.logp(t)).cuda() for t in range(wl.T)]
    eager = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, toks, poff, soff)
    for t in range(wl.T):
        eager.step(dev[t])
    want_out = [a.tobytes() for a in eager.outputs()]
    want_state = {n: a.tobytes() for n, a in eager.state().items()}
    want_fin = [np.asarray(a).tobytes() for a in eager.finalize()]
    want_stop = eager.finished().tobytes()
    eager.close()

    side = torch.cuda.Stream()
    ses = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, toks, poff, soff, stream=side)
    with torch.cuda.stream(side):
        ses.step(dev[0])
    torch.cuda.synchronize()
    after_step0 = ses.workspace.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for t in range(1, wl.T):
            ses.step(dev[t])
    torch.cuda.synchronize()
    for replay in range(3):
        ses.workspace.copy_(after_step0)                  # eager work between the replays
        for o in (ses.out_token, ses.out_backptr, ses.out_score, ses.out_flags):
            o.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        torch.cuda.synchronize()
        assert [a.tobytes() for a in ses.outputs()] == want_out, replay
        assert {n: a.tobytes() for n, a in ses.state().items()} == want_state, replay
        assert ses.finished().tobytes() == want_stop, replay
        assert [np.asarray(a).tobytes() for a in ses.finalize()] == want_fin, replay
    ses.close()


def test_ctxs_that_come_and_go_without_waiting():
    """dba_init does not wait for the GPU: ctxs that are destroyed before it has read their constraints, on two
    streams and from two threads, do not disturb those that follow, which get their host memory."""
    import threading
    import torch
    from paper_1804_06609_amd.session import Session
    jobs = []
    for i, (B, k, V) in enumerate([(3, 5, 300), (40, 3, 200), (300, 2, 60), (2, 20, 500)]):
        wl = si.make_small(8900 + i, B, k, V, 6, max_phrases=4, max_len=3, dup_prob=0.3)
        wl.eos_switch = 3
        dev = [torch.from_numpy(wl.logp(t)).cuda() for t in range(wl.T)]
        ses = Session(B, k, V, wl.T, wl.eos_id, wl.pad_id, *wl.csr())
        for t in range(wl.T):
            ses.step(dev[t])
        want = [np.asarray(a).tobytes() for a in ses.finalize()] + [ses.finished().tobytes()]
        ses.close()
        jobs.append((wl, dev, want))
    torch.cuda.synchronize()
    wrong = []

    def work(first):
        import paper_1804_06609_amd as dba
        stream = torch.cuda.Stream()
        for rep in range(12):
            wl, dev, want = jobs[(first + rep) % len(jobs)]
            other = jobs[(first + rep + 1) % len(jobs)][0]
            keep = []                                      # (device memory outlives the ctxs below: theirs may still be under way)
            with torch.cuda.stream(stream):
                for _ in range(3):
                    gone = Session(other.B, other.k, other.V, other.T, other.eos_id, other.pad_id, *other.csr(), stream=stream)
                    dba.dba_destroy(gone.ctx)
                    gone.ctx = None
                    keep.append(gone)
                ses = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, *wl.csr(), stream=stream)
                for t in range(wl.T):
                    ses.step(dev[t])
                    ses.finished()
                got = [np.asarray(a).tobytes() for a in ses.finalize()] + [ses.finished().tobytes()]
                ses.close()
            if got != want:
                wrong.append((first, rep))
            stream.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not wrong


@pytest.mark.parametrize("B,N", [(4000, 5), (4100, 5), (500, 400)])
def test_batches_with_and_without_a_block_of_host_memory(B, N):
    """Constraints, stopping flags and results pass through host memory that kernels use themselves, up to a megabyte;
    beyond, and tokens of more than 512 KB, through copies."""
    import harness
    wl = si.make_small(8950, B, 2, 40, 5, max_phrases=2, max_len=2, dup_prob=0.3)
    wl.T = N
    wl.eos_switch = 2
    harness.run_parity(wl, T=5, oracle_sentences=[0, 1, 63, 64, B // 2, B - 1])


def _one_launch_decode(wl, dev, stream, first, waves=0):
    import paper_1804_06609_amd as dba
    from paper_1804_06609_amd.session import Session
    ses = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, *wl.csr(), stream=stream,
                  options={dba.DBA_OPT_MERGE_WAVES: waves})
    return ses, dba.dba_debug_sentences_first(ses.ctx, first)


@pytest.mark.parametrize("B,k,V,fmt,one", [
    (256, 1, 300, None, True), (512, 1, 300, None, True), (513, 1, 300, None, False), (34, 15, 9000, None, True), (16, 32, 2100, "bf16", True), (17, 31, 700, None, False), (85, 3, 1200, "f16", True), (32, 8, 1000, None, True), (28, 9, 4100, "bf16", True),
    (256, 1, 4097, None, True), (512, 1, 4097, None, True), (85, 3, 6200, "f16", True), (32, 8, 1025, None, True), (1, 5, 1025, None, True),
    (23, 11, 8200, None, True), (21, 12, 2000, None, True), (16, 16, 16500, "f16", True), (15, 17, 700, None, True), (8, 32, 8300, None, True),
    (7, 33, 600, None, False), (3, 20, 33001, None, True), (1, 5, 1000, None, True), (2, 32, 40000, "bf16", True)])
def test_steps_of_one_launch(B, k, V, fmt, one):
    """Small steps take one launch, whose sentences wait for their rows; or, if the rows are slow to start (forced here by
    numbering the sentences first), a row takes the sentence on.  Both against the two launches, every step; the
    formats and the step with its own scratch mixed."""
    import torch
    wl = si.make_small(9100 + V, B, k, V, 6, max_phrases=4, max_len=3, dup_prob=0.3)
    wl.eos_switch = 3
    tdt = {None: torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[fmt]
    dev = [torch.from_numpy(wl.logp(t)).cuda().to(tdt) for t in range(wl.T)]
    stream = torch.cuda.current_stream()
    two, is_one = _one_launch_decode(wl, dev, stream, False, waves=8)
    assert not is_one
    others = [_one_launch_decode(wl, dev, stream, first) for first in (False, True)]
    assert all(o[1] == one for o in others)
    for t in range(wl.T):
        two.step(dev[t])
        want = [a.tobytes() for a in two.outputs()] + [a.tobytes() for a in two.state().values()]
        for i, (ses, _) in enumerate(others):
            ses.step(dev[t], noalloc=(t + i) % 3 == 2)
            got = [a.tobytes() for a in ses.outputs()] + [a.tobytes() for a in ses.state().values()]
            assert got == want, (t, i)
    want = [np.asarray(a).tobytes() for a in two.finalize()]
    for ses, _ in others:
        assert [np.asarray(a).tobytes() for a in ses.finalize()] == want
        ses.close()
    two.close()


def test_steps_of_one_launch_side_by_side():
    """Six decodes on six streams, interleaved, two of them with the sentences first, beside a seventh that keeps
    the GPU busy with many rows: the results of each alone."""
    import torch
    from paper_1804_06609_amd.session import Session
    jobs = []
    for i, (B, k, V) in enumerate([(16, 10, 8200), (50, 5, 900), (1, 20, 33000), (8, 32, 3000), (85, 3, 500), (24, 7, 9001)]):
        wl = si.make_small(9200 + i, B, k, V, 8, max_phrases=4, max_len=3, dup_prob=0.3)
        wl.eos_switch = 5
        jobs.append((wl, [torch.from_numpy(wl.logp(t)).cuda() for t in range(wl.T)]))
    big = si.make_small(9300, 200, 20, 2000, 40, max_phrases=4, max_len=3)
    big_lp = torch.from_numpy(big.logp(0)).cuda()
    alone = []
    for wl, dev in jobs:
        ses, _ = _one_launch_decode(wl, dev, torch.cuda.current_stream(), False)
        for t in range(wl.T):
            ses.step(dev[t])
        alone.append([a.tobytes() for a in ses.outputs()] + [np.asarray(a).tobytes() for a in ses.finalize()])
        ses.close()
    torch.cuda.synchronize()
    for rep in range(4):
        streams = [torch.cuda.Stream() for _ in range(7)]
        busy = Session(big.B, big.k, big.V, big.T, big.eos_id, big.pad_id, *big.csr(), stream=streams[6])
        running = [_one_launch_decode(wl, dev, s, i % 3 == 2)[0] for i, ((wl, dev), s) in enumerate(zip(jobs, streams))]
        for t in range(8):
            for _ in range(5):
                busy.step(big_lp)
            for ses, (wl, dev) in zip(running, jobs):
                ses.step(dev[t])
        for ses, want in zip(running, alone):
            assert [a.tobytes() for a in ses.outputs()] + [np.asarray(a).tobytes() for a in ses.finalize()] == want, rep
            ses.close()
        busy.close()


@pytest.mark.parametrize("first", [1, 2])
@pytest.mark.parametrize("B,k,V,fmt", [(8, 9, 200, None), (40, 12, 500, None), (16, 10, 32000, None), (20, 24, 3000, None),
                                       (2, 32, 40000, "bf16"), (26, 10, 33000, "f16"), (3, 20, 300001, None), (769, 1, 700, None), (512, 1, 4097, None)])
def test_sentences_that_give_up_waiting(B, k, V, fmt, first):
    """A sentence's workgroup that looks for the rows' keys once and gives up (a limit of 0 looks set by the host; in
    earnest it runs out where rows take unusually long): the row that ends last takes the sentence on, or the
    workgroup goes on if all have ended.  Nothing is lost or left behind: the results of two launches, at every step
    and with the ordinary limit after."""
    import torch
    wl = si.make_small(9400 + V, B, k, V, 12, max_phrases=4, max_len=3, dup_prob=0.3)
    wl.eos_switch = 7
    tdt = {None: torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[fmt]
    dev = [torch.from_numpy(wl.logp(t)).cuda().to(tdt) for t in range(wl.T)]
    stream = torch.cuda.current_stream()
    import paper_1804_06609_amd as dba
    two, _ = _one_launch_decode(wl, dev, stream, 0, waves=8)
    ses, one = _one_launch_decode(wl, dev, stream, first)
    code = {None: dba.DBA_LOGP_F32, "f16": dba.DBA_LOGP_F16, "bf16": dba.DBA_LOGP_BF16}[fmt]
    assert one and dba.dba_debug_launches(B, k, V, code) == 1 and not dba.dba_debug_per_sentence(B, k, V, code)
    for t in range(wl.T):
        dba.dba_debug_sentences_first(ses.ctx, first if t % 4 != 3 else 0)
        two.step(dev[t])
        ses.step(dev[t])
        want = [a.tobytes() for a in two.outputs()] + [a.tobytes() for a in two.state().values()]
        assert [a.tobytes() for a in ses.outputs()] + [a.tobytes() for a in ses.state().values()] == want, t
    assert [np.asarray(a).tobytes() for a in ses.finalize()] == [np.asarray(a).tobytes() for a in two.finalize()]
    ses.close()
    two.close()


@pytest.mark.parametrize("B,k,V", [(3, 5, 300), (60, 20, 500), (300, 2, 60)])
def test_a_workspace_is_free_once_its_ctx_is_destroyed(B, k, V):
    """dba_init returns before the GPU has come to it; a ctx that is destroyed without a step gives its workspace back
    only when nothing of dba_init can write to it any more, on whatever stream it is used next."""
    import torch
    import paper_1804_06609_amd as dba
    wl = si.make_small(9500 + B, B, k, V, 4, max_phrases=3, max_len=3)
    nbytes = dba.dba_workspace_bytes(B, k, V, 4, dba.DBA_MAX_CONS_TOKENS)
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    a = torch.randn(4096, 4096, device="cuda")
    a @ a
    torch.cuda.synchronize()
    for option in (None, 99):
        with torch.cuda.stream(stream):
            for _ in range(20):                            # some milliseconds ahead of dba_init on its stream
                a @ a
        ctx = dba.dba_init(B, k, V, 4, wl.eos_id, wl.pad_id, *wl.csr(), base, nbytes, stream.cuda_stream)
        if option is not None:                             # (why a ctx may go without a step)
            with pytest.raises(dba.DbaError):
                dba.dba_set_option(ctx, option, 1.0)
        dba.dba_destroy(ctx)
        with torch.cuda.stream(other):
            ws.fill_(0x5A)
        other.synchronize()
        torch.cuda.synchronize()
        assert bool((ws == 0x5A).all()), option


def test_destroying_a_ctx_leaves_a_capture_alone():
    """dba_destroy between the begin and the end of a capture on the ctx's own stream, while dba_init is still under way."""
    import torch
    import paper_1804_06609_amd as dba
    wl = si.make_small(9550, 4, 5, 300, 4, max_phrases=3, max_len=3)
    nbytes = dba.dba_workspace_bytes(4, 5, 300, 4, dba.DBA_MAX_CONS_TOKENS)
    ws = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    base = (ws.data_ptr() + 255) // 256 * 256
    a, x = torch.randn(4096, 4096, device="cuda"), torch.zeros(64, device="cuda")
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        a @ a
        x.add_(0)
        stream.synchronize()
        for _ in range(20):
            a @ a
        ctx = dba.dba_init(4, 5, 300, 4, wl.eos_id, wl.pad_id, *wl.csr(), base, nbytes, stream.cuda_stream)
        graph.capture_begin()
        x.add_(1)
        dba.dba_destroy(ctx)
        graph.capture_end()
        for _ in range(3):
            graph.replay()
    torch.cuda.synchronize()
    assert bool((x == 3).all())


def test_blocks_of_host_memory_are_freed_beside_a_capture():
    """Four ctxs with a megabyte of host memory each are destroyed, two megabytes of it freed, while another stream is being
    captured: the capture is none the worse, nor is the decode that comes next."""
    import torch
    from paper_1804_06609_amd.session import Session
    wl = si.make_small(9560, 3000, 2, 40, 2, max_phrases=2, max_len=2)
    lp = [torch.from_numpy(wl.logp(t)).cuda() for t in range(2)]
    mine, other = torch.cuda.Stream(), torch.cuda.Stream()

    def decode():
        ses = Session(wl.B, wl.k, wl.V, wl.T, wl.eos_id, wl.pad_id, *wl.csr(), stream=mine)
        for t in range(2):
            ses.step(lp[t])
        return ses

    torch.cuda.synchronize()
    held = [decode() for _ in range(4)]
    want = [[np.asarray(a).tobytes() for a in s.finalize()] for s in held]
    assert all(w == want[0] for w in want)
    mine.synchronize()
    x, graph = torch.zeros(64, device="cuda"), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    import paper_1804_06609_amd as dba
    with torch.cuda.stream(other):
        graph.capture_begin(capture_error_mode="global")
        x.add_(1)
        for s in held:
            dba.dba_destroy(s.ctx)
            s.ctx = None
        x.add_(1)
        graph.capture_end()
        for _ in range(2):
            graph.replay()
    torch.cuda.synchronize()
    assert bool((x == 4).all())
    ses = decode()
    assert [np.asarray(a).tobytes() for a in ses.finalize()] == want[0]
    ses.close()


def test_one_launch_and_two_by_turns():
    """With k > 16 the element type decides (32 KB a row): steps of one ctx that take one launch and two by turns, eager
    and replayed from a graph, leave nothing behind for each other; an element type and back, the library's own scratch among them."""
    import torch
    import paper_1804_06609_amd as dba
    B, k, V, T = 6, 20, 9000, 9
    assert (dba.dba_debug_launches(B, k, V, dba.DBA_LOGP_F32), dba.dba_debug_launches(B, k, V, dba.DBA_LOGP_F16)) == (1, 2)
    wl = si.make_small(9600, B, k, V, 3 * T, max_phrases=4, max_len=3, dup_prob=0.3)
    wl.eos_switch = 7
    dev = [torch.from_numpy(wl.logp(t)).cuda().to(torch.float16 if t % 3 == 1 else torch.float32) for t in range(T)]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        two, _ = _one_launch_decode(wl, dev, stream, 0, waves=8)
        ses, one = _one_launch_decode(wl, dev, stream, 0)
        assert one
        for t in range(T):
            two.step(dev[t])
            ses.step(dev[t], noalloc=t % 4 == 1)
            want = [a.tobytes() for a in two.outputs()] + [a.tobytes() for a in two.state().values()]
            assert [a.tobytes() for a in ses.outputs()] + [a.tobytes() for a in ses.state().values()] == want, t
        # a step of one launch from a graph, behind eager steps of two
        graph = torch.cuda.CUDAGraph()
        stream.synchronize()
        graph.capture_begin()
        ses.step(dev[0])
        graph.capture_end()
        two.step(dev[0])
        want = [a.tobytes() for a in two.outputs()]
        for _ in range(3):
            graph.replay()
            assert [a.tobytes() for a in ses.outputs()] == want
        for t in (1, 2):
            two.step(dev[t])
            ses.step(dev[t])
            assert [a.tobytes() for a in ses.outputs()] == [a.tobytes() for a in two.outputs()], t
        ses.close()
        two.close()
