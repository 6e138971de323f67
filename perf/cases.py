"""Workloads by which the speed of this library is measured.

One pass is what a translation program does for a batch: it opens a `Session` for the batch's
constraints (dba_init), takes one DBA step per time step on the decoder's log-probs, which are on the
GPU already, and reads the translations at the end (dba_finalize).  The log-probs stand in for a
decoder's: Zipf-distributed tokens with N(0,1) noise, normalised, end-of-sentence unlikely until late
in the decode.  Several tensors are used in rotation, more than the GPU's last-level cache holds
wherever a decoder's output would not fit it either.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1804_06609_amd as dba
from paper_1804_06609_amd.session import Session

PAD, EOS, FIRST_FREE = 0, 2, 4                 # ids 1 and 3 are reserved too
EARLY, LATE = 6, 2                             # tensors in rotation before / after end-of-sentence becomes likely
ELEM = {"f32": 4, "f16": 2, "bf16": 2}
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
PRUNE = 20.0                                   # the threshold of the paper's experiments


def _case(B, k, V, steps, dtype="f32", cons=(0, 32), zipf=1.1, late=0.9, mode="", decodes=1):
    """B sentences, beam k, vocabulary V; every sentence has `cons` (lowest, highest) constraint tokens in
    phrases of up to five; end-of-sentence becomes likely after the share `late` of the steps.
    mode: "" the bare algorithm; "loop" the paper's decoding settings with the stopping test after every
    step; "gbs" bank sizes without adjustment; "noalloc" steps through dba_step_noalloc.
    decodes: independent batches in flight, each on a stream of its own."""
    return {"B": B, "k": k, "V": V, "steps": steps, "dtype": dtype, "cons_lo": cons[0], "cons_hi": cons[1],
            "zipf": zipf, "late": late, "mode": mode, "decodes": decodes}


def listed():
    return [
        # the smallest call: one sentence, a toy vocabulary, beam 5 - launches and latencies only
        dict(_case(1, 5, 1000, 20, cons=(2, 2)), name="toy_sentence"),
        # interactive translation: one sentence, beam 10, a subword vocabulary of 32k
        dict(_case(1, 10, 32000, 60, cons=(4, 12)), name="one_sentence"),
        # a small batch with a few terminology phrases each
        dict(_case(16, 10, 32000, 80, cons=(1, 16)), name="small_batch"),
        # the headline shape: batch 64, beam 20, 32 constraint tokens a sentence
        dict(_case(64, 20, 32000, 100, cons=(32, 32)), name="batch64"),
        # the same from a decoder that hands over bf16
        dict(_case(64, 20, 32000, 100, dtype="bf16", cons=(32, 32)), name="batch64_bf16"),
        # offline translation with a wide beam and a large batch, fp32 and fp16
        dict(_case(128, 64, 50000, 120, zipf=0.9), name="wide_beam"),
        dict(_case(128, 64, 50000, 120, dtype="f16", zipf=0.9), name="wide_beam_f16"),
        # vocabularies whose rows do not start on 16 bytes; the first through the step that brings its own scratch
        dict(_case(24, 7, 50001, 60, cons=(0, 8), mode="noalloc"), name="odd_vocab"),
        dict(_case(96, 12, 32003, 60, dtype="bf16", cons=(0, 24)), name="odd_vocab_bf16"),
        # a decoding loop with the paper's settings: per-word scores, pruning, best completed hypothesis
        # remembered, the stopping test asked for after every step
        dict(_case(8, 10, 32000, 60, cons=(1, 12), late=1 / 3, mode="loop"), name="decode_loop"),
        # grid beam search as simulated inside the method: beam 4 (C + 1), C = 7, no adjustment
        dict(_case(64, 32, 32000, 60, cons=(7, 7), mode="gbs"), name="gbs_simulation"),
        # a server with three batches in flight (smaller workgroups in the second launch, as recommended there)
        dict(_case(64, 20, 32000, 60, cons=(32, 32), decodes=3), name="three_in_flight"),
    ]


def draw(rng: random.Random):
    """One more case of these ranges: 1 to 128 sentences, beam 3 to 64, 1000 to 64000 tokens (odd ones
    among them), every element type and way of calling; never more bytes than the largest listed case."""
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    mode = rng.choice(["", "", "", "loop", "gbs", "noalloc"])
    decodes = rng.choice([1, 1, 1, 2, 3]) if mode == "" else 1
    lo = rng.randint(0, 15 if mode == "gbs" else 16)
    hi, k = (lo, 4 * (lo + 1)) if mode == "gbs" else (lo + rng.randint(0, 16), spread(3, 64))
    c = _case(spread(1, 128 // decodes), k, spread(1000, 64000), rng.randint(20, 120),
              dtype=rng.choice(["f32", "f32", "f16", "bf16"]), cons=(lo, hi),
              zipf=rng.choice([0.9, 1.1]), late=1 / 3 if mode == "loop" else 0.9, mode=mode, decodes=decodes)
    most = 128 * 64 * 50000 * 4 * 120
    while c["decodes"] * c["B"] * c["k"] * c["V"] * ELEM[c["dtype"]] * c["steps"] > most:
        c["steps"] = c["steps"] * 3 // 4
    return c


def _constraints(case, seed):
    """[decode][sentence][phrase][token]"""
    rng = random.Random(seed * 7919 + 17)
    out = []
    for _ in range(case["decodes"]):
        batch = []
        for _ in range(case["B"]):
            left = rng.randint(case["cons_lo"], case["cons_hi"])
            sent = []
            while left > 0:
                n = min(left, 1 if case["mode"] == "gbs" else rng.randint(1, 5))
                sent.append([rng.randrange(FIRST_FREE, case["V"]) for _ in range(n)])
                left -= n
            batch.append(sent)
        out.append(batch)
    return out


def _csr(batch):
    toks, poff, soff = [], [0], [0]
    for sent in batch:
        for phrase in sent:
            toks.extend(phrase)
            poff.append(len(toks))
        soff.append(len(poff) - 1)
    return tuple(np.asarray(a, dtype=np.int32) for a in (toks, poff, soff))


def _logprobs(case, seed):
    """[decode][tensor], each [B, k, V] on the GPU: EARLY tensors, then LATE ones with end-of-sentence likely."""
    B, k, V = case["B"], case["k"], case["V"]
    gen = torch.Generator(device="cuda").manual_seed(seed * 1000003 + 5)
    rank = torch.empty(V, device="cuda")
    rank[torch.randperm(V, generator=gen, device="cuda")] = torch.arange(1, V + 1, device="cuda", dtype=torch.float32)
    bias = -case["zipf"] * rank.log()
    bias[[PAD, 1, 3]] = -case["zipf"] * math.log(V)
    out = []
    for _ in range(case["decodes"]):
        mine = []
        for i in range(EARLY + LATE):
            bias[EOS] = -30.0 if i < EARLY else 2.0
            lp = torch.empty((B, k, V), dtype=TORCH[case["dtype"]], device="cuda")
            part = max(1, 50_000_000 // (k * V))
            for b in range(0, B, part):
                x = torch.randn((min(part, B - b), k, V), generator=gen, device="cuda")
                lp[b:b + part] = torch.log_softmax(x.add_(bias), dim=-1)
            mine.append(lp)
        out.append(mine)
    return out


def _tensor_at(case, t):
    switch = int(case["steps"] * case["late"])
    return t % EARLY if t < switch else EARLY + t % LATE


def prepare(case, seed):
    options = {}
    if case["mode"] == "loop":
        options = {dba.DBA_OPT_NORMALIZE_FINISHED: 1, dba.DBA_OPT_PRUNE_THRESHOLD: PRUNE,
                   dba.DBA_OPT_TRACK_COMPLETED: 1}
    elif case["mode"] == "gbs":
        options = {dba.DBA_OPT_ADJUSTMENT: 0}
    if case["decodes"] > 1:
        options[dba.DBA_OPT_MERGE_WAVES] = 4
    return {"case": case, "options": options, "csr": [_csr(b) for b in _constraints(case, seed)],
            "logp": _logprobs(case, seed),
            "streams": [torch.cuda.Stream() for _ in range(case["decodes"])] if case["decodes"] > 1 else [None]}


def run(state):
    case = state["case"]
    noalloc, loop = case["mode"] == "noalloc", case["mode"] == "loop"
    jobs = [Session(case["B"], case["k"], case["V"], case["steps"], EOS, PAD, *csr, stream=st,
                    options=state["options"]) for csr, st in zip(state["csr"], state["streams"])]
    for t in range(case["steps"]):
        i = _tensor_at(case, t)
        for ses, lp in zip(jobs, state["logp"]):
            ses.step(lp[i], noalloc=noalloc)
        if loop and (jobs[0].finished() & dba.DBA_STOP_ALL).all():     # every hypothesis is completed
            break
    out = []
    for ses in jobs:
        tokens, length, score, status = ses.finalize()
        out.append({"beam_token": ses.out_token, "beam_parent": ses.out_backptr, "beam_score": ses.out_score,
                    "beam_flags": ses.out_flags, "tokens": tokens, "length": length, "score": score,
                    "status": status})
        ses.close()
    return out


def work(case):
    """Every live beam row's log-probs once per step (the first step has one live row a sentence), and the new
    beam written.  Where decoding stops early, only the steps before end-of-sentence becomes likely count:
    what follows depends on the inputs, and completed rows are not read."""
    steps = int(case["steps"] * case["late"]) if case["mode"] == "loop" else case["steps"]
    rows = case["B"] * (1 + (steps - 1) * case["k"])
    beam = case["B"] * case["k"] * steps * 13              # token, parent, score, flags
    return {"bytes": case["decodes"] * (rows * case["V"] * ELEM[case["dtype"]] + beam),
            "flops": case["decodes"] * rows * case["V"]}   # one addition per log-prob


def tolerance(case):
    # A score is by definition one fp32 addition per step and every choice is on those sums with a fixed
    # tie rule, so two correct implementations agree in every bit.
    return "exact"


def exact(case, seed):
    """The scores `run` returns, from a plain statement of the method: sums in 64 bits, each rounded to fp32
    as the method defines a score.  The beam's choices depend on every rounding, so nothing else is meaningful."""
    B, k, V, steps = case["B"], case["k"], case["V"], case["steps"]
    if case["decodes"] * B * k * steps > 60_000 or B * k * V > 20_000_000:
        return None
    loop = case["mode"] == "loop"
    f32 = np.float32
    out = []
    for cons, logp in zip(_constraints(case, seed), _logprobs(case, seed)):
        # a hypothesis: (score, complete phrases, phrase under way, its tokens met, finished, length)
        beams = [[(f32(0), frozenset(), -1, 0, False, 0)] for _ in range(B)]
        record = [None] * B
        for t in range(steps):
            lp = logp[_tensor_at(case, t)]
            prev = torch.full((B, k), -math.inf, dtype=torch.float64)
            for b, beam in enumerate(beams):
                for h, y in enumerate(beam):
                    if not y[4]:
                        prev[b, h] = float(y[0])
            sums = torch.empty((B, k, V), device="cuda")
            for b in range(B):
                sums[b] = (prev[b].cuda()[:, None] + lp[b].double()).float()
                for h, y in enumerate(beams[b]):
                    if len(y[1]) < len(cons[b]):
                        sums[b, h, EOS] = -math.inf
            tops, ids = torch.sort(sums, dim=-1, descending=True, stable=True)
            tops, ids = tops[..., :k].cpu().numpy(), ids[..., :k].cpu().numpy()
            wanted = [[_placeable(cons[b], y) for y in beams[b]] for b in range(B)]
            at = [(b, h, w) for b in range(B) for h in range(len(beams[b])) for w in wanted[b][h]]
            got = sums[tuple(torch.tensor(x, device="cuda") for x in zip(*at))].cpu().numpy() if at else []
            extra = [[] for _ in range(B)]
            for (b, h, w), s in zip(at, got):
                extra[b].append((s, h, w))
            for b in range(B):
                best, cands = [], {(h, w): s for s, h, w in extra[b] if s > -math.inf}
                for h, y in enumerate(beams[b]):
                    row = [(y[0], h, PAD)] if y[4] else [(tops[b, h, i], h, int(ids[b, h, i])) for i in range(k)]
                    row = [x for x in row if x[0] > -math.inf]
                    best += row
                    cands.update({(h, w): s for s, h, w in row[:1]})
                best.sort(key=lambda x: (-x[0], x[1], x[2]))
                cands.update({(h, w): s for s, h, w in best[:k]})
                beams[b] = _select(case, cons[b], beams[b], cands)
                if loop:
                    done = [y for y in beams[b] if y[4]]
                    top = max([y[0] for y in done], default=None)
                    if top is not None and (record[b] is None or top > record[b]):
                        record[b] = top
            if loop and all(beam and all(y[4] for y in beam) for beam in beams):
                break
        score = np.full(B, -math.inf)
        for b, beam in enumerate(beams):
            done = [y for y in beam if y[4]]
            if loop and record[b] is not None:
                score[b] = record[b]
            elif done:
                score[b] = max(done, key=lambda y: y[0] if loop else f32(y[0] / f32(y[5])))[0]
            elif beam:
                score[b] = max(beam, key=lambda y: (_met(cons[b], y), y[0]))[0]
        final = np.full((B, k), -math.inf)
        for b, beam in enumerate(beams):
            final[b, :len(beam)] = [y[0] for y in beam]
        out.append({"beam_token": None, "beam_parent": None, "beam_score": final, "beam_flags": None, "tokens": None,
                    "length": None, "score": score, "status": None})
    return out


def _met(cons, y):
    return sum(len(cons[p]) for p in y[1]) + y[3]


def _placeable(cons, y):
    """Constraint tokens a hypothesis may place now."""
    if y[4]:
        return set()
    firsts = {cons[p][0] for p in range(len(cons)) if p not in y[1] and p != y[2]}
    return firsts | ({cons[y[2]][y[3]]} if y[2] >= 0 else set())


def _add(case, cons, y, w, s):
    """The hypothesis `y` extended by token w, with the sum s."""
    score, whole, p, n, fin, length = y
    if fin:
        return y
    if p >= 0 and cons[p][n] == w:
        n += 1
    else:
        p, n = -1, 0
        for q in range(len(cons)):
            if q not in whole and cons[q][0] == w:
                p, n = q, 1
                break
    if p >= 0 and n == len(cons[p]):
        whole, p, n = whole | {p}, -1, 0
    return (s, whole, p, n, w == EOS, length + 1)


def _select(case, cons, beam, cands):
    """The new beam: bank sizes by constraints met, the best of every bank, best first."""
    k, C = case["k"], sum(len(p) for p in cons)
    banks = [[] for _ in range(C + 1)]
    for (h, w), s in cands.items():
        y = _add(case, cons, beam[h], w, s)
        banks[_met(cons, y)].append((s, h, w, y))
    count = [len(x) for x in banks]
    size = [k // (C + 1)] * C + [k // (C + 1) + k % (C + 1)]
    if case["mode"] == "gbs":
        size = [min(a, c) for a, c in zip(size, count)]
    else:
        for d in [i for i in range(C + 1) if size[i] > count[i]]:
            spare, size[d] = size[d] - count[d], count[d]
            for dist in range(1, C + 1):
                for x in (d + dist, d - dist):
                    if 0 <= x <= C and size[x] < count[x]:
                        give = min(spare, count[x] - size[x])
                        size[x] += give
                        spare -= give
    new = []
    for bank, n in zip(banks, size):
        new += sorted(bank, key=lambda x: (-x[0], x[1], x[2]))[:n]
    new.sort(key=lambda x: (-x[0], x[1], x[2]))
    if case["mode"] != "loop":
        return [x[3] for x in new]
    f32 = np.float32
    beam2 = [(f32(y[0] / f32(y[5])),) + y[1:] if y[4] and not beam[h][4] else y for _, h, _, y in new]
    done = [y[0] for y in beam2 if y[4]]
    if done:
        bar = f32(max(done) - f32(PRUNE))
        beam2 = [y for y in beam2 if y[0] >= bar]
    return beam2
