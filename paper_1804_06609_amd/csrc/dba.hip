// libdba: C-ABI implementation (see include/dba.h) and the gfx950 kernels' entry points.
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "../../include/dba.h"
#include "../../include/dba_debug.h"
#include "dba_kernels.hpp"
#include "host_blocks.hpp"

using namespace dba;

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------
// Stream phase of one beam row (sentence b, slot h) by one workgroup of NW waves: leaves the row's
// sorted top keys in p.rowlists and the keys of its constraint tokens in p.conskeys.
// U = 16-byte loads each lane keeps in flight per tile; FMT = element type of the log-probs.
// logp, V, k, first_step are what the first loads need; the kernels take them as leading scalar
// arguments, which the hardware hands over in registers at wave start (kernel-argument preload),
// so that the first two tiles are requested before any argument has been read from memory.
// TO: where the keys go.  kInMemory; kHandedOver, the same to a workgroup that runs now; kInLds, sm.key[slot] (rows of one wave).
// wave: of the row's NW; turn: which of them finishes the row, modulo NW; early: what else to request, right behind the first two tiles.
template <int U, int FMT, int NW, int D, int TO, typename Smem, typename Early>
__device__ __forceinline__ void stream_phase(const StepParams &p, const void *logp, int V, int k, int first_step, int b, int h,
                                             int wave, int turn, int slot, Smem &sm, Early early)
{
    typedef typename Logp<FMT>::elem_t elem_t;
    static_assert((TO == kInLds) == (NW == 1), "a row of one wave");
    const int row = b * k + h;
    const int lane = lane_id();
    constexpr int nwaves = NW;
    const bool gatherer = wave == nwaves - 1;     // this wave also fetches the constraint tokens

    // the first two tiles of the row are requested before anything else: they need nothing of
    // the hypothesis, and the loads of the hypothesis (uniform, hence scalar loads the wave has to
    // wait for one after the other) would otherwise hold them back
    const elem_t *__restrict__ logp_row = static_cast<const elem_t *>(logp) + (size_t)row * (size_t)V;
    RowStream<U, FMT, D> rs;
    const bool known_empty = first_step && h != 0;   // decoder-init leaves slots 1.. empty
    if (!known_empty) rs.begin(logp_row, V, wave, nwaves);
    __builtin_amdgcn_sched_barrier(0);
    early();
    // then the hypothesis and its constraint bookkeeping (one wave, one lane per phrase)
    const Sentence &sent = p.sentences[b];
    const Hyp hyp = p.beam[row];
    const int phrases = sent.nphr;
    // The flags come by a vector load, which returns after those of the two tiles: whatever depends on them, the scattered
    // gathers of the constraint tokens' log-probs above all, is then behind the tiles of the rows beside this one and not among
    // them (per step, by a scalar load / like this: 798 rows of 16760 fp32 23.6 / 22.6 us, 768 of 16000 23.45 / 22.0, 800, k = 20,
    // 19.6 / 18.6, 160 of 32000 12.25 / 12.1; ten rows of 32000, which have the chip to themselves, 10.15 / 10.4).
    int zero = 0;
    asm volatile("" : "+v"(zero));
    const uint32_t state_ld = (&p.beam[row].state)[zero];
    const int fin_wave = turn & (nwaves - 1);
    const bool finisher = wave == fin_wave;
    u64 g_sfl = 0, t_bucket = 0;
    int g_ftok = -1, t_btok = -1;
    if (gatherer || finisher) g_ftok = sent.first_tok[lane];
    if (gatherer) g_sfl = sent.same_first_lower[lane];
    if (finisher) {
        // lane j: the phrases whose first token has low six bits j, and that token where they agree on it
        t_bucket = sent.first_bucket[lane];
        t_btok = sent.bucket_tok[lane];
    }

    asm volatile("" : : "s"(phrases));                   // (waited for together with the hypothesis)
    const float prev = hyp.score;
    const uint32_t state = (uint32_t)__builtin_amdgcn_readfirstlane((int)state_ld);
    const int fin = flags_of(state), ipq = ipq_of(state);
    const uint32_t code_base = (uint32_t)h << p.tok_bits;

    RowTop st;
    st.list = 0;
    st.thr = kLowestFinite;
    u64 ckey = 0;
    int parked = 0;
    if (prev > -INFINITY && !(fin & kFinFinished) && !known_empty) {
        // Alg. 2 inner loop / Sec. 3.1 item 2: the hypothesis extended by each constraint token
        // it may place now; the log-prob is one 4-byte read per token, in flight during the stream
        int cw = -1, cbank = 0;
        if (gatherer)
            cw = expandable_entry(phrases, __popcll(hyp.met), hyp.inc, ipq < 0 ? -1 : (ipq >> 8), ipq < 0 ? 0 : (ipq & 255), hyp.nxt,
                                  g_ftok, g_sfl, cbank);
        const float cx = cw >= 0 ? Logp<FMT>::widen_one(logp_row[cw]) : -INFINITY;
        // Sec. 3.3: no end-of-sentence before all constraints are met
        const int eos_block = (fin & kFinEosBlocked) ? p.eos_id : -1;
        parked = rs.template run<NW>(prev, eos_block, code_base, k, wave, slot, sm, st);
        const float cs = prev + cx;
        if (cw >= 0 && cs > -INFINITY)
            ckey = pack_sel(p.met_bits, cbank, ord_from_float(cs), code_base | (uint32_t)cw);
    } else if (prev > -INFINITY && wave == 0 && lane == 0) {
        // a finished hypothesis stays on the beam: its one continuation is the pad token
        // at log-prob +0.0, score carried unchanged
        st.list = make_key(prev + 0.0f, code_base | (uint32_t)p.pad_id);
    }
    if (gatherer && TO != kInLds) {
        if constexpr (TO == kHandedOver) {
            if (lane < phrases) hand_over(p.conskeys + (size_t)row * kMaxCons + lane, ckey ? ckey : kNoKey);
        } else {
            p.conskeys[(size_t)row * kMaxCons + lane] = ckey;
        }
    }
    u64 acc;
    if constexpr (NW == 1) acc = finish_row_of_one_wave(sm.key[slot], st.list, parked);
    else acc = finish_row(sm, st.list, parked, wave, fin_wave);
    if (finisher) {
        // Handed on as selection keys: every listed sum with the bank it would land in - the
        // constraints met once the hypothesis has emitted that token (add(), Sec. 3.1).  Each lane
        // looks its own token up in the sentence's table of first tokens, which the lanes of this
        // wave hold (lane j = bucket j): the phrases it could begin, then the count.
        // (every lane takes every step, so that any lane's table entry can be read)
        const int nmet = __popcll(hyp.met);
        const bool extends = !(fin & kFinFinished) && acc != 0;      // not the carried-over key of a finished row
        const int w = extends ? (int)(key_flat(acc) & ((1u << p.tok_bits) - 1u)) : 0;
        const int same = __shfl(t_btok, w & 63, kWave);
        const u64 bucket = ((u64)(uint32_t)__shfl((int)(uint32_t)(t_bucket >> 32), w & 63, kWave) << 32) |
                           (u64)(uint32_t)__shfl((int)(uint32_t)t_bucket, w & 63, kWave);
        u64 match = (extends && same == w) ? bucket : 0;
        u64 todo = (extends && same == -2) ? bucket : 0;   // the bucket's phrases begin differently: one by one
        while (__ballot(todo != 0)) {
            const int j = todo ? __ffsll((long long)todo) - 1 : 0;
            const int first = __shfl(g_ftok, j, kWave);
            if (todo && first == w) match |= 1ull << j;
            todo &= todo - 1;
        }
        const int bank = !extends ? nmet
                                  : nmet_after(nmet, ipq < 0 ? -1 : (ipq >> 8), ipq < 0 ? 0 : (ipq & 255), w == hyp.nxt, match,
                                               hyp.inc);
        const u64 key = sel_from_rowkey(p.met_bits, bank, acc);
        if constexpr (TO == kInLds) {
            sm.key[slot][lane] = key;
            sm.key[slot][kWave + lane] = ckey;
        } else if constexpr (TO == kHandedOver) {
            if (lane < k) hand_over(p.rowlists + (size_t)row * kWave + lane, key ? key : kNoKey);
        } else {
            p.rowlists[(size_t)row * kWave + lane] = key;
        }
    }
}

// First launch of a step.  Grid: B * k workgroups of NW waves, one per beam row.  Workgroups are dealt
// out to the chip's eight dies (XCDs, each with an L2 of its own) in turn, so consecutive numbers
// mean consecutive dies: where rows_abreast says so (rows below 512000 bytes, or few of them), the first B & ~7 sentences are
// numbered eight abreast, slot by slot, and a die streams all rows of every eighth sentence - one stretch of
// memory after the other - instead of every eighth row (8192 rows of 50000, k = 64: 269.7 -> 262.7 us per step in fp32, 151.5 -> 146.5 with
// fp16; 0.1-0.3 us at 1152 to 2048 rows of 32000).  The other sentences, the last B & 7 or all of them, are
// numbered row by row over all dies, which keeps the dies evenly loaded.
// k_first = k | first_step << 16; rows_abreast = (B & ~7) * k or 0; inv_k = ceil(2^32 / k): with fewer than
// 2^22 rows and k <= 64, the high half of n * inv_k is n / k.
template <int U, int FMT, int NW, int D>
__global__ __launch_bounds__(NW * kWave) void dba_stream_kernel(const void *logp, int V, int k_first, uint32_t rows_abreast,
                                                               uint32_t inv_k, const StepParams p)
{
    __shared__ StreamSmem<NW> sm;
    const uint32_t k = (uint32_t)k_first & 0xFFFFu, n = blockIdx.x;
    const bool abreast = n < rows_abreast;
    const uint32_t m = abreast ? n >> 3 : n;
    const uint32_t q = k == 1 ? m : __umulhi(m, inv_k);
    const int b = (int)(abreast ? q * 8u + (n & 7u) : q), h = (int)(m - q * k);
    // workgroups are dealt out round-robin over the 256 compute units, so the ones sharing a
    // compute unit differ in (number / 256): let that pick the wave (hence the SIMD) that finishes the row
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    stream_phase<U, FMT, NW, D, kInMemory>(p, logp, V, (int)k, k_first >> 16, b, h, wave, (int)(blockIdx.x >> 8), wave, sm, [] {});
}

// Both phases in one launch, where the sentences' workgroups find room beside the rows (one_launch_shape).  Grid: B * k workgroups for
// the rows, then B that each take a sentence through the merge phase.  Such a step is a chain of latencies, and the end of one kernel,
// the start of the next and its wait for the row lists were 2.2 us of it; here a sentence's workgroup has its tables in LDS before the
// rows are through and reads their places in the row lists again and again until all are filled (a store is seen
// there after 0.6 to 0.9 us).  Per step, two launches / one: ten rows of 32000 11.1 / 10.2 us, 160 13.0 / 11.8, 168 of 50001 14.05 / 12.9, 240 of
// 9000 11.45 / 10.5, 192 of 32000 with k = 16 13.6 / 12.5, 256 with k = 32 16.15 / 15.2, 400 rows of 8000 12.6 / 11.45, 500 of 32000 18.75 / 17.65.
//
// Every wait ends, and with the right answer.  A row waits for nothing; when its keys have reached memory it counts itself
// among the sentence's ended rows.  A sentence's workgroup that has looked for the keys most_tries times - the rows may be
// long, or have not started because other work holds the chip - says so in the atomic step that tells it how many rows have ended.  If all
// have, their keys are there; if not, it leaves, and the row that ends last finds that said and takes the sentence on itself.
// (Rows could always do so, without a workgroup for the sentence; its tables and its code then come cold: as slow as two
// launches.)
// rows_order: B * k, and from bit 31 whether the sentences' workgroups are numbered first (for tests of the other way).
template <int U, int FMT, int NW, int D, int ROWS, int MW, int J>
__global__ __launch_bounds__(NW * kWave) void dba_step_kernel(const void *logp, int V, int k_first, uint32_t rows_abreast,
                                                             uint32_t inv_k, uint32_t rows_order, uint32_t inv_k16, int most_tries,
                                                             const StepParams p)
{
    extern __shared__ __align__(16) unsigned char dyn_smem[];
    __shared__ int role;
    StreamSmem<NW> &ss = *reinterpret_cast<StreamSmem<NW> *>(dyn_smem);
    MergeSmem<MW> &ms = *reinterpret_cast<MergeSmem<MW> *>(dyn_smem);
    u64 *cand = reinterpret_cast<u64 *>(dyn_smem + (sizeof(MergeSmem<MW>) + 15) / 16 * 16);
    const uint32_t k = (uint32_t)k_first & 0xFFFFu, rows = rows_order & 0x7FFFFFFFu;
    const uint32_t n = blockIdx.x - (rows_order >> 31 ? (k == 1 ? rows : __umulhi(rows, inv_k)) : 0u);     // (wraps below the first row)
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), tid = (int)threadIdx.x;
    int b;
    bool all_ended = false;
    if (n < rows) {
        const bool abreast = n < rows_abreast;
        const uint32_t m = abreast ? n >> 3 : n;
        const uint32_t q = k == 1 ? m : __umulhi(m, inv_k);
        b = (int)(abreast ? q * 8u + (n & 7u) : q);
        const int h = (int)(m - q * k);
        stream_phase<U, FMT, NW, D, kHandedOver>(p, logp, V, (int)k, k_first >> 16, b, h, wave, (int)(blockIdx.x >> 8), wave, ss,
                                                 [] {});
        // (each wave waits until the keys it has handed over are in memory, where their agent-scope stores put them)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0)
        __syncthreads();                                   // (and everyone has left the row's LDS)
        if (wave == 0 && lane_id() == 0)
            role = __hip_atomic_fetch_add(&p.best[b].ended, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   (kGivenUp | (int)(k - 1));
        __syncthreads();
        if (!role) return;
        all_ended = true;
    } else {
        b = (int)((rows_order >> 31) ? blockIdx.x : n - rows);
    }
    MergeTables tables;
    int P = 0;
    if (wave < MW) {
        P = tables.request(p, b, (int)k, tid);
        clear_for_merge(p, tid, MW * kWave, ms, cand);
        tables.store((int)k, tid, ms);
    }
    __syncthreads();
    if (wave >= MW) return;
    merge_phase<ROWS, MW, J, kHandedOver>(p, p.rowlists, p.conskeys, (int)k, inv_k16, b, ms, cand, P, most_tries, all_ended);
}

// Both phases of steps of short rows and narrow beams: one workgroup per sentence, a wave per row (k <= 8), so that nothing is
// handed over through memory and no wave of a row waits for another.  Such a step is one chain of latencies; here it is as long as
// one wave takes for a row, with eight on four SIMDs, which is why it pays only for few bytes a sentence.  Per step, one launch with a
// workgroup per row and one per sentence / this: 5 rows of 1000 fp32 7.95 / 6.9 us, one of 1000 7.45 / 6.25, 8 of 1024 7.75 / 7.3, 256 x 5 of 1000
// 9.95 / 8.2; but 5 of 3000 7.75 / 8.1, 8 of 2000 7.85 / 8.35, 8 of 4000 8.1 / 9.6, and with sixteen waves 10 of 2000 8.8 / 9.7, 16 of 4000
// 9.1 / 11.0.
template <int FMT>
__global__ __launch_bounds__(kSentenceWaves * kWave) void dba_sentence_kernel(const void *logp, int V, int k_first, uint32_t inv_k16,
                                                                             const StepParams p)
{
    extern __shared__ __align__(16) unsigned char dyn_smem[];
    __shared__ SentenceSmem sm;
    constexpr int MW = 4;
    MergeSmem<MW> &ms = *reinterpret_cast<MergeSmem<MW> *>(dyn_smem);
    u64 *cand = reinterpret_cast<u64 *>(dyn_smem + (sizeof(MergeSmem<MW>) + 15) / 16 * 16);
    const int k = k_first & 0xFFFF, b = (int)blockIdx.x, tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    MergeTables tables;
    int P = 0;
    auto early = [&] {
        if (wave < MW) P = tables.request(p, b, k, tid);
    };
    if (wave < k) stream_phase<kTileLoads, FMT, 1, 2, kInLds>(p, logp, V, k, k_first >> 16, b, wave, 0, 0, wave, sm, early);
    else early();
    if (wave < MW) {
        clear_for_merge(p, tid, MW * kWave, ms, cand);
        tables.store(k, tid, ms);
    }
    __syncthreads();
    if (wave >= MW) return;
    merge_phase<2, MW, 1, kInLds>(p, sm.key[0], sm.key[0] + kWave, k, inv_k16, b, ms, cand, P, 0, false);
}

// Second launch of a step: the merge phase.  Grid: one workgroup of MW waves per sentence, each wave
// taking up to ROWS beam rows (k <= ROWS * MW); J > 0: and holding J entries per lane of all the sentence's lists
// (k * k <= 64 * J).  The pointers to the row lists and the beam width (k_inv = k | inv_k << 16) come first:
// they are all the first loads need.
template <int ROWS, int MW, int J>
__global__ __launch_bounds__(MW * kWave) void dba_merge_kernel(const u64 *rowlists, const u64 *conskeys, uint32_t k_inv,
                                                               const StepParams p)
{
    extern __shared__ __align__(16) unsigned char dyn_smem[];
    __shared__ MergeSmem<MW> sm;
    merge_phase<ROWS, MW, J, kInMemory>(p, rowlists, conskeys, (int)(k_inv & 0xFFFFu), k_inv >> 16, (int)blockIdx.x, sm,
                                           reinterpret_cast<u64 *>(dyn_smem), 0, 0, false);
}

// Reference read: the largest element of each row, one workgroup per row, with the tile order and
// the two-tiles-in-flight non-temporal 128-bit loads of the stream phase and nothing else.  Its
// duration is what this chip takes to deliver the [rows, V] tensor once; the step is compared
// with it.
__global__ __launch_bounds__(kBlock) void dba_row_max_kernel(const float *__restrict__ src, int V,
                                                             float *__restrict__ out)
{
    typedef float v4f __attribute__((ext_vector_type(4)));
    constexpr int U = 4;
    __shared__ float part[kWavesPerBlock];
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    const v4f *vec = reinterpret_cast<const v4f *>(src + (size_t)blockIdx.x * V);
    const int nv = V >> 2, per = kWave * U, ntiles = (nv + per - 1) / per;
    const float ninf = -__builtin_inff();
    v4f a[U], b[U];
    auto load = [&](v4f(&x)[U], int tl) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = tl * per + u * kWave + lane;
            x[u] = i < nv ? __builtin_nontemporal_load(vec + i) : v4f{ninf, ninf, ninf, ninf};
        }
    };
    float m = ninf;
    auto fold = [&](v4f(&x)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) m = fmaxf(m, fmaxf(fmaxf(x[u].x, x[u].y), fmaxf(x[u].z, x[u].w)));
    };
    int tl = wave;
    if (tl < ntiles) load(a, tl);
    if (tl + kWavesPerBlock < ntiles) load(b, tl + kWavesPerBlock);
    while (tl < ntiles) {
        fold(a);
        if (tl + 2 * kWavesPerBlock < ntiles) load(a, tl + 2 * kWavesPerBlock);
        tl += kWavesPerBlock;
        if (tl >= ntiles) break;
        fold(b);
        if (tl + 2 * kWavesPerBlock < ntiles) load(b, tl + 2 * kWavesPerBlock);
        tl += kWavesPerBlock;
    }
    for (int d = 32; d > 0; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, kWave));
    if (lane == 0) part[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWavesPerBlock; ++w) m = fmaxf(m, part[w]);
        out[blockIdx.x] = m;
    }
}


// Diagnostic: the wavefront selection primitives on caller-provided keys, one wave per case.
// in: keys[128] per case, vals[64] per case.  out[0:64] = sort of keys[0:64];
// out[64:128] = merge of sort(keys[0:64]) and sort(keys[64:128]); out[128:192] = the first
// list after inserting keys[64..71] one at a time; out[192:256] = low word: the 64 greatest high
// words of both sorted lists (32-bit merge), high word: the greatest high word left out;
// fout[0:64] = sort of vals.
__global__ void dba_wave_select_kernel(int n_cases, const u64 *keys, const float *vals, u64 *out,
                                       float *fout)
{
    const int i = blockIdx.x;
    if (i >= n_cases) return;
    const int lane = lane_id();
    const u64 a = sort64_desc<u64>(keys[(size_t)i * 128 + lane]);
    const u64 b = sort64_desc<u64>(keys[(size_t)i * 128 + 64 + lane]);
    out[(size_t)i * 256 + lane] = a;
    out[(size_t)i * 256 + 64 + lane] = merge_desc<u64>(a, b);
    u64 l = a;
    for (int j = 0; j < 8; ++j) {
        const u64 x = keys[(size_t)i * 128 + 64 + j];
        l = insert_desc(l, x);
    }
    out[(size_t)i * 256 + 128 + lane] = l;
    uint32_t fell = 0;
    const uint32_t hi = merge32_desc((uint32_t)(a >> 32), (uint32_t)(b >> 32), fell);
    out[(size_t)i * 256 + 192 + lane] = ((u64)wave_max_u32(fell) << 32) | hi;
    fout[(size_t)i * 64 + lane] = float_from_ord(sort64_desc<uint32_t>(ord_from_float(vals[(size_t)i * 64 + lane])));
}

// The constraints of a sentence as the host hands them over: one word per place, token id | kBeginsPhrase, or kNoToken.
constexpr uint32_t kBeginsPhrase = 0x80000000u, kNoToken = 0x40000000u;

// decoder-init: slot 0 of every sentence is a live, empty hypothesis with score +0.0; and the sentence's tables, one
// wave per sentence, lane = place of a token, then phrase.  Its time is one trip to host memory for the words.  seen
// (may be null): host word per sentence, set once the sentence's words have been read and all that is written for it here is in
// memory, where no later write-back can land on what a next owner of the workspace puts there.
__global__ __launch_bounds__(kWave) void dba_init_kernel(int B, int k, const uint32_t *words, uint32_t *seen, StepParams p)
{
    __shared__ int off[kMaxCons], first[kMaxCons];
    const int b = (int)blockIdx.x, lane = lane_id();
    const size_t at = (size_t)b * kMaxCons + lane;
    const uint32_t word = __hip_atomic_load(words + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    // (past the L2, like every store here)
    auto put = [](auto *to, auto value) { __hip_atomic_store(to, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (p.rowlists)                                        // steps of one launch: all places empty, while the words are on their way
        for (int h = 0; h < k; ++h) {
            put(p.rowlists + ((size_t)b * k + h) * kWave + lane, (u64)0);
            put(p.conskeys + ((size_t)b * k + h) * kWave + lane, (u64)0);
        }
    const bool valid = (word & kNoToken) == 0, begins = valid && (word & kBeginsPhrase) != 0;
    const int tok = valid ? (int)(word & ~kBeginsPhrase) : 0;
    const u64 starts = __ballot(begins);
    const int C = (int)__popcll(__ballot(valid)), P = (int)__popcll(starts);
    if (begins) {
        off[lanes_before(starts)] = lane;
        first[lanes_before(starts)] = tok;
    }
    __syncthreads();
    const int ftok = lane < P ? first[lane] : -1;
    u64 same_lower = 0, bucket = 0;
    int btok = -1;
    for (int j = 0; j < P; ++j) {
        const int f = __builtin_amdgcn_readlane(ftok, j);
        if (j < lane && f == ftok) same_lower |= 1ull << j;
        if ((f & 63) == lane) {
            bucket |= 1ull << j;
            btok = btok == -1 || btok == f ? f : -2;
        }
    }
    Sentence *s = const_cast<Sentence *>(p.sentences) + b;
    put(s->tok + lane, tok);
    put(s->phr_off + lane, lane < P ? off[lane] : lane == P ? C : 0);
    put(s->first_tok + lane, ftok);
    put(s->same_first_lower + lane, same_lower);
    put(s->first_bucket + lane, bucket);
    put(s->bucket_tok + lane, btok);
    if (lane == 0) {
        put(s->phr_off + kMaxCons, P == kMaxCons ? C : 0);
        put(&s->nphr, P);
        put(p.all_finished + b, (uint8_t)0);
    }
    static_assert(sizeof(BestCompleted) == 4 * sizeof(u64), "four words");
    if (lane < 4) put(reinterpret_cast<u64 *>(p.best + b) + lane, (u64)0);
    if (lane < k) {
        const size_t i = (size_t)b * k + lane;
        put(&p.beam_nxt[i].score, lane == 0 ? 0.0f : -INFINITY);
        put(&p.beam_nxt[i].state, state_word((lane == 0 && C > 0) ? kFinEosBlocked : 0, -1));
        put(&p.beam_nxt[i].len, 0);
        put(&p.beam_nxt[i].nxt, -1);
        put(&p.beam_nxt[i].met, (u64)0);
        put(&p.beam_nxt[i].inc, (lane == 0 && P > 0) ? (P == 64 ? ~0ull : ((1ull << P) - 1ull)) : 0ull);
    }
    if (seen) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): all of it is in memory
        if (lane == 0) __hip_atomic_store(seen + b, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// The stopping flags on their way to host memory, four sentences a word.
__global__ __launch_bounds__(kBlock) void dba_flags_kernel(int words, const uint32_t *flags, uint32_t *out)
{
    for (int i = threadIdx.x; i < words; i += kBlock) out[i] = flags[i];
}

// End of decoding (Sec. 3.3, length normalisation of Sec. 4): one workgroup per sentence.
// best != null: the record of the best completed hypothesis seen on any beam decides, if there is one.
//
// The back-pointers form one chain over all steps; followed in memory every link costs a trip there (71 us
// for 64 sentences of 100 steps, one thread each).  Here the eight waves fetch the parents of all slots of
// kFinSteps steps at once, one row of a beam per load, into LDS; one wave then reads rows that do not depend on the
// chain, lane = slot, and follows it with lane reads.  The tokens along it are fetched 64 at a time.
// (The call, copies to the host included: 172 -> 117 us there, 236 -> 126 for 128 sentences of 120 steps, k = 64.)
constexpr int kFinWaves = 8, kFinRows = 16, kFinSteps = kFinWaves * kFinRows;

__global__ __launch_bounds__(kFinWaves * kWave) void dba_finalize_kernel(
    int B, int k, int T, int N, int pad_id, int normalized, const int32_t *hist_token, const int32_t *hist_backptr,
    const Hyp *beam, const BestCompleted *best_rec,
    int32_t *out_tokens, int32_t *out_len, float *out_score, int32_t *out_status)
{
    __shared__ uint8_t parent[kFinSteps][kWave];
    const int b = (int)blockIdx.x, lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    int32_t *toks = out_tokens + (size_t)b * N;
    auto at = [&](int t, int slot) { return ((size_t)t * B + b) * k + slot; };
    // parents of steps hi - kFinSteps + 1 .. hi, row hi - r in parent[r]
    int row[kFinRows];
    auto fetch = [&](int hi) {
#pragma unroll
        for (int i = 0; i < kFinRows; ++i) {
            const int t = hi - (i * kFinWaves + wave);
            row[i] = 0;
            if (t >= 0 && lane < k) row[i] = hist_backptr[at(t, lane)];
        }
    };
    fetch(T - 1);                                          // (the last steps are needed nearly always)

    // which hypothesis: every wave finds out for itself, lane = slot
    int status = 0, length = 0, last = -1, slot = 0;
    float value = -INFINITY;
    if (T >= 1) {
        if (best_rec && best_rec[b].have) {
            const BestCompleted r = best_rec[b];
            status = 1;
            length = r.len;
            value = r.score;
            last = r.step;
            slot = r.slot;
        } else {
            const size_t o = (size_t)b * k + (lane < k ? lane : 0);
            const float s = beam[o].score;
            const int l = beam[o].len;
            const bool live = lane < k && s > -INFINITY, done = live && (flags_of(beam[o].state) & kFinFinished) != 0;
            const u64 any_done = __ballot(done), any_live = __ballot(live);
            u64 among = any_live;                          // slots still in question; ties go to the lowest
            uint32_t image = 0;
            if (any_done) {
                // per-word score; already held by the beam when completed hypotheses are stored that way
                status = 1;
                if (done) image = ord_from_float(normalized ? s : __fdiv_rn(s, (float)l));
                among = any_done;
            } else if (any_live) {
                const uint32_t n = live ? 1u + (uint32_t)__popcll(beam[o].met) : 0u;
                const uint32_t most = wave_max_uniform(n);     // (every lane takes part)
                among = __ballot(live && n == most);
                if ((among >> lane) & 1ull) image = ord_from_float(s);
            }
            if (among) {
                const uint32_t top = wave_max_uniform(image);
                slot = __ffsll((long long)__ballot(((among >> lane) & 1ull) && image == top)) - 1;
                length = __builtin_amdgcn_readlane(l, slot);
                value = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(s), slot));
                last = T - 1;
            }
        }
    }
    length = __builtin_amdgcn_readfirstlane(length);
    last = __builtin_amdgcn_readfirstlane(last);
    slot = __builtin_amdgcn_readfirstlane(slot);
    if (threadIdx.x == 0) {
        out_len[b] = length;
        out_score[b] = value;
        out_status[b] = status;
    }
    const int ntoks = min(min(length, last + 1), N);       // steps 0 .. ntoks-1 give a token each
    for (int i = max(ntoks, 0) + (int)threadIdx.x; i < N; i += kFinWaves * kWave) toks[i] = pad_id;

    for (int hi = T - 1; hi >= 0 && last >= 0; hi -= kFinSteps) {
        if (hi != T - 1) fetch(hi);
#pragma unroll
        for (int i = 0; i < kFinRows; ++i) parent[i * kFinWaves + wave][lane] = (uint8_t)row[i];
        __syncthreads();
        if (wave == 0) {
            for (int t0 = min(hi, last); t0 > hi - kFinSteps && t0 >= 0; t0 -= kWave) {
                int mine = 0;                              // lane j: the slot at step t0 - j
                const int n = min(min(kWave, t0 + 1), t0 - (hi - kFinSteps));
                for (int j0 = 0; j0 < n; j0 += 8) {
                    int p[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) p[j] = parent[min(hi - t0 + j0 + j, kFinSteps - 1)][lane];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        if (lane == j0 + j) mine = slot;
                        if (j0 + j < n) slot = __builtin_amdgcn_readlane(p[j], slot & (kWave - 1));
                    }
                }
                const int t = t0 - lane;
                if (lane < n && t < ntoks) toks[t] = hist_token[at(t, min(mine, k - 1))];
            }
        }
        __syncthreads();
    }
}

// Diagnostic: the allocation of Sec. 3.2 alone, one wavefront per case.
__global__ void dba_allocate_kernel(int n_cases, int adjust, const int32_t *kk, const int32_t *CC,
                                    const int32_t *cnt, int32_t *alloc)
{
    const int i = blockIdx.x;
    if (i >= n_cases) return;
    const int lane = lane_id();
    const int C = CC[i];
    const int c = cnt[(size_t)i * 65 + lane];
    const int c64 = cnt[(size_t)i * 65 + 64];
    int a64;
    const int a = allocate_wave(kk[i], C, c, c64, a64, adjust != 0);
    alloc[(size_t)i * 65 + lane] = lane <= C ? a : 0;
    if (lane == 0) alloc[(size_t)i * 65 + 64] = C == 64 ? a64 : 0;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace {

thread_local char g_init_error[256] = "";

constexpr size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct Layout {
    size_t beam[2], sentences, rowlists, conskeys;
    size_t place_lists, place_keys;     // the same for steps of one launch, empty between steps
    size_t hist_token, hist_backptr;
    size_t fin_tokens, fin_len, fin_score, fin_status, all_finished, best;
    size_t total;
};

constexpr size_t kComputeUnits = 256;
constexpr size_t kOneLaunchRows = 22 * kComputeUnits / 4;   // no step of more beam rows takes one launch

// Grows with B, k and N and goes by nothing else, so that a workspace made for the largest job serves every smaller one: a shape
// has its places for steps of one launch whether it takes such steps or not.
Layout make_layout(size_t B, size_t k, size_t N)
{
    Layout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off = align_up(off + bytes, 256);
        return at;
    };
    for (int i = 0; i < 2; ++i) L.beam[i] = take(B * k * sizeof(Hyp));
    L.sentences = take(B * sizeof(Sentence));
    L.rowlists = take(B * k * kWave * sizeof(u64));
    L.conskeys = take(B * k * kMaxCons * sizeof(u64));
    const size_t places = std::min(B * k, kOneLaunchRows);
    L.place_lists = take(places * kWave * sizeof(u64));
    L.place_keys = take(places * kMaxCons * sizeof(u64));
    L.hist_token = take(N * B * k * sizeof(int32_t));
    L.hist_backptr = take(N * B * k * sizeof(int32_t));
    L.fin_tokens = take(B * N * sizeof(int32_t));
    L.fin_len = take(B * sizeof(int32_t));
    L.fin_score = take(B * sizeof(float));
    L.fin_status = take(B * sizeof(int32_t));
    L.all_finished = take(B);
    L.best = take(B * sizeof(BestCompleted));
    L.total = off;
    return L;
}

// Up to this many bytes of tokens dba_finalize brings over together with the other results: 58 against 74 us with the
// tokens on their own for 512000 bytes into ordinary memory, 57 against 50 into pinned memory; 78 / 75 and 77 / 53 at 716800,
// 810 / 520 and 810 / 200 at 8 MB.
bool staged_tokens(size_t B, size_t N) { return B * N * 4 <= 512 * 1024; }

constexpr size_t kLdsPerUnit = 160 * 1024;
constexpr size_t kLdsPerLaunch = 64 * 1024;   // what a launch may ask for as it is

// LDS to add to a stream-phase workgroup of NW waves so that no more than n <= MOST of them fit a compute unit
template <int NW, int MOST>
constexpr size_t spread_lds(size_t n)
{
    static_assert(sizeof(StreamSmem<NW>) <= kLdsPerUnit / (MOST + 1), "a workgroup's own LDS leaves room for MOST + 1 of them");
    return align_up(kLdsPerUnit / (n + 1) + 1 - sizeof(StreamSmem<NW>), 256);
}

// Where steps may take one launch, whatever their rows are made of: up to k = 16, where four waves merge as fast as eight, while a
// compute unit has five or six rows of four waves (seven waves of this kernel fit a SIMD, by its scalar registers, and the sentences'
// workgroups need room beside the rows); with two rows a unit up to k = 32, where the rows have eight waves.  Per step, two launches /
// one: 768 rows of 32000 fp32, k = 12, 24.2 / 23.2 us, 1152 of 32003 bf16 20.9 / 19.5, 1280, k = 16, 32.8 / 32.2, 1275 of 16000 22.0 / 20.8, 1024
// of 8000 14.5 / 13.9, 960 of 2000 11.7 / 10.8, 600 of 1000 11.0 / 10.5; but 1700 of 32000 41.6 / 43.3, 1600 of 2000 13.2 / 14.6, 5000 of 2000
// 22.0 / 24.5, and with k = 20 to 32 and four waves 1280 of 32000 34.2 / 34.3, 2048 49.6 / 51.1.  Vocabularies of a few
// hundred keep two launches beyond two rows a unit, where one would be less again: 600 rows of 300 9.85 / 7.7, 1024, k = 8, 10.5 / 8.2, 1408, k = 16, 11.75 /
// 10.8, as from 512 tokens on, 1408 of 520, k = 16, 11.8 / 10.85.
bool one_launch_shape(size_t B, size_t k, size_t V)
{
    const size_t rows = B * k;
    if (rows <= 2 * kComputeUnits) return k <= 32;
    return rows <= kOneLaunchRows && (k <= 16 ? V >= 512 : k <= 28 && V >= 4096);
}

// How the stream phase of a step is launched: one workgroup per beam row, and
struct StreamPlan {
    bool one;               // launch does for the whole step, if the options leave it open,
    bool sentence;          // with one workgroup per sentence
    int waves;              // of a workgroup: 4 or 8
    int tiles;              // of 4 KB that each wave keeps in flight
    size_t spare_lds;       // LDS a workgroup asks for and does not use, which keeps others off its compute unit
    uint32_t rows_abreast;  // rows of the sentences that are numbered eight abreast
};

// free: the options leave the number of launches open
StreamPlan stream_plan(size_t B, size_t k, size_t V, unsigned elem, bool free)
{
    StreamPlan plan;
    const size_t rows = B * k, row_bytes = V * elem;
    // Sentences eight abreast (see the kernel) where rows are shorter than 512000 bytes: the rows a die streams at a
    // time lie one after the other (per step, k = 64, fp32, eight abreast / row by row: 64 sentences of 70000 tokens
    // 183.1 / 189.2 us, 98304 252.9 / 256.4, 110000 283.6 / 292.4, 125000 322.6 / 328.0; 64 of 65536 the other way, 174.9 / 172.9).
    // Beyond, they gain nothing (128000 334.2 / 330.0, 131000 343.2 / 340.2), and rows a large power of two apart
    // keep asking the same part of the die's L2 (64 of 131072 376.6 / 331.6, 16 of 262144 217.2 / 183.6) - but only
    // where a die has many of them at a time: below two rows per compute unit eight abreast stays ahead (32 sentences,
    // k = 8, 131072 tokens 28.3 / 29.5 us, 34 and 159134 45.5 / 46.3, 16, k = 20, 131072 41.5 / 41.8; 8, k = 64, 131072 the other
    // way, 59.3 / 57.9).
    plan.rows_abreast = row_bytes < 512000 || rows < 2 * kComputeUnits ? (uint32_t)((B & ~(size_t)7) * k) : 0;
    // Waves per beam row (measured on MI355X, fp32 and 16-bit inputs, 10 to 8192 rows): eight where the
    // grid cannot fill the chip by itself (at most two rows per compute unit) and a row has work for
    // them, and where rows are long (from 160 KB on: the floor then rests on a larger share of the
    // row and fewer sums are looked at closely); four otherwise - with rows of 64-128 KB and
    // thousands of them, twice the workgroups per compute unit stream faster than twice the waves.
    // Eight also where that lets a step of k = 17 to 28 with short rows take one launch (see below).
    const bool wide_short = free && rows <= 2 * kComputeUnits && k > 16 && k <= 28 && elem == 4 && row_bytes <= 28 * 1024;
    plan.waves = ((rows <= 2 * kComputeUnits && (row_bytes >= 32768 || wide_short)) || row_bytes >= 163840) ? 8 : 4;
    // One launch for the whole step where the shape allows it and a row's workgroup has the waves to merge with: beyond k = 16
    // eight; beyond two rows a compute unit as long as their waves leave room.  Per step, two launches / one, 16 to 512 rows of 100 to 32000 elements:
    // with k up to 8 0.4 to 1.4 us less, 9 to 11 0.1 to 0.9, 12 to 16 0.6 to 1.4; k = 17 to 32 with eight waves 0.7 to 1.35 (500 rows of
    // 32000, k = 20, 19.95 / 18.8; 256 rows, k = 32, 16.5 / 15.45), but with four waves up to 0.35 more at k = 18, 0.5 at 24, 0.9 at 28 and 1.2 at
    // 32.  So short rows get eight too, though most of these have no tile, to k = 28 (fp32, two launches with four / one with eight: 200
    // rows of 2000, k = 20, 10.3 / 9.7 us, 126 of 4000, k = 18, 10.8 / 9.75, 504 11.7 / 10.8, 448 of 7000, k = 28, 13.0 / 12.2; 512 of 5000, k = 32, 12.8 /
    // 13.5; 16-bit rows gain less, 240 of 6000, k = 20, 11.15 / 10.7, and are left as they are; so are rows of 28 to 32 KB, where one
    // launch with eight waves would be less as well: 144 of 7800, k = 24, 11.85 / 10.65, 500 of 7500, k = 20, 12.75 / 12.0, 504 of 8100, k = 28, 13.65 / 12.9).
    // Beyond two rows a unit 16-bit rows also with k = 17 to 28 and four waves: there are half the bytes in front of what one launch
    // saves (bf16, 544 rows of 32000, k = 17, 18.35 / 17.6, 1080, k = 24, 22.75 / 22.0, 1200 of 8000, k = 20, 15.9 / 15.2, 1400 of 16000, k =
    // 28, 21.45 / 20.9; k = 32 equal).  But three such decodes side by side are 3 to 4 % slower than with two launches where the rows are 64 KB (3 x 1280 of 32000, k =
    // 20, 40.9 / 42.5, 3 x 1152 of 32003, k = 12, 37.1 / 38.5; two of them 33.1 / 30.9 and 29.8 / 28.2, three with rows of 32 KB 26.4 / 23.1): the sentences' workgroups hold room that
    // rows of the others could have, whatever LDS is left unused, however often they look and whenever they give up.  fp32 stays at two, where the difference is
    // small and changes sign: 1080 of 12000, k = 18, 18.1 / 17.8, 527 of 32000, k = 17, 23.15 / 22.5, 960 of 16000, k = 24, equal, 1280 of 32000, k = 20, 34.0 / 34.25, 1400 of
    // 24000, k = 28, 31.35 / 31.65.
    plan.one = free && one_launch_shape(B, k, V) &&
               (rows <= 2 * kComputeUnits ? k <= 16 || plan.waves == 8
                                          : rows * plan.waves <= 22 * kComputeUnits && (k <= 16 || (elem == 2 && plan.waves == 4)));
    // One workgroup for a whole sentence where its rows are short and few: eight tiles in all (a partial one takes as long as a whole one; per step,
    // a workgroup per row / per sentence, 40 sentences, fp32: k = 8, 1024 tokens 8.15 / 7.75 us, 4, 2048 7.85 / 7.6, 5, 1000 8.2 / 7.55, but 5, 1638 8.3 / 8.55,
    // 3, 2730 8.1 / 8.25), and no more sentences than three for a compute unit (700, k = 2, 1000 tokens 10.5 / 8.95; 1300, k = 1, 11.3 / 14.5).
    const size_t tiles = (row_bytes + 4095) / 4096;
    plan.sentence = plan.one && k * tiles <= kSentenceWaves && tiles <= 4 && B <= 3 * kComputeUnits;
    // Rows side by side on a compute unit.  More than a unit's even share leaves others short, and lets a
    // second decode's rows in beside the first one's: where the grid fills the chip, no more than that share
    // (three decodes of 64 x 20 rows of 32000 in flight: 84 against 94 us for three steps, one of them alone
    // unchanged; 1152 rows of 32003 bf16: 22.8 against 23.1 us per step).  Where rows follow one another, six
    // waves per SIMD instead of the eight that fit: fewer streams at a time then serve memory better (8192 rows
    // of 50000, k = 64: 263 against 267 us per step in fp32, 146 against 148.5 with fp16; 8000 rows of 32000 bf16: 92.2
    // against 93.3; 2048 rows of 32000, all resident with eight: 50.9 against 49.6) - but only from 48 KB on: shorter rows
    // are latency more than traffic, and take all eight (2200 rows of 8000 fp32: 24.7 against 26.2 us per step with six, 8000
    // rows 54.1 against 58.5, 8192 of 2000 41.8 against 48.7, 8000 of 16000 bf16 60.1 against 65.8; at 48000 bytes 0 to 4 %
    // less up to 4000 rows, 0 to 1.4 % more at 8000 and above).  Workgroups are kept apart by LDS they do not use; at
    // least a tenth of a unit's LDS stays free for other work.
    const size_t share = (rows + kComputeUnits - 1) / kComputeUnits;
    plan.spare_lds = plan.one            ? 0               // (the sentences' workgroups are to find room beside the rows)
                     : plan.waves == 8 ? (share > 4 ? spread_lds<8, 3>(3) : 0)
                     : share <= 4 || share == 8 || (share > 8 && row_bytes < 49152) ? 0
                                                : spread_lds<4, 7>(share < 8 ? share : 6);
    // Tiles in flight per wave: four where every row has a compute unit to itself and its latencies show
    // (per step: 14.7 -> 13.7 us for 160 rows of 32000 fp32, 16.0 -> 15.0 for 168 of 50001, 26.6 -> 25.0 for 240 of
    // 100000); two beyond (480 rows of 50000: 24.8 against 25.8 with four).  In one launch the registers of two tiles leave
    // room for a sentence's workgroup beside two rows (59 against 89; per step, four / two: 400 rows of 32000 fp32 18.3 / 17.65 us, 320
    // 17.1 / 16.8, 480 of 50000 25.7 / 25.05, 400 of 58000 26.1 / 25.25, 400 of 32000 bf16 16.25 / 15.75, 480 of 65000 bf16 20.35 / 19.45; four
    // decodes of 512 rows of 32000 bf16 side by side 35.1 / 29.7), but long rows are traffic more than latency again, from
    // seven tiles a wave on, six with two elements in the place of one (240 KB: fp32 22.55 / 22.65 and 28.1 / 28.25, bf16 21.55 / 22.85;
    // 200 KB: bf16 20.35 / 20.85 and 26.55 / 26.8; 400 KB: fp32 30.05 / 31.2 and 39.45 / 40.0, at 260 and 500 rows).
    const bool long_rows = row_bytes >= (elem == 4 ? 7u : 6u) * 8 * 4096;
    plan.tiles = plan.waves == 8 && (rows <= kComputeUnits || (plan.one && rows <= 2 * kComputeUnits && long_rows)) ? 4 : 2;
    return plan;
}

// Whether any step of this shape hands its keys over in places that must be empty: the element type decides, step by step.
bool hands_over(size_t B, size_t k, size_t V)
{
    for (const unsigned elem : {4u, 2u}) {
        const StreamPlan plan = stream_plan(B, k, V, elem, true);
        if (plan.one && !plan.sentence) return true;
    }
    return false;
}

// How often a sentence's workgroup looks for the rows' keys: a look takes about a microsecond, and the rows two to four times
// less than these, as many as at 2 TB/s.  Beyond, the row that ends last takes the sentence on, which costs the step the 2 us
// that one launch saves.
int most_tries(size_t rows, size_t row_bytes) { return 64 + (int)std::min(rows * row_bytes >> 21, (size_t)1 << 20); }

int bits_for(int v)   // bits needed to hold values 0..v
{
    int n = 0;
    while ((1 << n) <= v) ++n;
    return n;
}

}  // namespace

// ---------------------------------------------------------------------------
// scratch owned by the library, for dba_step_noalloc
// ---------------------------------------------------------------------------
// The two arrays that pass a step's results from its first launch to its second (every row's list
// and its constraint keys, 64 keys of 8 bytes each) for up to DBA_NOALLOC_MAX_ROWS beam rows: 8 MiB,
// present once on every GPU the library runs on, until the process ends.
constexpr size_t kStaticRows = DBA_NOALLOC_MAX_ROWS;
constexpr size_t kStaticListBytes = kStaticRows * kWave * sizeof(u64);
constexpr size_t kStaticScratchBytes = kStaticListBytes + kStaticRows * kMaxCons * sizeof(u64);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];       // device address of `scratch` on each GPU (its name is a host-side stand-in)
std::mutex g_scratch_mutex;

// Device address of `scratch` on the current device: asked for once per device, kept afterwards.
hipError_t static_scratch(void **out)
{
    *out = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> hold(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

namespace {

// For calls that are no part of a stream capture which this or another thread may have under way.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool exchanged = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    RelaxedCapture() = default;
    RelaxedCapture(const RelaxedCapture &) = delete;
    RelaxedCapture &operator=(const RelaxedCapture &) = delete;
    ~RelaxedCapture()
    {
        if (exchanged) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
};

// Pinned host memory that kernels read and write themselves: a copy to or from ordinary host memory costs about 8
// us and a wait of its own (a decode with the stopping test asked for after each of its 21 steps, 8 x 10 x 32000: 814 -> 641
// us; one of 100 steps, 64 x 20 x 32000: 3360 -> 3294).  A ctx holds one block from dba_init to dba_destroy; blocks are kept for the next
// ctx, of any thread and device, and what is more than the store keeps is freed.  No kernel uses a block any more when it
// comes back, or its words tell when (put_when).
struct PinnedMemory {
    static void *allocate(size_t n)
    {
        const RelaxedCapture relaxed;
        void *p = nullptr;
        if (hipHostMalloc(&p, n, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess) return p;
        (void)hipGetLastError();
        return nullptr;
    }
    static void release(void *p)                           // (waits for the GPU)
    {
        const RelaxedCapture relaxed;
        if (hipHostFree(p) != hipSuccess) (void)hipGetLastError();
    }
};

HostBlocks<PinnedMemory> &host_blocks()
{
    static auto *blocks = new HostBlocks<PinnedMemory>;    // (outlives every ctx: never destroyed)
    return *blocks;
}

// A launch that tells how it went, so that of one that failed it is known that no kernel of it is under way: hipGetLastError, behind the <<< >>> form,
// may tell of an earlier call on this thread, of whomever, and takes that error from its owner.  (Nor does this one pass its grid through the runtime first: a step's call takes 2.85 instead of 3.05
// us with one launch and 5.27 instead of 5.65 with two, which is the time of a step where short ones of several decodes alternate.)
template <typename... P, typename... A>
hipError_t launch(void (*kernel)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream, const A &...a)
{
    auto with = [&](P... arg) {
        void *args[] = {&arg...};
        return hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, args, lds, stream);
    };
    return with(a...);
}

}  // namespace

struct dba_ctx {
    int B, k, V, N, eos_id, pad_id;
    int met_bits;
    int tok_bits;
    int max_phrases;
    int steps;
    int adjust;                         // DBA_OPT_ADJUSTMENT
    int normalize;                      // DBA_OPT_NORMALIZE_FINISHED
    float prune;                        // DBA_OPT_PRUNE_THRESHOLD (< 0: off)
    int track;                          // DBA_OPT_TRACK_COMPLETED
    int merge_waves;                    // DBA_OPT_MERGE_WAVES (0: chosen here)
    int device;                         // the device that was current at dba_init
    unsigned char *lib_scratch;         // this device's copy of the library's own scratch (null: not resolved)
    int cand_cap;                       // candidates of one sentence at most, in whole chunks of 64
    size_t dyn_smem;
    unsigned char *ws;
    Layout L;
    HostBlock block;                    // seen words [B] (then what steps tell), stopping flags [B], then constraint words / results (p null: none)
    size_t block_flags, block_data;     // offsets in it
    bool one_launch;                    // the row lists are empty between steps, which may then be one launch each
    int give_up;                        // dba_debug_sentences_first
    bool init_under_way;                // the kernel of dba_init may not be through: nothing has waited for it yet
    // Once the stopping flags have been asked for, steps write them to the block themselves: no kernel of its own has to bring them over.
    // (a decode of 21 steps asked after each, 8 x 10 x 32000: 614 -> 589 us; the rest of a question is the wait for the stream, 8 us of it
    // after the last store).  Not those recorded into a graph, which may run when the ctx is gone, and none from there on: a replay may be what ran last.
    bool asked, recorded;
    int told;                           // steps taken when the last one that did so had been launched (0: none),
    bool told_under_way;                // and whether nothing has waited for it yet
    hipStream_t stream;
    char err[256];
};

namespace {

int fail(dba_ctx *ctx, int code, const char *fmt, ...)
{
    char *dst = ctx ? ctx->err : g_init_error;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(dst, 256, fmt, ap);
    va_end(ap);
    return code;
}

bool shape_ok(int B, int k, int V, int N, int max_cons)
{
    return B >= 1 && B <= 65535 && k >= 1 && k <= DBA_MAX_BEAM && V >= 1 && N >= 1 && k <= V && max_cons >= 0 &&
           max_cons <= DBA_MAX_CONS_TOKENS;
}

template <typename T>
T *at(dba_ctx *c, size_t off)
{
    return reinterpret_cast<T *>(c->ws + off);
}

void set_tables(dba_ctx *c, StepParams &p)
{
    const Layout &L = c->L;
    p.sentences = at<Sentence>(c, L.sentences);
    p.all_finished = at<uint8_t>(c, L.all_finished);
    p.best = at<BestCompleted>(c, L.best);
}

// the kernel of dba_init sets a word of the block for every sentence when it is through with it
bool init_is_through(const dba_ctx *c)
{
    const uint32_t *seen = reinterpret_cast<const uint32_t *>(c->block.p);
    for (int b = 0; seen && b < c->B; ++b)
        if (__atomic_load_n(seen + b, __ATOMIC_RELAXED) == 0) return false;
    return true;
}

}  // namespace

extern "C" {

DBA_API size_t dba_workspace_bytes(int B, int k, int V, int N, int max_cons_tokens)
{
    if (!shape_ok(B, k, V, N, max_cons_tokens)) return 0;
    return make_layout((size_t)B, (size_t)k, (size_t)N).total;
}

// dba_init proper; may throw std::bad_alloc from its host tables (caught by dba_init)
static int init_impl(dba_ctx **out, int B, int k, int V, int N, int eos_id, int pad_id,
                     const int32_t *cons_tokens, const int32_t *phrase_offsets,
                     const int32_t *sent_offsets, void *workspace_dev, size_t workspace_bytes,
                     void *hip_stream)
{
    if (!out) return fail(nullptr, DBA_EINVAL, "dba_init: out is NULL");
    *out = nullptr;
    if (!shape_ok(B, k, V, N, 0))
        return fail(nullptr, DBA_EINVAL,
                    "dba_init: need 1 <= B <= 65535, V,N >= 1 and 1 <= k <= %d, k <= V (got B=%d k=%d V=%d N=%d)",
                    DBA_MAX_BEAM, B, k, V, N);
    if (eos_id < 0 || eos_id >= V || pad_id < 0 || pad_id >= V || eos_id == pad_id)
        return fail(nullptr, DBA_EINVAL, "dba_init: eos_id/pad_id must be distinct ids in [0,V)");
    if (!sent_offsets || !phrase_offsets)
        return fail(nullptr, DBA_EINVAL, "dba_init: sent_offsets / phrase_offsets is NULL");
    if (!workspace_dev) return fail(nullptr, DBA_EINVAL, "dba_init: workspace_dev is NULL");
    if (reinterpret_cast<uintptr_t>(workspace_dev) % 256 != 0)
        return fail(nullptr, DBA_EINVAL, "dba_init: workspace_dev must be 256-byte aligned");

    // constraints -> fixed-stride per-sentence tables
    if (sent_offsets[0] != 0 || phrase_offsets[0] != 0)
        return fail(nullptr, DBA_EINVAL, "dba_init: offsets must start at 0");
    // sent_offsets[B] is the length of phrase_offsets minus one: nothing beyond it is read
    for (int b = 0; b < B; ++b)
        if (sent_offsets[b + 1] < sent_offsets[b])
            return fail(nullptr, DBA_EINVAL, "dba_init: sent_offsets decreases at %d", b);
    // The constraint words go to a block of host memory that the kernel of dba_init reads itself, or, where there
    // is none (large batches), through a copy to the workspace.  (Opening a session, the caller's allocations included, with
    // all tables made on the host, copied and waited for / like this: one sentence 51 / 38 us, 64 sentences 119 / 48.)
    const Layout L = make_layout((size_t)B, (size_t)k, (size_t)N);
    const size_t words_bytes = (size_t)B * kMaxCons * sizeof(uint32_t);
    struct Holder {
        HostBlock block;
        ~Holder() { host_blocks().put(block); }
    } held;
    const size_t block_flags = (size_t)B * sizeof(uint32_t), block_data = align_up(block_flags + (size_t)B, 256);
    const size_t results_bytes = L.fin_status + (size_t)B * 4 - (staged_tokens((size_t)B, (size_t)N) ? L.fin_tokens : L.fin_len);
    held.block = host_blocks().get(block_data + std::max(words_bytes, results_bytes));
    std::vector<uint32_t> own_words;
    if (!held.block.p) own_words.resize((size_t)B * kMaxCons);
    uint32_t *words = held.block.p ? reinterpret_cast<uint32_t *>(held.block.p + block_data) : own_words.data();
    std::fill(words, words + (size_t)B * kMaxCons, kNoToken);
    int max_tokens = 0, max_phrases = 0;
    for (int b = 0; b < B; ++b) {
        const int p0 = sent_offsets[b], p1 = sent_offsets[b + 1];
        const int t0 = phrase_offsets[p0];
        int n = 0;
        for (int p = p0; p < p1; ++p) {
            const int a = phrase_offsets[p], e = phrase_offsets[p + 1];
            if (e <= a) return fail(nullptr, DBA_EINVAL, "dba_init: phrase %d is empty or offsets decrease", p);
            if (a - t0 != n)
                return fail(nullptr, DBA_EINVAL, "dba_init: phrase offsets of sentence %d are not contiguous", b);
            if (n + (e - a) > DBA_MAX_CONS_TOKENS)
                return fail(nullptr, DBA_EINVAL, "dba_init: sentence %d has more than %d constraint tokens", b,
                            DBA_MAX_CONS_TOKENS);
            if (!cons_tokens) return fail(nullptr, DBA_EINVAL, "dba_init: cons_tokens is NULL");
            for (int i = a; i < e; ++i) {
                const int w = cons_tokens[i];
                if (w < 0 || w >= V)
                    return fail(nullptr, DBA_EINVAL, "dba_init: constraint token %d outside [0,V)", w);
                if (w == eos_id || w == pad_id)
                    return fail(nullptr, DBA_EINVAL, "dba_init: eos_id/pad_id cannot be a constraint token");
                words[(size_t)b * kMaxCons + n++] = (uint32_t)w | (i == a ? kBeginsPhrase : 0u);
            }
        }
        if (n > max_tokens) max_tokens = n;
        if (p1 - p0 > max_phrases) max_phrases = p1 - p0;
    }
    // a coordinate is (slot << tok_bits) | token; with the bank it must fit the 32 bits the
    // selection key has beside the score
    const int met_bits = bits_for(max_tokens);
    const int tok_bits = bits_for(V - 1) < 1 ? 1 : bits_for(V - 1);
    const int slot_bits = bits_for(k - 1);
    if (met_bits + slot_bits + tok_bits > 32 || tok_bits > 24)
        return fail(nullptr, DBA_EINVAL,
                    "dba_init: bits(k-1)=%d + bits(V-1)=%d + bits(max constraint tokens)=%d exceed the 32-bit "
                    "coordinate field of the selection key (or V > 2^24)", slot_bits, tok_bits, met_bits);

    if (workspace_bytes < L.total)
        return fail(nullptr, DBA_ENOMEM, "dba_init: workspace has %zu bytes, %zu needed", workspace_bytes, L.total);

    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(static_cast<hipStream_t>(hip_stream), &capture) != hipSuccess) (void)hipGetLastError();
    else if (capture != hipStreamCaptureStatusNone)
        return fail(nullptr, DBA_EHIP, "dba_init: HIP error: %s", hipGetErrorString(hipErrorStreamCaptureUnsupported));
    dba_ctx *c = new (std::nothrow) dba_ctx();
    if (!c) return fail(nullptr, DBA_ENOMEM, "dba_init: out of host memory");
    c->B = B; c->k = k; c->V = V; c->N = N; c->eos_id = eos_id; c->pad_id = pad_id;
    c->met_bits = met_bits;
    c->tok_bits = tok_bits;
    c->max_phrases = max_phrases;
    c->steps = 0;
    c->ws = static_cast<unsigned char *>(workspace_dev);
    c->L = L;
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->adjust = 1;
    c->normalize = 0;
    c->prune = -1.0f;
    c->track = 0;
    c->merge_waves = 0;
    c->device = -1;
    (void)hipGetDevice(&c->device);
    void *own = nullptr;
    (void)static_scratch(&own);          // dba_step_noalloc asks again (and reports) if this failed
    c->lib_scratch = static_cast<unsigned char *>(own);
    // candidates of one sentence: at most k best + k row bests + k * phrases constraint tokens,
    // in whole chunks of 64 keys
    const int ncand_max = (k * (max_phrases + 2) + kWave - 1) / kWave * kWave;
    c->cand_cap = ncand_max;
    constexpr size_t most_cand = (size_t)DBA_MAX_BEAM * (DBA_MAX_CONS_TOKENS + 2) * sizeof(u64) + kMostLeft * (sizeof(u64) + sizeof(int));
    static_assert(sizeof(MergeSmem<16>) + 16 + most_cand <= kLdsPerLaunch, "k = 64 with 64 phrases: 45 KB beside the merge phase's own 18");
    c->dyn_smem = (size_t)ncand_max * sizeof(u64) + (ncand_max > 4 * kWave ? kMostLeft * (sizeof(u64) + sizeof(int)) : 0);

    // (without a block the words pass through the row lists' place, which is large enough and not in use yet)
    hipError_t e = hipSuccess;
    uint32_t *seen = nullptr;
    if (held.block.p) {
        seen = reinterpret_cast<uint32_t *>(held.block.p);
        memset(seen, 0, (size_t)B * sizeof(uint32_t));
    } else {
        e = hipMemcpyAsync(c->ws + L.rowlists, words, words_bytes, hipMemcpyHostToDevice, c->stream);
        words = at<uint32_t>(c, L.rowlists);
    }
    if (e == hipSuccess) {
        StepParams p = {};
        set_tables(c, p);
        p.beam_nxt = at<Hyp>(c, L.beam[0]);
        c->one_launch = seen != nullptr && one_launch_shape((size_t)B, (size_t)k, (size_t)V);
        if (c->one_launch && hands_over((size_t)B, (size_t)k, (size_t)V)) {
            p.rowlists = at<u64>(c, L.place_lists);
            p.conskeys = at<u64>(c, L.place_keys);
        }
        e = launch(dba_init_kernel, (unsigned)B, kWave, 0, c->stream, B, k, words, seen, p);
    }
    if (e == hipSuccess && !seen) e = hipStreamSynchronize(c->stream);   // the words are freed on return
    if (e != hipSuccess) {
        const int rc = fail(nullptr, DBA_EHIP, "dba_init: HIP error: %s", hipGetErrorString(e));
        delete c;
        return rc;
    }
    c->block = held.block;
    c->block_flags = block_flags;
    c->block_data = block_data;
    c->init_under_way = seen != nullptr;
    held.block.p = nullptr;
    *out = c;
    return DBA_OK;
}

DBA_API int dba_init(dba_ctx **out, int B, int k, int V, int N, int eos_id, int pad_id,
             const int32_t *cons_tokens, const int32_t *phrase_offsets,
             const int32_t *sent_offsets, void *workspace_dev, size_t workspace_bytes,
             void *hip_stream)
{
    try {
        return init_impl(out, B, k, V, N, eos_id, pad_id, cons_tokens, phrase_offsets, sent_offsets,
                         workspace_dev, workspace_bytes, hip_stream);
    } catch (...) {                                        // nothing crosses the C boundary
        if (out) *out = nullptr;
        return fail(nullptr, DBA_ENOMEM, "dba_init: out of host memory");
    }
}

DBA_API int dba_step(dba_ctx *c, const float *logp_dev, int32_t *out_token_dev, int32_t *out_backptr_dev,
             float *out_score_dev, uint8_t *out_flags_dev)
{
    return dba_step_fmt(c, logp_dev, DBA_LOGP_F32, out_token_dev, out_backptr_dev, out_score_dev, out_flags_dev);
}

// One step.  own_scratch: the row lists and constraint keys go through the library's own scratch
// (given here as its device address) instead of the workspace.
static int step_impl(dba_ctx *c, const void *logp_dev, int logp_format, int32_t *out_token_dev,
                     int32_t *out_backptr_dev, float *out_score_dev, uint8_t *out_flags_dev,
                     unsigned char *own_scratch)
{
    if (!c) return DBA_EINVAL;
    if (!logp_dev) return fail(c, DBA_EINVAL, "dba_step: logp_dev is NULL");
    if (logp_format != DBA_LOGP_F32 && logp_format != DBA_LOGP_F16 && logp_format != DBA_LOGP_BF16)
        return fail(c, DBA_EINVAL, "dba_step: unknown log-prob format %d", logp_format);
    const unsigned elem = logp_format == DBA_LOGP_F32 ? 4u : 2u;
    if (reinterpret_cast<uintptr_t>(logp_dev) % elem != 0)
        return fail(c, DBA_EINVAL, "dba_step: logp_dev must be aligned to its element size (%u bytes)", elem);
    if (c->steps >= c->N) return fail(c, DBA_ESTATE, "dba_step: all N=%d steps have been taken", c->N);

    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (!c->recorded && (hipStreamIsCapturing(c->stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone)) {
        if (capture == hipStreamCaptureStatusNone) (void)hipGetLastError();
        c->recorded = true;
    }
    const bool tells = c->asked && !c->recorded && c->block.p;
    // one workgroup per beam row, 4 loads of 16 bytes per lane and tile, two or four 4 KB tiles in flight per wave
    const StreamPlan plan = stream_plan((size_t)c->B, (size_t)c->k, (size_t)c->V, elem, c->one_launch && c->merge_waves == 0);
    const int cur = c->steps & 1;
    const Layout &L = c->L;
    StepParams p;
    p.B = c->B; p.k = c->k; p.V = c->V;
    p.eos_id = c->eos_id; p.pad_id = c->pad_id;
    p.met_bits = c->met_bits;
    p.tok_bits = c->tok_bits;
    p.first_step = c->steps == 0 ? 1 : 0;
    p.cand_cap = c->cand_cap;
    p.adjust = c->adjust;
    p.normalize = c->normalize;
    p.prune = c->prune;
    p.track = c->track;
    p.step = c->steps;
    p.logp = logp_dev;
    p.beam = at<Hyp>(c, L.beam[cur]);
    p.beam_nxt = at<Hyp>(c, L.beam[cur ^ 1]);
    set_tables(c, p);
    p.rowlists = own_scratch ? reinterpret_cast<u64 *>(own_scratch) : at<u64>(c, L.rowlists);
    p.conskeys = own_scratch ? reinterpret_cast<u64 *>(own_scratch + kStaticListBytes) : at<u64>(c, L.conskeys);
    p.told = tells ? reinterpret_cast<uint32_t *>(c->block.p) : nullptr;
    p.out_token = out_token_dev;
    p.out_backptr = out_backptr_dev;
    p.out_score = out_score_dev;
    p.out_flags = out_flags_dev;
    const size_t hrow = (size_t)c->steps * c->B * c->k;
    p.hist_token = at<int32_t>(c, L.hist_token) + hrow;
    p.hist_backptr = at<int32_t>(c, L.hist_backptr) + hrow;

    hipError_t e = hipSuccess;
    const dim3 grid((unsigned)c->B * (unsigned)c->k);
    const uint32_t inv_k = (uint32_t)(((1ull << 32) + (unsigned)c->k - 1) / (unsigned)c->k);
    const int kf = p.k | (p.first_step << 16);
    const uint32_t inv_k16 = (uint32_t)(c->k == 1 ? 65535 : 65536 / c->k + 1);
    if (plan.sentence) {
        const size_t lds = align_up(sizeof(MergeSmem<4>), 16) + c->dyn_smem;
        static_assert(sizeof(SentenceSmem) + sizeof(MergeSmem<4>) + 16 + (size_t)kSentenceWaves * (DBA_MAX_CONS_TOKENS + 2) * sizeof(u64) + 64 * sizeof(u64) +
                      kMostLeft * (sizeof(u64) + sizeof(int)) <= kLdsPerLaunch, "beside the rows' LDS");
#define SENTENCE(FMT) e = launch(dba_sentence_kernel<FMT>, (unsigned)c->B, kSentenceWaves * kWave, lds, c->stream, p.logp, p.V, kf, inv_k16, p)
        switch (logp_format) {
            case DBA_LOGP_F16: SENTENCE(kFmtF16); break;
            case DBA_LOGP_BF16: SENTENCE(kFmtBF16); break;
            default: SENTENCE(kFmtF32); break;
        }
#undef SENTENCE
    } else if (plan.one) {
        // (places that no step of two launches writes to: they are empty between steps, whatever the steps before took)
        p.rowlists = at<u64>(c, L.place_lists);
        p.conskeys = at<u64>(c, L.place_keys);
        const dim3 sblock((unsigned)(plan.waves * kWave)), sgrid((unsigned)c->B * (unsigned)(c->k + 1));
        const int mw = c->k <= 16 || plan.waves == 4 ? 4 : 8;
        const size_t lds = std::max(plan.waves == 8 ? sizeof(StreamSmem<8>) : sizeof(StreamSmem<4>),
                                    align_up(mw == 4 ? sizeof(MergeSmem<4>) : sizeof(MergeSmem<8>), 16) + c->dyn_smem);
        const int tries = c->give_up ? 0 : most_tries((size_t)c->B * (size_t)c->k, (size_t)c->V * elem);
        const uint32_t rows_order = (unsigned)c->B * (unsigned)c->k | ((c->give_up & 1) ? 0x80000000u : 0u);
#define ONE(FMT, NW, D, ROWS, MW, J)                                                                                       \
    e = launch(dba_step_kernel<kTileLoads, FMT, NW, D, ROWS, MW, J>, sgrid, sblock, lds, c->stream, p.logp, p.V, kf, plan.rows_abreast, \
               inv_k, rows_order, inv_k16, tries, p)
#define ONE_ANY(NW, D, ROWS, MW, J)                                       \
    switch (logp_format) {                                      \
        case DBA_LOGP_F16: ONE(kFmtF16, NW, D, ROWS, MW, J); break;       \
        case DBA_LOGP_BF16: ONE(kFmtBF16, NW, D, ROWS, MW, J); break;     \
        default: ONE(kFmtF32, NW, D, ROWS, MW, J); break;                 \
    }
#define ONE_16(NW, D, ROWS, MW, J)                                        \
    switch (logp_format) {                                      \
        case DBA_LOGP_F16: ONE(kFmtF16, NW, D, ROWS, MW, J); break;       \
        default: ONE(kFmtBF16, NW, D, ROWS, MW, J); break;                \
    }
        if (plan.waves == 8 && plan.tiles == 4) {
            if (c->k <= 8) ONE_ANY(8, 4, 2, 4, 1)
            else if (c->k <= 11) ONE_ANY(8, 4, 4, 4, 2)
            else if (c->k <= 16) ONE_ANY(8, 4, 4, 4, -1)
            else ONE_ANY(8, 4, 4, 8, -1)
        } else if (plan.waves == 8) {
            if (c->k <= 8) ONE_ANY(8, 2, 2, 4, 1)
            else if (c->k <= 11) ONE_ANY(8, 2, 4, 4, 2)
            else if (c->k <= 16) ONE_ANY(8, 2, 4, 4, -1)
            else ONE_ANY(8, 2, 4, 8, -1)
        } else {
            if (c->k <= 8) ONE_ANY(4, 2, 2, 4, 1)
            else if (c->k <= 11) ONE_ANY(4, 2, 4, 4, 2)
            else if (c->k <= 16) ONE_ANY(4, 2, 4, 4, -1)
            else ONE_16(4, 2, 8, 4, -1)
        }
#undef ONE_16
#undef ONE_ANY
#undef ONE
    } else {
        const dim3 sblock((unsigned)(plan.waves * kWave));
#define STREAM(FMT, NW, D)                                                                                              \
    e = launch(dba_stream_kernel<kTileLoads, FMT, NW, D>, grid, sblock, plan.spare_lds, c->stream, p.logp, p.V, kf, plan.rows_abreast, inv_k, p)
#define STREAM_ANY(NW, D)                                       \
    switch (logp_format) {                                      \
        case DBA_LOGP_F16: STREAM(kFmtF16, NW, D); break;       \
        case DBA_LOGP_BF16: STREAM(kFmtBF16, NW, D); break;     \
        default: STREAM(kFmtF32, NW, D); break;                 \
    }
        if (plan.waves == 8 && plan.tiles == 4) {
            STREAM_ANY(8, 4)
        } else if (plan.waves == 8) {
            STREAM_ANY(8, 2)
        } else {
            STREAM_ANY(4, 2)
        }
#undef STREAM_ANY
#undef STREAM
        // The merge phase is compiled for (rows per wave, waves, entries per lane).  Unless the caller fixes the
        // waves: four up to k = 16, eight up to 32, sixteen beyond (16 sentences of 2000 tokens, k = 64: 18.1 us per step with
        // eight, 17.4 with sixteen; 4 of 32000 21.45 / 20.95 - as long as every sentence has a compute unit to itself: 256 of 1000, k =
        // 64, 91.8 / 91.0, but 257 87.9 / 92.3, 1000 292.9 / 306.2, 300 of 8000 bf16 100.4 / 105.0; fewer lists per wave to merge and to scan, more waves to rank
        // candidates, at the price of a deeper tree where the waves' lists are joined; one decode, per step: 22.1 / 22.3 us with
        // four / eight waves at k = 12, 14.7 / 14.7 at k = 16; merge kernel 7.7 / 7.0 us at k = 20, 19.3 / 14.6 at k = 64).
        // Up to k = 11 every wave holds the k * k entries that matter, one or two a lane, and finds the bar by
        // itself (16 sentences, k = 10: 14.6 against 14.9 us per step with merged lists); with four and more a
        // lane the bisection's counts cost more than merging (k = 16: 15.4 against 15.3, with bf16, where
        // scores tie, 15.3 against 14.7; k = 20: 35.2 against 33.1; k = 32: 56.1 against 49.5).  From there to
        // k = 32 two rows share a register (k = 16: 14.9 against 15.4; k = 20: 32.6 against 33.1, with bf16 22.7 against
        // 23.4; k = 32: 49.1 against 49.6); beyond, a row's list needs all 64 lanes.
        const dim3 mgrid((unsigned)c->B);
        const int mw = c->merge_waves ? c->merge_waves : (c->k <= 16 ? 4 : c->k <= 32 || c->B > (int)kComputeUnits ? 8 : 16);
        const uint32_t k_inv = (uint32_t)c->k | inv_k16 << 16;
#define MERGE(ROWS, MW, J) \
    e = launch(dba_merge_kernel<ROWS, MW, J>, mgrid, MW * kWave, c->dyn_smem, c->stream, p.rowlists, p.conskeys, k_inv, p)
        if (e != hipSuccess) {
            // (nothing to merge)
        } else if (mw == 4) {
            if (c->k <= 8) MERGE(2, 4, 1);
            else if (c->k <= 11) MERGE(4, 4, 2);
            else if (c->k <= 16) MERGE(4, 4, -1);
            else if (c->k <= 32) MERGE(8, 4, -1);
            else MERGE(16, 4, 0);
        } else if (mw == 16) {
            MERGE(4, 16, 0);
        } else {
            if (c->k <= 8) MERGE(2, 8, 1);
            else if (c->k <= 11) MERGE(2, 8, 2);
            else if (c->k <= 32) MERGE(4, 8, -1);
            else MERGE(8, 8, 0);
        }
#undef MERGE
    }
    // (nothing that writes to the block has been launched then: the words to wait for are still those of the step before)
    if (e != hipSuccess) return fail(c, DBA_EHIP, "dba_step: launch failed: %s", hipGetErrorString(e));
    c->steps += 1;
    if (tells) {
        c->told = c->steps;
        c->told_under_way = true;
    }
    return DBA_OK;
}

DBA_API int dba_step_fmt(dba_ctx *c, const void *logp_dev, int logp_format, int32_t *out_token_dev,
                         int32_t *out_backptr_dev, float *out_score_dev, uint8_t *out_flags_dev)
{
    return step_impl(c, logp_dev, logp_format, out_token_dev, out_backptr_dev, out_score_dev, out_flags_dev,
                     nullptr);
}

DBA_API int dba_step_noalloc(dba_ctx *c, const void *logp_dev, int logp_format, int32_t *out_token_dev,
                             int32_t *out_backptr_dev, float *out_score_dev, uint8_t *out_flags_dev)
{
    if (!c) return DBA_EINVAL;
    if ((size_t)c->B * (size_t)c->k > kStaticRows)
        return fail(c, DBA_EINVAL,
                    "dba_step_noalloc: B*k = %zu beam rows exceed the %zu rows (DBA_NOALLOC_MAX_ROWS) the "
                    "library's own scratch holds; use dba_step / dba_step_fmt",
                    (size_t)c->B * (size_t)c->k, kStaticRows);
    if (!c->lib_scratch) {
        int dev = -1;
        if (hipGetDevice(&dev) != hipSuccess || dev != c->device)
            return fail(c, DBA_ESTATE, "dba_step_noalloc: the device of dba_init (%d) must be current", c->device);
        void *own = nullptr;
        const hipError_t e = static_scratch(&own);
        if (e != hipSuccess)
            return fail(c, DBA_EHIP, "dba_step_noalloc: the library's scratch has no device address: %s",
                        hipGetErrorString(e));
        c->lib_scratch = static_cast<unsigned char *>(own);
    }
    return step_impl(c, logp_dev, logp_format, out_token_dev, out_backptr_dev, out_score_dev, out_flags_dev,
                     c->lib_scratch);
}

DBA_API int dba_finalize(dba_ctx *c, int32_t *out_tokens_host, int32_t *out_len_host, float *out_score_host,
                 int32_t *out_status_host)
{
    if (!c) return DBA_EINVAL;
    if (!out_tokens_host || !out_len_host || !out_score_host || !out_status_host)
        return fail(c, DBA_EINVAL, "dba_finalize: an output pointer is NULL");
    const Layout &L = c->L;
    const int cur = c->steps & 1;
    const size_t B = (size_t)c->B, tokens_bytes = B * c->N * 4;
    const bool staged = staged_tokens(B, (size_t)c->N);
    // The four results lie side by side, small ones all in the block, where the kernel writes them; tokens beyond
    // stay in the workspace and go straight to the caller's array.  Without a block one copy takes what the block would
    // hold (5000 sentences, 20 steps: 71 us, 91 with a copy each); without host memory for that, each goes straight.
    const size_t first = staged ? L.fin_tokens : L.fin_len, bytes = L.fin_status + B * 4 - first;
    unsigned char *here = c->block.p ? c->block.p + c->block_data : nullptr;
    struct Free {
        unsigned char *p;
        ~Free() { free(p); }
    } copied{here ? nullptr : static_cast<unsigned char *>(malloc(bytes))};
    auto place = [&](size_t off) {
        return reinterpret_cast<int32_t *>(here && off >= first ? here + (off - first) : c->ws + off);
    };
    hipError_t e = launch(dba_finalize_kernel, (unsigned)c->B, kFinWaves * kWave, 0, c->stream, c->B, c->k, c->steps, c->N, c->pad_id,
                          c->normalize, at<int32_t>(c, L.hist_token), at<int32_t>(c, L.hist_backptr), at<Hyp>(c, L.beam[cur]),
                          c->track ? at<BestCompleted>(c, L.best) : nullptr, place(L.fin_tokens), place(L.fin_len),
                          reinterpret_cast<float *>(place(L.fin_score)), place(L.fin_status));
    auto fetch = [&](void *to, size_t off, size_t n) {
        if (e == hipSuccess && !((here || copied.p) && off >= first))
            e = hipMemcpyAsync(to, c->ws + off, n, hipMemcpyDeviceToHost, c->stream);
    };
    fetch(out_tokens_host, L.fin_tokens, tokens_bytes);
    fetch(out_len_host, L.fin_len, B * 4);
    fetch(out_score_host, L.fin_score, B * 4);
    fetch(out_status_host, L.fin_status, B * 4);
    if (e == hipSuccess && copied.p) e = hipMemcpyAsync(copied.p, c->ws + first, bytes, hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        if (here) c->block.p = nullptr;                    // (a kernel may still write to it: never used again)
        return fail(c, DBA_EHIP, "dba_finalize: HIP error: %s", hipGetErrorString(e));
    }
    c->init_under_way = c->told_under_way = false;
    if (const unsigned char *from = here ? here : copied.p) {
        if (staged) memcpy(out_tokens_host, from, tokens_bytes);
        memcpy(out_len_host, from + (L.fin_len - first), B * 4);
        memcpy(out_score_host, from + (L.fin_score - first), B * 4);
        memcpy(out_status_host, from + (L.fin_status - first), B * 4);
    }
    return DBA_OK;
}

DBA_API int dba_get_state(dba_ctx *c, float *score_host, uint64_t *met_mask_host, int32_t *inprog_phrase_host,
                  int32_t *inprog_pos_host, int32_t *length_host, uint8_t *flags_host)
{
    if (!c) return DBA_EINVAL;
    const Layout &L = c->L;
    const int cur = c->steps & 1;
    const size_t n = (size_t)c->B * c->k;
    Hyp *beam = static_cast<Hyp *>(malloc(n * sizeof(Hyp)));
    if (!beam) return fail(c, DBA_ENOMEM, "dba_get_state: out of host memory");
    struct Free {
        Hyp *p;
        ~Free() { free(p); }
    } guard{beam};
    hipError_t e = hipMemcpyAsync(beam, at<Hyp>(c, L.beam[cur]), n * sizeof(Hyp), hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return fail(c, DBA_EHIP, "dba_get_state: HIP error: %s", hipGetErrorString(e));
    c->init_under_way = c->told_under_way = false;
    for (size_t i = 0; i < n; ++i) {
        const Hyp &y = beam[i];
        const int ipq = ipq_of(y.state);
        if (score_host) score_host[i] = y.score;
        if (met_mask_host) met_mask_host[i] = y.met;
        if (inprog_phrase_host) inprog_phrase_host[i] = ipq < 0 ? -1 : (ipq >> 8);
        if (inprog_pos_host) inprog_pos_host[i] = ipq < 0 ? 0 : (ipq & 255);
        if (length_host) length_host[i] = y.len;
        if (flags_host)
            flags_host[i] = (uint8_t)(((flags_of(y.state) & kFinFinished) ? DBA_FLAG_FINISHED : 0) | (y.score > -INFINITY ? 0 : DBA_FLAG_DEAD));
    }
    return DBA_OK;
}

DBA_API int dba_steps_done(const dba_ctx *c) { return c ? c->steps : DBA_EINVAL; }

DBA_API int dba_set_option(dba_ctx *c, int option, double value)
{
    if (!c) return DBA_EINVAL;
    if (c->steps != 0) return fail(c, DBA_ESTATE, "dba_set_option: options are fixed once the first step is taken");
    if (value != value) return fail(c, DBA_EINVAL, "dba_set_option: the value is not a number");
    switch (option) {
        case DBA_OPT_ADJUSTMENT: c->adjust = value != 0.0 ? 1 : 0; return DBA_OK;
        case DBA_OPT_NORMALIZE_FINISHED: c->normalize = value != 0.0 ? 1 : 0; return DBA_OK;
        case DBA_OPT_PRUNE_THRESHOLD: c->prune = value < 0.0 ? -1.0f : (float)value; return DBA_OK;
        case DBA_OPT_TRACK_COMPLETED: c->track = value != 0.0 ? 1 : 0; return DBA_OK;
        case DBA_OPT_MERGE_WAVES:
            if (value != 0.0 && value != 4.0 && value != 8.0)
                return fail(c, DBA_EINVAL, "dba_set_option: DBA_OPT_MERGE_WAVES takes 0, 4 or 8");
            c->merge_waves = (int)value;
            return DBA_OK;
        default: return fail(c, DBA_EINVAL, "dba_set_option: unknown option %d", option);
    }
}

DBA_API int dba_get_finished(dba_ctx *c, uint8_t *all_finished_host)
{
    if (!c) return DBA_EINVAL;
    if (!all_finished_host) return fail(c, DBA_EINVAL, "dba_get_finished: the output pointer is NULL");
    const uint8_t *flags = at<uint8_t>(c, c->L.all_finished);
    uint8_t *here = c->block.p ? c->block.p + c->block_flags : nullptr;
    const bool told = here && !c->recorded && c->steps > 0 && c->told == c->steps;     // the last step has written them
    hipError_t e = hipSuccess;
    if (here && !told) {
        e = launch(dba_flags_kernel, 1, kBlock, 0, c->stream, (c->B + 3) / 4, reinterpret_cast<const uint32_t *>(flags),
                   reinterpret_cast<uint32_t *>(here));
    } else if (!here) {
        e = hipMemcpyAsync(all_finished_host, flags, (size_t)c->B, hipMemcpyDeviceToHost, c->stream);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        c->block.p = nullptr;                              // (a kernel may still write to it: never used again)
        return fail(c, DBA_EHIP, "dba_get_finished: HIP error: %s", hipGetErrorString(e));
    }
    c->init_under_way = c->told_under_way = false;
    const uint32_t *words = reinterpret_cast<const uint32_t *>(c->block.p);
    for (int b = 0; told && b < c->B; ++b) all_finished_host[b] = (uint8_t)(__atomic_load_n(words + b, __ATOMIC_RELAXED) & 3u);
    if (here && !told) memcpy(all_finished_host, here, (size_t)c->B);
    c->asked = true;
    return DBA_OK;
}

DBA_API void dba_destroy(dba_ctx *c)
{
    if (!c) return;
    // a ctx that goes before the GPU is through with its dba_init: the workspace and the block are given back only then
    if (c->init_under_way && !init_is_through(c)) {
        const RelaxedCapture relaxed;
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(c->stream, &capture) != hipSuccess) (void)hipGetLastError();
        if (capture != hipStreamCaptureStatusNone) {       // (what was enqueued before the capture began runs all the same)
            while (!init_is_through(c)) std::this_thread::yield();
        } else if (hipStreamSynchronize(c->stream) != hipSuccess) {
            (void)hipGetLastError();
            c->block.p = nullptr;                          // (never used again)
        }
    }
    // Nor does the block go to the next ctx while a step may still write to it: it goes when every sentence's word is the one that the
    // last such step leaves there.  (The stream may be gone by now, and a step may be behind work that waits for this thread.)
    if (c->told_under_way) host_blocks().put_when(c->block, (uint32_t)c->B, (uint32_t)c->told << 2, ~3u);
    else host_blocks().put(c->block);
    delete c;
}

DBA_API const char *dba_last_error(const dba_ctx *c) { return c ? c->err : g_init_error; }

DBA_API int dba_debug_allocate(int n_cases, int adjust, const int32_t *k_host, const int32_t *C_host, const int32_t *cnt_host,
                       int32_t *alloc_host, void *scratch_dev, size_t scratch_bytes, void *hip_stream)
{
    if (n_cases < 1 || !k_host || !C_host || !cnt_host || !alloc_host || !scratch_dev)
        return fail(nullptr, DBA_EINVAL, "dba_debug_allocate: bad argument");
    const size_t n = (size_t)n_cases;
    if (scratch_bytes < n * 132 * 4) return fail(nullptr, DBA_ENOMEM, "dba_debug_allocate: scratch too small");
    for (size_t i = 0; i < n; ++i)
        if (k_host[i] < 1 || k_host[i] > DBA_MAX_BEAM || C_host[i] < 0 || C_host[i] > DBA_MAX_CONS_TOKENS)
            return fail(nullptr, DBA_EINVAL, "dba_debug_allocate: case %zu out of range", i);
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    int32_t *d_k = static_cast<int32_t *>(scratch_dev);
    int32_t *d_C = d_k + n;
    int32_t *d_cnt = d_C + n;
    int32_t *d_alloc = d_cnt + n * 65;
    hipError_t e = hipMemcpyAsync(d_k, k_host, n * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(d_C, C_host, n * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(d_cnt, cnt_host, n * 65 * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = launch(dba_allocate_kernel, (unsigned)n_cases, kWave, 0, s, n_cases, adjust, d_k, d_C, d_cnt, d_alloc);
    if (e == hipSuccess) e = hipMemcpyAsync(alloc_host, d_alloc, n * 65 * 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(nullptr, DBA_EHIP, "dba_debug_allocate: HIP error: %s", hipGetErrorString(e));
    return DBA_OK;
}

DBA_API int dba_debug_wave_select(int n_cases, const uint64_t *keys_host, const float *vals_host,
                                  uint64_t *out_host, float *fout_host, void *scratch_dev,
                                  size_t scratch_bytes, void *hip_stream)
{
    if (n_cases < 1 || !keys_host || !vals_host || !out_host || !fout_host || !scratch_dev)
        return fail(nullptr, DBA_EINVAL, "dba_debug_wave_select: bad argument");
    const size_t n = (size_t)n_cases;
    if (scratch_bytes < n * (128 * 8 + 256 * 8 + 64 * 4 + 64 * 4))
        return fail(nullptr, DBA_ENOMEM, "dba_debug_wave_select: scratch too small");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    u64 *d_keys = static_cast<u64 *>(scratch_dev);
    u64 *d_out = d_keys + n * 128;
    float *d_vals = reinterpret_cast<float *>(d_out + n * 256);
    float *d_fout = d_vals + n * 64;
    hipError_t e = hipMemcpyAsync(d_keys, keys_host, n * 128 * 8, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(d_vals, vals_host, n * 64 * 4, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = launch(dba_wave_select_kernel, (unsigned)n_cases, kWave, 0, s, n_cases, d_keys, d_vals, d_out, d_fout);
    if (e == hipSuccess) e = hipMemcpyAsync(out_host, d_out, n * 256 * 8, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(fout_host, d_fout, n * 64 * 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(nullptr, DBA_EHIP, "dba_debug_wave_select: HIP error: %s", hipGetErrorString(e));
    return DBA_OK;
}

DBA_API int dba_debug_sentences_first(dba_ctx *c, int on)
{
    if (!c) return DBA_EINVAL;
    c->give_up = on;
    return c->one_launch && c->merge_waves == 0 ? 1 : 0;
}

DBA_API int dba_debug_launches(int B, int k, int V, int logp_format)
{
    if (!shape_ok(B, k, V, 1, 0) || logp_format < DBA_LOGP_F32 || logp_format > DBA_LOGP_BF16)
        return fail(nullptr, DBA_EINVAL, "dba_debug_launches: bad argument");
    return stream_plan((size_t)B, (size_t)k, (size_t)V, logp_format == DBA_LOGP_F32 ? 4u : 2u, true).one ? 1 : 2;
}

DBA_API int dba_debug_per_sentence(int B, int k, int V, int logp_format)
{
    if (!shape_ok(B, k, V, 1, 0) || logp_format < DBA_LOGP_F32 || logp_format > DBA_LOGP_BF16)
        return fail(nullptr, DBA_EINVAL, "dba_debug_per_sentence: bad argument");
    return stream_plan((size_t)B, (size_t)k, (size_t)V, logp_format == DBA_LOGP_F32 ? 4u : 2u, true).sentence ? 1 : 0;
}

DBA_API int dba_debug_stream_plan(int B, int k, int V, int logp_format, int32_t *plan_host)
{
    if (!shape_ok(B, k, V, 1, 0) || !plan_host || logp_format < DBA_LOGP_F32 || logp_format > DBA_LOGP_BF16)
        return fail(nullptr, DBA_EINVAL, "dba_debug_stream_plan: bad argument");
    const StreamPlan plan = stream_plan((size_t)B, (size_t)k, (size_t)V, logp_format == DBA_LOGP_F32 ? 4u : 2u, true);
    plan_host[0] = plan.waves;
    plan_host[1] = plan.tiles;
    plan_host[2] = (int32_t)((plan.waves == 8 ? sizeof(StreamSmem<8>) : sizeof(StreamSmem<4>)) + plan.spare_lds);
    plan_host[3] = (int32_t)plan.rows_abreast;
    return DBA_OK;
}

DBA_API int dba_debug_row_max(const float *src_dev, int rows, int V, float *out_max_dev, void *hip_stream)
{
    if (!src_dev || !out_max_dev || rows < 1 || V < 4 || (V & 3))
        return fail(nullptr, DBA_EINVAL, "dba_debug_row_max: bad argument (V must be a multiple of 4)");
    if (reinterpret_cast<uintptr_t>(src_dev) & 15)
        return fail(nullptr, DBA_EINVAL, "dba_debug_row_max: src_dev must be 16-byte aligned");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const hipError_t e = launch(dba_row_max_kernel, (unsigned)rows, kBlock, 0, s, src_dev, V, out_max_dev);
    if (e != hipSuccess) return fail(nullptr, DBA_EHIP, "dba_debug_row_max: HIP error: %s", hipGetErrorString(e));
    return DBA_OK;
}

}  // extern "C"
