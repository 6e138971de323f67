// Device side of the DBA step (Post & Vilar 2018, Alg. 2, Sec. 3.1-3.3) for gfx950.
//
// Two phases per step, one launch each, or both in one where rows are few:
//   stream phase  one workgroup per beam row (b,h): a single pass over the V
//                 log-probs of that row - score add, end-of-sentence mask,
//                 exact top-k of the row (which holds the row's best token
//                 and its share of the sentence's top-k) written as one sorted
//                 64-key list per row - plus the row's expandable constraint
//                 tokens (Alg. 2 inner loop): which they are and their sums;
//                 every key of either kind carries the bank it would land in
//                 (the constraints met after add(), Sec. 3.1): selection keys;
//   merge phase   one workgroup per sentence: the bar of the sentence's top-k
//                 from the row lists, dedup, bank counts, allocation with
//                 adjustment, selection, the state transition add() in full
//                 for the winners, new beam.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "wave_topk.hpp"

namespace dba {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int kMaxBeam = 64;
constexpr int kMaxCons = 64;          // constraint tokens (and phrases) per sentence
constexpr int kBlock = 256;           // threads per workgroup of the small helper kernels
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kTileLoads = 4;         // 16-byte loads per lane and tile in the stream phase
constexpr int kFmtF32 = 0;            // element type of the log-probs: fp32,
constexpr int kFmtF16 = 1;            // IEEE binary16,
constexpr int kFmtBF16 = 2;           // bfloat16 (the 16-bit types are widened exactly; the sum is fp32)
constexpr int kFinFinished = 1;       // beam-state flag: the hypothesis has generated end-of-sentence
constexpr int kFinEosBlocked = 4;     // beam-state flag: constraints unmet, end-of-sentence not allowed (Sec. 3.3)

// One hypothesis of a beam in memory, two 16-byte words: who needs all of it has two loads or stores, and a kernel one pointer (an
// array for each member, seven loads and stores and seven pointers, and seven pointers to the constraints' tables filled the scalar
// registers of both phases: 15 to 51 of them spilled in the kernels of one launch, now 2 to 16; none in
// the second of two, but with four merge waves fixed by the caller beyond k = 16: 13, and 35 beyond 32.  Per step, before / now: one sentence of five rows of 1000 8.55 / 8.2 us, ten of 32000 10.6 / 10.4, 160 rows 12.4 / 12.1, 168 of 50001 13.0 / 12.7,
// 595 of 24157 18.95 / 18.35, 1280 of 32000 32.2 / 32.0).
struct __attribute__((aligned(16))) Hyp {
    float score;                      // -inf: empty slot
    uint32_t state;                   // kFin* flags | (phrase under way * 256 + tokens met in it, + 1; 0: none) << 8
    int len;
    int nxt;                          // next token of the phrase under way (-1: none)
    u64 met;                          // bit i = constraint token i met
    u64 inc;                          // bit j = phrase j is not complete
};
__host__ __device__ __forceinline__ uint32_t state_word(int flags, int ipq) { return (uint32_t)flags | (uint32_t)(ipq + 1) << 8; }
__host__ __device__ __forceinline__ int flags_of(uint32_t state) { return (int)(state & 255u); }
// phrase under way * 256 + tokens met in it, or -1
__host__ __device__ __forceinline__ int ipq_of(uint32_t state) { return (int)(state >> 8) - 1; }

// The constraints of one sentence in memory, made by dba_init.
struct __attribute__((aligned(64))) Sentence {
    u64 same_first_lower[kMaxCons];   // phrase j: the lower phrases with the same first token
    u64 first_bucket[kMaxCons];       // bucket w & 63: the phrases whose first token has these low six bits
    int32_t bucket_tok[kMaxCons];     // that first token if the bucket's phrases agree on it; -1 none, -2 they differ
    int32_t first_tok[kMaxCons];      // first token of phrase j
    int32_t tok[kMaxCons];            // the tokens, phrase after phrase
    int32_t phr_off[kMaxCons + 1];    // token offset of each phrase, phr_off[nphr] = tokens in all
    int32_t nphr;                     // phrases
};

struct StepParams {
    int B, k, V;
    int eos_id, pad_id;
    int met_bits;                     // width of the bank field in the packed selection key
    int tok_bits;                     // width of the token field of a coordinate: (h << tok_bits) | w
    int first_step;                   // 1: the beam is the initial one (only slot 0 of a sentence is live)
    int cand_cap;                     // candidate keys the merge phase's dynamic LDS holds (a multiple of 64)
    int adjust;                       // 0: bank sizes stay at the base split (Sec. 5)
    int normalize;                    // 1: a hypothesis completing now is stored with sum / length (Sec. 4)
    float prune;                      // >= 0: threshold pruning against the best completed hypothesis (Sec. 4)
    int track;                        // 1: keep a record of the best completed hypothesis seen on any beam (Sec. 3.3)
    int step;                         // index of this step, from 0
    const void *logp;                 // [B,k,V] in the element type the kernel is instantiated for
    const Hyp *beam;                  // [B,k]  before the step,
    Hyp *beam_nxt;                    //        and after it
    const Sentence *sentences;        // [B]    the constraints
    // scratch
    u64 *rowlists;                    // [B*k,64] every row's best sums, decreasing, as selection-key bodies
    u64 *conskeys;                    // [B*k,64] selection keys (bank, score image, ~flat) of the
                                      //          row's expandable constraint tokens, 0 = none
    // outputs (each may be null)
    int32_t *out_token, *out_backptr;
    float *out_score;
    uint8_t *out_flags;
    int32_t *hist_token, *hist_backptr;   // row t of the history, [B,k]
    uint8_t *all_finished;            // [B] bit 0: the new beam is not empty and every hypothesis on it is completed;
                                      //     bit 1: some hypothesis on it is completed
    uint32_t *told;                   // [B] host memory that takes the same, | steps taken << 2 (null: the host does not ask)
    struct BestCompleted *best;       // [B] the record kept under `track`
};

// The best completed hypothesis a sentence has had on any of its beams so far (Sec. 3.3: the answer is
// the best-scoring finished hypothesis; Sec. 4 ranks completed hypotheses by score per word).
struct __attribute__((aligned(32))) BestCompleted {
    int have;          // 0: nothing completed yet
    int step, slot;    // where it was first seen: the beam after step `step`, place `slot`
    int len;           // its length, end-of-sentence included
    float q;           // its score per word
    float score;       // its score as that beam held it
    int ended;         // rows of the step under way that have ended (steps of one launch; 0 between steps)
    int pad;
};

// constraints of one sentence: token ids phrase after phrase, phrase p = tok[poff[p] .. poff[p+1])
struct ConsTab {
    int tok[kMaxCons];
    int poff[kMaxCons + 1];
};

// one hypothesis of the beam before the step, as the merge phase keeps it in LDS (two 16-byte reads)
struct __attribute__((aligned(16))) HypState {
    u64 met;       // bit i = constraint token i met
    u64 inc;       // bit j = phrase j not complete
    int ipq;       // phrase under way * 256 + tokens met in it, or -1
    int nxt;       // next token of the phrase under way (-1: none under way)
    int len;
    int misc;      // finished flag | constraints met << 8
};

constexpr int kMostLeft = 1024;        // candidates there is room for after those that cannot be among their bank's best are gone
// LDS of a merge-phase workgroup of MW waves (one sentence): 4, 8 or 16 are used
template <int MW>
struct MergeSmem {
    uint32_t ws[MW][kWave];           // every wave's best score images
    uint32_t wf[MW][kWave];           // and the greatest images its merges dropped
    uint32_t ws2[MW][kWave];          // every wave's best low words among tied keys
    HypState hyp[kMaxBeam];
    u64 sel[kMaxBeam];
    int slot[kMaxBeam];               // place in the new beam of the selected key i
    ConsTab ct;
    u64 fbucket[kMaxCons];            // phrases by the low six bits of their first token
    int btok[kMaxCons];               // and that token where a bucket's phrases agree on it (-1 none, -2 they differ)
    // per bank (constraints met, 0..64); sized for every value the 7-bit bank field of a key can hold
    int cnt[2 * kMaxCons];
    int alloc[2 * kMaxCons];
    int start[2 * kMaxCons];          // candidates in higher banks
    int first[2 * kMaxCons];          // slots of lower banks: where the bank's selected keys go in `sel`
    uint32_t bar_score;               // with eight waves: the score image of the bar of the k best, from the waves that join the lists,
    int bar_need;                     // and the places left for keys that tie at that score (-1: no tie to settle)
    int ncand;
    int nsel;
    int nleft;                        // candidates that can still be among their bank's best
    int verdict;                      // steps of one launch, once a wave has run out of looks for the rows' keys (below)
    u64 kept;                         // pruning: bit i = the hypothesis at place i of the new beam stays
};

// ---------------------------------------------------------------------------
// stream phase
// ---------------------------------------------------------------------------
struct RowTop {
    u64 list;      // this lane's entry of the wave's decreasing top-64
    float thr;     // sums below this cannot reach the row's top k; only ever raised, and never below
                   // -FLT_MAX, so that "s >= thr" also rejects -inf sums
};

constexpr float kLowestFinite = -3.402823466e+38f;

__device__ __forceinline__ void refresh_threshold(RowTop &st, int kk)
{
    const u64 kth = read_lane(st.list, kk - 1);
    if (kth != 0) st.thr = fmaxf(st.thr, float_from_ord((uint32_t)(kth >> 32)));
}

// lanes below the caller's in the mask m
__device__ __forceinline__ int lanes_before(u64 m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

constexpr int kGroupCap = 128;        // 16-byte groups one wave can set aside in LDS,
constexpr int kKeyCap = 128;          // and keys it can park there

// Where the floor of a row (below) is taken from cells: the greatest elements of as many neighbouring lanes as the workgroup
// has waves, 64 cells if every wave has a tile, fewer in shorter rows.  One sort of the cells does for the row, instead of
// one of every wave's 64 lane maxima and another, or merges with every other wave's list.  The k-th greatest of 64
// cells lets 64 ln(64 / (64 - k)) of the sampled elements through instead of little more than k: 18 at k = 16, 24 at 20, 44 at 32, 63
// at 40, 89 at 48.  So: not for more than five eighths of the cells (1280 rows of 10000, k = 64: 28.6 us per step with cells,
// 23.8 without), and with four waves, where the other way is one more sort, wide beams only if the floor
// rests on the whole row (2400 rows of 9000 fp16, k = 20: 22.5 / 23.5; 2048 of 8000 fp32, k = 32: 22.8 / 23.4; but 1280 of 32000 bf16, k =
// 20: 23.5 / 23.2; 2048 of 32000 fp32, k = 32: 49.3 / 49.0).  160 rows of 32000 fp32, k = 10: 13.4 / 13.9; with eight waves 192, k = 32,
// 15.8 / 17.2, 1024 of 100000 bf16, k = 32, 42.2 / 44.4.
// Nor for more than the cells that hold an element, which can be fewer in rows of one tile or two (1872 rows of 131 fp16, k = 8:
// four cells hold any, and a floor from sixteen was none, 15.6 us against 14.15): groups are dealt out lane by lane, and
// with three tiles more lanes have one than five eighths of the cells need.
template <int NW, int U>
__device__ __forceinline__ bool floor_from_cells(int k, int ngroups, int ntiles)
{
    return 8 * k <= 5 * (kWave / NW) * min(NW, ntiles) && (NW == 8 || k <= 16 || ntiles <= 2 * NW) &&
           k * NW <= ngroups - (ntiles - 1) * (kWave * (U - 1));
}

// Keys of one wave folded into its sorted list 64 at a time: one 64-lane sort and one merge per
// chunk instead of one serial insert per key.
__device__ __forceinline__ u64 fold_keys(u64 list, const u64 *keys, int cnt)
{
    const int lane = lane_id();
    for (int base = 0; base < cnt; base += kWave) {
        const u64 key = (base + lane < cnt) ? keys[base + lane] : 0ull;
        list = merge_desc<u64>(list, sort64_desc<u64>(key));
    }
    return list;
}

// max of four finite-or-infinite floats in two instructions (the inputs are never NaN, so the
// quieting moves a generic fmaxf would add are not needed)
__device__ __forceinline__ float max4(const v4f &x)
{
    float m;
    asm("v_max3_f32 %0, %1, %2, %3\n\tv_max_f32 %0, %0, %4" : "=&v"(m) : "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w));
    return m;
}

// ---- element formats of the log-prob tensor ----------------------------------------------
// A lane reads 16 bytes at a time: a "group" of G consecutive elements.  Every format answers
// three questions about a group: may any of its elements reach the threshold (cheap, and
// allowed to say yes too often, never no wrongly; the threshold comes as a bound on the elements
// themselves, worked out only when it changes), what are its G elements as fp32 (exact), and
// which single fp32 value is certainly not above the group's greatest element (for the
// threshold floor).  The sum itself is always one fp32 addition prev + element.
template <int FMT>
struct Logp;

template <>
struct Logp<kFmtF32> {
    static constexpr int G = 4;
    typedef float elem_t;
    typedef v4f vec_t;
    struct Quick {
        float xmin;       // no element below this reaches the threshold; never below -FLT_MAX
    };
    static __device__ __forceinline__ vec_t neg_inf() { return v4f{-INFINITY, -INFINITY, -INFINITY, -INFINITY}; }
    // fl(prev + x) >= thr needs prev + x >= thr - ulp(thr), and d = fl(thr - prev) is off by at most
    // ulp(d): both are below 2^-22 of the magnitudes, and three roundings of that size fit what is
    // left (the last term covers sums in the subnormal range).
    static __device__ __forceinline__ Quick quick(float prev, float thr)
    {
        const float d = thr - prev;
        const float x = d - ((fabsf(thr) + fabsf(d)) * 0x1p-22f + 0x1p-126f);
        return Quick{x >= kLowestFinite ? x : kLowestFinite};
    }
    // the least x with fl(prev + x) >= thr exactly, by bisection between the bound above and one as far on the other side
    static __device__ __forceinline__ Quick quick_exact(float prev, float thr)
    {
        const float d = thr - prev;
        uint32_t lo = ord_from_float(quick(prev, thr).xmin);
        uint32_t hi = ord_from_float(d + ((fabsf(thr) + fabsf(d)) * 0x1p-22f + 0x1p-126f));
        while (lo < hi) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            if (prev + float_from_ord(mid) >= thr) hi = mid;
            else lo = mid + 1;
        }
        return Quick{float_from_ord(lo)};
    }
    static __device__ __forceinline__ bool may_reach(const vec_t &x, const Quick &q) { return max4(x) >= q.xmin; }
    static __device__ __forceinline__ void widen(const vec_t &x, float (&f)[G])
    {
        f[0] = x.x;
        f[1] = x.y;
        f[2] = x.z;
        f[3] = x.w;
    }
    static __device__ __forceinline__ float some_element_at_most_max(const vec_t &x) { return max4(x); }
    static __device__ __forceinline__ float widen_one(elem_t e) { return e; }
    typedef float lone_t;
    static __device__ __forceinline__ float widen_lone(lone_t e) { return e; }
};

// The two 16-bit formats are sign-magnitude like fp32, so among negative values a greater bit
// pattern is a smaller number, and every non-negative pattern is below every negative one:
// "element >= bound" for a negative bound is "pattern <= pattern of the bound" on unsigned
// 16-bit integers.  The quick test therefore needs no conversion at all: the unsigned minimum
// of the group's eight patterns (packed 16-bit minima) against one precomputed pattern.
template <int FMT>
struct Logp16 {
    static constexpr int G = 8;
    typedef uint16_t elem_t;
    typedef v4u vec_t;
    static constexpr uint32_t kNegInf = FMT == kFmtF16 ? 0xFC00u : 0xFF80u;
    struct Quick {
        uint32_t umax2;   // greatest pattern whose sum still reaches the threshold, twice (0xFFFF: test everything)
    };
    static __device__ __forceinline__ vec_t neg_inf()
    {
        const uint32_t w = kNegInf | (kNegInf << 16);
        return v4u{w, w, w, w};
    }
    static __device__ __forceinline__ float widen_bits(uint32_t h)
    {
        if constexpr (FMT == kFmtBF16) return __uint_as_float(h << 16);
        else return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
    }
    static __device__ __forceinline__ float widen_one(elem_t e) { return widen_bits(e); }
    typedef uint32_t lone_t;
    static __device__ __forceinline__ float widen_lone(lone_t e) { return widen_bits(e); }
    // round-to-nearest pattern of a negative finite fp32 (a starting point only: quick() corrects it)
    static __device__ __forceinline__ uint32_t narrow_bits(float d)
    {
        if constexpr (FMT == kFmtBF16) {
            const uint32_t u = __float_as_uint(d);
            return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
        } else {
            return (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)d);
        }
    }
    // umax = the pattern of the smallest element x with fp32(prev + x) >= thr, found exactly: a
    // rounded guess, then single steps while the next smaller element still reaches thr, then
    // single steps back while the element itself does not.  If the steps run out on the way
    // down, everything is tested (never wrong, only slower).  thr never decreases, so a value
    // computed for an older thr stays valid.
    static __device__ __forceinline__ Quick quick(float prev, float thr)
    {
        const float d = thr - prev;
        if (!(d < 0.0f)) return Quick{~0u};
        uint32_t u = narrow_bits(d);
        if (u < 0x8000u) u = 0x8000u;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (prev + widen_bits(u + 1u) >= thr) ++u;
        if (prev + widen_bits(u + 1u) >= thr) return Quick{~0u};
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (u >= 0x8000u && !(prev + widen_bits(u) >= thr)) --u;
        return Quick{u | (u << 16)};
    }
    static __device__ __forceinline__ Quick quick_exact(float prev, float thr) { return quick(prev, thr); }
    // unsigned minimum of the eight patterns, in both halves of the result
    static __device__ __forceinline__ uint32_t min_pattern_twice(const vec_t &x)
    {
        uint32_t r, t;
        asm("v_pk_min_u16 %0, %2, %3\n\tv_pk_min_u16 %1, %4, %5\n\tv_pk_min_u16 %0, %0, %1\n\t"
            "v_pk_min_u16 %0, %0, %0 op_sel:[0,1] op_sel_hi:[1,0]"
            : "=&v"(r), "=&v"(t)
            : "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w));
        return r;
    }
    // (m, m) <= (umax, umax) as 32-bit numbers is m <= umax
    static __device__ __forceinline__ bool may_reach(const vec_t &x, const Quick &q)
    {
        return min_pattern_twice(x) <= q.umax2;
    }
    static __device__ __forceinline__ void widen(const vec_t &x, float (&f)[G])
    {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = widen_bits(w[i] & 0xFFFFu);
            f[2 * i + 1] = widen_bits(w[i] >> 16);
        }
    }
    // the element with the smallest pattern: the greatest one if none is positive, else some
    // positive one - in both cases an element of the group
    static __device__ __forceinline__ float some_element_at_most_max(const vec_t &x)
    {
        return widen_bits(min_pattern_twice(x) & 0xFFFFu);
    }
};
template <>
struct Logp<kFmtF16> : Logp16<kFmtF16> {};
template <>
struct Logp<kFmtBF16> : Logp16<kFmtBF16> {};

// The log-probs are read exactly once: non-temporal loads keep them from displacing
// anything useful in the caches.
constexpr int kNonTemporal = 2;       // cache-policy bit of a buffer load on gfx950
constexpr int kRawBuffer = 0x00027000;// last word of a buffer descriptor: 32-bit data, no swizzle

// LDS shared by the waves of one row's workgroup during the stream phase.
template <int NW>
struct StreamSmem {
    v4u group[NW][kGroupCap];           // groups set aside: the 16 bytes as they were read,
    uint32_t coord[NW][kGroupCap];      // and the coordinate of the first element
    u64 key[NW][kKeyCap];               // keys parked for the end of the row
    u64 wl[NW][kWave];                  // the waves' lists, for the final merge
    uint32_t boot[NW][kWave];           // maxima of every wave's first tiles (order images), of its lanes, sorted, or of its cells
    int parked[NW];                     // end of the row: keys each wave has parked,
    int has_list[NW];                   // and whether it holds a list from earlier folds
};

// LDS of a workgroup that streams all rows of a sentence, a wave each.  At the end of its row a wave leaves the row's list in the
// first 64 of its keys and the keys of its constraint tokens in the others.
constexpr int kSentenceWaves = 8;
struct SentenceSmem {
    v4u group[kSentenceWaves][kGroupCap];
    uint32_t coord[kSentenceWaves][kGroupCap];
    u64 key[kSentenceWaves][kKeyCap];
};
static_assert(kKeyCap == kWave + kMaxCons, "a list and the constraint keys");

// The groups a wave has set aside, element by element: sums that reach the threshold are parked as keys,
// and the keys are folded into the wave's list whenever they would overflow (the threshold then
// rises).  Reached only where the k best groups hold more keys than there is room for (few elements, many ties): kept
// small, not fast.
template <int FMT>
__device__ __forceinline__ void drain_groups(RowTop &st, int &parked, const v4u *group, const uint32_t *coord, u64 *key,
                                             int cnt, float prev, uint32_t no_coord, int kk)
{
    typedef Logp<FMT> F;
    const int lane = lane_id();
    const typename F::elem_t *elem = reinterpret_cast<const typename F::elem_t *>(group);
#pragma unroll 1
    for (int base = 0; base < cnt; base += kWave) {
        const int i = base + lane;
        const uint32_t at = i < cnt ? coord[i] : 0u;
#pragma unroll 1
        for (int c = 0; c < F::G; ++c) {
            const float s =
                i < cnt && at + (uint32_t)c != no_coord ? prev + F::widen_one(elem[i * F::G + c]) : -INFINITY;
            const u64 m = __ballot(s >= st.thr);
            const int n = __popcll(m);
            if (parked + n > kKeyCap) {
                st.list = fold_keys(st.list, key, parked);
                parked = 0;
                refresh_threshold(st, kk);
            }
            if ((m >> lane) & 1ull) key[parked + lanes_before(m)] = make_key(s, at + (uint32_t)c);
            parked += n;
        }
    }
}

// One wave's share of one row: tiles wave, wave+nwaves, ... of 64*U groups of 16 bytes each.
// Must be called by every thread of the workgroup (it contains one barrier).
//
// s = prev + logp is a single fp32 add (a 16-bit log-prob is widened exactly first).  A group is
// set aside only if the sum of one of its elements can still reach the row's k best (>=: a later
// element may tie the k-th score and win on the coordinate); Logp<FMT>::may_reach decides that
// for a whole 16-byte group at once.  What is set aside is the group as it was read: one vote and two
// LDS writes, whatever the number of elements in it.  Its elements are looked at one by one only at the
// end of the row, 64 groups side by side, so that nothing but the quick test stands between a tile's
// arrival and the request that refills its registers.  What bounds this phase besides memory is the issue
// slots that about 4k near candidates per row take (against handling them one element at a time as
// they pass: stream kernel 27.8 -> 27.0 us at 1280 rows of 32000 fp32, k = 20, 18.6 -> 16.7 us with bf16;
// 261 -> 256 us at 8192 rows of 50000 fp32, k = 64, 149 -> 137 us with fp16).
//
// Thresholds.  (1) Every lane takes an element of its share of the wave's first two tiles (the
// greatest, where the format finds it cheaply); the k-th greatest of the workgroup's
// values, of single lanes or of cells of a few, is a floor: k different lanes hold an element at
// least that large, so nothing below it can be among the row's k best.  About k * V / (elements of those first tiles) elements of the row reach
// it, so a wide beam over a long row (k = 64: from about 256000 fp32 elements on) or over a row of a single tile, whose
// floor is near the least of 64 values, fills a wave's room, and so does a row whose best sums tie in great number.
// (2) Such a wave makes room: of the groups it has set aside the k-th greatest stands for k elements of the row and is
// a floor as well; the k best groups stay, and the fast loop goes on behind the tile that found no room (per step, against
// leaving the fast loop for good and reading the rest 64 groups at a time: 64 rows of 524288 fp32, k = 64: 129 -> 65
// us; 1024 rows of 2000 bf16, k = 64: 29.0 -> 24.6; 320 rows of 1000 fp32, k = 20: 18.7 -> 13.4; 1280 rows of 32000 equal
// elements 245 -> 42, a quarter of them equal and best 93 -> 43).  (3) Keys that find no room at the end of the row, several
// elements to a group, are folded into the wave's sorted list, whose k-th entry bounds its share of the row.  The row's
// best element is never below any bound, so it always survives.
//
// Whatever is rare is kept out of the fast loop: one place that looks into groups one element at
// a time, no end-of-sentence test per tile, and a copy of the loop for the tiles behind one that found no room
// (a single loop that returns to its start keeps its tiles' registers through all that is rare, and costs rows that
// never come there 0.2 to 0.4 us).  53-55 vector registers and at most 80 scalar ones let eight waves share a SIMD
// (2048 rows of 32000, k = 32: 50.6 -> 49.5 us per step; 168 rows of 50001: 17.6 -> 17.2).
// D = tiles in flight per wave.  The first two are requested before anything else; the others once both have
// arrived, while the floor is worked out - asked for at the start they would only queue in front of other
// waves' first tiles, and the floor waits for those (160 rows of 32000: 15.2 instead of 13.7 us per step).
template <int U, int FMT, int D>
struct RowStream {
    typedef Logp<FMT> F;
    typedef typename F::vec_t vec_t;
    typedef typename F::elem_t elem_t;
    static constexpr int G = F::G;

    const elem_t *row;
    const vec_t *vec;
    int V, head, nv, tail, ntiles;        // nv: groups in the row's aligned body
    __amdgpu_buffer_rsrc_t body;
    vec_t tile_[D][U];
    typename F::lone_t lone;   // wave 0: this lane's element outside the aligned body, if there is one, as it is read

    // Requests a tile.  The descriptor ends with the row's aligned body, so lanes beyond it read nothing and get 0:
    // a partial tile needs neither a branch nor switched-off lanes when it is requested, only to be blanked when it is looked at,
    // and the waits of the loop count the same loads on every way through it.  (Requested under a lane mask instead, into
    // registers that were filled first, it came after the floor and waited: per step, 160 rows of 32000 fp32 13.4 -> 13.2 us, 240
    // of 9000 11.65 -> 11.2, 1280 of 32000 bf16 23.4 -> 23.2, 1152 of 32003 bf16 21.75 -> 21.55; the partial tile at the
    // front of the row instead: 13.1, 11.2, 23.2, 22.7, as the floor then rests on less.)
    __device__ __forceinline__ void load(int tile, vec_t (&x)[U]) const
    {
#pragma unroll
        for (int u = 0; u < U; ++u)
            x[u] = __builtin_bit_cast(vec_t, __builtin_amdgcn_raw_buffer_load_b128(
                body, (int)sizeof(vec_t) * (tile * (kWave * U) + u * kWave + lane_id()), 0, kNonTemporal));
    }
    // The groups that a partial tile does not have read as if no element could reach the threshold.
    __device__ __forceinline__ void blank(int tile, vec_t (&x)[U]) const
    {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (tile * (kWave * U) + u * kWave + lane_id() >= nv) x[u] = F::neg_inf();
    }

    // Issues the loads of this wave's first two tiles.  Needs nothing of the hypothesis, so it
    // runs before the beam state has arrived.
    __device__ __forceinline__ void begin(const elem_t *__restrict__ row_, int V_, int wave, int nwaves)
    {
        const int lane = lane_id();
        row = row_;
        V = V_;
        const uintptr_t addr = reinterpret_cast<uintptr_t>(row);
        head = (int)(((16u - (unsigned)(addr & 15u)) & 15u) / (unsigned)sizeof(elem_t));
        if (head > V) head = V;
        nv = (V - head) / G;
        tail = V - head - nv * G;
        vec = reinterpret_cast<const vec_t *>(row + head);
        ntiles = (nv + kWave * U - 1) / (kWave * U);
        body = __builtin_amdgcn_make_buffer_rsrc(const_cast<vec_t *>(vec), 0, nv * (int)sizeof(vec_t), kRawBuffer);
        // (A wave that has no tile requests none: its requests would read nothing, but take their turn.  Per step, many rows of one
        // tile or two: 2010 of 1296 fp32 with most of them empty 9.5 -> 8.6 us, 8192 of 1000, k = 64, 55.8 -> 54.4, 320 of 2000 9.8 ->
        // 9.4.  The second tile shares the branch: in one of its own the wait for the first would be for both, 2123
        // rows of 6910 bf16 19.8 -> 20.0.  The branch costs rows that need none up to 0.2 us: 1162 of 7214 bf16 14.9 -> 15.1.)
        if (wave < ntiles) {
#pragma unroll
            for (int d = 0; d < 2; ++d) load(wave + d * nwaves, tile_[d]);
        }
        lone = 0;
        if (wave == 0 && lane < head + tail) lone = row[lone_at(lane)];
    }

    // position of the lane's element before the first / after the last 16-byte aligned group (rows whose
    // length or start is not a multiple of one group): fewer than two groups of them, one per lane
    __device__ __forceinline__ int lone_at(int lane) const
    {
        return lane < head ? lane : head + nv * G + (lane - head);
    }

    // slot: the wave's places in sm (which other rows' waves may share).
    // Returns the number of keys left parked in sm.key[slot] (not yet folded into st.list).
    template <int NW, typename Smem>
    __device__ __forceinline__ int run(float prev, int eos_block, uint32_t flat_base, int kk, int wave, int slot, Smem &sm,
                                       RowTop &st);
};

template <int U, int FMT, int D>
template <int NW, typename Smem>
__device__ __forceinline__ int RowStream<U, FMT, D>::run(float prev, int eos_block, uint32_t flat_base, int kk,
                                                         int wave, int slot, Smem &sm, RowTop &st)
{
    constexpr int nwaves = NW;
    constexpr bool LL = D > 2 || NW == 1; // few waves about: exchanges of the shortest latency
    const int lane = lane_id();
    const int nfull = nv / (kWave * U);
    const uint32_t lane_coord = flat_base + (uint32_t)(head + G * lane);
    // Sec. 3.3: while constraints are unmet the end-of-sentence entry does not exist: its group takes no part in
    // the floor, and the entry is passed over where groups are looked at element by element
    const uint32_t no_coord = eos_block >= 0 ? flat_base + (uint32_t)eos_block : ~0u;
    uint32_t boot = ord_from_float(-INFINITY);
    if (wave < ntiles) {
        // the first two tiles take part in the floor (8 KB per wave)
        float lane_max = -INFINITY;
        auto offer = [&](vec_t (&t)[U], int tile) {
            if (tile == nfull) blank(tile, t);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t off = no_coord - (lane_coord + (uint32_t)(G * kWave * u) + (uint32_t)(G * U * kWave) * (uint32_t)tile);
                const float mu = off < (uint32_t)G ? -INFINITY : F::some_element_at_most_max(t[u]);
                asm("v_max_f32 %0, %1, %2" : "=v"(lane_max) : "v"(lane_max), "v"(mu));
            }
        };
        offer(tile_[0], wave);
        if (wave + nwaves < ntiles) offer(tile_[1], wave + nwaves);
        asm volatile("" : "+v"(lane_max));                 // (both tiles are here before more is requested)
#pragma unroll
        for (int d = 2; d < D; ++d) load(wave + d * nwaves, tile_[d]);
        boot = ord_from_float(prev + lane_max);
    }
    // Any k values that different lanes hold give a valid floor
    constexpr int share = kWave / nwaves;              // entries of every wave that fit one 64-lane sort
    if constexpr (NW == 1) {
        boot = sort64_minmax_desc(boot);
    } else if (floor_from_cells<NW, U>(kk, nv, ntiles)) {
        boot = max_of_lanes<nwaves>(boot);
        if (lane % nwaves == 0) sm.boot[wave][lane / nwaves] = boot;
        __syncthreads();
        boot = sm.boot[lane / share][lane % share];
        boot = LL ? sort64_minmax_desc(boot) : sort64_desc<uint32_t, false>(boot);
    } else {
        if (NW == 8 || wave < ntiles) boot = sort64_desc<uint32_t, LL>(boot);      // (the others hold the same in every lane)
        sm.boot[wave][lane] = boot;
        __syncthreads();
        const int lists = min(nwaves, ntiles);             // (the other waves hold nothing)
        if (lists > 3 && 4 * kk <= 3 * lists * share) {
            // the best `share` of every wave's list, sorted once: the k-th of them is the k-th of all unless one
            // wave holds more than `share` of the k greatest (then it is a little lower).  Of one to three lists, as rows of so
            // many tiles have, all is kept: a merge each is no longer than the sort, and `share` of each would be fewer than k, no floor
            // at all (per step, rows of one tile, k = 20 to 32: 96 of 1000 fp32 12.7 -> 9.7 us, 512 14.2 -> 11.5, 500 of 2000 bf16 15.6 -> 12.0)
            boot = sort64_desc<uint32_t, LL>(sm.boot[lane / share][lane % share]);
        } else {
            const int own = wave < lists ? wave : 0;
            if (wave >= lists) boot = sm.boot[0][lane];
            for (int w = 0; w < lists; ++w)
                if (w != own) boot = merge_desc<uint32_t, LL>(boot, sm.boot[w][lane]);
        }
    }
    st.thr = fmaxf(float_from_ord((uint32_t)__builtin_amdgcn_readlane((int)boot, kk - 1)), kLowestFinite);
    typename F::Quick quick = F::quick(prev, st.thr);
    v4u *group = sm.group[slot];
    uint32_t *coord = sm.coord[slot];
    u64 *key = sm.key[slot];
    int cnt = 0, parked = 0;              // groups set aside, keys parked
    auto set_aside = [&](const vec_t &x, bool mine, u64 m, uint32_t at) {
        if (mine) {
            const int pos = cnt + lanes_before(m);
            group[pos] = __builtin_bit_cast(v4u, x);
            coord[pos] = at;
        }
        // (no instruction: keeps this join of lanes apart from the uniform branches behind it, which would
        // otherwise be taken for branches of single lanes and kept in ten more scalar registers: seven waves a SIMD)
        __builtin_amdgcn_wave_barrier();
        cnt += __popcll(m);
    };
    // the elements outside the aligned body (fewer than two groups of them) are parked as keys at once
    if (wave == 0 && head + tail > 0) {
        const uint32_t at = flat_base + (uint32_t)lone_at(lane);
        // (16 bits are widened here and not where they are read: the wait for them there would also be one for the tiles
        // requested before; 1152 rows of 32003 bf16 21.1 -> 20.75 us per step)
        if constexpr (G > 4) asm volatile("" : "+v"(lone));
        const float s = lane < head + tail && at != no_coord ? prev + F::widen_lone(lone) : -INFINITY;
        const u64 m = __ballot(s >= st.thr);
        if ((m >> lane) & 1ull) key[lanes_before(m)] = make_key(s, at);
        parked = __popcll(m);
    }
    const int parked_alone = parked;
    // one tile: test its U groups, set aside what may belong to the top k.  False: no room for them.
    auto examine = [&](vec_t (&t)[U], int tile) {
        if (tile == nfull) blank(tile, t);
        bool mine[U];
        u64 m[U], any = 0;
        int n = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            mine[u] = F::may_reach(t[u], quick);
            m[u] = __ballot(mine[u]);
            any |= m[u];
            n += __popcll(m[u]);
        }
        if (any == 0) return true;
        if (__builtin_expect(cnt + n > kGroupCap, 0)) return false;
        const uint32_t at0 = lane_coord + (uint32_t)(G * U * kWave) * (uint32_t)tile;
#pragma unroll
        for (int u = 0; u < U; ++u) set_aside(t[u], mine[u], m[u], at0 + (uint32_t)(G * kWave * u));
        return true;
    };
    // Makes room: leaves the k best groups, k <= 64 of at most 128.  The k-th greatest of the groups' greatest sums is a floor
    // (the bar); groups below it go.  A wave comes by its groups in the order of their coordinates, so of the groups
    // that only tie at the bar the first few, up to k in all, are enough, and once there are k, a later element has to be
    // better than the bar: a sum that only ties would lose to all of them.  (Groups move down within one wave, whose
    // LDS operations keep their order: 64 at a time, all of them read before any is written.)
    auto make_room = [&]() {
        uint32_t image[2];
        int l = lane;                                      // (taken anew: what follows from it would otherwise be kept in
        asm volatile("" : "+v"(l));                        // registers through the loops around this, 58 instead of 55)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = j * kWave + l;
            image[j] = 0;
            if (i < cnt) {
                const uint32_t at = coord[i];
                float f[G], best = -INFINITY;
                F::widen(__builtin_bit_cast(vec_t, group[i]), f);
#pragma unroll
                for (int c = 0; c < G; ++c)
                    if (at + (uint32_t)c != no_coord) best = fmaxf(best, prev + f[c]);
                image[j] = ord_from_float(best);
            }
        }
        int reach;
        const uint32_t tau = kth_greatest<2>(image, kk, reach), old = ord_from_float(st.thr), bar = tau > old ? tau : old;
        const u64 better0 = __ballot(image[0] > bar), better1 = __ballot(image[1] > bar);
        const u64 tied0 = __ballot(image[0] == bar), tied1 = __ballot(image[1] == bar);
        const int left = kk - __popcll(better0) - __popcll(better1), ties0 = __popcll(tied0);
        st.thr = float_from_ord(bar);
        const int ties = ties0 + (int)__popcll(tied1);
        cnt = 0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int i = j * kWave + l;
            const v4u bytes = group[i];
            const uint32_t at = coord[i];
            const bool keep = image[j] > bar || (image[j] == bar && (j ? ties0 : 0) + lanes_before(j ? tied1 : tied0) < left);
            set_aside(__builtin_bit_cast(vec_t, bytes), keep, __ballot(keep), at);
        }
        // (where many tie the bound has to be exact: the rounded one lets through what ties)
        quick = ties > left ? F::quick_exact(prev, float_from_ord(bar + 1))
                            : F::quick(prev, float_from_ord(bar + (ties == left ? 1u : 0u)));
    };
    int tl = wave;                        // tile to look at next
    // a tile's registers are refilled as soon as it has been looked at, N tiles ahead
    auto stream = [&](auto &t) {
        constexpr int N = sizeof(t) / sizeof(t[0]);
        bool room = true;
        while (room && tl < ntiles) {
#pragma unroll
            for (int d = 0; d < N; ++d) {
                if (tl >= ntiles) break;
                room = examine(t[d], tl);
                if (!room) break;
                if (tl + N * nwaves < ntiles) load(tl + N * nwaves, t[d]);
                tl += nwaves;
            }
        }
    };
    stream(tile_);
    if (__builtin_expect(tl < ntiles, 0)) {
        vec_t next[2][U];
        do {
            // no room for this tile's groups: they are read again and taken in columns of 64, with room made in between
            vec_t x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int g = (tl * U + u) * kWave + lane;
                x[u] = g < nv ? vec[g] : F::neg_inf();
            }
            const uint32_t at0 = lane_coord + (uint32_t)(G * U * kWave) * (uint32_t)tl;
            for (int u0 = 0;;) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool mine = F::may_reach(x[u], quick);
                    const u64 m = __ballot(mine);
                    if (u == u0 && cnt + (int)__popcll(m) <= kGroupCap) {
                        set_aside(x[u], mine, m, at0 + (uint32_t)(G * kWave * u));
                        u0 = u + 1;
                    }
                }
                if (u0 == U) break;
                make_room();
            }
            tl += nwaves;
#pragma unroll
            for (int d = 0; d < 2; ++d) load(tl + d * nwaves, next[d]);
            stream(next);
        } while (tl < ntiles);
    }
    // the elements of the groups set aside, 64 groups side by side: every lane counts its own, a
    // prefix sum over the wave gives it its places
    bool tightened = false;
    for (int base = 0; base < cnt; base += kWave) {
        const int i = base + lane;
        const bool mine = i < cnt;
        const uint32_t at = mine ? coord[i] : 0u;
        float f[G];
        F::widen(mine ? __builtin_bit_cast(vec_t, group[i]) : F::neg_inf(), f);
        int n = 0;
#pragma unroll
        for (int c = 0; c < G; ++c) {
            f[c] = at + (uint32_t)c == no_coord ? -INFINITY : prev + f[c];
            n += f[c] >= st.thr ? 1 : 0;
        }
        const int incl = wave_inclusive_sum(n);
        const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
        if (__builtin_expect(parked + total > kKeyCap, 0)) {
            if (tightened || cnt <= kk) {
                // many elements to a group: the rest one by one, with folds
                drain_groups<FMT>(st, parked, group + base, coord + base, key, cnt - base, prev, no_coord, kk);
                break;
            }
            tightened = true;                              // once more from the first group, with the floor the groups give
            make_room();
            parked = parked_alone;
            base = -kWave;
            continue;
        }
        int pos = parked + incl - n;
#pragma unroll
        for (int c = 0; c < G; ++c)
            if (f[c] >= st.thr) key[pos++] = make_key(f[c], at + (uint32_t)c);
        parked += total;
    }
    return parked;
}

// End of a row.  Each wave arrives with a sorted list from earlier folds (usually none: with
// the floor in place a wave parks a few dozen keys per row and never has to fold) and the
// keys it has parked.  The parked keys of all waves are pooled and sorted in chunks
// of 64 - one chunk in the common case, sorted by one wave - instead of one sort per wave plus
// a merge per wave.  The wave that finishes the row (fin_wave) rotates with the row index, so
// that the rows sharing a compute unit finish on different SIMDs.  Returns the row's list to
// the lanes of fin_wave.  Called by every thread of the workgroup (one or two barriers).
template <int NW>
__device__ __forceinline__ u64 finish_row(StreamSmem<NW> &sm, u64 list, int parked, int wave, int fin_wave)
{
    constexpr int nwaves = NW;
    const int lane = lane_id();
    const bool mine_has = read_lane(list, 0) != 0;
    if (lane == 0) {
        sm.parked[wave] = parked;
        sm.has_list[wave] = mine_has ? 1 : 0;
    }
    __syncthreads();
    // keys parked by waves 0..w-1 (pre[w]); all of them (n)
    int pre[NW + 1];
    int any = 0;
    pre[0] = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        pre[w + 1] = pre[w] + sm.parked[w];
        any |= sm.has_list[w];
    }
    const int n = __builtin_amdgcn_readfirstlane(pre[NW]);
    any = __builtin_amdgcn_readfirstlane(any);
    const int nchunks = (n + kWave - 1) >> 6;
    u64 part = 0;
    bool have = false;
    for (int c = (wave - fin_wave) & (nwaves - 1); c < nchunks; c += nwaves) {
        const int i = c * kWave + lane;
        u64 key = 0;
        if (i < n) {
            int w = 0, first = 0;
#pragma unroll
            for (int j = 1; j < NW; ++j)
                if (i >= pre[j]) {
                    w = j;
                    first = pre[j];
                }
            key = sm.key[w][i - first];
        }
        const u64 sorted = sort_first_desc<u64, true>(key, n - c * kWave);
        part = have ? merge_desc<u64, true>(part, sorted) : sorted;
        have = true;
    }
    if (nchunks <= 1 && !any) return part;            // the whole row was one chunk of fin_wave's
    if (mine_has) {
        part = have ? merge_desc<u64, true>(part, list) : list;
        have = true;
    }
    sm.wl[wave][lane] = part;
    __syncthreads();
    if (wave == fin_wave) {
        for (int w = 1; w < nwaves; ++w) {
            const u64 other = sm.wl[(wave + w) & (nwaves - 1)][lane];
            if (read_lane(other, 0) != 0) {
                part = have ? merge_desc<u64, true>(part, other) : other;
                have = true;
            }
        }
    }
    return part;
}

// The same for a row of one wave.
__device__ __forceinline__ u64 finish_row_of_one_wave(const u64 *keys, u64 list, int parked)
{
    const int lane = lane_id(), n = __builtin_amdgcn_readfirstlane(parked);
    for (int base = 0; base < n; base += kWave) {
        const u64 sorted = sort_first_desc<u64, true>(base + lane < n ? keys[base + lane] : 0ull, n - base);
        list = read_lane(list, 0) != 0 ? merge_desc<u64, true>(list, sorted) : sorted;
    }
    return list;
}

// ---------------------------------------------------------------------------
// constraint bookkeeping (Sec. 3.1): in-order phrases, one phrase under way
// ---------------------------------------------------------------------------
// Wave-wide, one lane per phrase: what the hypothesis (nmet tokens met, incomplete phrases inc,
// phrase ip under way with iq tokens met and next token nxt) may place now (Alg. 2 inner loop,
// Sec. 3.1 item 2) - the next token of the phrase under way, the first token of a phrase
// neither complete nor under way.  Of equal tokens only the lowest phrase keeps its entry
// (they are one coordinate).  Returns the lane's token or -1, and in bank the constraints met
// once it is placed: nmet+1 if it continues the phrase under way or no phrase is under way,
// else the phrase under way is unwound first (Sec. 3.1, last paragraph).
// ftok = first token of the lane's phrase, sfl = lower phrases with the same first token.
__device__ __forceinline__ int expandable_entry(int P, int nmet, u64 inc, int ip, int iq, int nxt, int ftok,
                                                u64 sfl, int &bank)
{
    const int lane = lane_id();
    const bool offers_first = lane < P && ((inc >> lane) & 1ull) && lane != ip;
    const u64 F = __ballot(offers_first);
    int w = -1;
    if (lane == ip) w = nxt;
    else if (offers_first && !(sfl & F)) w = ftok;
    if (ip >= 0) {
        const u64 E = __ballot(w >= 0 && lane != ip && w == nxt);   // at most one lane
        if (E) {
            const int lowest = __ffsll((long long)E) - 1;
            if (lowest < ip) {
                if (lane == ip) w = -1;
            } else if (lane == lowest) {
                w = -1;
            }
        }
    }
    bank = (ip < 0 || lane == ip || w == nxt) ? nmet + 1 : nmet - iq + 1;
    return w;
}

// ---------------------------------------------------------------------------
// allocation (Sec. 3.2) on one wavefront, registers only
// ---------------------------------------------------------------------------
// Lane x holds bank x (x < 64); bank 64 is carried wave-uniform.  c = candidates
// in the bank; returns the slots of the lane's bank and writes bank 64's to a64.
// Base split: floor(k/(C+1)) each, remainder to bank C.  Adjustment: banks with
// more slots than candidates, in ascending order, keep what they can fill and
// pass the rest to banks with spare candidates, nearest first, the higher
// neighbour before the lower, as much as each can take.
// adjust = false (Sec. 5): the base split stays; a bank keeps only the slots it can fill.
// One chain of dependent steps per donor, and early in a decode most banks are empty donors: a
// donor's hand-outs are one prefix sum and one lane exchange, or, where it has one or two slots or one or two
// banks can take any, a few bit scans each (16 sentences with 1 to 16 constraints, k = 10: with the counted
// ranks and the bar of each wave's own, 15.5 -> 14.6 us per step).
__device__ __forceinline__ int allocate_wave(int k, int C, int c, int c64, int &a64, bool adjust)
{
    const int lane = lane_id();
    const int base = k / (C + 1);
    const int rem = k - base * (C + 1);
    int a = (lane <= C) ? base + (lane == C ? rem : 0) : 0;
    a64 = (C == 64) ? base + rem : 0;
    if (lane > C) c = 0;
    if (C < 64) c64 = 0;
    if (!adjust) {
        a64 = min(a64, c64);
        return min(a, c);
    }

    if (C == 64) {
        // 65 banks share k <= 64 slots: the base split gives all of them to bank 64, the only donor, and what it
        // cannot fill goes to the nearest banks below, each taking what those above it have left
        const int left = max(0, k - c64), incl = wave_inclusive_sum(c);
        a64 = min(k, c64);
        return min(c, max(0, left - (__builtin_amdgcn_readlane(incl, kWave - 1) - incl)));
    }
    u64 donors = __ballot(a > c);                         // fixed before the hand-outs begin: a receiver never becomes one
    int need = max(0, c - a);
    u64 receivers = __ballot(need > 0);
    const int last_donor = donors ? 63 - __clzll((long long)donors) : -1;
    while (donors != 0 && receivers != 0) {
        const int b = __ffsll((long long)donors) - 1;
        const bool all_below = (receivers >> b) == 0, all_above = (receivers & (~0ull >> (63 - last_donor))) == 0;
        if (all_below || all_above) {
            // every donor that is left hands to the same banks in the same order, downwards from the highest or upwards
            // from the lowest: early in a decode, when nearly all banks are empty donors above a few full ones, one prefix
            // sum instead of up to 32 rounds (4.4 of the merge phase's 17 us with 128 sentences, k = 64)
            const int spare = wave_inclusive_sum(((donors >> lane) & 1ull) ? a - c : 0);
            const int incl = wave_inclusive_sum(need);
            const int served = all_below ? __builtin_amdgcn_readlane(incl, kWave - 1) - incl : incl - need;
            need -= min(need, max(0, __builtin_amdgcn_readlane(spare, kWave - 1) - served));
            break;
        }
        donors &= donors - 1;
        int e = __builtin_amdgcn_readlane(a - c, b);
        if (e > 2 && __popcll(receivers) > 2) {
            // all receivers at once: what those served before bank x need is a sum over the banks between
            // x and its mirror image in b, b's side of which counts first
            const int incl = wave_inclusive_sum(need), y = 2 * b - lane;
            const int mirror = __shfl(incl, min(max(y, 0), kWave - 1), kWave), q = y < 0 ? 0 : mirror;
            const int before = lane > b ? incl - need - q : q - incl;
            need -= min(need, max(0, e - before));
            receivers = __ballot(need > 0);
            continue;
        }
        // few slots or few receivers: the nearest receiver on either side is a bit scan away
        while (e > 0 && receivers != 0) {
            const u64 above = receivers >> b, below = receivers & ((1ull << b) - 1ull);   // b itself is none
            const int up = above ? __ffsll((long long)above) - 1 : kWave;
            const int dn = below ? b - (63 - __clzll((long long)below)) : kWave;
            const int x = up <= dn ? b + up : b - dn;
            const int n = __builtin_amdgcn_readlane(need, x), g = min(n, e);
            if (lane == x) need = n - g;
            e -= g;
            if (g == n) receivers &= ~(1ull << x);
        }
    }
    return c - need;                                      // donors keep what they can fill, receivers got the rest
}

// ---------------------------------------------------------------------------
// merge phase
// ---------------------------------------------------------------------------
__device__ __forceinline__ u64 pack_sel(int met_bits, int bank, uint32_t ord, uint32_t flat)
{
    const int fb = 32 - met_bits;
    const uint32_t flatmask = fb >= 32 ? 0xFFFFFFFFu : ((1u << fb) - 1u);
    u64 v = ((u64)ord << fb) | (u64)(flatmask - flat);
    if (met_bits) v |= (u64)bank << (64 - met_bits);
    return v;
}

// stream-phase key (score image << 32 | ~flat) -> selection key in bank `bank` (its body - score image
// << fb | ~flat in fb bits - orders like the stream-phase key); 0 stays 0
__device__ __forceinline__ u64 sel_from_rowkey(int met_bits, int bank, u64 key)
{
    if (key == 0) return 0;
    return pack_sel(met_bits, bank, (uint32_t)(key >> 32), key_flat(key));
}

// The phrases whose first token is w (w < 0: none), as a bit mask.  Every lane looks its own
// token up in the bucket of the token's low six bits: one trip to LDS where the bucket's
// phrases all begin with the same token (nearly always), else they are compared one by one.
template <typename Smem>
__device__ __forceinline__ u64 first_token_matches(int w, const Smem &sm)
{
    if (w < 0) return 0;
    const int same = sm.btok[w & 63];
    u64 todo = sm.fbucket[w & 63];
    if (same == w) return todo;
    u64 mine = 0;
    if (same == -2) {
        while (todo) {
            const int j = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            if (sm.ct.tok[sm.ct.poff[j]] == w) mine |= 1ull << j;
        }
    }
    return mine;
}

// Constraints met after a hypothesis (nmet met, phrase ip under way with iq tokens) emits a
// token: is_next = it continues the phrase under way; match = phrases it could begin;
// inc = phrases not complete.
__device__ __forceinline__ int nmet_after(int nmet, int ip, int iq, bool is_next, u64 match, u64 inc)
{
    if (ip >= 0 && is_next) return nmet + 1;
    const int base = ip >= 0 ? nmet - iq : nmet;          // a broken phrase is unwound
    return base + ((match & inc) ? 1 : 0);
}

// The 64 greatest 32-bit keys of the rows of one wave (row i of the wave = list(i), a
// decreasing list; rows are dealt out to the waves in turn, those from k on are empty).  Two
// chains of merges run side by side, so that their instructions interleave, and are joined at
// the end.  A list whose head is below place `kth` of the chain it would join cannot change
// places 0..kth of the result and is skipped; apart from that the result is exact.
template <int R, int MW, typename List>
__device__ __forceinline__ uint32_t wave_best64(int wave, int k, int kth, List list, uint32_t &fell)
{
    uint32_t a0 = wave < k ? list(0) : 0u;
    uint32_t a1 = (R > 1 && wave + MW < k) ? list(R > 1 ? 1 : 0) : 0u;
#pragma unroll
    for (int i = 2; i < R; i += 2) {
        if (wave + i * MW < k) {               // wave-uniform
            const bool pair = i + 1 < R && wave + (i + 1) * MW < k;
            const uint32_t s0 = list(i);
            const uint32_t s1 = pair ? list(i + 1 < R ? i + 1 : i) : 0u;
            const uint32_t h0 = (uint32_t)__builtin_amdgcn_readlane((int)s0, 0);
            const uint32_t h1 = (uint32_t)__builtin_amdgcn_readlane((int)s1, 0);
            const bool n0 = h0 != 0 && h0 >= (uint32_t)__builtin_amdgcn_readlane((int)a0, kth);
            const bool n1 = h1 != 0 && h1 >= (uint32_t)__builtin_amdgcn_readlane((int)a1, kth);
            if (n0 && n1) {
                a0 = merge32_desc(a0, s0, fell);
                a1 = merge32_desc(a1, s1, fell);
            } else if (n0) {
                a0 = merge32_desc(a0, s0, fell);
            } else if (n1) {
                a1 = merge32_desc(a1, s1, fell);
            }
        }
    }
    return __builtin_amdgcn_readlane((int)a1, 0) != 0 ? merge32_desc(a0, a1, fell) : a0;
}

// The 64 greatest keys of the lists the MW waves have left in buf (after a barrier), for the
// calling wave: a tree of merges whose independent pairs run side by side.
template <int MW>
__device__ __forceinline__ uint32_t join_best64(const uint32_t (*buf)[kWave], int wave, int lane, uint32_t &fell)
{
    uint32_t o[MW];
#pragma unroll
    for (int w = 0; w < MW; ++w) o[w] = buf[(wave + w) & (MW - 1)][lane];
#pragma unroll
    for (int span = 1; span < MW; span *= 2)
#pragma unroll
        for (int w = 0; w + span < MW; w += 2 * span) o[w] = merge32_desc(o[w], o[w + span], fell);
    return o[0];
}

// The same where most lists are expected to be empty (an empty list costs nothing), in every
// wave; one barrier.
template <int MW>
__device__ __forceinline__ uint32_t block_best64_sparse(uint32_t (&buf)[MW][kWave], int wave, int lane,
                                                        uint32_t mine, uint32_t &fell)
{
    buf[wave][lane] = mine;
    __syncthreads();
    uint32_t acc = mine;
#pragma unroll
    for (int w = 1; w < MW; ++w) {
        const uint32_t other = buf[(wave + w) & (MW - 1)][lane];
        if (__builtin_amdgcn_readlane((int)other, 0) != 0) acc = merge32_desc(acc, other, fell);
    }
    return acc;
}

// The same for lists of at most 32 keys, two side by side in a register: the 32 greatest of the N registers
// of a wave, in both halves.
template <int N>
__device__ __forceinline__ uint32_t best32_of(uint32_t (&o)[N], uint32_t &fell)
{
#pragma unroll
    for (int span = 1; span < N; span *= 2)
#pragma unroll
        for (int w = 0; w + span < N; w += 2 * span) o[w] = merge32_halves(o[w], o[w + span], fell);
    return join32_halves(o[0], fell);
}

// ---- hand-over inside one launch --------------------------------------------------------
// A place of the row lists and constraint keys is 0 while it is empty, kNoKey if there is no key for it.
constexpr u64 kNoKey = 1;             // (no key is 1: the score image of a finite sum is not 0)
constexpr int kGivenUp = 1 << 16;     // in BestCompleted::ended: the sentence is left to the row that ends last
constexpr int kLastTries = 1 << 16;   // where all rows have ended: their keys are in memory, the first look finds them (a damaged
                                      // workspace costs a wrong beam, not an endless wait)
constexpr int kAsked = 1, kGoesOn = 2, kLeaves = 3;    // MergeSmem::verdict

// A wave of sentence b's workgroup has run out of looks for its rows' keys.  The first one to do so tells the rows, in the
// atomic step that tells it how many have ended: if all, their keys are there (true); if not, the last one will find
// that said and take the sentence on (false).  The other waves go by what it was told.
__device__ __forceinline__ bool all_rows_ended(const StepParams &p, int b, int k, int &told)
{
    int verdict = 0;
    if (lane_id() == 0) {
        if (atomicCAS(&told, 0, kAsked) == 0) {
            const int ended = __hip_atomic_fetch_or(&p.best[b].ended, kGivenUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&told, ended == k ? kGoesOn : kLeaves, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        do verdict = __hip_atomic_load(&told, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while (verdict == kAsked);
    }
    return __builtin_amdgcn_readfirstlane(verdict) == kGoesOn;
}

__device__ __forceinline__ void hand_over(u64 *to, u64 key)
{
    __hip_atomic_store(to, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 handed_over(const u64 *from)
{
    return __hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The sentence's tables and beam on their way from memory to LDS, one entry a thread: every load
// is issued before the first one is waited for (clamped indices instead of branches).
struct MergeTables {
    int poff, tok, btok;
    u64 bucket;
    v4u lo, hi;                        // the two halves of a Hyp
    __device__ __forceinline__ int request(const StepParams &p, int b, int k, int tid)
    {
        const int lane = lane_id(), t64 = tid < kMaxCons ? tid : kMaxCons;
        const v4u *hyp = reinterpret_cast<const v4u *>(p.beam + ((size_t)b * k + (tid < k ? tid : k - 1)));
        const Sentence &s = p.sentences[b];
        poff = s.phr_off[t64];
        tok = s.tok[lane];
        const int P = s.nphr;
        bucket = s.first_bucket[lane];
        btok = s.bucket_tok[lane];
        lo = hyp[0];
        hi = hyp[1];
        return P;
    }
    template <typename Smem>
    __device__ __forceinline__ void store(int k, int tid, Smem &sm) const
    {
        if (tid <= kMaxCons) sm.ct.poff[tid] = poff;
        if (tid < kMaxCons) {
            sm.ct.tok[tid] = tok;
            sm.fbucket[tid] = bucket;
            sm.btok[tid] = btok;
        }
        if (tid < k) {
            HypState hs;
            hs.met = (u64)hi.y << 32 | hi.x;
            hs.inc = (u64)hi.w << 32 | hi.z;
            hs.ipq = ipq_of(lo.y);
            hs.nxt = (int)lo.w;
            hs.len = (int)lo.z;
            hs.misc = (flags_of(lo.y) & kFinFinished) | (__popcll(hs.met) << 8);
            sm.hyp[tid] = hs;
        }
    }
};

// the counters and the candidate buffer, by the first `threads` threads
template <typename Smem>
__device__ __forceinline__ void clear_for_merge(const StepParams &p, int tid, int threads, Smem &sm, u64 *cand)
{
    if (tid < 2 * kMaxCons) {
        sm.cnt[tid] = 0;
        sm.alloc[tid] = 0;                             // banks beyond the sentence's get no slot
        sm.start[tid] = 0;
        sm.first[tid] = 0;
    }
    if (tid < kMaxCons) sm.sel[tid] = 0;               // places beyond the last selected key compare as empty
    if (tid == 0) {
        sm.ncand = 0;
        sm.nsel = 0;
        sm.nleft = 0;
        sm.verdict = 0;
        sm.kept = 0;
    }
    for (int i = tid; i < p.cand_cap; i += threads) cand[i] = 0;
}

// MW: waves of the sentence's workgroup; ROWS: beam rows per wave the code is laid out for
// (k <= MW * ROWS; wave w takes rows w, w + MW, ...): the loops over a wave's rows are unrolled, so a
// smaller bound keeps the code of small beams short.
// J: where k * k <= 64 * J, every wave holds the k best of all the sentence's rows, J per lane (the entries that
// can be among the sentence's k best), and finds the bar by itself; J = 0: a wave holds the lists of its own
// rows and the waves' lists are merged; J = -1, k <= 32: the same with two rows to a register, which
// halves the merges, the registers looked through for candidates and the LDS they pass through.
// rowlists, conskeys, k, inv_k: what the first loads need (p.rowlists, p.conskeys, p.k; floor(2^16 / k) + 1,
// with which i * inv_k >> 16 is i / k for i < k * k, k <= 32).
// SRC: where the keys come from.  kInMemory, an earlier launch has left them there; kHandedOver, workgroups that run now (most_tries: how
// often a wave looks for them before it asks whether to go on; if not, the workgroup leaves and has written nothing.  all_ended:
// the sentence was left to this workgroup, a row's, as every row has ended); kInLds, the other waves of this workgroup, rowlists
// and conskeys point to those of its first row.  Tables and counters are in LDS already, but for kInMemory.
// (kHandedOver leaves the places empty, as it found them.)
constexpr int kInMemory = 0, kHandedOver = 1, kInLds = 2;

template <int ROWS, int MW, int J, int SRC>
__device__ __forceinline__ void merge_phase(const StepParams &p, const u64 *rowlists, const u64 *conskeys, int k,
                                            uint32_t inv_k, int b, MergeSmem<MW> &sm, u64 *cand, int P_here, int most_tries,
                                            bool all_ended)
{
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // in a scalar register: row guards are scalar branches
    // places of the lists of the sentence's row h
    auto at_row = [&](int h) { return SRC == kInLds ? (size_t)(h * kKeyCap) : ((size_t)b * k + h) * kWave; };
    // the row lists first: the chain of this phase starts with them, and their addresses need nothing
    // that has to be read from memory first
    constexpr bool kPacked = J > 0;
    constexpr bool kHalves = J < 0;
    constexpr int kRowsPerWave = ROWS;
    constexpr int kLists = kPacked ? J : (kHalves ? ROWS / 2 : ROWS);
    u64 rl[kLists], ck[kRowsPerWave];
    uint32_t head_bits = 0;                                // packed: bit j = this lane's entry j is a row's best
    if constexpr (SRC == kHandedOver) {
        // Handed over by workgroups that run now: read again until every place this wave looks at is filled (ONE's tables
        // and counters are in LDS already).  Only places that are still empty are asked for again: a look takes as long as its
        // requests, the keys are seen half a look late, and at the end it is one row that all wait for.  (Per step, all places asked for in
        // every look / this, and the heads of the lists by lane reads instead of loads of their own: 5 rows of 1000 8.5 / 7.9 us, ten of
        // 32000 10.5 / 10.2, 160 12.15 / 11.75, 168 of 50001 12.9 / 12.65, 612 of 4872 12.05 / 11.4, 595 of 24157 17.2 / 16.8.)
        static_assert(kPacked || kHalves, "lists of up to 32 keys");
        u64 miss[kLists], cmiss[kRowsPerWave];             // lanes whose place is empty
        const u64 *from[kLists], *cfrom[kRowsPerWave];
#pragma unroll
        for (int i = 0; i < kLists; ++i) {
            bool mine;
            uint32_t at;
            if constexpr (kPacked) {
                const uint32_t e = (uint32_t)(i * kWave + lane), h = (e * inv_k) >> 16;
                mine = e < (uint32_t)(k * k);
                head_bits |= (mine && e == h * (uint32_t)k ? 1u : 0u) << i;
                at = h * kWave + (e - h * (uint32_t)k);
            } else {
                const int h = wave + (2 * i + (lane >> 5)) * MW;
                mine = h < k && (lane & 31) < k;
                at = (uint32_t)(h * kWave + (lane & 31));
            }
            rl[i] = kNoKey;
            miss[i] = __ballot(mine);
            from[i] = rowlists + ((size_t)b * k * kWave + at);
        }
#pragma unroll
        for (int i = 0; i < kRowsPerWave; ++i) {
            const int h = wave + i * MW;
            ck[i] = kNoKey;
            cmiss[i] = __ballot(h < k && lane < P_here);
            cfrom[i] = conskeys + (((size_t)b * k + h) * kWave + lane);
        }
        bool last = all_ended;
        for (int tries = last ? kLastTries : most_tries;; --tries) {
#pragma unroll
            for (int i = 0; i < kLists; ++i)
                if (miss[i] != 0 && ((miss[i] >> lane) & 1ull)) rl[i] = handed_over(from[i]);
#pragma unroll
            for (int i = 0; i < kRowsPerWave; ++i)
                if (cmiss[i] != 0 && ((cmiss[i] >> lane) & 1ull)) ck[i] = handed_over(cfrom[i]);
            u64 any = 0;
#pragma unroll
            for (int i = 0; i < kLists; ++i) any |= miss[i] = __ballot(rl[i] == 0);
#pragma unroll
            for (int i = 0; i < kRowsPerWave; ++i) any |= cmiss[i] = __ballot(ck[i] == 0);
            if (any == 0) break;
            if (tries <= 0) {
                if (last || !all_rows_ended(p, b, k, sm.verdict)) break;
                last = true;
                tries = kLastTries;
            }
        }
#pragma unroll
        for (int i = 0; i < kLists; ++i) rl[i] = rl[i] == kNoKey ? 0 : rl[i];
#pragma unroll
        for (int i = 0; i < kRowsPerWave; ++i) ck[i] = ck[i] == kNoKey ? 0 : ck[i];
    } else {
        // left by an earlier launch or by the other waves: there already
        if constexpr (kPacked) {
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const uint32_t i = (uint32_t)(j * kWave + lane);
                rl[j] = 0;
                if (i < (uint32_t)(k * k)) {
                    const uint32_t h = (i * inv_k) >> 16, at = i - h * (uint32_t)k;
                    head_bits |= (at == 0 ? 1u : 0u) << j;
                    rl[j] = rowlists[at_row((int)h) + at];
                }
            }
        } else if constexpr (kHalves) {
            // register i: rows wave + 2 i MW and wave + (2 i + 1) MW
#pragma unroll
            for (int i = 0; i < kLists; ++i) {
                const int h = wave + (2 * i + (lane >> 5)) * MW;
                rl[i] = 0;
                if (h < k && (lane & 31) < k) rl[i] = rowlists[at_row(h) + (lane & 31)];
            }
        } else {
#pragma unroll
            for (int i = 0; i < kLists; ++i) {
                const int h = wave + i * MW;
                rl[i] = 0;
                if (h < k) rl[i] = rowlists[at_row(h) + lane];
            }
        }
#pragma unroll
        for (int i = 0; i < kRowsPerWave; ++i) {
            const int h = wave + i * MW;
            ck[i] = 0;
            if (h < k) ck[i] = conskeys[at_row(h) + lane];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    const int mb = p.met_bits;
    const int sel_shift = 64 - mb;
    const u64 body_mask = mb ? ((1ull << sel_shift) - 1ull) : ~0ull;
    const int fb = 32 - mb;
    const uint32_t flatmask = fb >= 32 ? 0xFFFFFFFFu : ((1u << fb) - 1u);
    const uint32_t tokmask = (1u << p.tok_bits) - 1u;

    MergeTables tables;
    int P = P_here;
    if constexpr (SRC == kInMemory) {
        P = tables.request(p, b, k, tid);
        clear_for_merge(p, tid, MW * kWave, sm, cand);
        if (kPacked) __syncthreads();
        // the lists are pinned here, or their loads would be moved down to the conditional code that uses them
#pragma unroll
        for (int i = 0; i < kLists; ++i) asm volatile("" : "+v"(rl[i]));
#pragma unroll
        for (int i = 0; i < kRowsPerWave; ++i) asm volatile("" : "+v"(ck[i]));
    }
    // ---- source 1: the sentence's k best (Sec. 3.1 item 1) = top k of the union of the row
    // lists.  All that is needed of them is the bar tau a key has to reach to be among them.
    // The k-th best SCORE comes from merging the 32-bit score images alone.  If the keys with
    // that score or a better one are exactly k, that is the bar.  Otherwise several keys tie
    // for the last places: the same merge over the low words (the coordinates, complemented)
    // of the keys with that score finds the last one that gets in. -------------------------
    uint32_t tau_s = 0;
    bool settled = true;
    int need = 0;                                          // places left for keys that tie at the bar's score
    uint32_t fell = 0, accs = 0;
    if constexpr (kPacked) {
        // Every wave for itself: no exchange between waves (one LDS round trip and one barrier cost as much as
        // three steps of the bisection).
        uint32_t image[J];
#pragma unroll
        for (int j = 0; j < J; ++j) image[j] = (uint32_t)(rl[j] >> fb);
        int reach;
        tau_s = kth_greatest<J>(image, k, reach);
        settled = tau_s == 0 || reach == k;
    } else if constexpr (kHalves) {
        uint32_t image[kLists];
#pragma unroll
        for (int i = 0; i < kLists; ++i) image[i] = (uint32_t)(rl[i] >> fb);
        accs = best32_of(image, fell);
    } else {
        accs = wave_best64<kRowsPerWave, MW>(wave, k, k - 1, [&](int i) { return (uint32_t)(rl[i] >> fb); }, fell);
    }
    // the sentence's tables and beam go to LDS only now: their loads were issued after those of the
    // row lists and arrive later, and the merges above needed none of them
    if constexpr (SRC == kInMemory) tables.store(k, tid, sm);
    // the waves' lists of 32, two to a register
    auto joined32 = [&](uint32_t *buf, uint32_t mine) {
        if (lane < 32) buf[wave * 32 + lane] = mine;
        __syncthreads();
        uint32_t o[MW / 2];
#pragma unroll
        for (int i = 0; i < MW / 2; ++i) o[i] = buf[i * kWave + lane];
        return best32_of(o, fell);
    };
    if constexpr (kHalves) {
        if (k == 32) sm.wf[wave][lane] = fell;
        accs = joined32(&sm.ws[0][0], accs);
        tau_s = (uint32_t)__builtin_amdgcn_readlane((int)accs, k - 1);
        if (tau_s != 0) {
            settled = (int)__popcll(__ballot(accs >= tau_s) & 0xFFFFFFFFull) == k;  // places k.. hold lower scores
            if (settled && k == 32) {
                // every place is taken: a tie may hide among the keys the merges dropped
                for (int w = 0; w < MW; ++w) {
                    const uint32_t f = sm.wf[w][lane];
                    fell = fell > f ? fell : f;
                }
                settled = wave_max_uniform(fell) < tau_s;
            }
        }
        need = k - __popcll(__ballot(accs > tau_s) & 0xFFFFFFFFull);
    } else if constexpr (!kPacked) {
        sm.wf[wave][lane] = fell;
        sm.ws[wave][lane] = accs;
        __syncthreads();
        // The sentence's best score images, lane i = i-th best, from the waves' lists.  With eight
        // waves two share a SIMD, and the join is the same work in every wave: the first four (one
        // per SIMD) do it and hand the outcome to the others.
        constexpr int kJoiners = MW < 4 ? MW : 4;
        if constexpr (MW > 8) {
            // in two rounds: four lists in each of four waves, then the four results
            if (wave < kJoiners) {
                accs = merge32_desc(merge32_desc(sm.ws[4 * wave][lane], sm.ws[4 * wave + 1][lane], fell),
                                    merge32_desc(sm.ws[4 * wave + 2][lane], sm.ws[4 * wave + 3][lane], fell), fell);
                sm.wf[wave][lane] = fell;
                sm.ws2[wave][lane] = accs;
            }
            __syncthreads();
        }
        if (wave < kJoiners) {
            accs = MW > 8 ? join_best64<4>(sm.ws2, wave, lane, fell) : join_best64<MW>(sm.ws, wave, lane, fell);
            tau_s = (uint32_t)__builtin_amdgcn_readlane((int)accs, k - 1);
            if (tau_s != 0) {
                settled = (int)__popcll(__ballot(accs >= tau_s)) == k;  // places k.. hold lower scores
                if (settled && k == kWave) {
                    // every place is taken: a tie may hide among the keys the merges dropped
                    for (int w = 1; w < MW; ++w) {
                        const uint32_t f = sm.wf[(wave + w) & (MW - 1)][lane];
                        fell = fell > f ? fell : f;
                    }
                    settled = wave_max_u32(fell) < tau_s;
                }
            }
            need = k - __popcll(__ballot(accs > tau_s));
            if (MW > kJoiners && tid == 0) {
                sm.bar_score = tau_s;
                sm.bar_need = settled ? -1 : need;
            }
        }
        if (MW > kJoiners) {
            __syncthreads();
            tau_s = sm.bar_score;
            need = sm.bar_need;
            settled = need < 0;
        }
    }
    // tau = what a selection-key body has to reach to be among the k best; 0 while fewer than
    // k finite sums exist, in which case every finite sum is among them.
    u64 tau = (u64)tau_s << fb;
    if (!settled) {                                        // the same decision in every wave
        const uint32_t low_bias = fb < 32 ? 1u : 0u;       // (a low word may be 0 where it has fewer than 32 bits)
        uint32_t tau_l;
        if constexpr (kPacked) {
            uint32_t low[J];
            int above = 0, reach;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const uint32_t hi = (uint32_t)(rl[j] >> fb);
                above += (int)__popcll(__ballot(hi > tau_s));
                low[j] = hi == tau_s ? ((uint32_t)rl[j] & flatmask) + low_bias : 0u;
            }
            need = k - above;
            tau_l = kth_greatest<J>(low, need, reach);
        } else if constexpr (kHalves) {
            uint32_t low[kLists];
#pragma unroll
            for (int i = 0; i < kLists; ++i) {
                // the tied keys of a decreasing list are neighbours: move them to the front of their half
                const uint32_t hi = (uint32_t)(rl[i] >> fb);
                const uint32_t lo = hi == tau_s ? ((uint32_t)rl[i] & flatmask) + low_bias : 0u;
                const u64 better = __ballot(hi > tau_s);
                const int to = (lane & 31) + (int)__popc((uint32_t)(better >> (lane & 32)));
                const uint32_t moved = (uint32_t)__shfl((int)lo, (lane & 32) | (to & 31), kWave);
                low[i] = to < 32 ? moved : 0u;
            }
            const uint32_t accl = joined32(&sm.ws2[0][0], best32_of(low, fell));
            tau_l = (uint32_t)__builtin_amdgcn_readlane((int)accl, need - 1);
        } else {
            uint32_t unused = 0;
            uint32_t accl = wave_best64<kRowsPerWave, MW>(wave, k, need - 1, [&](int i) {
                // the tied keys of a decreasing list are neighbours: move them to the front
                const uint32_t hi = (uint32_t)(rl[i] >> fb);
                if (__ballot(hi == tau_s) == 0) return 0u;     // most rows hold none
                const int first = __popcll(__ballot(hi > tau_s));
                const uint32_t lo = hi == tau_s ? ((uint32_t)rl[i] & flatmask) + low_bias : 0u;
                const uint32_t moved = (uint32_t)__shfl((int)lo, (lane + first) & (kWave - 1), kWave);
                return lane + first < kWave ? moved : 0u;
            }, unused);
            accl = block_best64_sparse<MW>(sm.ws2, wave, lane, accl, unused);
            tau_l = (uint32_t)__builtin_amdgcn_readlane((int)accl, need - 1);
        }
        tau = ((u64)tau_s << fb) | (u64)(tau_l - low_bias);
    }

    // ---- candidates, deduplicated by construction: the k best; a row's best (item 3, the
    // head of its list) unless among the k best; an expandable constraint token (item 2)
    // unless among the k best or equal to its row's best (the table never offers one token
    // twice for a hypothesis).  Each wave collects what its own rows give to sources 1 and 3
    // (in a decreasing list the keys that reach tau come first), works out their banks with
    // add() (Sec. 3.1), counts its candidates, reserves room with one atomic and writes them.
    // Lanes count what they hold themselves; two prefix sums over the wave then give every lane
    // its places (no wave-wide vote per row).
    const bool by_score = settled && tau_s != 0;
    // a constraint token is a candidate while below tau.  Where tau stands for a score alone,
    // one with exactly that score is among the k best only if its row's list holds it (every
    // listed key with that score is): those pass for now and are looked up below.
    const u64 below = by_score ? tau + (1ull << fb) : tau;
    const u64 from = tau > 1 ? tau : 1ull;                 // what a listed key has to reach; a row's best need not
    uint32_t gm = 0, cm = 0;                               // bit i: this lane's key i of the lists / of constraint tokens is kept
    bool some_tied = false;
#pragma unroll
    for (int i = 0; i < kLists; ++i) {
        const bool head = kPacked ? ((head_bits >> i) & 1u) != 0 : (kHalves ? (lane & 31) == 0 : lane == 0);
        gm |= ((rl[i] & body_mask) >= (head ? 1ull : from) ? 1u : 0u) << i;    // (an empty place holds 0)
    }
    if (tau != 0) {                                        // (else all finite sums are listed: none is left for source 2)
#pragma unroll
        for (int i = 0; i < kRowsPerWave; ++i) {
            if (wave + i * MW < k) {
                u64 best;
                if constexpr (kPacked) {
                    const int e = (wave + i * MW) * k;
                    best = read_lane(rl[0], e & (kWave - 1));
#pragma unroll
                    for (int j = 1; j < J; ++j) best = e >= j * kWave ? read_lane(rl[j], e & (kWave - 1)) : best;
                } else {
                    best = kHalves ? read_lane(rl[i / 2], (i & 1) * 32) : read_lane(rl[kPacked ? 0 : i], 0);
                }
                best &= body_mask;
                const u64 body = ck[i] & body_mask;
                const bool valid = body - 1 < below - 1 && body != best;      // (an empty place holds 0)
                cm |= (valid ? 1u : 0u) << i;
                if (by_score) some_tied |= valid && body >= tau;
            }
        }
    }
    if (__ballot(some_tied)) {                             // rare
#pragma unroll
        for (int i = 0; i < kRowsPerWave; ++i) {
            const int h = wave + i * MW;
            if (h < k) {
                const u64 body = ck[i] & body_mask;
                // (places from k on cannot be among the k best)
                const u64 listed = lane >= k ? 0ull
                                   : SRC == kHandedOver ? handed_over(rowlists + at_row(h) + lane)
                                   : (kPacked || kHalves) ? rowlists[at_row(h) + lane] : rl[kPacked ? 0 : i];
                u64 tied = __ballot(((cm >> i) & 1u) != 0 && body >= tau);
                while (tied) {
                    const int l = __ffsll((long long)tied) - 1;
                    tied &= tied - 1;
                    const u64 one = read_lane(body, l);
                    if (__ballot((listed & body_mask) == one) != 0 && lane == l) cm &= ~(1u << i);
                }
            }
        }
    }
    // Both kinds of key arrive with their bank (the constraints met once the token is placed, worked
    // out with add() by the row's own workgroup, Sec. 3.1), so a kept key goes straight to its place.
    // The counts cannot exceed the room (at most k keys reach tau, a row adds one more only if none of
    // its keys does, the host sized `cand` for every source) as long as the row lists are what the
    // stream phase writes: decreasing, distinct keys.  A wave that finds otherwise writes nothing: a
    // damaged list costs a wrong beam, not a stray write.  (The bank tables hold every value the
    // bank field of a key can take.)
    const int c = __popc(cm);                              // this lane's keys from source 2
    const int c_incl = wave_inclusive_sum(c);
    const int c_all = __builtin_amdgcn_readlane(c_incl, kWave - 1);
    int listed_all = 0, room = c_all;                      // packed: every wave knows all kept keys of the lists
    int g = 0, g_incl = 0;
    if constexpr (kPacked) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const u64 mask = __ballot(((gm >> j) & 1u) != 0);
            if (j % MW == wave && ((gm >> j) & 1u) != 0) {
                const int to = listed_all + lanes_before(mask);
                if (to < p.cand_cap) {
                    cand[to] = rl[j];
                    atomicAdd(&sm.cnt[mb ? (int)(rl[j] >> sel_shift) : 0], 1);    // bank = constraints met (Sec. 3.1)
                }
            }
            listed_all += (int)__popcll(mask);
        }
    } else {
        g = __popc(gm);                                    // this lane's keys from sources 1 and 3
        g_incl = wave_inclusive_sum(g);
        room += __builtin_amdgcn_readlane(g_incl, kWave - 1);
    }
    int at = 0;
    if (lane == 0 && room > 0) at = atomicAdd(&sm.ncand, room);
    at = listed_all + __builtin_amdgcn_readfirstlane(at);
    if (at + room <= p.cand_cap) {
        if constexpr (!kPacked) {
            int to = at + g_incl - g;
#pragma unroll
            for (int i = 0; i < kLists; ++i) {
                if ((gm >> i) & 1u) {
                    cand[to++] = rl[i];
                    atomicAdd(&sm.cnt[mb ? (int)(rl[i] >> sel_shift) : 0], 1);
                }
            }
        }
        int to = at + room - c_all + c_incl - c;
#pragma unroll
        for (int i = 0; i < kRowsPerWave; ++i) {
            if (wave + i * MW < k && ((cm >> i) & 1u)) {
                cand[to++] = ck[i];
                atomicAdd(&sm.cnt[mb ? (int)(ck[i] >> sel_shift) : 0], 1);
            }
        }
    }
    __syncthreads();                                       // tables and beam are in LDS too
    const int C = sm.ct.poff[P];
    const int ncand = min(listed_all + sm.ncand, p.cand_cap);
    const int nchunks = (ncand + kWave - 1) >> 6;

    // ---- slots per bank (Sec. 3.2) --------------------------------------------------------
    if (wave == 0) {
        const int c = sm.cnt[lane];
        const int c64 = sm.cnt[kMaxCons];
        int a64;
        const int a = allocate_wave(k, C, c, c64, a64, p.adjust != 0);
        sm.alloc[lane] = a;
        const int cc = lane <= C ? c : 0;
        const int incl = wave_inclusive_sum(cc);          // candidates in banks <= lane
        const int slots = wave_inclusive_sum(a);
        const int total63 = __builtin_amdgcn_readlane(incl, 63);
        const int slots63 = __builtin_amdgcn_readlane(slots, 63);
        const int c64v = C == 64 ? c64 : 0;
        sm.start[lane] = (total63 - incl) + c64v;         // candidates in higher banks
        sm.first[lane] = slots - a;
        if (lane == 0) {
            sm.alloc[kMaxCons] = a64;
            sm.start[kMaxCons] = 0;
            sm.first[kMaxCons] = slots63;
            sm.nsel = slots63 + a64;
        }
    }
    // ---- every candidate's place in the order (bank desc, score desc, coordinate asc), then within a
    // bank the best alloc[bank] are taken (Sec. 3.1/3.2) -------------------------------------
    auto select = [&](u64 mine, int rank) {
        const int bank = mb ? (int)(mine >> sel_shift) : 0;
        const int place = rank - sm.start[bank];
        if ((uint32_t)place < (uint32_t)sm.alloc[bank]) sm.sel[min(sm.first[bank] + place, kMaxBeam - 1)] = mine & body_mask;
    };
    constexpr int kCounters = MW - 1;                      // waves that count while wave 0 allocates
    // Up to here counting (n / lanes-per-candidate compares, no chain) is shorter than a 64-lane sort and
    // searches in the other chunks; at twice as many candidates it is longer (64 sentences, k = 32, 100 to 200
    // candidates: merge kernel 7.7 us with this limit, 8.3 with twice it, 7.6 sorted throughout; k = 20, about 80 of
    // them in most steps: 6.6 against 7.2 us sorted throughout).
    constexpr int kCountLimit = MW >= 8 ? 112 : 96;
    if (ncand <= kCountLimit) {
        // Few candidates (the usual case): the rank is the number of greater keys, counted over all of them.  A wave
        // takes 16 or 32 candidates, four or two lanes each, the lanes of a candidate each count a share.
        static_assert(kCountLimit <= 32 * kCounters, "every candidate has its lanes");
        const int each = ncand <= 16 * kCounters ? 16 : 32;
        const int share = kWave / each;                    // lanes per candidate
        const int i = (wave - 1) * each + (lane & (each - 1));
        u64 mine = 0;
        int rank = 0;
        if (wave > 0 && (wave - 1) * each < ncand) {
            mine = i < ncand ? cand[i] : 0ull;
            const u64 *key = cand + lane / each;
            for (int j = 0; j < ncand; j += 4 * share)     // (places from ncand to the next multiple of 16 hold 0)
                rank += (key[j] > mine ? 1 : 0) + (key[j + share] > mine ? 1 : 0) + (key[j + 2 * share] > mine ? 1 : 0) +
                        (key[j + 3 * share] > mine ? 1 : 0);
            rank += (int)xor_lane_u32<32, true>((uint32_t)rank);
            if (each == 16) rank += (int)xor_lane_u32<16, true>((uint32_t)rank);
        }
        __syncthreads();
        if (mine != 0 && lane < each) select(mine, rank);
    } else {
        // chunks of 64 are sorted by one wave each (wave 0, busy with the allocation, last); a
        // candidate's rank is the sum over the chunks of the keys greater than it, by a search with three probes a round
        const int my_first = MW - 1 - wave;
        for (int c = my_first; c < nchunks; c += MW) {
            const int i = c * kWave + lane;
            cand[i] = sort64_desc<u64, true>(i < ncand ? cand[i] : 0ull);
        }
        __syncthreads();
        // how many keys of chunks c0 .. c0 + 3 are greater; four searches at a time, so that their LDS reads overlap
        auto greater = [&](u64 mine, int c0) {
            int pos[4];
            bool full[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int c2 = min(c0 + q, nchunks - 1);      // out of range: ignored below
                pos[q] = 0;
                full[q] = cand[c2 * kWave + 63] > mine;
            }
            // three probes a round (quarters, then sixteenths, then single places): three
            // dependent trips to LDS instead of six
#pragma unroll
            for (int step = 16; step >= 1; step >>= 2) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u64 *at0 = cand + min(c0 + q, nchunks - 1) * kWave + pos[q] - 1;
                    const int above = (at0[step] > mine ? 1 : 0) + (at0[2 * step] > mine ? 1 : 0) +
                                      (at0[3 * step] > mine ? 1 : 0);
                    pos[q] += step * above;
                }
            }
            int sum = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (c0 + q < nchunks) sum += full[q] ? 64 : pos[q];
            return sum;
        };
        bool ranked = false;
        if (nchunks > 4) {
            // Many candidates (a wide beam with many constraints, up to a thousand early in a decode): only those
            // that are among their bank's first alloc[bank] in their own chunk can be among them in all, and only those are ranked,
            // a block of 64 of them against four chunks at a time.  (Every candidate against every chunk, five trips to LDS for
            // a block and four chunks, took 6 of 17.6 us in the slowest of 128 sentences, k = 64, 32 constraint tokens; all its
            // steps 145.5 -> 144.0 us in fp16.)  With four chunks or fewer the extra two barriers cost what they save.
            u64 *left = cand + p.cand_cap;
            int *ranks = reinterpret_cast<int *>(left + kMostLeft);
            for (int c = my_first; c < nchunks; c += MW) {
                const u64 mine = cand[c * kWave + lane];
                const int bank = mb ? (int)(mine >> sel_shift) : 0;
                const int below = (int)dpp_mov<kDppWaveShr1>((uint32_t)bank);    // (by every lane: a lane that is switched off reads as 0)
                const u64 starts = __ballot(lane == 0 || below != bank);
                const int first = 63 - __clzll((long long)(starts & (~0ull >> (63 - lane))));
                const bool keep = mine != 0 && lane - first < sm.alloc[bank];
                const u64 kept = __ballot(keep);
                int at = 0;
                if (lane == 0 && kept != 0) at = atomicAdd(&sm.nleft, (int)__popcll(kept));
                const int to = __builtin_amdgcn_readfirstlane(at) + lanes_before(kept);
                if (keep && to < kMostLeft) {
                    left[to] = mine;
                    ranks[to] = 0;
                }
            }
            __syncthreads();
            const int n = __builtin_amdgcn_readfirstlane(sm.nleft);
            if (n <= kMostLeft) {
                ranked = true;
                const int blocks = (n + kWave - 1) >> 6;
                int c0 = 0, block = wave;
                for (;;) {
                    while (block >= blocks && c0 < nchunks) {
                        block -= blocks;
                        c0 += 4;
                    }
                    if (c0 >= nchunks) break;
                    const int i = block * kWave + lane;
                    if (i < n) atomicAdd(&ranks[i], greater(left[i], c0));
                    block += MW;
                }
                __syncthreads();
                for (int i = tid; i < n; i += MW * kWave) select(left[i], ranks[i]);
            }
        }
        if (!ranked) {
            for (int c = my_first; c < nchunks; c += MW) {
                const u64 mine = cand[c * kWave + lane];
                int rank = 0;
                for (int c0 = 0; c0 < nchunks; c0 += 4) rank += greater(mine, c0);
                if (mine != 0) select(mine, rank);
            }
        }
    }
    __syncthreads();

    const int nsel = min(sm.nsel, k);
    if constexpr (SRC == kHandedOver) {
        const int verdict = __builtin_amdgcn_readfirstlane(sm.verdict);
        if (verdict == kLeaves) return;
        // once the last row has counted itself, the next step finds no row ended,
        if (wave == 2 && lane == 0)
            __hip_atomic_fetch_add(&p.best[b].ended, -(k + (all_ended || verdict == kGoesOn ? kGivenUp : 0)), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
    if constexpr (SRC == kHandedOver) {
        // and the places empty
        if (wave >= 2) {
            for (int h = wave - 2; h < k; h += MW - 2) {
                const size_t o = ((size_t)b * k + h) * kWave + lane;
                if (lane < k) hand_over(p.rowlists + o, 0);
                if (lane < P) hand_over(p.conskeys + o, 0);
            }
        }
    }

    // ---- new beam, best first (Sec. 3.1); empty slots last ---------------------------------
    // One lane per selected candidate.  Its place in the new beam is the number of selected keys greater
    // than its own (at most 64 uniform LDS reads: cheaper than a 64-lane sort); wave 1 counts that
    // while wave 0 takes the hypotheses through add().
    const bool live = lane < nsel;
    const u64 mine = (wave <= 1 && live) ? sm.sel[lane] : 0ull;
    if (wave == 1) {
        int slot = 0;
        for (int j = 0; j < nsel; j += 4)                 // (kMaxBeam is a multiple of 4; unused places hold 0)
            slot += (sm.sel[j] > mine ? 1 : 0) + (sm.sel[j + 1] > mine ? 1 : 0) + (sm.sel[j + 2] > mine ? 1 : 0) +
                    (sm.sel[j + 3] > mine ? 1 : 0);
        sm.slot[lane] = slot;
    }
    int token = p.pad_id, parent = -1, length = 0, ipq2 = -1, nxt2 = -1;
    float score = -INFINITY;
    u64 met2 = 0, inc2 = 0;
    uint8_t flags = 2, fin2 = 0;
    if (wave == 0) {
        if (live) {
            const uint32_t code = flatmask - ((uint32_t)mine & flatmask);
            parent = (int)(code >> p.tok_bits);
            token = (int)(code & tokmask);
            score = float_from_ord((uint32_t)(mine >> fb));
        }
        const u64 match = first_token_matches(live ? token : -1, sm);
        if (live) {
            const HypState hs = sm.hyp[min(parent, kMaxBeam - 1)];
            met2 = hs.met;
            inc2 = hs.inc;
            const int ipq = hs.ipq;
            int ip = ipq < 0 ? -1 : (ipq >> 8), iq = ipq < 0 ? 0 : (ipq & 255);
            const bool pfin = (hs.misc & kFinFinished) != 0;
            if (!pfin) {
                // add(token), Sec. 3.1: advance the phrase under way, or unwind it and let the
                // token begin the lowest-index incomplete phrase that starts with it
                if (ip >= 0 && token == hs.nxt) {
                    const int o = sm.ct.poff[ip];
                    met2 |= 1ull << (o + iq);
                    ++iq;
                    if (o + iq == sm.ct.poff[ip + 1]) {
                        inc2 &= ~(1ull << ip);
                        ip = -1;
                        iq = 0;
                    }
                } else {
                    if (ip >= 0) {
                        met2 &= ~(((1ull << iq) - 1ull) << sm.ct.poff[ip]);
                        ip = -1;
                        iq = 0;
                    }
                    const u64 startable = match & hs.inc;
                    if (startable) {
                        const int j = __ffsll((long long)startable) - 1;
                        const int o = sm.ct.poff[j];
                        met2 |= 1ull << o;
                        if (sm.ct.poff[j + 1] - o > 1) {
                            ip = j;
                            iq = 1;
                        } else {
                            inc2 &= ~(1ull << j);
                        }
                    }
                }
            }
            ipq2 = ip < 0 ? -1 : ((ip << 8) | iq);
            nxt2 = ip < 0 ? -1 : sm.ct.tok[sm.ct.poff[ip] + iq];
            fin2 = (pfin || token == p.eos_id) ? 1 : 0;
            length = pfin ? hs.len : hs.len + 1;
            flags = fin2;
            // Sec. 4: a hypothesis that completes now is kept with its score per word (one fp32
            // division, the length counts end-of-sentence); it competed with its raw sum above
            if (p.normalize && fin2 && !pfin) score = __fdiv_rn(score, (float)length);
        }
    }
    __syncthreads();
    if (wave == 0) {
        int slot = sm.slot[lane];
        // Sec. 4 / Sec. 6.3: hypotheses, completed or not, below (best completed - threshold) leave
        // the beam; the others close ranks
        bool keep = live;
        int nlive = nsel;
        if (p.prune >= 0.0f) {
            float best = (live && fin2) ? score : -INFINITY;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) best = fmaxf(best, __shfl_xor(best, d, kWave));
            if (best > -INFINITY) keep = live && score >= best - p.prune;
            if (keep) atomicOr(&sm.kept, 1ull << slot);
            // every lane's OR belongs to the one LDS instruction issued before this read
            const u64 km = __hip_atomic_load(&sm.kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            slot = __popcll(km & ((1ull << slot) - 1ull));
            nlive = __popcll(km);
        }
        const u64 open = __ballot(keep && !fin2);
        if (keep) {
            const size_t o = (size_t)b * k + slot;
            p.beam_nxt[o] = Hyp{score, state_word(fin2 | ((!fin2 && (int)__popcll(met2) < C) ? kFinEosBlocked : 0), ipq2),
                                length, nxt2, met2, inc2};
            p.hist_token[o] = token;
            p.hist_backptr[o] = parent;
            if (p.out_token) p.out_token[o] = token;
            if (p.out_backptr) p.out_backptr[o] = parent;
            if (p.out_score) p.out_score[o] = score;
            if (p.out_flags) p.out_flags[o] = flags;
        }
        if (lane >= nlive && lane < k) {                  // empty slots
            const size_t o = (size_t)b * k + lane;
            p.beam_nxt[o] = Hyp{-INFINITY, state_word(0, -1), 0, -1, 0, 0};
            p.hist_token[o] = p.pad_id;
            p.hist_backptr[o] = -1;
            if (p.out_token) p.out_token[o] = p.pad_id;
            if (p.out_backptr) p.out_backptr[o] = -1;
            if (p.out_score) p.out_score[o] = -INFINITY;
            if (p.out_flags) p.out_flags[o] = 2;
        }
        const u64 closed = __ballot(keep && fin2);
        if (p.track && closed != 0) {
            // Sec. 3.3: a completed hypothesis may lose its slot later on, so the best one seen so
            // far is remembered: value per word (the stored score where the beam already holds it
            // per word), replaced only by a strictly better one - the earliest step, then the
            // lowest slot keep a tie.  A hypothesis carried along compares equal to its own record.
            const bool cl = keep && fin2;
            const float q = !cl ? -INFINITY : (p.normalize ? score : __fdiv_rn(score, (float)length));
            float best = q;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) best = fmaxf(best, __shfl_xor(best, d, kWave));
            int first = (cl && q == best) ? slot : kWave;
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) first = min(first, __shfl_xor(first, d, kWave));
            if (cl && slot == first) {
                BestCompleted *r = p.best + b;
                if (!r->have || best > r->q) {
                    r->have = 1;
                    r->step = p.step;
                    r->slot = slot;
                    r->len = length;
                    r->q = best;
                    r->score = score;
                }
            }
        }
        if (lane == 0) {                                  // stopping tests: Sec. 4 (all), Sec. 6.3 (any)
            const uint8_t stop = (uint8_t)(((nlive > 0 && open == 0) ? 1 : 0) | (closed != 0 ? 2 : 0));
            p.all_finished[b] = stop;
            if (p.told)
                __hip_atomic_store(p.told + b, (uint32_t)(p.step + 1) << 2 | stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

}  // namespace dba
