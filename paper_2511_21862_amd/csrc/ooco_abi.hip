// Host side of libooco: context, argument validation, the work-list planner and the C ABI.
#include "../../include/ooco.h"
#include "ooco_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

using namespace ooco;

namespace {

thread_local char g_create_error[512] = "";

constexpr size_t kDefaultWorkspace = 128ull << 20;
constexpr size_t kPlanInts = 1u << 21;       // staging for cumulative arrays of very large batches
constexpr size_t kCounterInts = 1u << 20;    // arrival counters: num_seqs * num_kv_heads must fit
constexpr size_t kTraceWaves = 1u << 16;     // decode waves the trace buffer can hold
constexpr int kProfSlots = 1024;             // profiled calls between two ooco_profile_read
constexpr int kProfEvents = 6;               // events per profiled call

// ooco_attn_mixed_static: everything the kernels need beyond the caller's tensors lives in one fixed device array
// (arrival counters at the front, partial results behind them); see include/ooco.h
constexpr size_t kStaticScratchBytes = 16u << 20;
constexpr size_t kStaticCounterInts = 1u << 16;
constexpr int kStaticMaxDevices = 64;

}  // namespace

// One copy per GPU, at an address of its own on each; zero when the code object is loaded.  In host code the
// name below is only a handle for hipGetSymbolAddress, never a device address.  (No `used` attribute: the
// compiler gives a static device variable that host code refers to an externally visible symbol, which is what
// the runtime looks up; marked `used` it stays a local symbol and the lookup aborts.)
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
struct StaticDevice {
    void *ptr = nullptr;   // device address of `scratch` on this GPU
    int num_cus = 0;
};
std::mutex g_static_mu;
StaticDevice g_static_dev[kStaticMaxDevices];

// Address of this device's scratch array and its CU count, looked up once per device with that device current.
hipError_t static_device(StaticDevice &out, int &device)
{
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    if (device < 0 || device >= kStaticMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_static_mu);
    StaticDevice &d = g_static_dev[device];
    if (!d.ptr) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        int cus = 0;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
        if (e != hipSuccess) return e;
        d.num_cus = cus > 0 ? cus : 256;
        d.ptr = ptr;
    }
    out = d;
    return hipSuccess;
}
}  // namespace

namespace {
// Geometry and knobs the planner needs (no device state).
struct PlanGeometry {
    int Hq, Hkv, hd, BS, max_blocks_per_seq, num_cus;
    size_t ws_bytes;
    int64_t segments_opt;   // static runs; 0 = automatic
    int64_t tail_pct;       // share of the decode line handed out dynamically, in percent
    int64_t tail_blocks;    // KV blocks per dynamically fetched run
    int64_t pf_split_opt = 0;   // parts per prefill tile; 0 = automatic
    int64_t piece_pad = -1;     // line units charged for starting a piece (see build_plan); < 0 = automatic
    int64_t pf_waves_opt = 0;   // waves per prefill workgroup: 4, 8, or 0 = automatic
    int64_t pf_groups_opt = 0;  // key groups per prefill workgroup: 1, 4, or 0 = automatic
    int64_t coop_opt = 1;       // cooperative decode workgroups: 0 never, 1 by rule, 2 always
    int64_t lean_opt = 0;       // mixed batches: register-lean kernels (see HostPlan::lean)
    int64_t fused = 0;          // batches with both kinds of work run in the one-launch mixed kernel
    int64_t dec_cus_opt = 0;    // mixed kernel: compute units per XCD that decode; 0 = automatic
    int64_t pf_table_opt = 1;   // batches of at most kSortedTiles prefill tiles: tiles dispatched longest first across chunks
    uint16_t xcd_cw[kXcds] = {};   // cumulative XCD weights of the static runs; zeros = equal runs
};

// The compact plan: two cumulative arrays and a few scalars (see ooco_internal.h).
struct HostPlan {
    // (the two arrays live in storage the caller of build_plan provides, see PlanStorage)
    const int32_t *dcum = nullptr;   // [num_seqs+1] units of the decode line before each sequence (blocks + piece_pad per decode sequence)
    // prefill chunks, heaviest (most keys) first: pf[0..P] = query tiles before chunk k of that
    // order, pf[P+1+k] = sequence index of chunk k
    const int32_t *pf = nullptr;
    size_t pf_size = 0;              // 2 * num_pf + 1, + pf_table with the tile list
    int32_t pf_table = 0;            // > 0: pf goes on with that many (tile, part) entries in dispatch order (list_entry)
    int32_t num_pf = 0;
    int32_t dec_blocks = 0, static_blocks = 0, static_runs = 0, tail_runs = 0;   // in line units
    int32_t piece_pad = 0;
    int64_t kv_blocks = 0;       // KV blocks of all decode sequences
    uint16_t cw[kXcds] = {};     // XCD weights in force (RunLayout::cw)
    int32_t n_tiles = 0, total_q = 0, num_seqs = 0;
    int32_t pf_split = 1;        // parts a prefill tile's keys are cut into (with the tile list: the most any tile has)
    int64_t pf_slots = 0;        // partial-result slots of the split tiles per kv head (with the list: its leading entries that are parts)
    int32_t pf_waves = 4;        // waves per prefill workgroup (32 query columns each, of a key group)
    int32_t pf_groups = 1;       // key groups of a workgroup (1, or kKeyGroups in workgroups of eight waves)
    int32_t pf_col_waves() const { return pf_waves / pf_groups; }   // waves per tile of query columns
    int32_t pf_step_keys() const { return pf_groups > 1 ? 128 : 64; }   // keys of a workgroup's step
    // mixed batches (head_dim 128): the register-lean pair of kernels -- prefill workgroups of eight waves (176
    // registers, no software pipeline) and decode waves of 144 registers, four per compute unit -- so that a SIMD
    // holds two prefill waves and a decode wave at once
    int32_t lean = 0;
    int32_t dec_cus = 0;         // > 0: the batch runs in the mixed kernel with this many decoding compute units per XCD
    int64_t slots = 0;           // partial-result slots the decode kernel may touch
    // a batch with both kinds of work whose two kernels, one after the other, are estimated to take under 80 us: they
    // then run in sequence on the caller's stream (the fork and join of the second stream cost more than they gain)
    bool brief = false;
    bool two_streams = false;    // a batch with both kinds of work that runs faster as two kernels on two streams than in one launch
    bool near = false;           // step kernel: AttnParams::dec_near
    int32_t coop = 0;            // decode runs are worked on by workgroups of four waves (decode_coop_kernel); kCoopBySequence: run i is sequence i
    int32_t coop_waves = 4;      // waves of such a workgroup
    int32_t pf_units = 0;        // key groups beside decode work in one launch: the compute units that the prefill workgroups take
    int32_t nbi = 0;             // KV blocks per softmax step that the plan asks single decode waves for (0 = the kernel's default)
};

// XCD weights -> cumulative form; false if a weight is outside 1..255 or they differ by more than 4x.
bool xcd_weights_to_cw(const int32_t *w, uint16_t *cw)
{
    int32_t lo = 256, hi = 0, acc = 0;
    for (int k = 0; k < kXcds; ++k) {
        if (w[k] < 1 || w[k] > 255) return false;
        lo = std::min(lo, w[k]);
        hi = std::max(hi, w[k]);
        acc += w[k];
        cw[k] = (uint16_t)acc;
    }
    return hi <= 4 * lo;
}

size_t slot_bytes(const PlanGeometry &geo) { return (size_t)geo.Hq * (geo.hd + 2) * sizeof(float); }
// (one part of a split prefill tile, for one kv head)
size_t pf_part_bytes(const PlanGeometry &geo, const HostPlan &pl) { return (size_t)(32 * pl.pf_col_waves()) * (geo.hd + 2) * sizeof(float); }

// Where build_plan puts the plan's arrays: room for `seqs_cap` sequences, i.e. dcum [seqs_cap + 1],
// pf [2 * seqs_cap + 1 + kListEntries] and a work array order [seqs_cap].  build_plan itself allocates nothing.
struct PlanStorage {
    int32_t *dcum, *pf, *order;
    size_t seqs_cap;
};
PlanStorage carve_storage(int32_t *base, size_t seqs_cap)
{
    return PlanStorage{base, base + (seqs_cap + 1), base + (seqs_cap + 1) + (2 * seqs_cap + 1 + kListEntries), seqs_cap};
}
constexpr size_t storage_ints(size_t seqs_cap) { return (seqs_cap + 1) + (2 * seqs_cap + 1 + kListEntries) + seqs_cap; }

// Run layout of the decode block line (see ooco_internal.h): how many static runs, their XCD weights, the dynamic tail,
// the partial-result slots; fills out.static_runs / static_blocks / tail_runs / slots / cw / nbi.
// dec_blocks: units of the line (blocks + piece pads), kv_blocks: KV blocks of all decode sequences, dec_seqs: decode
// sequences that hold a block, max_blocks: blocks of the longest, pf_wgs: (tile, kv head) pairs of the batch's prefill
// part, lean: the batch runs the register-lean pair of kernels, dcum: the line, whose pads may grow here.
void plan_decode_runs(const PlanGeometry &geo, int num_seqs, int64_t dec_blocks, int64_t kv_blocks, int64_t dec_seqs, int64_t max_blocks,
                      int64_t pf_wgs, bool lean, int32_t *dcum, HostPlan &out)
{
    // static runs: by default three waves per CU (measured best on MI355X: enough loads in
    // flight to saturate HBM, few enough waves that start-up and partial results stay small)
    // and at least ~16 blocks of head_dim 128 per wave (a small batch is a chain of dependent blocks per wave:
    // one sequence of 512 blocks takes 27 us in 16 runs, 21 us in 32, 26 us in 64; eight sequences of 1121 blocks
    // 30 us in 36 runs, 25 us in 64)
    // (mixed kernel: eight decode waves on every decoding unit, one run each)
    int64_t wave_slots = lean ? std::max<int64_t>(1, (int64_t)geo.num_cus * 4 / geo.Hkv) : out.dec_cus == 99 ? std::max<int64_t>(1, (int64_t)geo.num_cus * 4 / geo.Hkv)
                               : out.dec_cus > 0 ? std::max<int64_t>(1, (int64_t)out.dec_cus * kXcds * 8 / geo.Hkv)
                                               : std::max<int64_t>(1, (int64_t)geo.num_cus * 3 / geo.Hkv);
    // A batch of SHORT sequences (24 blocks = 384 tokens on average, or fewer) is a line of many short pieces, each
    // with its own start (query vectors, first tiles): four waves per compute unit hide those better than three, and
    // one block per step wastes no padded step.  512 sequences of 128 tokens 58.5 -> 50.9 us, 900 of 64 71.9 -> 62.0,
    // 2048 of 256 403 -> 382, 1024 of 384 285 -> 275; 4096 of 512 tokens are faster with three waves (1430 / 1449 us).
    // Up to 16,384 tiles of them as many runs as sequences even if those hold fewer than 16 blocks, and, while there are fewer
    // than 2.5 waves per unit, two blocks per step: 32 sequences of 128 tokens 13.0 -> 10.2 us, 64 of 256 15.2 -> 13.2; 56 of 214
    // with one block 1.26 of the time, 64 of 166, 64/8 heads, 1.21.  More waves hide a piece's start by themselves, and a step
    // of one block has no empty half: 99 sequences of 169 tokens 13.5 -> 12.8, 216 of 202, 28/4 heads, 17.6 -> 16.8, 371 of 20..41,
    // 64/8 heads, 23.7 -> 21.2, 31 such batches 0.89 .. 1.0; 128 of 384 tokens, 24,576 tiles: 34.5 / 33.7 us.
    // A SMALL batch (at most 36,864 tiles, a tile being a (block, kv head) pair's 8 KiB of head_dim 128: with head_dim 64
    // twice as many blocks) cannot keep HBM busy anyway: what counts is the chain start -> steps of a wave -> partial
    // result -> merge.
    //   * One sequence, or sequences of more than 384 tokens on average of which at most two begin per run: its work is shared by
    //     the four waves of a workgroup (decode_coop_kernel), one workgroup per unit: one sequence of 1000 tokens 11.1 -> 7.8 us,
    //     of 4000 14.1 -> 10.0, of 16,000 24.1 -> 18.8, four of 2000..4000 20.1 -> 16.2.  Time over that of single waves, up to 0.5 /
    //     1 / 2 / more beginnings per run, 400 random batches: 0.73 / 0.88 / 0.95 / 0.97, us: 39 of 477..1908, 28/4 heads, 21.0 -> 18.3,
    //     24 of 885..1771, 64/8 heads, 27.6 -> 24.8; equal lengths 0.79 up to 0.5, then 0.90 .. 1.14 (one batch of another sweep 1.26), as
    //     single waves in as many runs cut nothing: half a one for them, and for lengths that differ by less than an eighth.
    //     Larger batches, however many begin per run: 0.93 / 0.96 / 0.97 / 0.97 up to 70,000 tiles, 0.97 .. 1.01 from there on (head_dim 64:
    //     0.97 and 0.99; equal lengths 0.97, left to single waves).
    //     Beside a prefill part, whose workgroups hold units that single waves would want too, up to one beginning per run, of
    //     equal lengths or not: 0.92 and 0.97; more 0.96 .. 1.01.
    //     Runs hold at least 16 blocks -- 8 where the sequences are of 64 blocks or fewer on average and so have few parts
    //     to merge (four of 500..1000 tokens 11.3 -> 8.5 us, but one of 4000 10.0 -> 12.3); 32 for sequences of more than
    //     512 blocks on average, whose many parts cost more than the shorter chain gains (one of 16,000 tokens, 64/8 heads,
    //     runs of 16 / 32 / 64 blocks 25.0 / 18.9 / 19.3), and beside a prefill part from 256 blocks on.
    //   * Else single waves, two blocks per step, two waves per unit.
    const int64_t tiles = kv_blocks * geo.Hkv * geo.hd / 128;
    const bool plain = !lean && out.dec_cus == 0 && dec_seqs > 0;
    const bool short_seqs = plain && kv_blocks <= 24 * dec_seqs;
    const bool small = plain && tiles <= 36864;
    const int64_t per_unit = std::max<int64_t>(1, (int64_t)geo.num_cus / geo.Hkv);   // runs that put one workgroup (of one kv head) on every unit
    const bool coop_can = plain && geo.tail_pct == 0 && geo.xcd_cw[kXcds - 1] == 0;
    const bool equal = max_blocks * dec_seqs == kv_blocks;
    const bool unequal = 8 * max_blocks * dec_seqs > 9 * kv_blocks;   // (by more than the cut of a run's ends)
    const bool coop_rule = short_seqs ? small && dec_seqs == 1
                           : pf_wgs > 0 ? tiles <= 70000 && dec_seqs <= per_unit
                           : small ? dec_seqs * (unequal ? 1 : 4) <= 2 * per_unit
                                   : tiles <= 70000 && (geo.hd == 128 || unequal);
    // A batch of short sequences takes one workgroup per (sequence, kv head) and cuts nothing: no partial results, no arrival
    // counters, no merge through memory.  Sequences of up to 768 tokens (48 blocks of head_dim 128: six steps of the four
    // waves; one of 1000 tokens is faster cut, 13.0 against 7.8 us), and by the number of workgroups per unit, against
    // single waves:
    //   * up to one: always (equal lengths 0.9 of the time, unequal ones 0.4..0.9).
    //   * up to two: but for equal lengths with head_dim 128 -- single waves, one run per sequence, cut nothing there either
    //     and start with one wave (64 sequences of 250 tokens, 8 kv heads, 14.9 against 12.2 us; unequal lengths 11.1
    //     against 13.9) --, and, without a prefill part, from 1.5 on but for sequences of more than 512 tokens that are much
    //     longer than the others (64 of median 150, longest 600: 1.09 of the time).
    //   * up to four, without a prefill part (whose workgroups would wait behind them: 128 of 60..200 tokens, 4 kv heads,
    //     beside 100 rows 23.0 against 20.3): unequal lengths in groups of so many heads that their partial results cost
    //     single waves most (256 of 62..250 tokens, 28/4 heads, 21.9 against 25.7; 640 of 150..600, 16/1 heads, 30.1
    //     against 38.3; 64/8 heads 0.75..1.0 of the time; 32/8 up to 2.5 workgroups 0.7..1.05, four 0.8..1.1; 32/32 0.9..1.3:
    //     smaller groups beyond that only up to 128 tokens, 0.75..1.0); up to 2.5 also equal ones of more than 384 tokens
    //     (0.8..0.98).
    const int64_t wgs = (int64_t)num_seqs * geo.Hkv, cus = geo.num_cus, g = geo.Hq / geo.Hkv;
    const int64_t longest = max_blocks * geo.hd;   // (in blocks of head_dim 1)
    const bool skewed = 5 * kv_blocks < 2 * max_blocks * dec_seqs;
    bool whole = longest <= 48 * 128;
    if (whole && wgs > 2 * cus) {
        const int64_t up_to = geo.hd == 64 ? (g >= 4 ? 32 : 8) : g >= 6 || (g >= 4 && 2 * wgs <= 5 * cus) ? 48 : 8;
        whole = pf_wgs == 0 && longest <= up_to * 128 && (equal ? 2 * wgs <= 5 * cus && longest > 24 * 128 : wgs <= 4 * cus);
    } else if (whole && wgs > cus) {
        whole = (geo.hd == 64 || !equal) && (pf_wgs > 0 || 2 * wgs <= 3 * cus || longest <= 32 * 128 || !skewed);
    }
    if (out.pf_units > 0) {
        // Beside prefill workgroups of key groups: workgroups of eight waves, one per unit that those leave.
        const int64_t left = std::max<int64_t>(1, (cus - out.pf_units) / geo.Hkv);
        out.coop_waves = 8;
        if (geo.segments_opt == 0 && longest <= 48 * 128 && num_seqs <= left) {
            out.coop = kCoopBySequence;
            out.static_runs = num_seqs;
            out.static_blocks = (int32_t)dec_blocks;
            return;
        }
        out.coop = 1;
    } else if (coop_can && geo.coop_opt && geo.segments_opt == 0 && whole) {
        out.coop = kCoopBySequence;
        out.static_runs = num_seqs;
        out.static_blocks = (int32_t)dec_blocks;
        return;
    }
    if (out.pf_units == 0) out.coop = coop_can && (geo.coop_opt >= 2 || (geo.coop_opt == 1 && coop_rule));
    if (!out.coop && geo.hd == 128 && short_seqs)
        out.nbi = tiles <= 16384 && 2 * dec_seqs * geo.Hkv < 5 * cus ? 2 : 1;
    else if (!out.coop && geo.hd == 128 && small)
        out.nbi = 2;
    int64_t min_blocks = 16 * 128 / geo.hd, at_least = 0;   // blocks of a run; runs whatever they hold
    if (out.coop) {
        // (beside a prefill part longer runs, which leave it units: one sequence of 16,000 tokens, 4 kv heads, beside
        // 100 rows 23.4 -> 16.9 us)
        wave_slots = out.pf_units > 0 ? std::max<int64_t>(1, (cus - out.pf_units) / geo.Hkv) : per_unit;
        min_blocks = kv_blocks > 512 * dec_seqs || (pf_wgs > 0 && kv_blocks > 256) ? 32 : pf_wgs > 0 || kv_blocks <= 16 || kv_blocks > 64 * dec_seqs ? 16 : 8;
        if (short_seqs) at_least = dec_seqs;
        // Starting a piece costs the whole workgroup, so it weighs more in the line: as much as 12 tiles of head_dim 128.
        // Pads of 3 / 6 / 12 / 24: sixteen sequences of 512..4096 tokens 31.5 / 31.1 / 30.6 / 30.5 us, sixteen of
        // 1000..2000 22.8 / 22.0 / 21.0 / 21.8; head_dim 64, pads of 6 / 12 / 24 / 36: 12.3 / 11.3 / 10.2 / 10.2.
        // Eight waves, beside key groups: 18 tiles.  60 random batches whose runs hold several pieces, time over the best of seven
        // pads of 3 / 6 / 9 / 12 / 18 / 24 / 30: 1.087 / 1.064 / 1.050 / 1.033 / 1.015 / 1.009 / 1.010, head_dim 64 (twice as many
        // units) 1.141 / 1.076 / 1.046 / 1.027 / 1.013 / 1.012 / 1.035.
        if (geo.piece_pad < 0) {
            const int32_t more = (out.coop_waves == 8 ? 5 : 3) * default_piece_pad(geo.hd);
            int32_t added = 0;
            for (int i = 0; i < num_seqs; ++i) {
                if (dcum[i + 1] + added > dcum[i]) added += more;   // (dcum[i] has its share already)
                dcum[i + 1] += added;
            }
            dec_blocks += added;
            out.dec_blocks = (int32_t)dec_blocks;
            out.piece_pad += more;
        }
    } else if (short_seqs && (geo.hd == 128 || small)) {
        wave_slots = std::max<int64_t>(1, (int64_t)geo.num_cus * 4 / geo.Hkv);
        min_blocks = 16;
        at_least = dec_seqs;
        // sequences of unequal lengths, of six blocks or more on average: runs that do not follow them anyway may as well
        // be short, up to two waves per unit (sixteen of 60..200 tokens 10.5 -> 8.6 us; head_dim 64: 64 of them
        // 18.7 -> 7.8; three waves per unit: 64 of 16..292 tokens, four layers, 48.9 -> 52.1).  Beside a prefill part
        // runs of 12 blocks (100 rows and 32 of 100..400 tokens, 4 kv heads, 14.7 us, with runs of 4 blocks 18.5).
        // No shorter than about the root of the longest sequence, though: one wave merges that one's parts, a quarter,
        // half or all of them in a row for groups of up to 4, 8 and 16 heads (16/1 heads, 128 sequences of median 250,
        // longest 1000 tokens, runs of 4 / 6 / 8 / 12 / 16 blocks 22.5 / 17.3 / 14.8 / 13.8 / 14.8; 127 of 30..300 and one
        // of 8000 in runs of 4 blocks 66.7, of 14 26.0).
        if (tiles <= 16384 && max_blocks * dec_seqs > kv_blocks + kv_blocks / 4 && kv_blocks >= 6 * dec_seqs) {
            const int64_t in_a_row = max_blocks * (g <= 4 ? 1 : g <= 8 ? 2 : 4) * geo.hd / 128;
            int64_t len = pf_wgs > 0 ? 12 : 4;
            while (8 * len * len < 5 * in_a_row) ++len;
            at_least = std::max(at_least, std::min<int64_t>((int64_t)geo.num_cus * 2 / geo.Hkv, kv_blocks / len));
        }
    } else if (small) {
        // (head_dim 64 keeps three: 363 sequences of 770 tokens on average 58.3 against 69.9 us with two)
        wave_slots = std::max<int64_t>(1, (int64_t)geo.num_cus * (geo.hd == 128 ? 2 : 3) / geo.Hkv);
        min_blocks = pf_wgs > 0 ? 24 : 16;
        // (head_dim 128, sequences of equal lengths: as many runs to each, so that no run holds the end of one and the start of the next --
        // 24 of 1000 tokens, 64/8 heads, in 48 runs 21.2 us, in 64 23.7; 40 of 768, 8 kv heads, in 40 23.2, cut 28.1 --
        // unless too few waves are left for long ones: 35 of 1536 in 35 runs 41.9, in 64 39.8)
        const int64_t odd = geo.hd == 128 && equal && wave_slots > dec_seqs ? wave_slots % dec_seqs : 0;
        if (8 * odd <= 3 * wave_slots || longest <= 48 * 128) wave_slots -= odd;
    }
    int64_t runs = geo.segments_opt > 0 ? geo.segments_opt
                                        : std::min<int64_t>(wave_slots, std::max<int64_t>((kv_blocks + min_blocks - 1) / min_blocks, at_least));
    runs = std::max<int64_t>(1, std::min<int64_t>(runs, dec_blocks));
    // (what prefill parts that were planned first leave of the workspace: they lie behind the slots, 256-byte aligned)
    const size_t pf_bytes = (size_t)out.pf_slots * geo.Hkv * pf_part_bytes(geo, out);
    const size_t ws_bytes = pf_bytes ? (geo.ws_bytes - std::min(geo.ws_bytes, pf_bytes)) / 256 * 256 : geo.ws_bytes;
    for (;;) {
        // weighted runs come in groups of one run per XCD
        bool weighted = geo.xcd_cw[kXcds - 1] != 0 && runs >= kXcds && out.dec_cus == 0;
        if (weighted) runs -= runs % kXcds;
        // dynamic tail: only when a static run is much longer than a tail run
        int64_t tail_blk = 0, tails = 0;
        if (geo.tail_pct > 0 && geo.tail_blocks > 0 && dec_blocks / runs >= 4 * geo.tail_blocks && out.dec_cus == 0) {
            tail_blk = std::min<int64_t>(dec_blocks - runs, dec_blocks * std::min<int64_t>(geo.tail_pct, 90) / 100);
            tails = (tail_blk + geo.tail_blocks - 1) / geo.tail_blocks;
            if (tails == 0) tail_blk = 0;
        }
        // ... and only for runs long enough that no weight (they differ by at most 4x) empties one
        if (dec_blocks - tail_blk < 16 * runs) weighted = false;
        // partial slots: (run index) + seq < runs + tails + num_seqs; one run never splits a sequence
        const int64_t slots = (runs + tails > 1) ? runs + tails + num_seqs : 0;
        if ((size_t)slots * slot_bytes(geo) <= ws_bytes || runs == 1) {
            if ((size_t)slots * slot_bytes(geo) > ws_bytes) {   // a single run, no tail, needs no slots
                tail_blk = tails = 0;
            }
            out.static_runs = (int32_t)runs;
            for (int k = 0; k < kXcds; ++k) out.cw[k] = weighted ? geo.xcd_cw[k] : 0;
            out.static_blocks = (int32_t)(dec_blocks - tail_blk);
            out.tail_runs = (int32_t)tails;
            out.slots = (runs + tails > 1) ? runs + tails + num_seqs : 0;
            break;
        }
        runs = (runs + 1) / 2;
    }
}

// What build_plan knows of the batch's prefill part when it decides how the tiles' keys are cut into parts.
struct PrefillFacts {
    int64_t tiles, tile_steps, max_tile_steps;   // tiles per kv head, their 64-key steps in all, steps of the longest
    size_t n_order;                              // prefill chunks
    const int32_t *st;                           // with the tile list: steps of the listed tiles, in list order
    int pf_waves;
    int64_t max_cols;                            // query columns of the widest tile
    int64_t dec_units;                           // units that the decode part needs, if it is planned later
    size_t dec_reserve;                          // workspace that the decode part may take, if it is planned later
    int64_t dec_blocks, kv_blocks;               // decode part: units of its line, KV blocks
    double pf_pairs;                             // visible (query row, key) pairs of all chunks
};

// Prefill tiles cut along the context when there are too few of them to occupy the GPU, or when a few of them are far
// longer than the rest: chooses the parts of every tile, rewrites the tile list as (tile, part) entries, fills
// out.pf_split / pf_slots / pf_table / pf_size.  `tab` is the tile list inside the plan's prefill array.
void plan_prefill_parts(const PlanGeometry &geo, const PrefillFacts &f, int32_t *const tab, HostPlan &out)
{
    const int64_t tiles = f.tiles, tile_steps = f.tile_steps, max_tile_steps = f.max_tile_steps;
    const size_t n_order = f.n_order;
    const int32_t *const st = f.st;
    const int pf_waves = f.pf_waves;
    const int64_t dec_blocks = f.dec_blocks, kv_blocks = f.kv_blocks;
    const double pf_pairs = f.pf_pairs;
    const int BS = geo.BS;
    const int64_t units = tiles * geo.Hkv;
    int64_t split = 1;
    const size_t part_bytes = pf_part_bytes(geo, out);
    const size_t left = geo.ws_bytes - std::min(geo.ws_bytes, std::max(f.dec_reserve, ((size_t)out.slots * slot_bytes(geo) + 255) / 256 * 256));
    const double cus = (double)geo.num_cus;
    // Estimated time in microseconds of a launch of w workgroups in all, the longest of them `longest` 64-key steps,
    // fitted to sweeps of 28 batches of equal chunks x 8 forced splits on MI355X (the choice is within 2.5 % of the best
    // forced split on every one of them, and better than any forced split on chunks of unequal contexts).  A workgroup's step takes 1.08 us while at most every other compute unit
    // holds a workgroup, 1.3 us with one workgroup on every unit, 1.95 us with two (the unit then completes a step
    // every 0.98 us, and further workgroups queue behind); the last workgroup of a tile merges the partial results
    // of its parts, which costs 2 us + 0.03 us per workgroup of the launch up to two per unit + 0.04 us for every
    // further one (their partial results then meet in memory at the same time).  The launch takes as long as its
    // average workgroup at the launch's occupancy or as its longest one beside what the others leave of a unit
    // (a chunk on a long context among chunks on short ones), whichever is more.
    auto step_us = [&](double r) {   // r = workgroups per compute unit
        if (r <= 0.5) return 1.08;
        if (r <= 1.0) return 1.08 + 0.44 * (r - 0.5);
        if (r <= 2.0) return 1.3 + 0.65 * (r - 1.0);
        return 0.975 * r;
    };
    // (the longest workgroup shares its unit with as many others as the launch has per unit, but no more than the
    // launch's work provides over its lifetime; a workgroup's start-up and epilogue, 2.5 us, come once per
    // workgroup that a unit holds at a time)
    // A compute unit holds ONE prefill workgroup, not two, when the workgroups have eight waves or when decode waves
    // share its registers (a batch with both kinds of work): such a workgroup counts as two, and beside decode
    // waves it never has a unit to itself.
    // (... a decode part, that is, which by its bytes lasts at least half as long as the prefill part by its FLOPs)
    const bool beside_decode = dec_blocks > 0 && !geo.fused &&
                               (double)kv_blocks * BS * 2.0 * geo.Hkv * geo.hd * 2.0 / 6.8e12 >= 0.5 * 4.0 * geo.Hq * geo.hd * pf_pairs / 1.05e15;
    const double wg_weight = beside_decode || pf_waves == 8 ? 2.0 : 1.0;
    const double all_steps = (double)tile_steps * geo.Hkv;   // 64-key steps of all workgroups together
    // w workgroups, w_big of them at least half as long as the longest one (`longest` steps), w_parts of them parts
    // of split tiles (which write partial results that the last of them merges)
    auto est = [&](double w, double w_big, double w_parts, double longest) {
        const bool merges = w_parts > 0.0;
        const double r = wg_weight * w / cus;
        const double beside = beside_decode ? 2.0 : std::min(std::min(r, 2.0), wg_weight * all_steps / (longest * cus));
        const double merge = merges ? 2.0 + 0.03 * std::min(w_parts, 2.0 * cus) + 0.04 * std::max(0.0, w_parts - 2.0 * cus) : 0.0;
        double average = all_steps / w * step_us(r);
        if (r > 2.0 && merges) {
            // more workgroups than fit at a time: the units work through them at full occupancy, and the long ones
            // go in rounds (up to four rounds count whole: the parts of a split tile are equally long, and 2.5
            // rounds of them take as long as 3; whole tiles of many lengths pack better than that)
            double rounds = wg_weight * w_big / (2.0 * cus);
            if (rounds <= 4.0) rounds = std::ceil(rounds - 1e-9);
            average = std::max(average, rounds * longest * 1.95);
        }
        return std::max(average, longest * step_us(beside)) + merge + 2.5 * std::ceil(std::min(r, 2.0));
    };
    // The same for k parts at head_dim 64, for batches without decode work: a workgroup has half the registers and LDS, so a unit
    // holds three; a step takes 0.95 us alone and hardly more beside others, the unit's steps 0.61 us at least whoever they
    // belong to, and the merge of a part reads half as much.  Fitted to 63 random batches of up to 512 tiles x 13 forced splits
    // (the choice is 2.3 % above the best of them on average, 14 % at worst; by the estimate above it was 7.6 and 54 %).  MI355X,
    // 32/4 heads (us): 615 rows on 1500 tokens 34.8 -> 21.9, 1036 on 1598 45.2 -> 34.7, 8 x 114 on 3800 66.0 -> 47.4.
    auto est64 = [&](double w, double w_parts, double longest, double k) {
        const double r = w / cus, beside = std::min(std::min(r, 1.15 * all_steps / (longest * cus)), 3.0);
        double body = std::max(longest * (beside <= 1.0 ? 0.945 : 0.95 + std::min(beside - 1.0, 0.15) / 3.0), all_steps / cus * 0.61);
        double rounds = r / 3.0;
        if (rounds > 1.0) {   // (parts are equally long: up to three rounds of them count whole)
            if (w_parts > 0.0 && rounds <= 3.0) rounds = std::ceil(rounds - 1e-9);
            body = std::max(body, rounds * all_steps / w * 0.82);
        }
        const double merge = w_parts > 0.0 ? std::max(1.5 + 0.3 * k, 0.64 + 0.29 * k + 2.03 * w_parts / cus) : 0.0;
        return 4.1 + 1.93 * std::min(r, 3.0) + body + merge;
    };
    // (below 16 steps the merge is most of what a split costs, and two workgroups keep a unit busy: the estimate above.  So it is
    // beside decode work, whose workgroups hold units as well: there the count of two per unit is kept, it was not fitted for three)
    const bool use64 = geo.hd == 64 && dec_blocks == 0 && out.pf_waves == 4 && max_tile_steps >= 16 && units < 2 * (int64_t)geo.num_cus;
    // With the tile list every tile gets parts by its own number of steps: the longest tile k parts, the others as
    // many as keep their parts no longer than that tile's (a tile of a short chunk stays whole beside a long one).
    // Without it (more than kSortedTiles tiles, or a forced value) every tile gets the same number.
    auto parts_of = [&](int64_t s, int64_t k, bool by_steps) -> int64_t {
        if (!by_steps) return std::min(k, s);
        const int64_t longest = (max_tile_steps + k - 1) / k;
        return std::min((s + longest - 1) / longest, s);
    };
    auto entries_of = [&](int64_t k, bool by_steps, int64_t *big = nullptr, int64_t *split_ones = nullptr) -> int64_t {
        const int64_t longest = (max_tile_steps + k - 1) / k;
        int64_t e = 0, b = 0, sp = 0;
        for (int64_t i = 0; i < tiles; ++i) {
            const int64_t parts = parts_of(st[i], k, by_steps);
            e += parts;
            if (2 * ((st[i] + parts - 1) / parts) >= longest) b += parts;
            if (parts > 1) sp += parts;
        }
        if (big) *big = b;
        if (split_ones) *split_ones = sp;
        return e;
    };
    // what a list of e entries, e_parts of them parts of split tiles, must fit: the kernel arguments; the counters
    // and the workspace (the parts come first in the list, and an entry's index is its partial-result slot)
    auto list_fits = [&](int64_t e, int64_t e_parts) {
        return e <= kListEntries && 2 * n_order + 1 + (size_t)e <= (size_t)kInlineSeqs + 1 &&
               e_parts * geo.Hkv <= kPrefillSplitUnits && (size_t)e_parts * geo.Hkv * part_bytes <= left;
    };
    bool by_steps = false;
    if (units <= kPrefillSplitUnits) {
        if (geo.pf_split_opt > 0) {
            split = std::min<int64_t>(std::min<int64_t>(geo.pf_split_opt, kMaxPrefillSplit), max_tile_steps);
        } else if (out.pf_table && out.pf_groups > 1) {
            by_steps = true;
            // Workgroups of several key groups: one per compute unit, so no more than those.  Time of a launch of r workgroups
            // per unit, the longest of L 128-key steps, in k parts, fitted to 934 batches of 1..8 equal chunks of 2..256 rows
            // on 0..30,000 cached tokens x 13 forced splits (the choice is 0.7 % above the best of them on average):
            // start-up and end 8.0 us (head_dim 64: 5.6), a step 1.06 .. 1.36 us by r (0.78 .. 0.98), the merge 2.0 us and
            // 0.21 per part, 0.36 with two waves' columns in it (1.5, 0.14, 0.24).
            const bool wide = geo.hd == 128;
            const double merge = (wide ? 0.21 : 0.14) + (f.max_cols > 32 ? (wide ? 0.15 : 0.10) : 0.0);
            auto est_groups = [&](int64_t wgs, int64_t longest, int64_t k) {
                const double r = std::min(1.0, (double)wgs / cus);
                const double step = !wide ? 0.78 + 0.2 * r : k > 1 ? 1.05 + 0.4 * r : 1.06 + 0.6 * std::max(0.0, r - 0.5);
                return (wide ? 8.0 : 5.6) + (double)longest * step + (k > 1 ? (wide ? 2.0 : 1.5) + merge * (double)k : 0.0);
            };
            // beside decode workgroups, one per unit that is left: the longer of the two
            const double dec_bytes = (double)kv_blocks * BS * 2.0 * geo.Hkv * geo.hd * 2.0;
            auto est_step = [&](int64_t wgs, int64_t longest, int64_t k) {
                const double t = est_groups(wgs, longest, k);
                if (kv_blocks == 0) return t;
                const double left_units = std::max(1.0, cus - (double)wgs);
                return std::max(t, 9.0 + dec_bytes / std::min(6.6e6, 0.030e6 * left_units)) + 0.1 * t;
            };
            double best = est_step(units, max_tile_steps, 1);
            int64_t worse = 0;
            for (int64_t k = 2; k <= kMaxGroupSplit && k <= max_tile_steps && worse < 8; ++k) {
                int64_t split_ones = 0;
                const int64_t e = entries_of(k, true, nullptr, &split_ones);
                if (e * geo.Hkv > geo.num_cus - (kv_blocks > 0 ? f.dec_units : 0) || !list_fits(e, split_ones)) break;
                const double t = est_step(e * geo.Hkv, (max_tile_steps + k - 1) / k, k);
                if (t < best) {
                    best = t;
                    split = k;
                    worse = 0;
                } else {
                    ++worse;
                }
            }
        } else if (out.pf_table) {
            by_steps = true;
            int64_t big = 0, split_ones = 0;
            (void)entries_of(1, true, &big);
            double best = use64 ? est64((double)units, 0.0, (double)max_tile_steps, 1.0)
                                : est((double)units, (double)(big * geo.Hkv), 0.0, (double)max_tile_steps);
            best *= 0.97;   // a split must win 3 %
            // (a launch of two or more workgroups per unit whose longest tile is no longer than the units' average
            // load cannot gain from more workgroups)
            // Beside a decode part that lasts longer anyway, parts beyond what hides the prefill part behind it only add
            // partial results to the memory traffic the decode part waits for: the fewest that do.  (48 sequences of
            // 500..4000 tokens, 8 kv heads, beside 2 x 120 rows on 600 tokens 83.5 -> 78.6 us, 4 x 60 on 1500 89.4 -> 82.3;
            // beside decode parts under 50 us, which start-up and merges stretch, the estimate's minimum stays best.)
            const double dec_us = (double)kv_blocks * BS * 2.0 * geo.Hkv * geo.hd * 2.0 / 6.8e6;
            const double hidden = pf_waves == 4 && !geo.fused && dec_us > 50.0 ? 0.8 * dec_us : 0.0;
            const bool full = best <= 0.97 * hidden ||
                              (wg_weight * (double)units >= 2.0 * cus && wg_weight * all_steps / cus * 0.975 >= (double)max_tile_steps * 1.95);
            for (int64_t k = 2; !full && k <= kMaxPrefillSplit && k <= max_tile_steps; ++k) {
                const int64_t e = entries_of(k, true, &big, &split_ones);
                if (!list_fits(e, split_ones)) break;
                const double longest = (double)((max_tile_steps + k - 1) / k);
                const double t = use64 ? est64((double)(e * geo.Hkv), (double)(split_ones * geo.Hkv), longest, (double)k)
                                       : est((double)(e * geo.Hkv), (double)(big * geo.Hkv), (double)(split_ones * geo.Hkv), longest);
                if (t < best) {
                    best = t;
                    split = k;
                    if (t <= hidden) break;
                } else if (k >= split + 4) {
                    break;   // (four values in a row without a gain: the estimate only grows from here)
                }
            }
        } else {
            const double steps = (double)tile_steps / (double)tiles;   // (every tile the same number of parts)
            double best = est((double)units, (double)units, 0.0, (double)max_tile_steps) * 0.97;
            for (int64_t sp = 2; sp <= kMaxPrefillSplit && sp <= (int64_t)steps; ++sp) {
                const double t = est((double)(units * sp), (double)(units * sp), (double)(units * sp), (double)((max_tile_steps + sp - 1) / sp));
                if (t < best) {
                    best = t;
                    split = sp;
                }
            }
        }
    }
    int64_t forced_parts = 0;
    if (out.pf_table && split > 1 && !by_steps && !list_fits(entries_of(split, false, nullptr, &forced_parts), forced_parts)) {
        // a forced number of parts whose list would not fit: the same parts without the list (chunk by chunk)
        out.pf_size -= (size_t)out.pf_table;
        out.pf_table = 0;
    }
    if (!out.pf_table)
        while (split > 1 && (size_t)units * (size_t)split * part_bytes > left) --split;
    if (out.pf_table && split > 1) {
        // (tile, part) entries: first the parts of the split tiles, then the whole tiles, each by decreasing number of
        // steps; the parts of a tile stay together, in part order; ties keep the chunk order and, inside a chunk,
        // the later tile first.  Sorted as plain numbers.
        uint64_t keys[kListEntries];
        size_t e = 0;
        int64_t most = 1;
        for (int64_t i = 0; i < tiles; ++i) {
            const int64_t s_i = st[i], parts = parts_of(s_i, split, by_steps), per = (s_i + parts - 1) / parts;
            most = std::max(most, parts);
            for (int64_t j = 0; j < parts; ++j)
                keys[e++] = ((uint64_t)(parts == 1) << 52) | ((uint64_t)(0xFFFFF - per) << 32) | ((uint32_t)entry_chunk(tab[i]) << 22) |
                            ((uint32_t)(1023 - entry_tile(tab[i])) << 12) | ((uint32_t)j << 6) | (uint32_t)(parts - 1);
        }
        std::sort(keys, keys + e);
        for (size_t i = 0; i < e; ++i) {
            const uint32_t k = (uint32_t)keys[i];
            tab[i] = list_entry((int)(k >> 22), 1023 - (int)((k >> 12) & 1023u), (int)((k >> 6) & 63u), (int)(k & 63u) + 1);
        }
        out.pf_size += e - (size_t)out.pf_table;
        out.pf_table = (int32_t)e;
        split = most;
        for (size_t i = 0; i < e && entry_parts(tab[i]) > 1; ++i) ++out.pf_slots;   // (the parts come first)
    } else if (split > 1) {
        out.pf_slots = tiles * split;
    }
    out.pf_split = (int32_t)split;
    // A launch of at most two four-wave workgroups per compute unit is one round: the hardware gives workgroups w
    // and w + CUs the same unit, and two workgroups that share a unit each advance at half its rate.  The tile
    // list then pairs the tile with the most steps with the one with the fewest, and so on (the second half of
    // the list ascending), so that every unit gets about the same number of steps: on MI355X one chunk of 2048
    // rows on 1662 cached tokens 102.1 -> 99.6 us, two of 1024 rows 67.5 -> 65.1 us (option "prefill_sorted" = 2
    // keeps the plain descending order).
    if (out.pf_table && geo.pf_table_opt == 1 && split == 1 && out.pf_waves == 4 && geo.num_cus % geo.Hkv == 0) {
        const int64_t half = geo.num_cus / geo.Hkv;   // tile positions whose workgroups arrive first on their unit
        if (tiles > half && tiles <= 2 * half) std::reverse(tab + half, tab + tiles);
    }
}

// Whether the prefill part of a batch runs in workgroups of key groups: eight waves, 64 query columns, each of the four groups
// walking a quarter of the keys, their results merged in LDS.  Such a workgroup has a compute unit to itself and takes
// 1.06 .. 1.36 us for 128 keys (one of four waves and 128 columns 1.08 .. 1.3 for 64), so it halves the chain of steps that
// bounds a batch of few tiles, and a tile of few columns wastes half as much; a batch that fills the units is better off with
// two workgroups of four waves on each.
//   * Without decode work, by the batch's load, 128-key steps of 64 columns per unit, against workgroups of four waves (699
//     random batches of up to 256 tiles of 64 columns on 256 units, nine head layouts): load up to 10: 0.80 of the time
//     (0.54 .. 1.03); 10..15: 0.88, but tiles of 65 to 90 columns on long contexts, which two workgroups then read twice, up
//     to 1.21; 15..25: 0.95 with up to 64 tiles and few unused columns, 1.0 (up to 1.7) with more, whose steps cannot be dealt
//     out evenly any more; above 25 1.07 and worse.  Fewer than three steps (head_dim 64: two) do not pay for the merge in LDS
//     (one step 6.4 -> 8.3 us, two 11.2 -> 10.3, with few columns 9.9 -> 10.3).
//   * Beside decode work (the step kernel, whose decode workgroups then have eight waves and a unit each too): where every
//     decode sequence finds a unit of its own or half of one, and the stream on the units that are left is no longer than the
//     prefill part or hardly longer than on all; not where the decode part alone decides the time (1713 random batches: 836
//     taken, 0.81 of the time, 39 of them more than 3 % slower, mostly by under a microsecond; one step more where one wave
//     holds all columns).
//   * "prefill_split" = 1, one workgroup per tile whatever its length, leaves only the chain, so any load (756 batches: 441
//     taken, 0.62 of the time, six of them more than 6 % slower).
//     With eight steps or more that chain decides the time also where the decode sequences have to share the units that
//     are left (120 batches of ooco_attn_mixed_static with more sequences than units: 48 taken, 0.61 of the time; us: 59
//     decodes of up to 1534 tokens beside 53 + 65 rows on 4728, 28/4 heads 95 -> 58; 128 beside 61 + 76 on 4518 107 -> 55;
//     with three or four steps 13.8 -> 15.8 .. 17.8, as they then wait for one another).  Where the decode part is the longer
//     one (54 batches at that edge, 0.78 of the time), it also takes ten steps at head_dim 128 (eight and nine: 0.85 .. 1.10,
//     us: 156 of up to 294 tokens beside 21 + 16 rows on 970, 28/4 heads 24.3 -> 26.6), and units enough that the decode part
//     takes less than 1.5 times as long as on all of them (71 on the 40 that 55 + 69 + 83 rows on 1700 leave, 64/8 heads 42.6
//     -> 50.0).
bool key_groups_pay(const PlanGeometry &geo, int num_seqs, const int32_t *h_seq_lens, const int32_t *h_query_start_loc)
{
    const int64_t g = geo.Hq / geo.Hkv, rows = prefill_tile_rows((int32_t)g, 8 / kKeyGroups);
    int64_t tiles = 0, steps = 0, longest = 0, widest = 0, n_dec = 0, dec_blk = 0;
    double cover = 0.0, used = 0.0;   // (row, step) pairs that the tiles have room for, and that the chunks have
    for (int i = 0; i < num_seqs; ++i) {
        const int64_t ql = (int64_t)h_query_start_loc[i + 1] - h_query_start_loc[i];
        if (ql == 1) {
            ++n_dec;
            dec_blk += ((int64_t)h_seq_lens[i] + geo.BS - 1) / geo.BS;
        }
        if (ql <= 1) continue;
        const int64_t t = (ql + rows - 1) / rows, s = ((int64_t)h_seq_lens[i] + 127) / 128;
        tiles += t;
        steps += t * s;
        cover += (double)(t * rows) * (double)s;
        used += (double)ql * (double)s;
        longest = std::max(longest, s);
        widest = std::max(widest, ql);
    }
    const int64_t units = tiles * geo.Hkv, load = steps * geo.Hkv, cus = geo.num_cus;
    const bool forced = geo.pf_groups_opt == kKeyGroups, whole = geo.pf_split_opt == 1;
    if (tiles == 0) return false;
    if (n_dec > 0) {
        // (the decode part in cooperative workgroups of the default run layout; a number of runs asked for is planned first,
        // with all of the workspace)
        if (geo.segments_opt && !forced) return false;
        if (!geo.coop_opt || geo.tail_pct || geo.xcd_cw[kXcds - 1] || num_seqs > kInlineSeqs / 2) return false;
        if (units + (whole && longest >= 8 ? 1 : n_dec) * geo.Hkv > cus) return false;
        if ((size_t)(cus / geo.Hkv + num_seqs + 1) * slot_bytes(geo) + 256 > geo.ws_bytes / 2) return false;
    }
    if (forced) return true;
    const int64_t enough = (geo.hd == 128 ? 3 : 2) + (n_dec > 0 && widest * g <= 32);
    // (without the tile list the parts of a tile are chosen for four waves: one chunk of 186 rows on 2760 tokens, 32/4 heads of
    // 64, five parts 21.8 us, key groups in one 24.2)
    if (units > cus || longest < enough || (geo.pf_split_opt > 0 && !whole) || !geo.pf_table_opt) return false;
    if (n_dec > 0) {
        // estimates in us, as in plan_prefill_parts
        const double bytes = (double)dec_blk * geo.BS * 2.0 * geo.Hkv * geo.hd * 2.0;
        const double dec_all = 9.0 + bytes / 6.6e6, dec_left = 9.0 + bytes / std::min(6.6e6, 0.030e6 * (double)(cus - units));
        const int64_t parts = whole ? 1 : std::max<int64_t>(1, std::min<int64_t>(kMaxGroupSplit, 4 * (cus - units) / (5 * units)));
        const double chain = (double)((longest + parts - 1) / parts), merge = parts > 1 ? 1.0 : 0.0, k = (double)parts;
        const double pf = geo.hd == 128 ? 8.0 + 1.2 * chain + merge * (2.0 + 0.3 * k) : 5.6 + 0.9 * chain + merge * (1.5 + 0.2 * k);
        if (dec_left > 1.35 * std::max(dec_all, pf) || pf < 0.7 * dec_all) return false;
        const bool shared_units = units + n_dec * geo.Hkv > cus;
        if (shared_units && dec_left > pf && (dec_left > 1.5 * dec_all || (geo.hd == 128 && longest < 10))) return false;
        if (!whole && parts == 1 && longest > 16) return false;   // (no unit left to cut a long tile)
    }
    return whole || load <= 10 * cus || (load <= 25 * cus && 4 * units <= cus && (widest <= rows || cover <= 1.2 * used));
}

// Validates the length arrays and builds the plan.  Pure host code, no allocation.
ooco_status build_plan(const PlanGeometry &geo, int num_seqs, const int32_t *h_seq_lens,
                       const int32_t *h_query_start_loc, const int32_t *h_ctx_lens, const PlanStorage &store,
                       HostPlan &out, char *err)
{
    auto bad = [&](ooco_status code, const char *fmt, ...) __attribute__((format(printf, 3, 4))) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(err, 512, fmt, ap);
        va_end(ap);
        return code;
    };
    out = HostPlan();
    if (num_seqs < 0) return bad(OOCO_EINVAL, "ooco_plan: num_seqs=%d", num_seqs);
    if (num_seqs > 0 && (!h_seq_lens || !h_query_start_loc || !h_ctx_lens))
        return bad(OOCO_EINVAL, "ooco_plan: NULL length array");
    const int BS = geo.BS;
    if (num_seqs > 0 && h_query_start_loc[0] != 0)
        return bad(OOCO_ESHAPE, "ooco_plan: query_start_loc[0]=%d, expected 0", h_query_start_loc[0]);
    if ((size_t)num_seqs > store.seqs_cap)
        return bad(OOCO_ENOMEM, "ooco_plan: %d sequences exceed the plan storage (%zu)", num_seqs, store.seqs_cap);
    out.num_seqs = num_seqs;
    int32_t *const dcum = store.dcum, *const pf = store.pf, *const order = store.order;
    out.dcum = dcum;
    out.pf = pf;
    std::fill(dcum, dcum + num_seqs + 1, 0);
    // The decode line: every decode sequence contributes piece_pad units followed by one unit per KV block.  The
    // runs cut the line into equal lengths, so a run that starts several pieces streams correspondingly fewer
    // blocks (starting a piece costs a wave about as long as streaming three 8 KiB tiles).
    int64_t dec_blocks = 0, kv_blocks = 0, tiles = 0, tile_steps = 0, max_tile_steps = 1;
    int64_t max_cols = 0;                        // query columns of the widest prefill tile
    int64_t dec_seqs = 0, max_dec_blocks = 0;    // decode sequences that hold at least one block, blocks of the longest
    double pf_pairs = 0.0;   // visible (query row, key) pairs of all prefill chunks
    const int64_t pad = geo.piece_pad < 0 ? default_piece_pad(geo.hd) : geo.piece_pad;
    // Waves per prefill workgroup.  Eight waves share every K/V tile staged in LDS among 256 query columns instead
    // of 128, which halves the traffic from L2 into the compute units.  Measured on MI355X it is no faster (that
    // traffic is not what bounds the kernel) and its 220-register waves leave no room for decode waves beside
    // them, so four waves are the default; eight (head_dim 128 only) stay selectable.
    // The register-lean pair for batches with both kinds of work (lean_opt 2 = whenever the batch is mixed; 1 = when
    // it pays: every compute unit gets at least one eight-wave prefill workgroup -- counting the parts of 16 or more
    // 64-key steps that tiles on a long context can be cut into --, and the prefill part, by itself,
    // would take between 0.30 and 2 times as long as the decode part -- estimated from the batch's FLOPs and bytes at 1.05 PFLOP/s
    // and 6.8 TB/s --, 0.50 with fewer than two workgroups per unit beside a decode part of up to 150 us).  MI355X, 250 random
    // batches, time of four-wave workgroups in one launch over that of the pair: with two workgroups per unit or a longer decode part
    // 0.95 below 0.30, 1.02 up to 0.75, 0.97 up to twice, 0.93 from there on (the pair's prefill workgroups have no software
    // pipeline: 9 % slower alone).  With fewer workgroups and short decode parts (its decode waves are 4 % slower alone, and it has
    // no cooperative ones) 0.93, inside the bounds too, where an earlier sweep had 1.01 and more: the line there is in need of
    // another.  32/8 heads, 128 decodes of 1.4 GB in all beside 8 x 512 rows 247 us; the long-context batch of 64/8 heads 1.57 ms,
    // with two kernels on two streams 1.8.
    bool lean = false;
    if (geo.lean_opt && geo.hd == 128 && !geo.fused && num_seqs > 0) {
        const int rows8 = prefill_tile_rows(geo.Hq / geo.Hkv, 8);
        int64_t n_dec = 0, tiles8 = 0, wgs8 = 0, dec_blk = 0;
        double pairs = 0.0;
        for (int i = 0; i < num_seqs; ++i) {
            const int64_t ql = (int64_t)h_query_start_loc[i + 1] - h_query_start_loc[i];
            n_dec += ql == 1;
            if (ql == 1) dec_blk += ((int64_t)h_seq_lens[i] + BS - 1) / BS;
            if (ql > 1) {
                const int64_t t8 = (ql + rows8 - 1) / rows8, parts = ((int64_t)h_seq_lens[i] + 63) / 64 / 16;
                tiles8 += t8;
                wgs8 += t8 * std::min<int64_t>(std::max<int64_t>(parts, 1), kMaxPrefillSplit);
                pairs += (double)ql * (double)h_ctx_lens[i] + (double)ql * (double)(ql + 1) / 2.0;
            }
        }
        const double t_pf = 4.0 * geo.Hq * geo.hd * pairs / 1.05e15;
        const double t_dec = (double)dec_blk * BS * 2.0 * geo.Hkv * geo.hd * 2.0 / 6.8e12;
        const double least = tiles8 * geo.Hkv >= 2 * (int64_t)geo.num_cus || t_dec > 150e-6 ? 0.30 : 0.50;
        const bool pays = wgs8 * geo.Hkv >= (int64_t)geo.num_cus && t_pf >= least * t_dec && t_pf <= 2.0 * t_dec;
        lean = n_dec > 0 && tiles8 > 0 && (geo.lean_opt >= 2 || pays);
    }
    out.lean = lean;
    const int pf_waves = geo.hd == 128 && (geo.pf_waves_opt == 8 || lean) ? 8 : 4;
    out.pf_waves = pf_waves;
    const int g = geo.Hq / geo.Hkv;
    if (geo.pf_groups_opt != 1 && !lean && !geo.fused && geo.pf_waves_opt == 0 && key_groups_pay(geo, num_seqs, h_seq_lens, h_query_start_loc))
        out.pf_groups = kKeyGroups, out.pf_waves = 8;
    const int step_keys = out.pf_step_keys();
    const int tile_rows = prefill_tile_rows(geo.Hq / geo.Hkv, out.pf_col_waves());
    for (int i = 0; i < num_seqs; ++i) {
        const int64_t ql = (int64_t)h_query_start_loc[i + 1] - h_query_start_loc[i];
        if (ql < 0) return bad(OOCO_ESHAPE, "ooco_plan: query_start_loc decreases at sequence %d", i);
        if (h_ctx_lens[i] < 0 || h_seq_lens[i] < 0)
            return bad(OOCO_ESHAPE, "ooco_plan: negative length at sequence %d", i);
        if ((int64_t)h_ctx_lens[i] + ql != h_seq_lens[i])
            return bad(OOCO_ESHAPE, "ooco_plan: sequence %d has ctx_len %d + q_len %lld != seq_len %d", i,
                       h_ctx_lens[i], (long long)ql, h_seq_lens[i]);
        const int64_t nb = ((int64_t)h_seq_lens[i] + BS - 1) / BS;
        if (nb > geo.max_blocks_per_seq)
            return bad(OOCO_ESHAPE, "ooco_plan: sequence %d needs %lld blocks > max_blocks_per_seq %d", i,
                       (long long)nb, geo.max_blocks_per_seq);
        if (ql == 1) {
            dec_blocks += nb + pad;
            kv_blocks += nb;
            dec_seqs += nb > 0;
            max_dec_blocks = std::max(max_dec_blocks, nb);
        }
        if (ql > 1) {
            pf_pairs += (double)ql * (double)h_ctx_lens[i] + (double)ql * (double)(ql + 1) / 2.0;
            tiles += (ql + tile_rows - 1) / tile_rows;
            max_cols = std::max(max_cols, std::min<int64_t>(ql, tile_rows) * g);
            for (int64_t t0 = 0; t0 < ql; t0 += tile_rows) {    // 64-key steps of every tile
                const int64_t nstep = ((int64_t)h_ctx_lens[i] + std::min<int64_t>(ql, t0 + tile_rows) + step_keys - 1) / step_keys;
                tile_steps += nstep;
                max_tile_steps = std::max(max_tile_steps, nstep);
            }
        }
        if (dec_blocks > 0x7FFFFFFF / 2 || tiles > 0x7FFFFFFF / 128)
            return bad(OOCO_ESHAPE, "ooco_plan: batch too large");
        dcum[(size_t)i + 1] = (int32_t)dec_blocks;
    }
    out.total_q = num_seqs > 0 ? h_query_start_loc[num_seqs] : 0;
    out.dec_blocks = (int32_t)dec_blocks;
    out.kv_blocks = kv_blocks;
    out.piece_pad = (int32_t)pad;
    out.n_tiles = (int32_t)tiles;
    // prefill chunks in order of decreasing sequence length: workgroups are dispatched in index
    // order, so the long ones start first and the short ones fill the end
    size_t n_order = 0;
    for (int i = 0; i < num_seqs; ++i)
        if (h_query_start_loc[i + 1] - h_query_start_loc[i] > 1) order[n_order++] = i;
    // (equal lengths keep their batch order; std::sort with the index as tie-break needs no temporary buffer)
    std::sort(order, order + n_order, [&](int32_t x, int32_t y) {
        return h_seq_lens[x] != h_seq_lens[y] ? h_seq_lens[x] > h_seq_lens[y] : x < y;
    });
    out.num_pf = (int32_t)n_order;
    out.pf_size = 2 * n_order + 1;
    std::fill(pf, pf + out.pf_size, 0);
    for (size_t k = 0; k < n_order; ++k) {
        const int64_t ql = (int64_t)h_query_start_loc[order[k] + 1] - h_query_start_loc[order[k]];
        pf[k + 1] = pf[k] + (int32_t)((ql + tile_rows - 1) / tile_rows);
        pf[n_order + 1 + k] = order[k];
    }
    int32_t st[kSortedTiles];   // with the tile list: 64-key steps of the listed tiles, in list order
    auto steps_of = [&](int32_t e) -> int64_t {   // 64-key steps of the tile a list entry names
        const int i = order[entry_chunk(e)];
        const int64_t ql = (int64_t)h_query_start_loc[i + 1] - h_query_start_loc[i], t0 = (int64_t)entry_tile(e) * tile_rows;
        return ((int64_t)h_ctx_lens[i] + std::min<int64_t>(ql, t0 + tile_rows) + step_keys - 1) / step_keys;
    };
    // A launch of few tiles is as long as its unluckiest compute unit is busy, and the hardware hands workgroups out
    // in index order to whichever unit has room: the tiles of ALL chunks go out by decreasing number of 64-key
    // steps (a chunk on a short context has fewer steps in its last tile than one on a long context in its first).
    // (only while the longer array still travels in the kernel arguments)
    if (geo.pf_table_opt && tiles > 0 && tiles <= kSortedTiles && 2 * n_order + 1 + (size_t)tiles <= (size_t)kInlineSeqs + 1) {
        // (ties keep the chunk order and, inside a chunk, the later tile first; sorted as plain numbers: steps
        // descending in the high half, chunk and descending tile below)
        int32_t *const tab = pf + out.pf_size;
        uint64_t keys[kSortedTiles];
        size_t n = 0;
        for (size_t k = 0; k < n_order; ++k)
            for (int32_t t = pf[k + 1] - pf[k] - 1; t >= 0; --t)
                keys[n++] = ((uint64_t)(0xFFFFF - steps_of(list_entry((int)k, t, 0, 1))) << 32) | (uint32_t)((k << 10) | (uint32_t)(1023 - t));
        std::sort(keys, keys + n);
        for (size_t i = 0; i < n; ++i) {
            tab[i] = list_entry((int)((uint32_t)keys[i] >> 10), 1023 - (int)((uint32_t)keys[i] & 1023u), 0, 1);
            st[i] = (int32_t)(0xFFFFF - (keys[i] >> 32));
        }
        out.pf_size += n;
        out.pf_table = (int32_t)n;
    }

    // ---- short mixed batches.  Measured on MI355X (32/8 heads): 1 x 64 rows + 4 decode sequences 50.7 us side by
    // side, 44.9 us in sequence; 1 x 128 + 8: 49.0 / 46.9; 2 x 128 + 32: 84.9 / 81.3; 4 x 128 + 64: 129.8 / 139.7 -- and
    // enqueueing the forked call costs the host 41 us against 8 us.  Estimate: each kernel's roofline time plus its
    // fixed cost (15 us decode, 12 us prefill).
    if (dec_blocks > 0 && tiles > 0) {
        const double t_dec = (double)kv_blocks * BS * 2.0 * geo.Hkv * geo.hd * 2.0 / 6.8e12 + 15e-6;
        const double t_pf = 4.0 * geo.Hq * geo.hd * pf_pairs / 1.05e15 + 12e-6;
        out.brief = t_dec + t_pf < 80e-6;
        // One launch for both kinds saves the second stream's fork and join (13 to 18 us of a call on an idle GPU), and its decode workgroups are
        // spread over the units a little less evenly than the decode kernel's single waves, which a long stream pays for:
        // 32/8 heads, 131 / 276 / 412 us of K/V at 6.8 TB/s beside 4 x 528 rows 172 -> 171, 321 -> 328, 461 -> 470 us; beside
        // 128 workgroups (1 x 512 rows) 164 -> 159, 316 -> 307, 460 -> 457.  (The register-lean pair gains at any length.  With the
        // prefill kernel as it is now one launch takes 0.96 of the time in those batches as well; the tests of the form with two streams
        // state this line.)
        out.two_streams = !lean && t_dec - 15e-6 > 180e-6 && tiles * geo.Hkv > geo.num_cus / 2;
    }
    // ---- one launch for both kinds of work: how many compute units of every XCD decode.  The decode part is
    // bound by HBM and reaches its bandwidth from a part of the units; the prefill part is bound by the matrix
    // cores and takes as long as its share of the units makes it.  The prefill units are sized so that they
    // finish with the decode stream (estimated from rates measured on MI355X: 6.8 TB/s, and 1.05 PFLOP/s on all
    // units), leaving the decode side at least kMinDecCus units per XCD; whoever finishes first helps the other.
    const int cus_per_xcd = std::max(1, geo.num_cus / kXcds);
    if (geo.fused && pf_waves == 4 && dec_blocks > 0 && tiles > 0 && cus_per_xcd >= 4 && geo.num_cus % kXcds == 0) {
        constexpr int kMinDecCus = 10;
        const double t_dec = (double)kv_blocks * BS * 2.0 * geo.Hkv * geo.hd * 2.0 / 6.8e12;
        const double t_pf = 4.0 * geo.Hq * geo.hd * pf_pairs / 1.05e15;
        int pf_cus = (int)std::ceil(cus_per_xcd * t_pf / std::max(t_dec, 1e-9));
        pf_cus = std::max(1, std::min(pf_cus, cus_per_xcd - std::min(kMinDecCus, cus_per_xcd / 2)));
        int dec = cus_per_xcd - pf_cus;
        if (geo.dec_cus_opt > 0) dec = (int)std::min<int64_t>(geo.dec_cus_opt, cus_per_xcd - 1);
        if (geo.dec_cus_opt == 99) dec = 99;   // every unit runs both kinds (one workgroup each): for measurements
        out.dec_cus = dec;
    }
    // ---- run layout of the decode block line (see plan_decode_runs); prefill tiles cut along the context (see
    // plan_prefill_parts).  Prefill workgroups of key groups come first: the decode part gets the units that they leave.
    const bool pf_first = out.pf_groups > 1 && dec_blocks > 0;
    auto plan_decode = [&]() {
        if (dec_blocks > 0) plan_decode_runs(geo, num_seqs, dec_blocks, kv_blocks, dec_seqs, max_dec_blocks, tiles * geo.Hkv, lean, dcum, out);
    };
    if (!pf_first) plan_decode();
    // The lean pair's decode waves of a workgroup side by side (half a percent of a long stream), but not where the longest
    // sequence is cut into more than 32 parts, whose merges then meet on one unit (see step_body): near / far by parts, 64/8
    // heads, 100,000 tokens: 16 0.99, 32 0.98, 43 1.04, 64 1.10, 128 1.17; 28/4 heads, 400,000: 32 1.02, 85 1.12, 128 1.24.
    out.near = lean && dec_blocks > 0 && max_dec_blocks * out.static_runs <= 32 * (int64_t)out.dec_blocks;
    if (tiles > 0) {
        const size_t reserve = pf_first ? (size_t)(geo.num_cus / geo.Hkv + num_seqs + 1) * slot_bytes(geo) + 256 : 0;
        const PrefillFacts facts = {tiles, tile_steps, max_tile_steps, n_order, st, out.pf_waves, max_cols, std::max<int64_t>(geo.Hkv, (dec_seqs * geo.Hkv + 1) / 2), reserve, dec_blocks, kv_blocks, pf_pairs};
        plan_prefill_parts(geo, facts, store.pf + (2 * (size_t)out.num_pf + 1), out);
    }
    if (pf_first) {
        // (where the arrays do not fit the kernel arguments together the parts run as two kernels, which have all units each:
        // ooco_attn_mixed_static, 16/1 heads, 159 decodes of 60..124 tokens beside 245 chunks of 2..4 rows on 1000..2500,
        // decode runs for the units that are left -> for all: 101 -> 47 us; four-wave prefill workgroups 56)
        if ((size_t)num_seqs + 1 + out.pf_size <= (size_t)kInlineSeqs + 1)
            out.pf_units = (int32_t)(out.pf_table ? (int64_t)out.pf_table * geo.Hkv : tiles * geo.Hkv * out.pf_split);
        plan_decode();
    }
    return OOCO_OK;
}

// Whether the plan's arrays ride in the kernel arguments (the mixed kernel, dec_cus > 0, takes both at once; the two separate
// kernels one each); else the kernels read them from device memory.
bool plan_in_args(const HostPlan &pl)
{
    const size_t n_cum = (size_t)pl.num_seqs + 1, room = (size_t)kInlineSeqs + 1;
    return pl.dec_cus > 0 ? n_cum + pl.pf_size <= room : n_cum <= room && pl.pf_size <= room;
}

// Whether the step kernel can run the plan: both kinds of work, both arrays together in the kernel arguments, no
// dynamic tail and no XCD weights, and decode waves that it is instantiated for (nbi: KV blocks per softmax step).
bool step_fits(const HostPlan &pl, int hd, bool coop, int nbi)
{
    return pl.n_tiles > 0 && pl.static_runs > 0 && pl.tail_runs == 0 && pl.cw[kXcds - 1] == 0 && pl.dec_cus == 0 &&
           (size_t)pl.num_seqs + 1 + pl.pf_size <= (size_t)kInlineSeqs + 1 &&
           (pl.pf_groups > 1 ? coop && pl.coop_waves == 8
            : pl.lean        ? hd == 128 && pl.pf_waves == 8
                             : pl.pf_waves == 4 && (coop || nbi == 2 || (nbi == 1 && hd == 128)));
}

// The plan's arrays in the kernel arguments, for kernels that take the decode part, the prefill part or both: the decode
// array, then the prefill array, or, where the plan has a tile list, only that, from the other end (AttnParams::list_row).
// The caller has seen to it that the arrays fit.
void fill_plan(const HostPlan &pl, bool dec, bool pf, KernArgs &ka)
{
    AttnParams &p = ka.p;
    const int64_t n_cum = dec ? (int64_t)pl.num_seqs + 1 : 0;
    p.list_row = 0;
    p.rows2d = 0;
    p.list_by_seq = pf && pl.pf_table > 0;
    if (dec) memcpy(ka.cum, pl.dcum, (size_t)n_cum * sizeof(int32_t));
    if (!pf) return;
    if (!pl.pf_table) {
        memcpy(ka.cum + n_cum, pl.pf, pl.pf_size * sizeof(int32_t));
        return;
    }
    if (dec && p.coop && n_cum + pl.static_runs + pl.pf_table <= kInlineSeqs + 1) p.rows2d = 1, p.list_row = (int16_t)pl.static_runs;
    const int32_t *const tab = pl.pf + 2 * pl.num_pf + 1, *const seqs = pl.pf + pl.num_pf + 1;
    int32_t *const top = ka.cum + kInlineSeqs - p.list_row;
    for (int32_t e = 0; e < pl.pf_table; ++e) top[-e] = list_entry(seqs[entry_chunk(tab[e])], entry_tile(tab[e]), entry_part(tab[e]), entry_parts(tab[e]));
}

// Pieces of the decode line as the kernel walks them (host mirror of the device logic).
struct Piece {
    int32_t seq, blk_begin, blk_end, slot, run;
};
std::vector<Piece> enumerate_pieces(const HostPlan &pl)
{
    std::vector<Piece> v;
    const RunLayout L = {pl.dec_blocks, pl.static_blocks, pl.static_runs, pl.tail_runs, pl.cw};
    for (int32_t k = 0; k < pl.static_runs + pl.tail_runs; ++k) {
        int32_t lo, hi;
        if (pl.coop == kCoopBySequence)
            lo = pl.dcum[(size_t)k], hi = pl.dcum[(size_t)k + 1];
        else
            run_bounds(L, k, lo, hi);
        if (lo >= hi) continue;
        int seq = 0;
        while (pl.dcum[(size_t)seq + 1] <= lo) ++seq;
        int64_t pos = lo;
        while (pos < hi) {
            while (pl.dcum[(size_t)seq + 1] <= pos) ++seq;
            const int64_t cs = pl.dcum[(size_t)seq], ce = pl.dcum[(size_t)seq + 1];
            const int64_t stop = std::min<int64_t>(hi, ce);
            const int64_t first = cs + pl.piece_pad, begin = std::max(pos, first);   // the blocks start at `first`
            if (begin < stop) {
                const bool whole = begin == first && stop == ce;
                v.push_back(Piece{seq, (int32_t)(begin - first), (int32_t)(stop - first), whole ? -1 : (int32_t)(k + seq),
                                  (int32_t)k});
            }
            pos = stop;
            ++seq;
        }
    }
    return v;
}
}  // namespace

struct ooco_ctx {
    int Hq = 0, Hkv = 0, g = 0, hd = 0, BS = 0;
    int64_t num_blocks = 0;
    int max_blocks_per_seq = 0;
    float scale = 0.f;
    int device = 0;
    int num_cus = 256;

    void *ws = nullptr;
    size_t ws_bytes = 0;
    bool own_ws = false;

    // streams that calls have put work on which uses the context's memory (workspace, counters, plan, sort buffer):
    // what ooco_ctx_destroy and ooco_trace_read wait for.  More than kMaxStreams different ones: the whole device.
    static constexpr int kMaxStreams = 4;
    hipStream_t used_streams[kMaxStreams] = {};
    int n_used_streams = 0;
    bool many_streams = false;
    hipStream_t last_stream = nullptr;
    void note_stream(hipStream_t st)
    {
        last_stream = st;
        for (int i = 0; i < n_used_streams; ++i)
            if (used_streams[i] == st) return;
        if (n_used_streams < kMaxStreams)
            used_streams[n_used_streams++] = st;
        else
            many_streams = true;
    }
    // Waits for everything the context has enqueued (its side stream is joined into the caller's stream by every call).
    hipError_t wait_for_own_work()
    {
        if (many_streams) return hipDeviceSynchronize();
        hipError_t first = hipSuccess;
        for (int i = 0; i < n_used_streams; ++i) {
            const hipError_t e = hipStreamSynchronize(used_streams[i]);
            if (first == hipSuccess) first = e;
        }
        return first;
    }

    int32_t *plan_h = nullptr;   // pinned host staging for batches beyond kInlineSeqs sequences
    int32_t *plan_d = nullptr;   // device copy of the two cumulative arrays
    int32_t *counters = nullptr; // arrival counters [kCounterInts], zero between calls
    hipEvent_t upload_done = nullptr;
    bool upload_pending = false;

    // current plan (its arrays live in plan_store)
    std::vector<int32_t> plan_store;
    HostPlan plan;
    bool plan_valid = false;
    bool plan_dirty = false;
    bool plan_one_shot = false;   // planned inside ooco_attn_mixed from device lengths
    bool plan_made = false;       // ctx->plan holds the numbers of the last plan made (current or used up)
    int64_t opt_plan_persistent = 0;   // an explicit plan serves every following call of the same shape

    // options
    int64_t opt_segments = 0;
    int64_t opt_tail_pct = 0;
    int64_t opt_tail_blocks = 8;
    uint32_t queue_base = 0;       // ticket value the next launch's tail runs start at
    int64_t opt_nbi = 0;
    int64_t opt_trace = 0;
    int64_t opt_rotate = 1;
    int64_t opt_pf_split = 0;
    int64_t opt_pf_table = 1;       // few prefill tiles: dispatched by decreasing number of steps across chunks
    int opt_copy_variant = 0;       // block copy: 10 x vectors per thread + non-temporal flag, 0 = default
    int64_t opt_decode_first = 1;   // mixed batches: enqueue the decode kernel before the prefill kernel
    int64_t opt_piece_pad = -1;   // < 0: automatic (3 tiles of head_dim 128, 12 in cooperative plans)
    int32_t *pf_counters = nullptr;   // [kPrefillSplitUnits] arrival counters of split prefill tiles, zero between calls
    uint16_t xcd_cw[kXcds] = {};   // option "xcd_weights"
    int64_t opt_overlap = 1;
    int64_t opt_copy_sort = 1;      // block copy: order the pairs by destination region on the device (0 never, 1 where the copy is large enough, 2 always)
    void *sort_buf = nullptr;       // [2 * sort_cap int64 (sorted dst, sorted src)] + temporary storage of the sort
    int64_t sort_cap = 0;           // pairs the buffer holds
    size_t sort_temp_bytes = 0;
    int64_t opt_append_parts = 0;   // KV append: workgroups per (sequence, block) pair, 0 = automatic
    int64_t opt_lean = 1;           // mixed batches: the register-lean kernels (0 never, 1 automatic, 2 always)
    int64_t opt_pf_waves = 0;       // waves per prefill workgroup: 0 = automatic, 4, 8
    int64_t opt_pf_groups = 0;      // key groups per prefill workgroup: 0 = automatic, 1, 4
    int64_t opt_merge_looks = 12;   // shared merge of a split tile: looks at the counter before an early part leaves
    int64_t opt_fused = 0;          // mixed batches in one launch (mixed kernel) instead of two kernels on two streams
    int64_t opt_coop = 1;           // cooperative decode workgroups (0 never, 1 by rule, 2 always)
    int64_t opt_step = 1;           // mixed batches in one launch of the step kernel (0 never, 1 by rule, 2 whenever it takes the plan)
    int64_t opt_dec_cus = 0;        // mixed kernel: decoding compute units per XCD, 0 = automatic
    hipStream_t side_stream = nullptr;   // default priority; carries the prefill kernel of mixed batches
    hipEvent_t fork_ev = nullptr, join_ev = nullptr;
    uint64_t *trace_d = nullptr;   // [kTraceWaves][4] decode-wave time stamps
    int64_t trace_waves = 0;       // waves of the last traced call
    int64_t opt_profile = 0;

    // per-kernel timing (option "profile"): kProfEvents events per call (decode start/end, prefill start/end,
    // call start/end), each pair recorded on the stream its kernel runs on
    std::vector<hipEvent_t> prof_ev;
    int64_t prof_calls = 0;

    KernArgs kargs;                      // staging of the kernel arguments of the current call
    std::vector<int32_t> h_len_scratch;   // for the plan-less path
    mutable char err[512] = "";
};

namespace {

// KV blocks per softmax step of the decode waves of the current plan.
int decode_nbi(const ooco_ctx *ctx)
{
    return ctx->opt_nbi ? (int)ctx->opt_nbi : ctx->plan.nbi ? ctx->plan.nbi : (ctx->hd == 64 ? 2 : 1);
}
// Whether its runs are worked on by cooperative workgroups (a number of blocks per step forced after the plan takes
// single waves on the same runs where it can).
int decode_coop(const ooco_ctx *ctx) { return ctx->plan.coop == kCoopBySequence || ctx->opt_nbi == 0 ? ctx->plan.coop : 0; }
// Whether the current plan runs in one launch of the step kernel ("overlap" 0 and 2 ask for two kernels).
bool runs_as_step(const ooco_ctx *ctx)
{
    return ctx->opt_step && ctx->opt_overlap == 1 && (ctx->opt_step >= 2 || !ctx->plan.two_streams) && step_fits(ctx->plan, ctx->hd, decode_coop(ctx) != 0, decode_nbi(ctx));
}

ooco_status fail(const ooco_ctx *ctx, ooco_status code, const char *fmt, ...)
{
    char *dst = ctx ? ctx->err : g_create_error;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(dst, 512, fmt, ap);
    va_end(ap);
    return code;
}


}  // namespace

extern "C" {

ooco_status ooco_ctx_create(ooco_ctx **out, int num_q_heads, int num_kv_heads, int head_dim, int block_size,
                            int64_t num_blocks, int max_blocks_per_seq, float softmax_scale, void *workspace,
                            size_t workspace_bytes)
{
    if (!out) return fail(nullptr, OOCO_EINVAL, "ooco_ctx_create: out is NULL");
    *out = nullptr;
    if (num_q_heads <= 0 || num_kv_heads <= 0 || num_q_heads % num_kv_heads != 0)
        return fail(nullptr, OOCO_ESHAPE, "ooco_ctx_create: num_q_heads=%d must be a positive multiple of num_kv_heads=%d",
                    num_q_heads, num_kv_heads);
    if (num_q_heads / num_kv_heads > 16)
        return fail(nullptr, OOCO_ESHAPE, "ooco_ctx_create: GQA group size %d > 16 is not supported",
                    num_q_heads / num_kv_heads);
    if (head_dim != 64 && head_dim != 128)
        return fail(nullptr, OOCO_ESHAPE, "ooco_ctx_create: head_dim=%d (supported: 64, 128)", head_dim);
    if (block_size != kBlockSize)
        return fail(nullptr, OOCO_ESHAPE, "ooco_ctx_create: block_size=%d (supported: %d)", block_size, kBlockSize);
    if (num_blocks <= 0 || max_blocks_per_seq <= 0)
        return fail(nullptr, OOCO_EINVAL, "ooco_ctx_create: num_blocks and max_blocks_per_seq must be positive");
    if (workspace && workspace_bytes == 0)
        return fail(nullptr, OOCO_EINVAL, "ooco_ctx_create: caller workspace given with workspace_bytes == 0");
    if (workspace && (reinterpret_cast<uintptr_t>(workspace) & 255u))
        return fail(nullptr, OOCO_EINVAL, "ooco_ctx_create: workspace must be 256-byte aligned");

    ooco_ctx *c = new (std::nothrow) ooco_ctx();
    if (!c) return fail(nullptr, OOCO_ENOMEM, "ooco_ctx_create: out of host memory");
    c->Hq = num_q_heads;
    c->Hkv = num_kv_heads;
    c->g = num_q_heads / num_kv_heads;
    c->hd = head_dim;
    c->BS = block_size;
    c->num_blocks = num_blocks;
    c->max_blocks_per_seq = max_blocks_per_seq;
    c->scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt((float)head_dim);

    hipError_t e = hipGetDevice(&c->device);
    if (e == hipSuccess) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) == hipSuccess && cus > 0)
            c->num_cus = cus;
    }
    if (e == hipSuccess) {
        if (workspace) {
            c->ws = workspace;
            c->ws_bytes = workspace_bytes;
        } else {
            c->ws_bytes = workspace_bytes ? workspace_bytes : kDefaultWorkspace;
            e = hipMalloc(&c->ws, c->ws_bytes);
            c->own_ws = (e == hipSuccess);
        }
    }
    if (e == hipSuccess) e = hipHostMalloc((void **)&c->plan_h, kPlanInts * sizeof(int32_t), hipHostMallocDefault);
    if (e == hipSuccess) e = hipMalloc((void **)&c->plan_d, kPlanInts * sizeof(int32_t));
    if (e == hipSuccess) e = hipMalloc((void **)&c->counters, kCounterInts * sizeof(int32_t));
    if (e == hipSuccess) e = hipMemset(c->counters, 0, kCounterInts * sizeof(int32_t));
    if (e == hipSuccess) e = hipMalloc((void **)&c->pf_counters, kPrefillSplitUnits * sizeof(int32_t));
    if (e == hipSuccess) e = hipMemset(c->pf_counters, 0, kPrefillSplitUnits * sizeof(int32_t));
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->upload_done, hipEventDisableTiming);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&c->side_stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->fork_ev, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->join_ev, hipEventDisableTiming);
    if (e != hipSuccess) {
        fail(nullptr, e == hipErrorOutOfMemory ? OOCO_ENOMEM : OOCO_EHIP, "ooco_ctx_create: %s", hipGetErrorString(e));
        ooco_status st = e == hipErrorOutOfMemory ? OOCO_ENOMEM : OOCO_EHIP;
        (void)hipGetLastError();
        if (c->upload_done) (void)hipEventDestroy(c->upload_done);
        if (c->fork_ev) (void)hipEventDestroy(c->fork_ev);
        if (c->join_ev) (void)hipEventDestroy(c->join_ev);
        if (c->side_stream) (void)hipStreamDestroy(c->side_stream);
        if (c->counters) (void)hipFree(c->counters);
        if (c->pf_counters) (void)hipFree(c->pf_counters);
        if (c->plan_d) (void)hipFree(c->plan_d);
        if (c->plan_h) (void)hipHostFree(c->plan_h);
        if (c->own_ws && c->ws) (void)hipFree(c->ws);
        delete c;
        return st;
    }
    *out = c;
    return OOCO_OK;
}

ooco_status ooco_ctx_destroy(ooco_ctx *ctx)
{
    if (!ctx) return OOCO_OK;
    if (ctx->upload_pending) (void)hipEventSynchronize(ctx->upload_done);
    (void)ctx->wait_for_own_work();
    if (ctx->side_stream) (void)hipStreamSynchronize(ctx->side_stream);
    if (ctx->upload_done) (void)hipEventDestroy(ctx->upload_done);
    if (ctx->fork_ev) (void)hipEventDestroy(ctx->fork_ev);
    if (ctx->join_ev) (void)hipEventDestroy(ctx->join_ev);
    if (ctx->side_stream) (void)hipStreamDestroy(ctx->side_stream);
    for (hipEvent_t x : ctx->prof_ev)
        if (x) (void)hipEventDestroy(x);
    if (ctx->trace_d) (void)hipFree(ctx->trace_d);
    if (ctx->sort_buf) (void)hipFree(ctx->sort_buf);
    if (ctx->counters) (void)hipFree(ctx->counters);
    if (ctx->pf_counters) (void)hipFree(ctx->pf_counters);
    if (ctx->plan_d) (void)hipFree(ctx->plan_d);
    if (ctx->plan_h) (void)hipHostFree(ctx->plan_h);
    if (ctx->own_ws && ctx->ws) (void)hipFree(ctx->ws);
    delete ctx;
    return OOCO_OK;
}

ooco_status ooco_trace_read(ooco_ctx *ctx, uint64_t *stamps, int64_t cap_waves, int64_t *waves)
{
    if (!ctx) return OOCO_EINVAL;
    if (!ctx->trace_d) return fail(ctx, OOCO_EINVAL, "ooco_trace_read: option \"trace\" was never enabled");
    hipError_t e = ctx->wait_for_own_work();
    const int64_t n = std::min<int64_t>(cap_waves, ctx->trace_waves);
    if (e == hipSuccess && stamps && n > 0)
        e = hipMemcpy(stamps, ctx->trace_d, (size_t)n * 4 * sizeof(uint64_t), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail(ctx, OOCO_EHIP, "ooco_trace_read: %s", hipGetErrorString(e));
    if (waves) *waves = ctx->trace_waves;
    return OOCO_OK;
}

ooco_status ooco_profile_read_calls(ooco_ctx *ctx, double *per_call_ms, int64_t cap, double *ms_sum, int64_t *calls)
{
    if (!ctx) return OOCO_EINVAL;
    if (cap < 0 || (cap > 0 && !per_call_ms)) return fail(ctx, OOCO_EINVAL, "ooco_profile_read_calls: bad per-call buffer");
    double sum[3] = {0.0, 0.0, 0.0};
    for (int64_t c = 0; c < ctx->prof_calls; ++c) {
        hipEvent_t *ev = ctx->prof_ev.data() + kProfEvents * c;
        // wait for the call's last record on either stream
        hipError_t e = hipEventSynchronize(ev[5]);
        if (e == hipSuccess) e = hipEventSynchronize(ev[3]);
        if (e == hipSuccess) e = hipEventSynchronize(ev[1]);
        // (prefill start, prefill end), (decode start, decode end), (call start, call end)
        static const int pairs[3][2] = {{2, 3}, {0, 1}, {4, 5}};
        for (int k = 0; k < 3 && e == hipSuccess; ++k) {
            float ms = 0.f;
            e = hipEventElapsedTime(&ms, ev[pairs[k][0]], ev[pairs[k][1]]);
            sum[k] += ms;
            if (c < cap) per_call_ms[3 * c + k] = ms;
        }
        if (e != hipSuccess) return fail(ctx, OOCO_EHIP, "ooco_profile_read: %s", hipGetErrorString(e));
    }
    if (ms_sum) ms_sum[0] = sum[0], ms_sum[1] = sum[1], ms_sum[2] = sum[2];
    if (calls) *calls = ctx->prof_calls;
    ctx->prof_calls = 0;
    return OOCO_OK;
}

ooco_status ooco_profile_read(ooco_ctx *ctx, double *ms_sum, int64_t *calls)
{
    return ooco_profile_read_calls(ctx, nullptr, 0, ms_sum, calls);
}

const char *ooco_last_error(const ooco_ctx *ctx) { return ctx ? ctx->err : g_create_error; }

ooco_status ooco_set_option(ooco_ctx *ctx, const char *name, int64_t value)
{
    if (!ctx) return OOCO_EINVAL;
    if (!name) return fail(ctx, OOCO_EINVAL, "ooco_set_option: name is NULL");
    if (value < 0) return fail(ctx, OOCO_EINVAL, "ooco_set_option: %s must be >= 0", name);
    if (!strcmp(name, "decode_segments"))
        ctx->opt_segments = value;
    else if (!strcmp(name, "decode_tail_pct"))
        ctx->opt_tail_pct = value;
    else if (!strcmp(name, "decode_tail_blocks"))
        ctx->opt_tail_blocks = value;
    else if (!strcmp(name, "prefill_split"))
        ctx->opt_pf_split = value;
    else if (!strcmp(name, "prefill_sorted"))
        ctx->opt_pf_table = value;
    else if (!strcmp(name, "decode_first"))
        ctx->opt_decode_first = value;
    else if (!strcmp(name, "prefill_waves")) {
        if (value != 0 && value != 4 && value != 8)
            return fail(ctx, OOCO_EINVAL, "ooco_set_option: prefill_waves must be 0 (automatic), 4 or 8");
        ctx->opt_pf_waves = value;
    }
    else if (!strcmp(name, "prefill_groups")) {
        if (value != 0 && value != 1 && value != kKeyGroups)
            return fail(ctx, OOCO_EINVAL, "ooco_set_option: prefill_groups must be 0 (automatic), 1 or 4");
        ctx->opt_pf_groups = value;
    }
    else if (!strcmp(name, "mixed_lean"))
        ctx->opt_lean = value;
    else if (!strcmp(name, "decode_coop"))
        ctx->opt_coop = value;
    else if (!strcmp(name, "mixed_fused"))
        ctx->opt_fused = value;
    else if (!strcmp(name, "mixed_dec_cus"))
        ctx->opt_dec_cus = value;
    else if (!strcmp(name, "decode_piece_pad")) {
        if (value > 64) return fail(ctx, OOCO_EINVAL, "ooco_set_option: decode_piece_pad must be 0..64");
        ctx->opt_piece_pad = value;
    }
    else if (!strcmp(name, "trace")) {
        if (value && !ctx->trace_d) {
            hipError_t e = hipMalloc((void **)&ctx->trace_d, kTraceWaves * 4 * sizeof(uint64_t));
            if (e != hipSuccess) return fail(ctx, OOCO_ENOMEM, "ooco_set_option: trace buffer: %s", hipGetErrorString(e));
        }
        ctx->opt_trace = value;
        return OOCO_OK;
    } else if (!strcmp(name, "copy_variant")) {
        static const int64_t known[] = {0, 10, 11, 20, 21, 40, 41, 80, 81};
        if (std::find(std::begin(known), std::end(known), value) == std::end(known))
            return fail(ctx, OOCO_EINVAL, "ooco_set_option: copy_variant must be one of 0, 10, 11, 20, 21, 40, 41, 80, 81");
        ctx->opt_copy_variant = (int)value;
        return OOCO_OK;
    } else if (!strcmp(name, "copy_sort")) {
        ctx->opt_copy_sort = value;
        return OOCO_OK;
    } else if (!strcmp(name, "append_parts")) {
        ctx->opt_append_parts = value;
        return OOCO_OK;
    } else if (!strcmp(name, "plan_persistent")) {
        ctx->opt_plan_persistent = value;
        return OOCO_OK;
    } else if (!strcmp(name, "overlap")) {
        ctx->opt_overlap = value;
        return OOCO_OK;
    } else if (!strcmp(name, "prefill_merge_looks")) {
        if (value > 100) return fail(ctx, OOCO_EINVAL, "ooco_set_option: prefill_merge_looks must be 0..100");
        ctx->opt_merge_looks = value;
        return OOCO_OK;
    } else if (!strcmp(name, "mixed_step")) {
        ctx->opt_step = value;
        return OOCO_OK;
    } else if (!strcmp(name, "rotate_heads")) {
        ctx->opt_rotate = value;
        return OOCO_OK;
    } else if (!strcmp(name, "xcd_weights")) {
        // eight relative weights, one byte each, XCD 0 in the lowest byte; 0 = equal runs
        int32_t w[kXcds];
        for (int k = 0; k < kXcds; ++k) w[k] = (int32_t)(((uint64_t)value >> (8 * k)) & 0xFFu);
        if (value == 0)
            for (int k = 0; k < kXcds; ++k) ctx->xcd_cw[k] = 0;
        else if (!xcd_weights_to_cw(w, ctx->xcd_cw)) {
            for (int k = 0; k < kXcds; ++k) ctx->xcd_cw[k] = 0;
            return fail(ctx, OOCO_EINVAL, "ooco_set_option: xcd_weights needs eight bytes in 1..255 that differ by at most 4x");
        }
    } else if (!strcmp(name, "decode_nbi")) {
        ctx->opt_nbi = value;
        return OOCO_OK;
    } else if (!strcmp(name, "profile")) {
        ctx->opt_profile = value;
        ctx->prof_calls = 0;
        return OOCO_OK;   // does not invalidate the plan
    }
    else
        return fail(ctx, OOCO_EINVAL, "ooco_set_option: unknown option '%s'", name);
    ctx->plan_valid = false;
    return OOCO_OK;
}

ooco_status ooco_plan(ooco_ctx *ctx, int num_seqs, const int32_t *h_seq_lens, const int32_t *h_query_start_loc,
                      const int32_t *h_ctx_lens)
{
    if (!ctx) return OOCO_EINVAL;
    ctx->plan_valid = false;
    PlanGeometry geo;
    geo.Hq = ctx->Hq;
    geo.Hkv = ctx->Hkv;
    geo.hd = ctx->hd;
    geo.BS = ctx->BS;
    geo.max_blocks_per_seq = ctx->max_blocks_per_seq;
    geo.num_cus = ctx->num_cus;
    geo.ws_bytes = ctx->ws_bytes;
    geo.segments_opt = ctx->opt_segments;
    geo.tail_pct = ctx->opt_tail_pct;
    geo.tail_blocks = ctx->opt_tail_blocks;
    geo.pf_split_opt = ctx->opt_pf_split;
    geo.piece_pad = ctx->opt_piece_pad;
    geo.pf_waves_opt = ctx->opt_pf_waves;
    geo.pf_groups_opt = ctx->opt_pf_groups;
    geo.lean_opt = ctx->opt_lean;
    geo.coop_opt = ctx->opt_nbi ? 0 : ctx->opt_coop;   // (a forced number of blocks per step asks for single waves)
    geo.fused = ctx->opt_fused && ctx->opt_overlap;
    geo.dec_cus_opt = ctx->opt_dec_cus;
    geo.pf_table_opt = ctx->opt_pf_table;
    for (int k = 0; k < kXcds; ++k) geo.xcd_cw[k] = ctx->xcd_cw[k];
    const size_t cap = (size_t)std::max(num_seqs, 0);
    if (ctx->plan_store.size() < storage_ints(cap)) ctx->plan_store.resize(storage_ints(cap));
    ooco_status st = build_plan(geo, num_seqs, h_seq_lens, h_query_start_loc, h_ctx_lens,
                                carve_storage(ctx->plan_store.data(), cap), ctx->plan, ctx->err);
    if (st != OOCO_OK) return st;
    if ((size_t)num_seqs * ctx->Hkv > kCounterInts - kMixedStateInts || 3 * ((size_t)num_seqs + 1) + kListEntries > kPlanInts)
        return fail(ctx, OOCO_ENOMEM, "ooco_plan: %d sequences exceed the context's counter/plan buffers", num_seqs);
    ctx->plan_valid = true;
    ctx->plan_made = true;
    ctx->plan_dirty = true;
    ctx->plan_one_shot = false;
    return OOCO_OK;
}

ooco_status ooco_plan_dry_run(int num_q_heads, int num_kv_heads, int head_dim, int block_size, int max_blocks_per_seq,
                              int num_cus, size_t workspace_bytes, int64_t decode_segments, int64_t decode_tail_pct,
                              int64_t decode_tail_blocks, int num_seqs,
                              const int32_t *h_seq_lens, const int32_t *h_query_start_loc, const int32_t *h_ctx_lens,
                              int32_t *decode_pieces_out, int64_t decode_cap, int32_t *prefill_tiles_out,
                              int64_t prefill_cap, int64_t *counts, char *msg, size_t msg_cap,
                              const int32_t *xcd_weights, int64_t prefill_split, int64_t decode_piece_pad)
{
    char err[512] = "";
    ooco_status st = OOCO_OK;
    HostPlan pl;
    std::vector<int32_t> store;
    if (num_q_heads <= 0 || num_kv_heads <= 0 || num_q_heads % num_kv_heads || (head_dim != 64 && head_dim != 128) ||
        block_size != kBlockSize || max_blocks_per_seq <= 0 || num_cus <= 0 || decode_segments < 0 ||
        decode_tail_pct < 0 || decode_tail_blocks < 0 || prefill_split < 0 || decode_piece_pad > 64) {
        snprintf(err, sizeof err, "ooco_plan_dry_run: bad geometry");
        st = OOCO_ESHAPE;
    } else {
        PlanGeometry geo;
        geo.Hq = num_q_heads;
        geo.Hkv = num_kv_heads;
        geo.hd = head_dim;
        geo.BS = block_size;
        geo.max_blocks_per_seq = max_blocks_per_seq;
        geo.num_cus = num_cus;
        geo.ws_bytes = workspace_bytes;
        geo.segments_opt = decode_segments;
        geo.tail_pct = decode_tail_pct;
        geo.tail_blocks = decode_tail_blocks;
        geo.pf_groups_opt = prefill_split >> 32;
        geo.pf_split_opt = prefill_split & 0xFFFFFFFF;
        if (geo.pf_groups_opt != 0 && geo.pf_groups_opt != 1 && geo.pf_groups_opt != kKeyGroups) {
            snprintf(err, sizeof err, "ooco_plan_dry_run: prefill groups (above bit 32 of prefill_split) must be 0 (automatic), 1 or 4");
            st = OOCO_EINVAL;
        }
        geo.lean_opt = 1;   // (the default of a context)
        geo.piece_pad = decode_piece_pad;
        if (xcd_weights && !xcd_weights_to_cw(xcd_weights, geo.xcd_cw)) {
            snprintf(err, sizeof err, "ooco_plan_dry_run: xcd_weights needs eight values in 1..255 that differ by at most 4x");
            st = OOCO_EINVAL;
        }
        if (st == OOCO_OK) {
            const size_t cap = (size_t)std::max(num_seqs, 0);
            store.resize(storage_ints(cap));
            st = build_plan(geo, num_seqs, h_seq_lens, h_query_start_loc, h_ctx_lens, carve_storage(store.data(), cap), pl, err);
        }
    }
    if (msg && msg_cap) snprintf(msg, msg_cap, "%s", err);
    if (st != OOCO_OK) return st;
    const std::vector<Piece> pieces = enumerate_pieces(pl);
    if (counts) {
        counts[0] = (int64_t)pieces.size();
        counts[1] = pl.n_tiles;
        counts[2] = pl.static_runs;
        counts[3] = pl.slots;
        counts[4] = pl.tail_runs;
        counts[5] = pl.pf_split;
    }
    if (decode_pieces_out)
        for (int64_t i = 0; i < std::min<int64_t>(decode_cap, (int64_t)pieces.size()); ++i) {
            const Piece &d = pieces[(size_t)i];
            int32_t *o = decode_pieces_out + 5 * i;
            o[0] = d.seq, o[1] = d.blk_begin, o[2] = d.blk_end, o[3] = d.slot, o[4] = d.run;
        }
    if (prefill_tiles_out) {
        // in dispatch order, derived from the plan's arrays the way the prefill kernel derives them
        const int tile_rows = prefill_tile_rows(num_q_heads / num_kv_heads, pl.pf_col_waves());
        const int32_t *const pf = pl.pf;
        const int P = pl.num_pf;
        // (with the tile list a tile is listed where its first part is dispatched)
        const int64_t n_list = pl.pf_table ? pl.pf_table : pl.n_tiles;
        int64_t idx = 0;
        for (int64_t pos = 0; pos < n_list && idx < prefill_cap; ++pos) {
            int k, t, parts;
            if (pl.pf_table) {
                const int32_t e = pf[2 * P + 1 + pos];
                if (entry_part(e) != 0) continue;
                k = entry_chunk(e);
                t = entry_tile(e);
                parts = entry_parts(e);
            } else {
                k = (int)(std::upper_bound(pf, pf + P + 1, (int32_t)pos) - pf) - 1;
                t = (pf[k + 1] - 1) - (int)pos;
                parts = pl.pf_split;
            }
            const int i = pf[P + 1 + k];
            const int q0 = h_query_start_loc[i], ql = h_query_start_loc[i + 1] - q0, t0 = t * tile_rows;
            int32_t *o = prefill_tiles_out + 5 * idx++;
            o[0] = i, o[1] = q0 + t0, o[2] = std::min(tile_rows, ql - t0), o[3] = h_ctx_lens[i] + t0;
            o[4] = (int32_t)std::min<int64_t>(parts, ((int64_t)o[3] + o[2] + pl.pf_step_keys() - 1) / pl.pf_step_keys());
        }
    }
    return OOCO_OK;
}

ooco_status ooco_plan_info(const ooco_ctx *ctx, int64_t *decode_waves, int64_t *prefill_tiles, int64_t *decode_blocks,
                           int64_t *workspace_used, int64_t *prefill_parts)
{
    if (!ctx) return OOCO_EINVAL;
    if (!ctx->plan_made) return fail(ctx, OOCO_EINVAL, "ooco_plan_info: no plan has been made");
    if (decode_waves) *decode_waves = ctx->plan.static_runs;
    if (prefill_tiles) *prefill_tiles = ctx->plan.n_tiles;
    if (decode_blocks) *decode_blocks = ctx->plan.kv_blocks;
    if (workspace_used) {
        size_t bytes = (size_t)ctx->plan.slots * (size_t)ctx->Hq * (ctx->hd + 2) * sizeof(float);
        if (ctx->plan.pf_split > 1)
            bytes = (bytes + 255) / 256 * 256 + (size_t)ctx->plan.pf_slots * ctx->Hkv * (size_t)(32 * ctx->plan.pf_col_waves()) *
                                                    (ctx->hd + 2) * sizeof(float);
        *workspace_used = (int64_t)bytes;
    }
    if (prefill_parts) *prefill_parts = ctx->plan.n_tiles > 0 ? ctx->plan.pf_split : 1;
    return OOCO_OK;
}

ooco_status ooco_plan_kernels(const ooco_ctx *ctx, char *names, size_t cap)
{
    if (!ctx) return OOCO_EINVAL;
    if (!ctx->plan_made) return fail(ctx, OOCO_EINVAL, "ooco_plan_kernels: no plan has been made");
    if (!names || cap == 0) return fail(ctx, OOCO_EINVAL, "ooco_plan_kernels: no buffer");
    // (by the conditions of launch_decode, launch_prefill and launch_step)
    const HostPlan &pl = ctx->plan;
    const bool dec = pl.static_runs > 0, pf = pl.n_tiles > 0;
    const bool coop = decode_coop(ctx) != 0, in_args = plan_in_args(pl), lean = pl.lean && ctx->hd == 128;
    const bool general = !in_args || (!coop && (pl.tail_runs > 0 || pl.cw[kXcds - 1] != 0));
    const int wanted = decode_nbi(ctx), blocks = coop ? 256 / ctx->hd : wanted == 2 || wanted == 4 ? wanted : 1;   // (in flight; of a step)
    char d[64] = "", f[64] = "";
    if (runs_as_step(ctx))
        snprintf(d, sizeof d, pl.pf_groups > 1 ? "step_kernel_groups<%d, %d>" : pl.lean ? "step_kernel_lean<%d>" : coop ? "step_kernel<%d, %d, true>" : "step_kernel<%d, %d, false>", ctx->hd,
                 blocks);
    else if (dec && pf && pl.dec_cus > 0)
        snprintf(d, sizeof d, "mixed_kernel<%d>", ctx->hd);
    else {
        if (dec && coop)
            snprintf(d, sizeof d, "decode_coop_kernel%s<%d, %d>", pl.coop_waves == 8 ? "_groups" : general ? "_general" : "", ctx->hd, blocks);
        else if (dec && lean)
            snprintf(d, sizeof d, "decode_kernel_lean%s<%d>", general ? "_general" : "", ctx->hd);
        else if (dec)
            snprintf(d, sizeof d, "decode_kernel%s<%d, %d>", general ? "_general" : "", ctx->hd, blocks);
        if (pf && (pl.pf_groups > 1 || (lean && pl.pf_waves == 8)))
            snprintf(f, sizeof f, pl.pf_groups > 1 ? "prefill_kernel_groups<%d>" : "prefill_kernel_lean<%d>", ctx->hd);
        else if (pf)
            snprintf(f, sizeof f, "prefill_kernel<%d, %d>", ctx->hd, pl.pf_waves);
    }
    snprintf(names, cap, "%s%s%s", d, d[0] && f[0] ? ";" : "", f);
    return OOCO_OK;
}

ooco_status ooco_attn_mixed(ooco_ctx *ctx, const void *q, const void *k_cache, const void *v_cache,
                            const int32_t *block_tables, const int32_t *seq_lens, const int32_t *query_start_loc,
                            const int32_t *ctx_lens, void *out, int num_seqs, int total_q_tokens, void *stream)
{
    if (!ctx) return OOCO_EINVAL;
    if (num_seqs < 0 || total_q_tokens < 0)
        return fail(ctx, OOCO_EINVAL, "ooco_attn_mixed: negative size (num_seqs=%d, total_q_tokens=%d)", num_seqs,
                    total_q_tokens);
    if (num_seqs == 0 || total_q_tokens == 0) return OOCO_OK;
    if (!q || !k_cache || !v_cache || !block_tables || !seq_lens || !query_start_loc || !ctx_lens || !out)
        return fail(ctx, OOCO_EINVAL, "ooco_attn_mixed: NULL pointer argument");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    ctx->note_stream(s);

    if (!ctx->plan_valid) {
        // No host plan for this batch: fetch the lengths and plan here (costs one stream sync).
        ctx->h_len_scratch.resize((size_t)3 * num_seqs + 1);
        int32_t *h_seq = ctx->h_len_scratch.data();
        int32_t *h_ctx = h_seq + num_seqs;
        int32_t *h_qsl = h_ctx + num_seqs;
        hipError_t e = hipMemcpyAsync(h_seq, seq_lens, sizeof(int32_t) * num_seqs, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipMemcpyAsync(h_ctx, ctx_lens, sizeof(int32_t) * num_seqs, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(h_qsl, query_start_loc, sizeof(int32_t) * (num_seqs + 1), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return fail(ctx, OOCO_EHIP, "ooco_attn_mixed: reading lengths: %s", hipGetErrorString(e));
        ooco_status st = ooco_plan(ctx, num_seqs, h_seq, h_qsl, h_ctx);
        if (st != OOCO_OK) return st;
        ctx->plan_one_shot = true;
    }
    const HostPlan &pl = ctx->plan;
    if (pl.num_seqs != num_seqs || pl.total_q != total_q_tokens) {
        if (ctx->plan_one_shot) {   // the plan made above from the device's lengths does not outlive this call
            ctx->plan_one_shot = false;
            ctx->plan_valid = false;
        }
        return fail(ctx, OOCO_ESHAPE, "ooco_attn_mixed: plan was made for %d sequences / %d query tokens, call has %d / %d",
                    pl.num_seqs, pl.total_q, num_seqs, total_q_tokens);
    }

    // The cumulative arrays ride in the kernel arguments; only very large batches need a copy.
    const size_t n_cum = (size_t)num_seqs + 1, n_pf = pl.pf_size;
    const bool inline_cum = plan_in_args(pl);
    if (!inline_cum && ctx->plan_dirty) {
        if (ctx->upload_pending) (void)hipEventSynchronize(ctx->upload_done);
        memcpy(ctx->plan_h, pl.dcum, n_cum * sizeof(int32_t));
        memcpy(ctx->plan_h + n_cum, pl.pf, n_pf * sizeof(int32_t));
        hipError_t e = hipMemcpyAsync(ctx->plan_d, ctx->plan_h, (n_cum + n_pf) * sizeof(int32_t), hipMemcpyHostToDevice, s);
        if (e == hipSuccess) e = hipEventRecord(ctx->upload_done, s);
        if (e != hipSuccess) return fail(ctx, OOCO_EHIP, "ooco_attn_mixed: plan upload: %s", hipGetErrorString(e));
        ctx->upload_pending = true;
    }
    ctx->plan_dirty = false;

    KernArgs &ka = ctx->kargs;
    AttnParams &p = ka.p;
    p.q = static_cast<const uint16_t *>(q);
    p.k_cache = static_cast<const uint16_t *>(k_cache);
    p.v_cache = static_cast<const uint16_t *>(v_cache);
    p.block_tables = block_tables;
    p.seq_lens = seq_lens;
    p.query_start_loc = query_start_loc;
    p.ctx_lens = ctx_lens;
    p.out = static_cast<uint16_t *>(out);
    p.part_acc = static_cast<float *>(ctx->ws);
    p.part_ml = p.part_acc + (size_t)pl.slots * ctx->Hq * ctx->hd;
    p.counters = ctx->counters;
    {
        const size_t dec_floats = ((size_t)pl.slots * ctx->Hq * (ctx->hd + 2) + 63) / 64 * 64;   // 256-byte aligned
        const size_t parts = (size_t)pl.pf_slots * ctx->Hkv;   // (what the planner checked against the workspace)
        p.pf_acc = static_cast<float *>(ctx->ws) + dec_floats;
        p.pf_ml = p.pf_acc + parts * (size_t)(32 * pl.pf_col_waves()) * ctx->hd;
        p.pf_counters = ctx->pf_counters;
        p.pf_split = (int16_t)pl.pf_split;
        p.pf_table = (int16_t)pl.pf_table;
        // (what the kernels will address, once more against what the context owns: a plan that does not fit is an error of
        // this library, reported instead of launched)
        const size_t pf_end = (dec_floats + parts * (size_t)(32 * pl.pf_col_waves()) * (ctx->hd + 2)) * sizeof(float);
        // (arrival counters: one per part-0 slot with the tile list, one per (tile, kv head) without it)
        const size_t pf_counters_used = pl.pf_table ? parts : (size_t)pl.n_tiles * ctx->Hkv;
        if ((pl.pf_split > 1 && (pf_end > ctx->ws_bytes || pf_counters_used > (size_t)kPrefillSplitUnits)) ||
            (size_t)pl.slots * ctx->Hq * (ctx->hd + 2) * sizeof(float) > ctx->ws_bytes)
            return fail(ctx, OOCO_EINVAL, "ooco_attn_mixed: internal error: the plan's partial results (%zu bytes) do not fit the workspace (%zu bytes)",
                        pf_end, ctx->ws_bytes);
    }
    // (the mixed kernel stamps once per workgroup, the decode kernel once per wave)
    // (a batch without decode work: once per prefill workgroup)
    const int64_t trace_rows = pl.dec_cus > 0 && pl.n_tiles > 0 ? 2 * (int64_t)ctx->num_cus
                               : pl.static_runs > 0           ? (int64_t)pl.static_runs * ctx->Hkv
                               : pl.pf_table                  ? (int64_t)pl.pf_table * ctx->Hkv
                                                              : (int64_t)pl.n_tiles * ctx->Hkv * pl.pf_split;
    const bool tracing = ctx->opt_trace && ctx->trace_d && (size_t)trace_rows <= kTraceWaves;
    p.trace = tracing ? ctx->trace_d : nullptr;
    if (tracing) ctx->trace_waves = trace_rows;
    p.Hq = ctx->Hq;
    p.Hkv = ctx->Hkv;
    p.g = ctx->g;
    p.g_magic = (uint16_t)(32768 / ctx->g + 1);
    p.hd = ctx->hd;
    p.max_blocks_per_seq = ctx->max_blocks_per_seq;
    p.scale_log2e = ctx->scale * 1.4426950408889634f;
    p.num_seqs = num_seqs;
    p.total_q = total_q_tokens;
    p.dec_blocks = pl.dec_blocks;
    p.piece_pad = pl.piece_pad;
    p.static_blocks = pl.static_blocks;
    p.static_runs = pl.static_runs;
    p.tail_runs = pl.tail_runs;
    p.queue = reinterpret_cast<uint32_t *>(ctx->counters + kCounterInts - 1);
    p.queue_base = ctx->queue_base;
    p.n_tiles = pl.n_tiles;
    p.num_pf = pl.num_pf;
    p.dec_cus = (int8_t)pl.dec_cus;
    p.pf_waves = (int8_t)pl.pf_waves;
    p.pf_groups = (int8_t)pl.pf_groups;
    p.nbi = (int8_t)std::min<int64_t>(ctx->opt_nbi ? ctx->opt_nbi : pl.nbi, 100);
    p.rotate_heads = (int8_t)(ctx->opt_rotate != 0);
    p.coop = (int8_t)decode_coop(ctx);
    p.coop_waves = (int8_t)pl.coop_waves;
    p.dec_near = (int8_t)pl.near;
    p.lean = (int8_t)pl.lean;
    for (int k = 0; k < kXcds; ++k) p.xcd_cw[k] = pl.cw[k];

    if (pl.tail_runs > 0) {
        // the ticket base of the dynamic tail is fixed when the call is enqueued: a replayed graph would hand out
        // tickets that lie beyond it and leave the tail runs undone
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
            return fail(ctx, OOCO_EINVAL, "ooco_attn_mixed: a plan with a dynamic tail (decode_tail_pct) cannot be captured into a graph");
    }
    hipEvent_t *ev = nullptr;
    hipError_t e = hipSuccess;
    if (ctx->opt_profile) {
        if (ctx->prof_calls >= kProfSlots)
            return fail(ctx, OOCO_EINVAL, "ooco_attn_mixed: more than %d profiled calls without ooco_profile_read",
                        kProfSlots);
        if (ctx->prof_ev.empty()) {
            ctx->prof_ev.assign((size_t)kProfEvents * kProfSlots, nullptr);
            for (auto &x : ctx->prof_ev)
                if (e == hipSuccess) e = hipEventCreate(&x);
            if (e != hipSuccess) return fail(ctx, OOCO_EHIP, "ooco_attn_mixed: %s", hipGetErrorString(e));
        }
        ev = ctx->prof_ev.data() + kProfEvents * ctx->prof_calls++;
    }
    // A mixed batch runs in one launch (the step kernel) where runs_as_step allows.  Else its two kernels run side by
    // side: the prefill kernel (matrix-core bound) goes to
    // the context's side stream, forked from and joined back into the caller's stream with events,
    // the decode kernel (HBM bound) stays on the caller's stream.  The decode kernel is enqueued first
    // (its three waves per compute unit take their places before the prefill workgroups fill the
    // register files; measured 1.5 % faster on a long-context mixed batch, no difference on a short one).
    // With per-kernel profiling on, the launch order and the streams stay exactly as they are without it (one launch
    // for both kinds of work counts as both): every kernel is bracketed by two events on the stream it runs on (ev[0..1] decode, ev[2..3] prefill)
    // and the whole call by two on the caller's stream (ev[4..5]), so the times are those of the kernels
    // as they run in the step.
    const bool mixed = pl.n_tiles > 0 && pl.static_runs > 0;
    // (option "mixed_fused": the persistent mixed kernel, whose compute units either decode or prefill -- the plan says how
    // many do which.  Both arrays of the plan travel together there, in the kernel arguments if they fit.)
    const bool fused = mixed && pl.dec_cus > 0;
    const bool step = runs_as_step(ctx);
    const bool overlap = mixed && !fused && !step && ctx->side_stream && (ctx->opt_overlap >= 2 || (ctx->opt_overlap == 1 && !pl.brief));
    hipStream_t ps = overlap ? ctx->side_stream : s;   // the stream of the prefill kernel
    // A split tile's merge is shared among its parts where all workgroups of the launch find a place at once (launch_step adds
    // its decode workgroups): two of four waves per compute unit.  Only with the tile list, whose counters lie a tile's parts
    // apart: without it those of 32 tiles share a line, and the waiting parts' looks delay the others (option "prefill_sorted" 0,
    // us, one merging part -> shared: 25 + 27 rows on 7000 tokens, 32/8 heads, 15 parts 31.4 -> 38.8; 32 + 40 on 6500, 64/8 heads,
    // six parts 34.6 -> 39.1).
    const int64_t pf_wgs = pl.pf_table ? (int64_t)pl.pf_table * ctx->Hkv : (int64_t)pl.n_tiles * ctx->Hkv * pl.pf_split;
    p.pf_share = pl.pf_table && pl.pf_split > 1 && pl.pf_waves == 4 && (step || !mixed) && pf_wgs <= 2 * (int64_t)ctx->num_cus ? (int8_t)(1 + ctx->opt_merge_looks) : (int8_t)0;
    auto mark = [&](int k, hipStream_t st) {
        if (ev && e == hipSuccess) e = hipEventRecord(ev[k], st);
    };
    auto run_prefill = [&]() {
        if (e == hipSuccess && pl.n_tiles > 0) {
            p.cum_dev = inline_cum ? nullptr : ctx->plan_d + n_cum;
            p.list_by_seq = 0;
            if (inline_cum) fill_plan(pl, false, true, ka);
        }
        mark(2, ps);
        if (e == hipSuccess && pl.n_tiles > 0) e = launch_prefill(ka, ps);
        mark(3, ps);
    };
    auto run_decode = [&]() {
        if (e == hipSuccess && pl.static_runs > 0) {
            p.cum_dev = inline_cum ? nullptr : ctx->plan_d;
            if (inline_cum) fill_plan(pl, true, false, ka);
        }
        mark(0, s);
        if (e == hipSuccess && pl.static_runs > 0) {
            e = launch_decode(ka, s);
            // every wave draws one ticket per tail run it takes plus one that tells it to stop
            if (e == hipSuccess && pl.tail_runs > 0)
                ctx->queue_base += (uint32_t)pl.tail_runs * (uint32_t)ctx->Hkv + (uint32_t)pl.static_runs * (uint32_t)ctx->Hkv;
        }
        mark(1, s);
    };
    mark(4, s);
    if (fused || step) {
        p.cum_dev = inline_cum ? nullptr : ctx->plan_d;
        if (step) {
            fill_plan(pl, true, true, ka);
        } else {
            p.list_by_seq = 0;   // (the mixed kernel takes the arrays one behind the other, as in device memory)
            if (inline_cum) {
                memcpy(ka.cum, pl.dcum, n_cum * sizeof(int32_t));
                memcpy(ka.cum + n_cum, pl.pf, n_pf * sizeof(int32_t));
            }
        }
        mark(0, s);
        mark(2, s);
        if (e == hipSuccess) e = fused ? launch_mixed(ka, ctx->num_cus, s) : launch_step(ka, ctx->num_cus, s);
        mark(1, s);
        mark(3, s);
    } else if (overlap) {
        // fork before anything else is enqueued, so that the side stream waits for nothing of this call
        if (e == hipSuccess) e = hipEventRecord(ctx->fork_ev, s);
        if (e == hipSuccess) e = hipStreamWaitEvent(ctx->side_stream, ctx->fork_ev, 0);
        if (ctx->opt_decode_first) {
            run_decode();
            run_prefill();
        } else {
            run_prefill();
            run_decode();
        }
        if (e == hipSuccess) e = hipEventRecord(ctx->join_ev, ctx->side_stream);
        if (e == hipSuccess) e = hipStreamWaitEvent(s, ctx->join_ev, 0);
    } else {
        run_prefill();
        run_decode();
    }
    mark(5, s);
    // A plan serves one call: the device length arrays are trusted to equal the planned host copies, and a caller
    // that advances the lengths between steps must plan again (option "plan_persistent" keeps an explicit plan).
    if (ctx->plan_one_shot || !ctx->opt_plan_persistent) {
        ctx->plan_one_shot = false;
        ctx->plan_valid = false;
    }
    if (e != hipSuccess) return fail(ctx, OOCO_EHIP, "ooco_attn_mixed: kernel launch: %s", hipGetErrorString(e));
    return OOCO_OK;
}

ooco_status ooco_attn_mixed_static(int num_q_heads, int num_kv_heads, int head_dim, int block_size, int max_blocks_per_seq,
                                   float softmax_scale, const int32_t *h_seq_lens, const int32_t *h_query_start_loc,
                                   const int32_t *h_ctx_lens, const void *q, const void *k_cache, const void *v_cache,
                                   const int32_t *block_tables, const int32_t *seq_lens, const int32_t *query_start_loc,
                                   const int32_t *ctx_lens, void *out, int num_seqs, int total_q_tokens, void *stream,
                                   char *msg, size_t msg_cap)
{
    char err[512] = "";
    auto bad = [&](ooco_status code, const char *fmt, ...) __attribute__((format(printf, 3, 4))) {
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(err, sizeof err, fmt, ap);
        va_end(ap);
        if (msg && msg_cap) snprintf(msg, msg_cap, "%s", err);
        return code;
    };
    if (msg && msg_cap) msg[0] = 0;
    if (num_seqs < 0 || total_q_tokens < 0)
        return bad(OOCO_EINVAL, "ooco_attn_mixed_static: negative size (num_seqs=%d, total_q_tokens=%d)", num_seqs, total_q_tokens);
    if (num_q_heads <= 0 || num_kv_heads <= 0 || num_q_heads % num_kv_heads != 0 || num_q_heads / num_kv_heads > 16 ||
        (head_dim != 64 && head_dim != 128) || block_size != kBlockSize || max_blocks_per_seq <= 0)
        return bad(OOCO_ESHAPE, "ooco_attn_mixed_static: unsupported geometry (heads %d/%d, head_dim %d, block_size %d, "
                                "max_blocks_per_seq %d)", num_q_heads, num_kv_heads, head_dim, block_size, max_blocks_per_seq);
    if (num_seqs == 0 || total_q_tokens == 0) return OOCO_OK;
    if (!q || !k_cache || !v_cache || !block_tables || !seq_lens || !query_start_loc || !ctx_lens || !out || !h_seq_lens ||
        !h_query_start_loc || !h_ctx_lens)
        return bad(OOCO_EINVAL, "ooco_attn_mixed_static: NULL pointer argument");
    if (num_seqs > kInlineSeqs)
        return bad(OOCO_ENOMEM, "ooco_attn_mixed_static: %d sequences exceed the maximum of %d", num_seqs, kInlineSeqs);
    if ((size_t)num_seqs * (size_t)num_kv_heads > kStaticCounterInts)
        return bad(OOCO_ENOMEM, "ooco_attn_mixed_static: %d sequences x %d kv heads exceed the %zu arrival counters", num_seqs,
                   num_kv_heads, kStaticCounterInts);
    StaticDevice dev;
    int device = 0;
    hipError_t e = static_device(dev, device);
    if (e != hipSuccess) return bad(OOCO_EHIP, "ooco_attn_mixed_static: scratch array: %s", hipGetErrorString(e));

    // plan on the stack: default run layout, no dynamic tail, prefill tiles never split (their partial results
    // would not fit the fixed array); a partial-result area too small for the wanted runs lowers their number
    PlanGeometry geo;
    geo.Hq = num_q_heads;
    geo.Hkv = num_kv_heads;
    geo.hd = head_dim;
    geo.BS = block_size;
    geo.max_blocks_per_seq = max_blocks_per_seq;
    geo.num_cus = dev.num_cus;
    geo.ws_bytes = kStaticScratchBytes - kStaticCounterInts * sizeof(int32_t);
    geo.segments_opt = 0;
    geo.tail_pct = 0;
    geo.tail_blocks = 0;
    geo.pf_split_opt = 1;
    int32_t store[storage_ints(kInlineSeqs)];
    HostPlan pl;
    ooco_status st = build_plan(geo, num_seqs, h_seq_lens, h_query_start_loc, h_ctx_lens, carve_storage(store, kInlineSeqs), pl, err);
    if (st != OOCO_OK) {
        if (msg && msg_cap) snprintf(msg, msg_cap, "%s", err);
        return st;
    }
    if (pl.total_q != total_q_tokens)
        return bad(OOCO_ESHAPE, "ooco_attn_mixed_static: query_start_loc ends at %d, call has %d query tokens", pl.total_q,
                   total_q_tokens);
    if ((size_t)pl.slots * slot_bytes(geo) > geo.ws_bytes)
        return bad(OOCO_ENOMEM, "ooco_attn_mixed_static: partial results of %lld slots exceed the scratch array", (long long)pl.slots);
    if (pl.pf_split != 1 || pl.pf_slots != 0)   // (this entry point has no area for parts of prefill tiles)
        return bad(OOCO_EINVAL, "ooco_attn_mixed_static: internal error: the plan splits prefill tiles");

    KernArgs ka;
    memset(&ka, 0, sizeof ka);
    AttnParams &p = ka.p;
    int32_t *const counters = static_cast<int32_t *>(dev.ptr);
    float *const partials = reinterpret_cast<float *>(static_cast<unsigned char *>(dev.ptr) + kStaticCounterInts * sizeof(int32_t));
    p.q = static_cast<const uint16_t *>(q);
    p.k_cache = static_cast<const uint16_t *>(k_cache);
    p.v_cache = static_cast<const uint16_t *>(v_cache);
    p.block_tables = block_tables;
    p.seq_lens = seq_lens;
    p.query_start_loc = query_start_loc;
    p.ctx_lens = ctx_lens;
    p.out = static_cast<uint16_t *>(out);
    p.part_acc = partials;
    p.part_ml = partials + (size_t)pl.slots * num_q_heads * head_dim;
    p.counters = counters;
    p.cum_dev = nullptr;
    p.trace = nullptr;
    p.Hq = num_q_heads;
    p.Hkv = num_kv_heads;
    p.g = num_q_heads / num_kv_heads;
    p.g_magic = (uint16_t)(32768 / p.g + 1);
    p.hd = head_dim;
    p.max_blocks_per_seq = max_blocks_per_seq;
    p.scale_log2e = (softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt((float)head_dim)) * 1.4426950408889634f;
    p.num_seqs = num_seqs;
    p.total_q = total_q_tokens;
    p.dec_blocks = pl.dec_blocks;
    p.piece_pad = pl.piece_pad;
    p.static_blocks = pl.static_blocks;
    p.static_runs = pl.static_runs;
    p.tail_runs = 0;
    p.queue = reinterpret_cast<uint32_t *>(counters + kStaticCounterInts - 1);   // (no tail runs: never touched)
    p.queue_base = 0;
    p.n_tiles = pl.n_tiles;
    p.num_pf = pl.num_pf;
    p.pf_waves = (int8_t)pl.pf_waves;
    p.pf_groups = (int8_t)pl.pf_groups;
    p.nbi = (int8_t)pl.nbi;
    p.coop = (int8_t)pl.coop;
    p.coop_waves = (int8_t)pl.coop_waves;
    p.dec_near = (int8_t)pl.near;
    p.rotate_heads = 1;
    p.pf_acc = nullptr;
    p.pf_ml = nullptr;
    p.pf_counters = nullptr;
    p.pf_split = 1;
    p.pf_share = 0;
    p.pf_table = (int16_t)pl.pf_table;

    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    // The array keeps whatever the last call on this GPU left: the arrival counters this call will count in
    // start at zero (a small fill kernel, not a memset node, so that the call can be captured into a graph).
    if (pl.slots > 0) e = launch_fill_zero(counters, (int64_t)num_seqs * num_kv_heads, s);
    if (e == hipSuccess && step_fits(pl, head_dim, pl.coop, pl.nbi ? pl.nbi : (head_dim == 64 ? 2 : 1))) {
        // both kinds of work side by side in one launch: a step of four decodes and one prompt 16.6 -> 11.4 us (7.5 with
        // whole sequences)
        fill_plan(pl, true, true, ka);
        e = launch_step(ka, dev.num_cus, s);
    } else {
        if (e == hipSuccess && pl.n_tiles > 0) {
            fill_plan(pl, false, true, ka);
            e = launch_prefill(ka, s);
        }
        if (e == hipSuccess && pl.static_runs > 0) {
            fill_plan(pl, true, false, ka);
            e = launch_decode(ka, s);
        }
    }
    if (e != hipSuccess) return bad(OOCO_EHIP, "ooco_attn_mixed_static: kernel launch: %s", hipGetErrorString(e));
    return OOCO_OK;
}

ooco_status ooco_kv_block_copy(ooco_ctx *ctx, const void *k_src, const void *v_src, void *k_dst, void *v_dst,
                               const int64_t *src_block_ids, const int64_t *dst_block_ids, int64_t num_pairs,
                               void *stream)
{
    if (!ctx) return OOCO_EINVAL;
    if (num_pairs < 0) return fail(ctx, OOCO_EINVAL, "ooco_kv_block_copy: num_pairs=%lld", (long long)num_pairs);
    if (num_pairs == 0) return OOCO_OK;
    if (!k_src || !v_src || !k_dst || !v_dst || !src_block_ids || !dst_block_ids)
        return fail(ctx, OOCO_EINVAL, "ooco_kv_block_copy: NULL pointer argument");
    constexpr int64_t kMaxCopyPairs = (int64_t)1 << 26;
    if (num_pairs > kMaxCopyPairs)
        return fail(ctx, OOCO_EINVAL, "ooco_kv_block_copy: num_pairs=%lld too large", (long long)num_pairs);
    const int64_t block_bytes = (int64_t)ctx->Hkv * ctx->BS * ctx->hd * 2;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    ctx->note_stream(s);
    hipError_t e = hipSuccess;
    // Large copies take their pairs in order of destination region (ordered on the device into a buffer of the context,
    // which grows on demand -- never while the stream is being captured, a captured copy keeps the caller's order).
    // The order is worth about an eighth of the copy's time and costs 6 us and 0.25 us per 1000 pairs in one workgroup, up
    // to kOrderPairsMax pairs, and 28 us and more in the radix sort beyond.  Measured on MI355X, unordered / ordered:
    // 8 kv heads of 128, 2048 pairs 53.0 / 51.6 us, 8192 209 / 187; 4 heads of 128, 4096 pairs 52.5 / 53.6, 8192 107 / 101;
    // 4 heads of 64, 8192 pairs 53.2 / 55.1, 16,384 106.1 / 105.5, 32,768 211 / 216 (radix), 65,536 427 / 405 (radix).
    // Below 2048 pairs, whose blocks are then of 96 KiB and more, slots handed out in ascending order lose what others gain:
    // 32 heads of 128, 1000 pairs 98.6 / 93.1 us, ascending 89.4 / 92.9; 2047 pairs 203.9 / 188.2, ascending 182.5 / 186.9.
    const int64_t bytes_one_way = 2 * num_pairs * block_bytes;
    const bool order_pays = num_pairs >= 2048 && bytes_one_way >= (num_pairs <= kOrderPairsMax ? (int64_t)192 << 20 : (int64_t)640 << 20);
    // (nor may a captured copy name the buffer a context has already: a later call frees it when it needs a larger one,
    // and replays would go on using the freed memory)
    bool ordered = ctx->opt_copy_sort >= 2 || (ctx->opt_copy_sort == 1 && order_pays);
    if (ordered) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        const hipError_t q = hipStreamIsCapturing(s, &cs);
        if (q != hipSuccess) (void)hipGetLastError();
        ordered = q == hipSuccess && cs == hipStreamCaptureStatusNone;
    }
    if (ordered) {
        bool ready = num_pairs <= ctx->sort_cap;
        if (!ready) {
            // (at least twice the last size, so that slowly growing copies do not reallocate every time)
            const int64_t cap = std::max({num_pairs, std::min(2 * ctx->sort_cap, kMaxCopyPairs), kOrderPairsMax});
            size_t temp = 0;
            if (sort_pairs_temp_bytes(cap, &temp) == hipSuccess) {
                // (work of earlier calls may still read the old buffer: wait for it before freeing)
                if (ctx->sort_buf) {
                    (void)hipStreamSynchronize(s);
                    (void)hipFree(ctx->sort_buf);
                    ctx->sort_buf = nullptr;
                    ctx->sort_cap = 0;
                }
                const size_t ids = ((size_t)cap * 2 * sizeof(int64_t) + 255) / 256 * 256;
                if (hipMalloc(&ctx->sort_buf, ids + temp) == hipSuccess) {
                    ctx->sort_cap = cap;
                    ctx->sort_temp_bytes = temp;
                    ready = true;
                } else {
                    (void)hipGetLastError();
                    ctx->sort_buf = nullptr;
                }
            }
        }
        if (ready) {
            int64_t *dst_sorted = static_cast<int64_t *>(ctx->sort_buf), *src_sorted = dst_sorted + ctx->sort_cap;
            void *temp = static_cast<unsigned char *>(ctx->sort_buf) + ((size_t)ctx->sort_cap * 2 * sizeof(int64_t) + 255) / 256 * 256;
            // (key = the low bits that number the blocks of this context's pool; the destination pool is that pool or
            // a smaller one)
            int bits = 1;
            while (bits < 32 && ((int64_t)1 << bits) < ctx->num_blocks) ++bits;
            e = num_pairs <= kOrderPairsMax ? launch_order_pairs(dst_block_ids, dst_sorted, src_block_ids, src_sorted, num_pairs, bits, s)
                                            : launch_sort_pairs(temp, ctx->sort_temp_bytes, dst_block_ids, dst_sorted, src_block_ids, src_sorted, num_pairs,
                                  bits, s);
            if (e == hipSuccess) {
                src_block_ids = src_sorted;
                dst_block_ids = dst_sorted;
            } else {
                (void)hipGetLastError();   // the sort did not start: copy in the caller's order
                e = hipSuccess;
            }
        }
    }
    if (e == hipSuccess)
        e = launch_block_copy(k_src, v_src, k_dst, v_dst, src_block_ids, dst_block_ids, num_pairs, block_bytes,
                              ctx->opt_copy_variant, s);
    if (e != hipSuccess) return fail(ctx, OOCO_EHIP, "ooco_kv_block_copy: kernel launch: %s", hipGetErrorString(e));
    return OOCO_OK;
}

ooco_status ooco_kv_append(ooco_ctx *ctx, const void *k_new, const void *v_new, void *k_cache, void *v_cache,
                           const int32_t *block_tables, const int32_t *query_start_loc, const int32_t *ctx_lens,
                           int num_seqs, int total_q_tokens, void *stream)
{
    if (!ctx) return OOCO_EINVAL;
    if (num_seqs < 0 || total_q_tokens < 0)
        return fail(ctx, OOCO_EINVAL, "ooco_kv_append: num_seqs=%d total_q_tokens=%d", num_seqs, total_q_tokens);
    if (num_seqs == 0 || total_q_tokens == 0) return OOCO_OK;
    if (!k_new || !v_new || !k_cache || !v_cache || !block_tables || !query_start_loc || !ctx_lens)
        return fail(ctx, OOCO_EINVAL, "ooco_kv_append: NULL pointer argument");
    hipError_t e = launch_kv_append(k_new, v_new, k_cache, v_cache, block_tables, query_start_loc, ctx_lens, num_seqs,
                                    total_q_tokens, ctx->Hkv, ctx->hd, ctx->max_blocks_per_seq, ctx->num_blocks,
                                    (int)ctx->opt_append_parts, ctx->num_cus, reinterpret_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail(ctx, OOCO_EHIP, "ooco_kv_append: kernel launch: %s", hipGetErrorString(e));
    return OOCO_OK;
}

}  // extern "C"
