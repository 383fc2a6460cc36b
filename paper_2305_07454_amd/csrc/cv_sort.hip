// cv_sort.hip -- cv_sort_records: stable order of raw records by
// (journey id, timestamp), the paper's unique index over all journeys
// (Methods, step (2)).
//
// Pipeline (all stream-ordered, no host synchronisation):
//   1. k_dict_insert  min/max timestamp; whether time never decreases within a
//                     shard in input order (then the key needs no time bits);
//                     the time offsets' common factor 2^a 5^b; distinct
//                     journey ids into an open-addressing hash set
//                     (run-deduplicated), batched: each id's slot tagged with
//                     its shard, an id met in two shards flagged;
//   2. k_dict_compact distinct ids -> list; its last block settles the journey
//                     count J, rank bits, time bits, key bits and passes;
//   3. launch_dict_order
//                     the list in signed order, batched: by (shard, id): by
//                     counting, sorted chunks and their join, or radix passes
//                     (cv_dictsort.h);
//   4.                and each id's dense rank in that order (the shard needs
//                     no bits of its own in the key unless an id spans shards);
//   5. k_pack_hist / k_pack_il   (grouped input, see JW: pack_grouped, and no pass after it)
//                     key = rank << t_bits | (ts - t_min) / factor (or the
//                     rank alone for time-ordered input) and the digit
//                     histograms of every radix pass in the same read; for
//                     interleaved input k_pack_il also regroups each tile by
//                     journey and packs the payload per record;
//   6. radix passes   ceil(key_bits / 8) stable scatter passes, one less with a
//                     9-bit first digit for a key of 8k + 1 bits (skipped on device);
//   7. k_gather / k_gather_feat
//                     perm, journey id from the dictionary, ts from the key
//                     when it survives packing, lat/lon/speed through perm or
//                     from the packed payload; k_gather_feat adds the
//                     kinematics.
#include <hip/hip_runtime.h>

#include "cv_device.h"
#include "cv_dictsort.h"
#include "cv_host.h"
#include "cv_kin.h"
#include "cv_radix.h"

using namespace cv;

namespace {

constexpr u64 EMPTY = 0x8000000000000000ull;  // INT64_MIN marks an empty slot
constexpr u64 SIGN = 0x8000000000000000ull;

struct SortMeta {
    u64 tmin_ord;
    u64 tmax_ord;
    u32 has_min;
    u32 overflow;
    u32 J;
    u32 list_count;
    u32 dict_n;
    u32 rank_bits;
    u32 t_bits;
    u32 key_bits;
    u32 passes;
    u32 range_err;
    u32 shard_bits;
    u32 ib;   // index bits of a packed key word
    u32 p0;   // first pass whose input words are packed (ib and p0 adjacent: the radix passes read both)
    u32 w0;   // bits of the first radix digit: 9 where that saves a pass (a key of 8k + 1 bits), else 8
    u32 big_n;   // dict_n when the radix passes are to sort the distinct ids, else 0
    u32 blocks_done;  // blocks of the compaction that have ended
    u32 n_runs;  // runs of equal ids in input order (counted by the dictionary insert)
    u32 unordered;  // a timestamp below its predecessor's (same shard) in input order
    u32 ts_dropped; // key = (shard, rank) only: the input is time-ordered within every shard
    u32 multi_shard; // batched: an id in more than one shard (ranks then in id order, shard bits in the key)
    u32 t_nd5;       // bit b: some time offset is not a multiple of 5^(b+1) (b < 3)
    u64 t_or;        // OR of every |ts - ts[0]|: its trailing zeros are the offsets' common power of two
    u32 t_sh;        // the key's time offset is (ts - t_min) / (2^t_sh * t_p5): the offsets'
    u32 t_p5;        //   common factor of the form 2^a 5^b (b <= 3), e.g. 1000 for 1 Hz in ms
    u32 grouped;     // the input's runs are whole journeys, in time order but for near neighbours (see JW)
    u32 sort_bits;   // key bits that the radix passes sort by: key_bits, or 0 where grouped
    u32 min_end, min_start;  // (plain form) the run of the id INT64_MIN, which has no slot
    u32 t_off;       // tickets of the run offsets
    u32 tickets[3 * MAX_PASSES];
};

__device__ __forceinline__ u32 bit_width64(u64 x) { return x ? 64u - (u32)__clzll((long long)x) : 0u; }

// What one block of the dictionary insert found in its records, stored by the
// block and joined by the last block of the compaction.  Adding it to one
// shared word instead serialised some 36 000 atomics on a few addresses:
// about 250 us of every sort, whatever its size.
struct InsPart {
    u64 lo, hi;  // least and largest time stamp (ordered image)
    u64 tor;     // OR of every |ts - ts[0]|
    u32 nd5, runs, down, multi;  // down: PD_*
};
constexpr u32 PD_DOWN = 1;  // a time stamp below its predecessor's
constexpr u32 PD_FAR = 2;   // not the near order that grouped input has

// Input of whole journeys (every id one run, as where journey files follow one
// another) whose runs are in time order but for neighbours at most JW records
// apart needs no radix pass: a record's place is its journey's start plus its
// place in the run, moved by the records within JW on either side that belong
// on the other side of it.  The insert decides it on the way: no inversion at
// a distance of JW + 1 to 2 JW + 1 within a run.  (That covers any distance:
// were the nearest inversion beyond JW, of records j < i, longer than
// 2 JW + 1, the record JW + 1 after j would be in an inversion beyond JW with
// one of them, a nearer one.)  Neighbours in a run have to lie less than
// JW_GAP apart, so that 32-bit differences compare exactly.  The insert of
// 123 M records takes 549 us with it (476 without; a wave that has seen its input
// to be otherwise goes on without it: 1 M shuffled 53 us as before), and the key
// packing and radix passes 0.65 + 0.18 ms where they took 0.75 + 2.44 (the whole
// call 9.19 -> 7.04 ms; 12.3 M: 1.15 -> 0.88).  A wave also ends it where it meets an id's
// second run: in bundled feeds (runs of a few records in time order, ids coming back)
// nothing else does, and every run's start and end went through the table (20 M
// records in runs of 5, 8 000 ids: insert and packing 1.64 ms, 0.76 now).
constexpr int JW = 3;
static_assert(JW >= 1 && JW <= 3, "the check's first part covers distances up to 3");
constexpr u64 JW_GAP = 1ull << 27;
static_assert((2 * JW + 1) * JW_GAP < (1ull << 31), "differences in a window fit 32 bits");
constexpr int JW_HEADS = 16;  // run starts per 64 records from which a wave takes its input for interleaved

// whether lanes l and l - d of a window lie in one run, as a lane mask: no run
// starts in the lanes after l - d up to l (h: the run starts of this window and
// the one before)
struct RunMask {
    u64 h, hp, none;  // none: starts within the last d lanes
    int d;
    __device__ __forceinline__ RunMask(u64 heads, u64 before) : h(heads), hp(before), none(0), d(0) {}
    __device__ __forceinline__ u64 next()  // for d = 1, 2, ...
    {
        none |= d ? (h << d) | (hp >> (WAVE - d)) : h;
        ++d;
        return ~none;
    }
};

// The sort's scratch in one launch: the meta words, the dictionary's empty
// slots and the region cleared to zero.
// used (nullable): the occupied slots' bits.
__global__ void __launch_bounds__(256) k_sort_begin(SortMeta* m, u64* __restrict__ table, u64 words,
                                                    u32* __restrict__ zero, u64 zwords, u32* __restrict__ used)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        SortMeta z = {};
        *m = z;
    }
    const u64 i0 = (u64)blockIdx.x * blockDim.x + threadIdx.x;
    const u64 stride = (u64)gridDim.x * blockDim.x;
    ulonglong2* t2 = (ulonglong2*)table;  // slots are 16-byte pairs
    for (u64 i = i0; i < words / 2; i += stride) t2[i] = make_ulonglong2(EMPTY, EMPTY);
    for (u64 i = i0; i < zwords; i += stride) zero[i] = 0u;
    if (used)
        for (u64 i = i0; i < words / 64; i += stride) used[i] = 0u;  // (two words per slot)
}

// The dictionary is an open-addressing table of 16-byte slots {id, rank}:
// the id word is claimed by CAS (EMPTY when free) and the rank word is filled
// in once the distinct ids are sorted, so that one 16-byte load per probe
// returns both.  An insert probes linearly from mix64(id); the caller reads the
// first slot (so that the first probes of many records are in flight
// together) and this continues from it.  A slot read as free is read again,
// past the XCD's L2, before the CAS: its line may have been cached while the
// slot was free, and by then most waves only need to see that the id is there
// (a CAS of every wave for every id, one after the other on the id's slot,
// was most of the insert of a small call).
__device__ __forceinline__ u64 slot_now(const u64* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A slot's first insert sets its bit of `used` (nullable), so that the ids are
// listed without reading a table that is mostly empty where the caller had to
// allow for an id per record.  Returns the id's slot, or ~0 when the table is full.
__device__ __forceinline__ void slot_used(u32* used, u64 h)
{
    if (used) atomicOr(&used[h / 32], 1u << (h % 32));
}
__device__ __forceinline__ u64 dict_insert_from(u64* table, u64 mask, u64 key, u64 h, u64 cur, u32* used)
{
    for (u64 probe = 0; probe <= mask; ++probe) {
        if (cur == EMPTY) cur = slot_now(&table[2 * h]);
        if (cur == key) return h;
        if (cur == EMPTY) {
            u64 prev =
                atomicCAS((unsigned long long*)&table[2 * h], (unsigned long long)EMPTY, (unsigned long long)key);
            if (prev == EMPTY) slot_used(used, h);
            if (prev == EMPTY || prev == key) return h;
        }
        h = (h + 1) & mask;
        cur = table[2 * h];
    }
    return ~0ull;
}

// Plain form: until the ranks are set, the second word of an id's slot holds
// where its run starts (high half) and ends (low half).  Only used where every
// id has one run.
__device__ __forceinline__ void run_store(u64* word, bool start, u32 at)
{
    __hip_atomic_store((u32*)word + (start ? 1 : 0), at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// the start of an id's run; false where another run's is there already (a wave that
// sees one id twice has seen that the input is not whole journeys)
__device__ __forceinline__ bool run_begin(u64* word, u32 at)
{
    if ((u32)(slot_now(word) >> 32) != (u32)(EMPTY >> 32)) return false;
    run_store(word, true, at);
    return true;
}
__device__ __forceinline__ u32 run_start(u64 w) { return (u32)(w >> 32); }
__device__ __forceinline__ u32 run_length(u64 w) { return (u32)w - (u32)(w >> 32); }
// the run of `key` ends before record `at`
__device__ __forceinline__ void run_end(u64* table, u64 mask, SortMeta* m, u64 key, u32 at, bool& full,
                                        u32* used)
{
    if (key == EMPTY) {
        m->min_end = at;
        return;
    }
    const u64 h = mix64(key) & mask;
    const u64 slot = dict_insert_from(table, mask, key, h, table[2 * h], used);
    if (slot == ~0ull) full = true;
    else run_store(&table[2 * slot + 1], false, at);
}

// Batched form: the insert of `key` for shard `sh`, continuing a probe at slot
// h whose entry e was read, also tags the slot's second word with the shard.
// A slot tagged with another shard means the id lies in two shards (multi).
// Both the inserter and a reader that finds the slot untagged tag it by
// compare-and-swap, so exactly one shard wins and any other sees it.
// Returns false when the table is full.
__device__ __forceinline__ bool dict_insert_tag(u64* table, u64 mask, u64 key, u64 h, ulonglong2 e, u64 sh,
                                                bool& multi, u32* used)
{
    const ulonglong2* t2 = (const ulonglong2*)table;
    for (u64 probe = 0; probe <= mask; ++probe) {
        if (e.x == EMPTY) {
            e.x = slot_now(&table[2 * h]);
            e.y = EMPTY;  // read again below
        }
        bool mine = e.x == key;
        if (!mine && e.x == EMPTY) {
            const u64 prev =
                atomicCAS((unsigned long long*)&table[2 * h], (unsigned long long)EMPTY, (unsigned long long)key);
            if (prev == EMPTY) slot_used(used, h);
            mine = prev == EMPTY || prev == key;
        }
        if (mine) {
            if (e.y == EMPTY) e.y = slot_now(&table[2 * h + 1]);
            if (e.y != sh) {
                const u64 old = atomicCAS((unsigned long long*)&table[2 * h + 1], (unsigned long long)EMPTY,
                                          (unsigned long long)sh);
                if (old != EMPTY && old != sh) multi = true;
            }
            return true;
        }
        h = (h + 1) & mask;
        e = t2[h];
    }
    return false;
}

// slot of `key`, or ~0 when absent
__device__ __forceinline__ u64 dict_find(const u64* table, u64 mask, u64 key)
{
    u64 h = mix64(key) & mask;
    for (u64 probe = 0; probe <= mask; ++probe) {
        u64 cur = table[2 * h];
        if (cur == key) return h;
        if (cur == EMPTY) return ~0ull;
        h = (h + 1) & mask;
    }
    return ~0ull;
}

// rank of `key` (0 when absent), one 16-byte load per probe
__device__ __forceinline__ u32 dict_rank_of(const u64* table, u64 mask, u64 key)
{
    const ulonglong2* t2 = (const ulonglong2*)table;
    u64 h = mix64(key) & mask;
    for (u64 probe = 0; probe <= mask; ++probe) {
        const ulonglong2 e = t2[h];
        if (e.x == key) return (u32)e.y;
        if (e.x == EMPTY) return 0u;
        h = (h + 1) & mask;
    }
    return 0u;
}

// Each wave of the dictionary kernels walks its own contiguous range of
// windows of 64 records and keeps the ids it met last in a small LDS cache
// (direct-mapped, DC slots per wave): in time-ordered input, where many
// journeys interleave, a window's ids mostly appeared in the windows just
// before, and the cache spares those records the probe of the global table.
// A slot is written by one lane only (the lanes that miss on a slot elect
// one through the owner word), so an entry is never a mix of two writes.
constexpr int DC = 512;   // slots per wave in the insert (24 KB of LDS per workgroup; 256: 0.3 ms slower on
                          // the interleaved batched feed)
constexpr int DCH = 128;  // slots per wave in the key packing for input in long runs (16 KB with the histograms)
constexpr int DCP = 256;  // slots per wave in the interleaved key packing (its 1 024-thread workgroups are
                          // one per CU at their register count, whatever the LDS)
constexpr int DPW = 4;  // windows whose ids and times are loaded together (plain form: 90 VGPRs, 5 waves per SIMD)

__device__ __forceinline__ void wave_range(u32 n, u64& wbeg, u64& wend)
{
    const u64 nw = (u64)gridDim.x * (blockDim.x / WAVE);
    const u64 nwin = ((u64)n + WAVE - 1) / WAVE;
    const u64 per = (nwin + nw - 1) / nw;
    wbeg = ((u64)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE) * per;
    wend = wbeg + per < nwin ? wbeg + per : nwin;
}

template <int C>
__device__ __forceinline__ u32 dict_cache_slot(u64 key)
{
    static_assert((C & (C - 1)) == 0 && C <= 4096, "power of two");
    return (u32)(mix64(key) >> (64 - __builtin_ctz(C)));  // the hash's top bits
}

// bits 0..2: |d| not a multiple of 5, 25, 125 (one remainder where it is one of 125)
__device__ __forceinline__ u32 not_div5(u64 ad)
{
    if ((ad >> 32) == 0) {
        const u32 x = (u32)ad % 125u;
        return x == 0 ? 0u : (x % 5u ? 1u : 0u) | (x % 25u ? 2u : 0u) | 4u;
    }
    return (ad % 5ull ? 1u : 0u) | (ad % 25ull ? 2u : 0u) | (ad % 125ull ? 4u : 0u);
}

// the key's time offset: (ts - t_min) divided by the offsets' common factor
// 2^sh 5^b (exact: every offset is a multiple of it)
__device__ __forceinline__ u64 time_offset(u64 toff, u32 sh, u32 p5)
{
    u64 q = toff >> sh;
    if (p5 == 5) q /= 5ull;
    else if (p5 == 25) q /= 25ull;
    else if (p5 == 125) q /= 125ull;
    return q;
}

__device__ __forceinline__ void part_join(InsPart& a, const InsPart& b)
{
    a.lo = b.lo < a.lo ? b.lo : a.lo;
    a.hi = b.hi > a.hi ? b.hi : a.hi;
    a.tor |= b.tor;
    a.nd5 |= b.nd5;
    a.runs += b.runs;
    a.down |= b.down;
    a.multi |= b.multi;
}

// the join of a wave's lanes, in every lane
__device__ __forceinline__ void part_wave_join(InsPart& p)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const InsPart o{(u64)__shfl_xor(p.lo, d, WAVE), (u64)__shfl_xor(p.hi, d, WAVE), (u64)__shfl_xor(p.tor, d, WAVE),
                        (u32)__shfl_xor(p.nd5, d, WAVE), (u32)__shfl_xor(p.runs, d, WAVE),
                        (u32)__shfl_xor(p.down, d, WAVE), (u32)__shfl_xor(p.multi, d, WAVE)};
        part_join(p, o);
    }
}

// Also checks whether the timestamps never decrease within a shard in input
// order: then every journey's records already come in time order, and a
// stable sort by (shard, journey) alone gives the (journey, time) order.
// SHARDS (the batched form) also tags every id's slot with its shard and
// flags an id met in two shards; a run of equal ids then ends at a shard
// start, and a window of a shard other than the one its wave's cache was
// filled in empties the cache (whose entries would skip the shard check); a
// window with a shard start inside goes without it.
// USED: the occupied slots' bits are kept.
template <bool SHARDS, bool USED>
__global__ void __launch_bounds__(256) k_dict_insert(const i64* __restrict__ jid, const i64* __restrict__ ts, u32 n,
                                                     u64* __restrict__ table, u64 mask, SortMeta* m,
                                                     InsPart* __restrict__ parts, const u64* __restrict__ soff,
                                                     u32 S, u32* used_)
{
    u32* used = USED ? used_ : nullptr;
    // (the batched form's 16-byte probes and shard checks take it to 4 waves
    // per SIMD, with 3 windows per round as with 4)
    constexpr int DP = DPW;
    __shared__ InsPart s_part[4];
    __shared__ u64 c_key[4][DC];
    __shared__ u32 c_own[4][DC];
    const int w = threadIdx.x / WAVE;
    const int l = lane_id();
    for (int i = l; i < DC; i += WAVE) c_key[w][i] = EMPTY;  // EMPTY is never looked up
    u64 lo = ~0ull, hi = 0;
    bool has_min = false, full = false, multi = false;
    u64 wbeg, wend;
    wave_range(n, wbeg, wend);
    i64 prevj = 0;  // last id of the previous window
    bool hp = false;
    // (plain form) the window before: time stamps, run starts, whether a time
    // stamp falls in it, inversions at 2 and 3; far: the input is not grouped (wave-uniform)
    u32 pt = 0;
    u64 ph_ = 0, pdown = ~0ull, pnear = ~0ull, far = 0;
    if (!SHARDS && wbeg < wend && wbeg > 0) {
        const u64 i = (wbeg - 1) * WAVE + l;
        const i64 j = jid[i];
        const i64 jb = lane_below(j);
        pt = (u32)ts[i];
        ph_ = __ballot(j != jb);
        prevj = lane_last(j);
        hp = true;
    }
    u32 runs = 0;   // records that start a run of equal ids (wave-uniform)
    // time of the record before the range (ordered form), then of each window's last
    u64 prevt = (wbeg < wend && wbeg > 0) ? ord_i64(ts[wbeg * WAVE - 1]) : 0ull;
    bool down = false;
    u32 shk = (S > 1 && wbeg < wend) ? shard_lower_bound(soff, S, wbeg * WAVE) : 0u;
    u32 csh = ~0u;  // the shard the wave's cache entries were met in (SHARDS)
    // the time offsets' common factor: every |ts - ts[0]| ORed together (its
    // trailing zeros) and which powers of five fail to divide one
    const u64 t0r = n ? ord_i64(ts[0]) : 0ull;
    const u64 nlast = ((u64)n - 1) / WAVE;  // the last record's window
    u64 tor = 0;
    u32 nd5 = 0;
    for (u64 w0 = wbeg; w0 < wend; w0 += DP) {
        i64 jv[DP];
        u64 tv[DP];
#pragma unroll
        for (int k = 0; k < DP; ++k) {
            u64 i = (w0 + k) * WAVE + l;
            i = i < n ? i : (u64)n - 1;  // past the end: a valid record, not used
            jv[k] = jid[i];
            tv[k] = ord_i64(ts[i]);
        }
        // shard starts of each window (lane masks) and the window's shard
        // when none starts inside it (~0 otherwise); wave-uniform
        u64 starts[DP];
        u32 wsh[DP];
#pragma unroll
        for (int k = 0; k < DP; ++k) {
            starts[k] = 0;
            wsh[k] = 0;
            if (S > 1 && w0 + k < wend) {
                const u32 k0 = __builtin_amdgcn_readfirstlane(shk);
                bool at_end = false;
                starts[k] = shard_starts_in(soff, S, shk, (w0 + k) * WAVE, at_end);
                wsh[k] = starts[k] ? ~0u : k0 - 1;
            }
        }
        // first the run starts of every window and, for each that misses the
        // cache, the first probe, issued together; then the inserts in order
        bool miss[DP];
        u64 ph[DP];
        ulonglong2 pe[DP];
        u64 heads[DP];  // run starts
        i64 jlast[DP];  // id before the window
#pragma unroll
        for (int k = 0; k < DP; ++k) {
            miss[k] = false;
            heads[k] = 0;
            jlast[k] = 0;
            if (w0 + k >= wend) continue;
            const u64 i = (w0 + k) * WAVE + l;
            const bool valid = i < n;
            const i64 j = jv[k];
            if (valid) {
                lo = tv[k] < lo ? tv[k] : lo;
                hi = tv[k] > hi ? tv[k] : hi;
                const u64 d = tv[k] - t0r;  // ts - ts[0] modulo 2^64 (the order map adds the same 2^63)
                const u64 ad = (i64)d < 0 ? 0ull - d : d;
                tor |= ad;
                if (nd5 != 7u) nd5 |= not_div5(ad);
            }
            const bool sstart = (starts[k] >> l) & 1ull;
            // time order against the record before (none before record 0
            // and before a shard's first record)
            const u64 tq = (u64)lane_below((i64)tv[k], (i64)prevt);
            if (valid && i > 0 && !sstart && tv[k] < tq) down = true;
            prevt = (u64)lane_last((i64)tv[k]);
            // a record repeating the id before it adds nothing (in the
            // batched form, unless a shard starts at it)
            const i64 jp = lane_below(j, prevj);
            const bool dup = (l > 0 || hp) && j == jp && !(SHARDS && sstart);
            jlast[k] = prevj;
            prevj = lane_last(j);
            hp = true;
            bool need = valid && !dup;
            heads[k] = __ballot(need);
            runs += (u32)__popcll(heads[k]);
            if (!SHARDS && !far) {
                // near order (JW): inversions at JW + 1 to 2 JW + 1, where a time
                // stamp falls at all; none where there are none at 2 and 3, as
                // with rows that changed places.  (Of records j < i in an inversion
                // at 4 or more, the record 2 after j is in one with i, nearer, or
                // with j, at 2: in this window, or among the last of the one before.)
                const u32 x = (u32)tv[k];
                const u64 vm = __ballot(valid);
                far |= __ballot(dup && tv[k] - tq + JW_GAP >= 2 * JW_GAP) & vm;
                const u64 falls = __ballot(tv[k] < tq) & ~heads[k] & vm;
                u64 near = 0;
                if (falls | pdown) {
                    RunMask rm(heads[k], ph_);
                    u32 y = x;
#pragma unroll
                    for (int d = 1; d <= 3; ++d) {
                        y = lane_below(y, (u32)__builtin_amdgcn_readlane((int)pt, WAVE - d));
                        const u64 in = rm.next() & vm;
                        if (d > 1) near |= __ballot((int)(x - y) < 0) & in;
                    }
                    if (near | pnear) {
#pragma unroll
                        for (int d = 4; d <= 2 * JW + 1; ++d) {
                            y = lane_below(y, (u32)__builtin_amdgcn_readlane((int)pt, WAVE - d));
                            const u64 in = rm.next() & vm;
                            if (d > JW) far |= __ballot((int)(x - y) < 0) & in;
                        }
                    }
                }
                if (__popcll(heads[k]) > JW_HEADS) far = 1;
                pdown = falls >> (WAVE - 2 * JW - 1);  // (those that the next window's pairs can span)
                pnear = near >> (WAVE - 2 * JW - 1);
                pt = x;
                ph_ = heads[k];
            }
            if (!SHARDS && heads[k] == 0) continue;  // (no hashing in the middle of a run)
            if (need && (u64)j == EMPTY) {
                has_min = true;
                if (!SHARDS) m->min_start = (u32)i;
                need = false;
            }
            // (an id of the cache is in the table, with the shard csh)
            const u32 cs = dict_cache_slot<DC>((u64)j);
            miss[k] = need && ((SHARDS && wsh[k] != csh) || c_key[w][cs] != (u64)j);
            if (!SHARDS && !far) far = __ballot(need && !miss[k]);  // an id's second run
            ph[k] = mix64((u64)j) & mask;
            if (SHARDS) {
                if (miss[k]) pe[k] = ((const ulonglong2*)table)[ph[k]];
            } else if (miss[k]) {
                pe[k].x = table[2 * ph[k]];
            }
        }
#pragma unroll
        for (int k = 0; k < DP; ++k) {
            if (w0 + k >= wend) break;
            if (SHARDS && wsh[k] != csh) {
                // the cache holds ids of one shard; none when a shard starts inside the window
                for (int i = l; i < DC; i += WAVE) c_key[w][i] = EMPTY;
                __builtin_amdgcn_wave_barrier();
                csh = wsh[k];
            }
            if (!SHARDS && heads[k] == 0 && w0 + k != nlast) continue;
            const bool cached = !SHARDS || csh != ~0u;
            const u64 j = (u64)jv[k];
            const u64 wi = (w0 + k) * WAVE;  // the window's first record
            const u32 cs = dict_cache_slot<DC>(j);
            // an earlier window of the round may have brought the id; of the
            // lanes that miss with one id, the one that owns its cache slot
            // inserts it (the first meetings of a table's few ids by every
            // wave at once are bound by atomics on the ids' slots)
            if (cached && miss[k]) miss[k] = c_key[w][cs] != j;
            if (__ballot(miss[k]) != 0) {
                if (miss[k]) c_own[w][cs] = (u32)l;
                __builtin_amdgcn_wave_barrier();
                const int own = miss[k] ? (int)c_own[w][cs] : l;
                const u64 jown = (u64)__shfl((i64)j, own, WAVE);
                bool again = false;  // the id's run here is its second
                if (miss[k] && (own == l || jown != j || !cached)) {
                    if (SHARDS) {
                        // the record's shard: the window's, or searched where a shard starts inside it
                        const u64 i = wi + l;
                        const u32 sh = wsh[k] != ~0u ? wsh[k] : shard_of(soff, S, i < n ? i : (u64)n - 1);
                        if (!dict_insert_tag(table, mask, j, ph[k], pe[k], (u64)sh, multi, used)) full = true;
                    } else {
                        const u64 slot = dict_insert_from(table, mask, j, ph[k], pe[k].x, used);
                        if (slot == ~0ull) full = true;
                        else if (!far) again = !run_begin(&table[2 * slot + 1], (u32)(wi + l));
                    }
                }
                if (!SHARDS) far |= __ballot(again);
                if (cached && miss[k] && own == l) c_key[w][cs] = j;
                __builtin_amdgcn_wave_barrier();
            }
            if (!SHARDS && !far) {
                // where the run before each run start ends; the last run
                const u64 jb = (u64)lane_below(jv[k], jlast[k]);
                if (((heads[k] >> l) & 1ull) && wi + l > 0) run_end(table, mask, m, jb, (u32)(wi + l), full, used);
                if (wi + l + 1 == n) run_end(table, mask, m, j, n, full, used);
            }
        }
    }
    if (has_min) atomicOr(&m->has_min, 1u);
    if (full) atomicOr(&m->overflow, 1u);
    // (runs is wave-uniform)
    InsPart wp{lo, hi, tor, nd5, l == 0 ? runs : 0u, (down ? PD_DOWN : 0u) | (far ? PD_FAR : 0u), SHARDS && multi ? 1u : 0u};
    part_wave_join(wp);
    if (l == 0) s_part[w] = wp;
    __syncthreads();
    if (threadIdx.x == 0) {
        InsPart p = s_part[0];
        for (int k = 1; k < (int)(blockDim.x / WAVE); ++k) part_join(p, s_part[k]);
        parts[blockIdx.x] = p;
    }
}

// Input whose runs of equal journey ids are short (journeys interleaved, as in
// a time-ordered feed) sends the gather through the sort's index to a separate
// memory segment per record and column; for such input the payload columns
// are first packed per record, so that the gather reads one 32-byte record.
constexpr u64 PAY_MIN_RUN = 8;  // mean run length below which the packed form is used
__device__ __forceinline__ bool pay_packed(const SortMeta* m, u32 n) { return (u64)m->n_runs * PAY_MIN_RUN > n; }

// The key's layout from the distinct ids (J) and the insert's findings (one thread).
// near: every run in near order (JW); res (nullable): the call's result, which is
// known from here on.
__device__ __forceinline__ void dict_meta(SortMeta* m, u32 J, u32 max_j, u32 n, u32 n_shards, u32 allow_wide,
                                          bool near, cv_result* res)
{
    m->J = J;
    if (J > max_j) m->overflow = 1;
    m->dict_n = J < max_j ? J : max_j;
    m->big_n = m->dict_n > DS_COUNT ? m->dict_n : 0u;
    u32 rb = J > 1 ? bit_width64((u64)J - 1) : 0;
    u64 span = n ? (unord_i64(m->tmax_ord) - (u64)unord_i64(m->tmin_ord)) : 0;
    // the offsets' common factor 2^a 5^b (1 when the time stamps are all equal)
    u32 a = m->t_or ? (u32)__ffsll((long long)m->t_or) - 1u : 0u;
    u32 p5 = (m->t_nd5 & 1u) ? 1u : (m->t_nd5 & 2u) ? 5u : (m->t_nd5 & 4u) ? 25u : 125u;
    if (!m->t_or) p5 = 1;
    m->t_sh = a;
    m->t_p5 = p5;
    span = (span >> a) / p5;
    // time-ordered input needs no time bits in the key (see the insert)
    m->ts_dropped = m->unordered ? 0u : 1u;
    u32 tb = m->ts_dropped ? 0u : bit_width64(span);
    // batched: when every id lies in one shard, ranks follow (shard, id) order
    // and already keep the shards apart; otherwise the shard goes above them
    // (the INT64_MIN id, which is never in the table, counts as such a case)
    if (n_shards > 1 && m->has_min) m->multi_shard = 1;
    const u32 sb = (n_shards > 1 && m->multi_shard) ? bit_width64((u64)n_shards - 1) : 0;
    m->rank_bits = rb;
    m->t_bits = tb;
    m->shard_bits = sb;
    u32 kb = sb + rb + tb;
    if (kb > 64) {
        m->range_err = 1;
        kb = 0;
    }
    m->key_bits = kb;
    // Packed words (key >> 8 p0) << ib | index replace the (key, index) pairs
    // from pass p0 on; p0 is the first digit boundary from which the rest of
    // the key and the index fit one word.  p0 < passes whenever p0 > 0.
    const u32 ib = n > 1 ? bit_width64((u64)n - 1) : 1u;
    m->ib = ib;
    const u32 p0 = kb + ib > 64 ? (kb + ib - 64 + RADIX_BITS - 1) / RADIX_BITS : 0u;
    m->p0 = p0;
    // a key of 8k + 1 bits, packed from the first pass, takes a 9-bit first
    // digit and k passes instead of k + 1
    const u32 w0 = (allow_wide && p0 == 0 && kb > RADIX_BITS && kb % RADIX_BITS == 1) ? RADIX_BITS + 1 : RADIX_BITS;
    m->w0 = w0;
    // whole journeys in near order: the key packing writes every word to its place
    const bool grouped = near && n_shards <= 1 && m->n_runs == J && p0 == 0 && !m->overflow && !m->range_err &&
                         !pay_packed(m, n);
    m->grouped = grouped;
    m->sort_bits = grouped ? 0u : kb;
    m->passes = m->sort_bits == 0 ? 0u : (kb <= w0 ? 1u : 1u + (kb - w0 + RADIX_BITS - 1) / RADIX_BITS);
    if (!res) return;
    cv_result r = {};
    r.status = m->range_err ? CV_ERR_RANGE : (m->overflow ? CV_ERR_CAPACITY : CV_OK);
    r.count = J;
    r.required = m->overflow ? J : 0;
    r.key_bits = kb;
    r.packed_pass = p0;
    r.flags = w0;  // bits of the first radix digit
    *res = r;
}

// The insert's per-block parts joined, then the key's layout from `ids` distinct
// ids (a whole block of B threads).
template <int B>
__device__ __forceinline__ void dict_settle(SortMeta* m, const InsPart* __restrict__ parts, u32 nparts, u32 ids,
                                            u32 max_j, u32 n, u32 n_shards, u32 allow_wide, cv_result* res)
{
    __shared__ InsPart s_part[B / WAVE];
    InsPart p{~0ull, 0, 0, 0, 0, 0, 0};
    for (u32 i = threadIdx.x; i < nparts; i += B) part_join(p, parts[i]);
    part_wave_join(p);
    if (lane_id() == 0) s_part[threadIdx.x / WAVE] = p;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < B / WAVE; ++k) part_join(p, s_part[k]);
    m->tmin_ord = p.lo;
    m->tmax_ord = p.hi;
    m->t_or = p.tor;
    m->t_nd5 = p.nd5;
    m->n_runs = p.runs;
    m->unordered = p.down & PD_DOWN;
    m->multi_shard = p.multi;
    dict_meta(m, ids, max_j, n, n_shards, allow_wide, !(p.down & PD_FAR), res);
}

// The dictionary's ids to a list (any order), with their slots' second words
// (batched: the ids' shards, else their runs), by their bits in `used` (nullable) or
// from the table.  Each thread takes `per` slots per round, so that a round's one claim
// of list places (atomics on one word, which serialise) covers 256 times as many.
// Large tables are mostly empty (a push allows for an id per record): 4 M slots take
// 74 us from the table, 31 by the bits, 512 k 20 and 10, and a serving session of
// eight pushes went from 3062 to 2829 us.  Small ones are up to half full: setting
// the bits costs as much as they save, and 16 slots to a thread 3 us more than 4.
// (16 slots of a table without bits are 256 bytes per thread: where the bits were kept
// only for tables that the records' key words could hold the bits of, 10 000 records
// with 16 M ids allowed took 681 us to sort, 249 with bits.)
constexpr u64 USED_MIN = 1u << 18;  // slots from which the bits are kept
inline __host__ __device__ u32 compact_slots(u64 slots) { return slots >= USED_MIN ? 16u : 4u; }
__global__ void __launch_bounds__(256) k_dict_compact(u64* __restrict__ table, u64 slots, u32 max_j,
                                                      SortMeta* m, u64* __restrict__ list, u64* __restrict__ tag,
                                                      const InsPart* __restrict__ parts, u32 nparts, u32 n,
                                                      u32 n_shards, u32 allow_wide, cv_result* res,
                                                      const u32* __restrict__ used)
{
    __shared__ u32 s_t[256 / WAVE];
    __shared__ u32 s_base;
    const u32 hm = m->has_min;
    if (blockIdx.x == 0 && threadIdx.x == 0 && hm && max_j > 0) {
        list[0] = EMPTY ^ SIGN;
        tag[0] = n_shards > 1 ? 0ull : ((u64)m->min_start << 32) | m->min_end;
    }
    const ulonglong2* t2 = (const ulonglong2*)table;
    const u32 per = compact_slots(slots);
    const u64 stride = (u64)gridDim.x * 256;
    for (u64 b = (u64)blockIdx.x * 256; b < slots / per; b += stride) {
        const u64 s0 = (b + threadIdx.x) * per;
        u32 mask = 0;
        if (s0 < slots) {
            if (used) {
                mask = (used[s0 / 32] >> (s0 % 32)) & ((1u << per) - 1u);
            } else {
                for (u32 q = 0; q < per; ++q) mask |= table[2 * (s0 + q)] != EMPTY ? 1u << q : 0u;
            }
        }
        u32 tot;
        const u32 ex = block_exclusive_sum<256>((u32)__popc(mask), s_t, tot);
        if (threadIdx.x == 0) s_base = tot ? atomicAdd(&m->list_count, tot) : 0u;
        __syncthreads();
        u32 pos = s_base + ex + hm;
        for (; mask; mask &= mask - 1) {
            const u64 sl = s0 + (u32)__ffs((int)mask) - 1;
            const ulonglong2 e = t2[sl];
            if (pos < max_j) {
                list[pos] = e.x ^ SIGN;
                tag[pos] = e.y;
            } else if (n_shards <= 1) {
                table[2 * sl + 1] = 0;  // an id beyond the capacity gets no rank: 0
            }
            ++pos;
        }
        __syncthreads();
    }
    // the last block to end settles the key (a launch less than a kernel of its own)
    if (threadIdx.x == 0) {
        __threadfence();
        s_base = atomicAdd(&m->blocks_done, 1u);
    }
    __syncthreads();
    if (s_base != gridDim.x - 1) return;
    __threadfence();
    dict_settle<256>(m, parts, nparts, atomicAdd(&m->list_count, 0u) + hm, max_j, n, n_shards, allow_wide,
                     res);
}

// writes rank r of the id (image) into its slot; the word that was there (the
// id's run in the plain form) goes to runs[r] (nullable)
__device__ __forceinline__ void dict_set_rank(u64* __restrict__ table, u64 mask, u64 image, u32 r, const SortMeta* m,
                                              u64* __restrict__ runs)
{
    const u64 k = image ^ SIGN;
    if (k == EMPTY) {  // INT64_MIN has no slot
        if (runs) runs[r] = ((u64)m->min_start << 32) | m->min_end;
        return;
    }
    const u64 slot = dict_find(table, mask, k);
    if (slot == ~0ull) return;
    if (runs) runs[r] = table[2 * slot + 1];
    table[2 * slot + 1] = r;
}

// Up to DS_COUNT distinct ids: their order into out, their ranks into the table;
// grouped input: where each journey's records go, as the difference to where
// its run lies, into delta (by rank).
template <bool SH>
__global__ void __launch_bounds__(DS_B) k_dict_count(const SortMeta* m, u64* __restrict__ table, u64 mask,
                                                     const u64* __restrict__ list, const u64* __restrict__ tag,
                                                     u64* __restrict__ out, u32* __restrict__ delta)
{
    const u32 n = m->dict_n;
    if (n > DS_COUNT) return;
    if (!SH && m->grouped) {
        ds_count_runs(list, tag, n, [&](u32 r, u64 id, u32 before, u64 run) {
            out[r] = id;
            delta[r] = before - run_start(run);
            dict_set_rank(table, mask, id, r, m, nullptr);
        });
        return;
    }
    ds_count<SH>(list, tag, n, SH && m->multi_shard, [&](u32 r, u64 id) {
        out[r] = id;
        dict_set_rank(table, mask, id, r, m, nullptr);
    });
}

// Grouped input of more than DS_COUNT ids: the same difference for every
// rank from the journeys' runs.  A block takes a contiguous range of ranks; the
// blocks before it (by ticket, so they run) leave their ranges' record counts in
// `sums`, which one wave reads together.
constexpr int OFF_BLOCKS = WAVE;
__global__ void __launch_bounds__(256) k_run_offsets(SortMeta* m, const u64* __restrict__ runs, u64* __restrict__ sums,
                                                     u32* __restrict__ delta)
{
    const u32 n = m->big_n;
    if (n == 0 || !m->grouped) return;
    __shared__ u32 s_tmp[256 / WAVE];
    __shared__ u32 s_b;
    if (threadIdx.x == 0) s_b = atomicAdd(&m->t_off, 1u);
    __syncthreads();
    const u32 b = s_b;
    const u32 per = (n + OFF_BLOCKS - 1) / OFF_BLOCKS;
    const u64 lo = (u64)b * per;
    const u32 a = lo < n ? (u32)lo : n, e = lo + per < n ? (u32)(lo + per) : n;
    u32 c = 0, tot;
    for (u32 r = a + threadIdx.x; r < e; r += 256) c += run_length(runs[r]);
    block_exclusive_sum<256>(c, s_tmp, tot);
    if (threadIdx.x == 0) lb_publish(&sums[b], LB_AGG | tot);
    u64 w = LB_AGG;
    if (lane_id() < (int)b) {
        while (((w = lb_peek(&sums[lane_id()])) & ~LB_VAL) == 0) __builtin_amdgcn_s_sleep(1);
    }
    const u32 got = wave_inclusive_sum((u32)(w & LB_VAL));
    u32 base = (u32)__builtin_amdgcn_readlane((int)got, WAVE - 1);
    for (u32 q = a; q < e; q += 256) {  // (the same trips in every thread)
        const u32 r = q + threadIdx.x;
        const u64 run = r < e ? runs[r] : 0ull;
        const u32 x = block_exclusive_sum<256>(run_length(run), s_tmp, tot);
        if (r < e) delta[r] = base + x - run_start(run);
        base += tot;
    }
}

// A step of the chunks' join (cv_dictsort.h); the last one also writes the ranks.
template <bool SH, bool LAST>
__global__ void __launch_bounds__(256) k_dict_join(const SortMeta* m, u64* __restrict__ table, u64 mask,
                                                   const u64* __restrict__ in, const u64* __restrict__ tin, u32 run,
                                                   u64* __restrict__ out, u64* __restrict__ tout,
                                                   u64* __restrict__ runs)
{
    const u32 n = m->big_n;
    ds_join<SH>(in, tin, n, run, out, tout, [&](u32 r, u64 id) {
        if (LAST) dict_set_rank(table, mask, id, r, m, runs);
    });
}

// Batched form, after the distinct ids are sorted: each id's shard (its slot's
// tag) as the key of a stable sort that brings the list into (shard, id)
// order; 0 for every id when an id lies in several shards, so that the list
// keeps id order.
__global__ void __launch_bounds__(256) k_dict_shardkey(const u64* __restrict__ sorted_list, const SortMeta* m,
                                                       const u64* __restrict__ table, u64 mask, u64* __restrict__ skey)
{
    const u32 dn = m->big_n;
    const bool multi = m->multi_shard != 0;
    for (u32 r = blockIdx.x * blockDim.x + threadIdx.x; r < dn; r += gridDim.x * blockDim.x) {
        const u64 k = sorted_list[r] ^ SIGN;
        u64 sh = 0;
        if (!multi && k != EMPTY) {
            const u64 slot = dict_find(table, mask, k);
            sh = slot != ~0ull ? table[2 * slot + 1] : 0ull;
        }
        skey[r] = sh;
    }
}

// Batched form: the list in (shard, id) order (perm: the stable sort's order of
// the id-sorted list) and each id's rank, its position in that order.
__global__ void __launch_bounds__(256) k_dict_final(const u64* __restrict__ sorted_list, const u32* __restrict__ perm,
                                                    const SortMeta* m, u64* __restrict__ table, u64 mask,
                                                    u64* __restrict__ final_list)
{
    const u32 dn = m->big_n;
    for (u32 r = blockIdx.x * blockDim.x + threadIdx.x; r < dn; r += gridDim.x * blockDim.x) {
        const u64 v = sorted_list[perm[r]];
        final_list[r] = v;
        dict_set_rank(table, mask, v, r, m, nullptr);
    }
}

__global__ void __launch_bounds__(256) k_dict_rank(const u64* __restrict__ sorted_list, const SortMeta* m,
                                                   u64* __restrict__ table, u64 mask, u64* __restrict__ out,
                                                   u64* __restrict__ runs)
{
    u32 dn = m->big_n;
    for (u32 r = blockIdx.x * blockDim.x + threadIdx.x; r < dn; r += gridDim.x * blockDim.x) {
        out[r] = sorted_list[r];
        dict_set_rank(table, mask, sorted_list[r], r, m, runs);
    }
}

// Waves walk contiguous windows of 64 records, so the journey-rank digits of a
// window are usually equal in every lane: such a digit is counted with one LDS
// add instead of 64 colliding ones.
// Each wave walks its own contiguous range of windows of 64 records, PW
// windows per round with their ids and times loaded together; the (id, rank)
// of a window's last record carries into the next window, so the dictionary
// is probed only where a run of equal ids starts, and the shard (batched form)
// is followed forward from the range's first one.  SHARDS = false compiles the
// plain form without the shard search.
// One input record's payload, packed (the form that gathers of every column read
// of interleaved input).
struct __attribute__((aligned(32))) PayRec {
    i64 ts;
    double lat, lon;
    float spd;
    u32 pad;
};

// rank of `key` continuing a probe sequence at slot h, whose entry e was read
__device__ __forceinline__ u32 dict_rank_from(const u64* table, u64 mask, u64 key, u64 h, ulonglong2 e)
{
    const ulonglong2* t2 = (const ulonglong2*)table;
    for (u64 probe = 0; probe <= mask; ++probe) {
        if (e.x == key) return (u32)e.y;
        if (e.x == EMPTY) return 0u;
        h = (h + 1) & mask;
        e = t2[h];
    }
    return 0u;
}

constexpr int PW = 8;

// Grouped input: every key word straight to its place in the sorted order.
// Pairs out of order at distance d are one lane mask per window (the same
// 32-bit differences as in the insert's check), and a record moves up by the
// pairs it is the later of and down by those it is the earlier of.  One read of
// the ids and times and one write of the words: 123 M records in 650 us, 4.6 TB/s.
__device__ __forceinline__ void pack_grouped(const i64* __restrict__ jid, const i64* __restrict__ ts, u32 n,
                                             const u64* __restrict__ table, u64 mask, const SortMeta* m,
                                             const u32* __restrict__ delta, u64* __restrict__ keys)
{
    const u32 tb = m->t_bits, ib = m->ib;
    const bool tdrop = m->ts_dropped != 0;
    const u64 tmin = (u64)unord_i64(m->tmin_ord);
    const u32 tsh = m->t_sh, tp5 = m->t_p5;
    const int l = lane_id();
    const u64 nw = (u64)gridDim.x * (blockDim.x / WAVE);
    const u64 nwin = ((u64)n + WAVE - 1) / WAVE;
    const u64 per = ((nwin + nw - 1) / nw + PW - 1) / PW * PW;  // windows per wave, whole rounds
    const u64 wbeg = ((u64)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE) * per;
    const u64 wend = wbeg + per < nwin ? wbeg + per : nwin;
    if (wbeg >= wend) return;
    // the window before: its last id, times and run starts
    i64 cj = 0;
    u32 pt = 0;
    u64 hp = 1;
    if (wbeg > 0) {
        const u64 i = (wbeg - 1) * WAVE + l;
        const i64 j = jid[i];
        const i64 jb = lane_below(j);
        pt = (u32)ts[i];
        hp = __ballot(j != jb);
        cj = lane_last(j);
    }
    u32 cr = 0, cd = 0;  // rank and difference of the run that a window goes on with
    bool fresh = true;   // not known yet
    for (u64 w0 = wbeg; w0 < wend; w0 += PW) {
        i64 jv[PW + 1], tv[PW + 1];
#pragma unroll
        for (int k = 0; k <= PW; ++k) {
            const u64 i = (w0 + k) * WAVE + l;
            const u64 c = i < n ? i : (u64)n - 1;  // past the end: a valid record, not used
            if (k < PW || l < JW) {
                jv[k] = jid[c];
                tv[k] = ts[c];
            } else {
                jv[k] = tv[k] = 0;
            }
        }
        u64 mc[JW], mn[JW];  // pairs out of order: this window's, the next one's
        u64 hc = 0;          // this window's run starts
#pragma unroll
        for (int d = 0; d < JW; ++d) mc[d] = mn[d] = 0;
#pragma unroll
        for (int k = 0; k <= PW; ++k) {
            // window k's run starts and pairs (past the end: starts)
            const u64 i = (w0 + k) * WAVE + l;
            const i64 jb = lane_below(jv[k], cj);
            const u64 h = __ballot(i == 0 || i >= n || jv[k] != jb);
            const u32 x = (u32)tv[k];
            RunMask rm(h, hp);
            u32 y = x;
#pragma unroll
            for (int d = 1; d <= JW; ++d) {
                y = lane_below(y, (u32)__builtin_amdgcn_readlane((int)pt, WAVE - d));
                mn[d - 1] = __ballot((int)(x - y) < 0) & rm.next();
            }
            if (k > 0) {
                // place window k - 1
                const u64 io = (w0 + k - 1) * WAVE + l;
                const u64 look = hc | (fresh ? 1ull : 0ull);
                u32 r = cr, dl = cd;
                if (look) {
                    if (((look >> l) & 1ull) && io < n) {
                        r = dict_rank_of(table, mask, (u64)jv[k - 1]);
                        dl = delta[r];
                    }
                    const u64 upto = look & (~0ull >> (63 - l));
                    const int src = upto ? 63 - __clzll((long long)upto) : 0;
                    const u32 rs = __shfl(r, src, WAVE), ds = __shfl(dl, src, WAVE);
                    r = upto ? rs : cr;
                    dl = upto ? ds : cd;
                    cr = (u32)__builtin_amdgcn_readlane((int)r, WAVE - 1);
                    cd = (u32)__builtin_amdgcn_readlane((int)dl, WAVE - 1);
                    fresh = false;
                }
                u32 at = (u32)io + dl;
                u64 any = 0;
#pragma unroll
                for (int d = 0; d < JW; ++d) any |= mc[d] | (mn[d] << (WAVE - 1 - d));
                if (any) {
#pragma unroll
                    for (int d = 0; d < JW; ++d) {
                        at -= (u32)(mc[d] >> l) & 1u;
                        at += (u32)(((mc[d] >> (d + 1)) | (mn[d] << (WAVE - 1 - d))) >> l) & 1u;
                    }
                }
                if (io < n && at < n) {
                    const u64 key = tdrop ? (u64)r
                                          : ((tb >= 64 ? 0ull : ((u64)r << tb)) |
                                             time_offset((u64)tv[k - 1] - tmin, tsh, tp5));
                    keys[at] = (key << ib) | io;
                }
            }
            if (k < PW) {
                hc = h;
                hp = h;
                pt = x;
                cj = lane_last(jv[k]);
#pragma unroll
                for (int d = 0; d < JW; ++d) mc[d] = mn[d];
            }
        }
    }
}

// Keys of every record with the digit histograms of every pass, for input in
// long runs of equal ids: each wave walks its own contiguous range of windows
// of 64 records, PW windows per round with their ids and times loaded
// together; the (id, rank) of a window's last record carries into the next
// window, so the dictionary is probed only where a run of equal ids starts
// (through the wave's cache), and the shard (batched form) is followed
// forward from the range's first one.  Returns at once for interleaved input
// (k_pack_il takes it).
template <bool SHARDS>
__global__ void __launch_bounds__(256) k_pack_hist(const i64* __restrict__ jid, const i64* __restrict__ ts, u32 n,
                                                   const u64* __restrict__ table, u64 mask, SortMeta* m,
                                                   u64* __restrict__ keys, u32* __restrict__ hist,
                                                   const u64* __restrict__ soff, u32 S, const u32* __restrict__ delta)
{
    __shared__ u32 s_h[HIST_WIDE_WORDS];  // digit counts, wide layout (first digit w0 bits)
    // per-wave cache of (id, rank) pairs, as in the dictionary insert
    __shared__ u64 c_key[4][DCH];
    __shared__ u32 c_rank[4][DCH], c_own[4][DCH];
    if (pay_packed(m, n)) return;
    if (!SHARDS && m->grouped) {
        pack_grouped(jid, ts, n, table, mask, m, delta, keys);
        return;
    }
    for (int i = threadIdx.x; i < HIST_WIDE_WORDS; i += blockDim.x) s_h[i] = 0;
    for (int i = threadIdx.x; i < 4 * DCH; i += blockDim.x) (&c_key[0][0])[i] = EMPTY;
    __syncthreads();
    const int wv_ = threadIdx.x / WAVE;
    const u32 tb = m->t_bits;
    const bool tdrop = m->ts_dropped != 0;
    const u32 np = m->passes;
    const u32 fdb = m->w0 == RADIX_BITS + 1 ? RADIX_BITS + 1 : RADIX_BITS;  // first digit bits
    const bool bad = m->range_err != 0;
    const u32 ib = m->ib;
    const bool packed = m->p0 == 0;
    const u64 tmin = (u64)unord_i64(m->tmin_ord);
    const u32 tsh = m->t_sh, tp5 = m->t_p5;
    const int l = lane_id();
    const u64 nw = (u64)gridDim.x * (blockDim.x / WAVE);
    const u64 nwin = ((u64)n + WAVE - 1) / WAVE;
    const u64 per = ((nwin + nw - 1) / nw + PW - 1) / PW * PW;  // windows per wave, whole rounds
    const u64 wbeg = ((u64)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE) * per;
    const u64 wend = wbeg + per < nwin ? wbeg + per : nwin;
    // id and rank of the previous window's last record
    bool hc = false;
    u64 cj = 0;
    u32 cr = 0;
    // shard of the current window's first record (batched form; wave-uniform)
    u32 shw = (SHARDS && wbeg < wend) ? shard_of(soff, S, wbeg * WAVE) : 0u;
    for (u64 w0 = wbeg; w0 < wend; w0 += PW) {
        u64 jv[PW], tv[PW];
#pragma unroll
        for (int k = 0; k < PW; ++k) {
            u64 i = (w0 + k) * WAVE + l;
            i = i < n ? i : (u64)n - 1;  // past the end: a valid record, not used
            jv[k] = (u64)jid[i];
            tv[k] = (u64)ts[i];
        }
#pragma unroll
        for (int k = 0; k < PW; ++k) {
            const u64 wi = w0 + k;
            if (wi >= wend) break;
            const u64 i = wi * WAVE + l;
            const bool valid = i < n;
            // only the first lane of each run of equal ids probes the dictionary;
            // the others take its rank (lane 0 continues the carried run)
            const u64 j = valid ? jv[k] : EMPTY;
            const u64 jp = lane_below(j);
            const bool runhead = l == 0 ? !(hc && j == cj) : j != jp;
            u32 r = 0;
            const bool look = valid && runhead && j != EMPTY;
            const u32 cs = dict_cache_slot<DCH>(j);
            bool miss = false;
            if (look) {
                if (c_key[wv_][cs] == j) {
                    r = c_rank[wv_][cs];
                } else {
                    r = dict_rank_of(table, mask, j);
                    miss = true;
                }
            }
            if (miss) c_own[wv_][cs] = (u32)l;
            __builtin_amdgcn_wave_barrier();
            if (miss && c_own[wv_][cs] == (u32)l) {
                c_key[wv_][cs] = j;
                c_rank[wv_][cs] = r;
            }
            __builtin_amdgcn_wave_barrier();
            const u64 heads = __ballot(runhead);
            const u64 upto = heads & (~0ull >> (63 - l));  // run starts at or below this lane
            const u32 rh = __shfl(r, upto ? 63 - __clzll((long long)upto) : 0, WAVE);
            r = upto ? rh : cr;
            cj = __shfl(j, WAVE - 1, WAVE);
            cr = __shfl(r, WAVE - 1, WAVE);
            hc = true;
            u64 key = 0;
            if (valid) {
                if (!bad) {
                    key = tdrop ? (u64)r : ((tb >= 64 ? 0ull : ((u64)r << tb)) | time_offset(tv[k] - tmin, tsh, tp5));
                    if (SHARDS && m->shard_bits) {
                        // the window's first shard, then forward to this record's
                        shw = __builtin_amdgcn_readfirstlane(shard_from(soff, S, shw, wi * WAVE));
                        const u32 sh = shard_from(soff, S, shw, i);
                        key |= (u64)sh << (m->rank_bits + tb);
                    }
                }
                keys[i] = packed ? ((key << ib) | i) : key;
            }
            const u64 vm = __ballot(valid);
            const int lead = __ffsll((long long)vm) - 1;
            for (u32 p = 0; p < np; ++p) {
                const u32 lo = p ? fdb + (p - 1) * RADIX_BITS : 0u;
                const u32 d = (u32)(key >> lo) & ((p ? RADIX : 1u << fdb) - 1u);
                u32* hp = s_h + hist_wide_off((int)p);
                const u32 d0 = __shfl(d, lead, WAVE);
                if (__ballot(valid && d != d0) == 0) {
                    if (l == lead) atomicAdd(&hp[d0], (u32)__popcll(vm));
                } else if (valid) {
                    atomicAdd(&hp[d], 1u);
                }
            }
        }
    }
    __syncthreads();
    for (u32 i = threadIdx.x; i < (u32)HIST_WIDE_WORDS; i += blockDim.x)
        if (s_h[i]) atomicAdd(&hist[i], s_h[i]);
}

// Keys and digit histograms for interleaved input (short runs of equal ids, as
// in a time-ordered feed), where nearly every record probes the dictionary:
// every block takes a contiguous range of tiles of PT records, and each
// record's first probe is issued with the tile's others before any is used.
// With `pay` (gathers of every column), the tile's records are also regrouped
// by the low byte of their journey rank (a stable local multisplit, so equal
// keys keep their input order): the key words and the packed payloads go to
// the regrouped positions, and each payload carries its input index.  After
// the sort, consecutive records of a journey then read consecutive payloads
// of each tile instead of one cache line per record.
constexpr int PT_B = 1024;               // threads per block (tiles of 4 096 records: half the per-tile scans and barriers of 2 048)
// Records per thread: fewer where tiles of 4 096 would leave most CUs without one
// (the whole preparation of 30 000 shuffled records with 1, 2 and 4: 37, 41 and 46 us;
// 125 000: 45, 48, 54; 250 000: 59, 57, 62; 500 000: 83, 81, 87; 1 M: 137, 132, 120).
inline int pack_items(u64 n) { return n <= (1u << 17) ? 1 : n <= (1u << 19) ? 2 : 4; }
template <bool SHARDS, int PT_I>
__global__ void __launch_bounds__(PT_B) k_pack_il(const i64* __restrict__ jid, const i64* __restrict__ ts,
                                                 const double* __restrict__ lat, const double* __restrict__ lon,
                                                 const float* __restrict__ spd, PayRec* __restrict__ pay, u32 n,
                                                 const u64* __restrict__ table, u64 mask, SortMeta* m,
                                                 u64* __restrict__ keys, u32* __restrict__ hist,
                                                 const u64* __restrict__ soff, u32 S)
{
    constexpr int PT = PT_B * PT_I;  // records per tile
    constexpr int NW = PT_B / WAVE;
    __shared__ u32 s_h[HIST_WIDE_WORDS];  // digit counts, wide layout (first digit w0 bits)
    __shared__ u64 c_key[NW][DCP];
    __shared__ u32 c_rank[NW][DCP], c_own[NW][DCP];
    __shared__ uint16_t s_whist[NW][RADIX];  // per-wave digit counts, then offsets
    __shared__ u32 s_start[RADIX];
    __shared__ u32 s_tmp[NW];
    if (!pay_packed(m, n)) return;
    for (int i = threadIdx.x; i < HIST_WIDE_WORDS; i += blockDim.x) s_h[i] = 0;
    for (int i = threadIdx.x; i < NW * DCP; i += blockDim.x) (&c_key[0][0])[i] = EMPTY;
    const int w = threadIdx.x / WAVE;
    const int l = lane_id();
    const u32 tb = m->t_bits;
    const bool tdrop = m->ts_dropped != 0;
    const u32 np = m->passes;
    const u32 fdb = m->w0 == RADIX_BITS + 1 ? RADIX_BITS + 1 : RADIX_BITS;  // first digit bits
    const bool bad = m->range_err != 0;
    const u32 ib = m->ib;
    const bool packed = m->p0 == 0;
    const bool group = pay != nullptr;
    const u32 rbits = m->rank_bits;
    const u32 sbits = m->shard_bits;  // 0: the ranks keep the shards apart
    // without time bits the first digit of a key is the low byte of its rank,
    // which the regrouping counts per tile: that pass's histogram is added
    // from those counts, one add per digit and tile
    const u32 p_first = (group && tdrop && !bad && rbits >= (u32)RADIX_BITS && np > 0 && fdb == RADIX_BITS) ? 1u : 0u;
    const u64 tmin = (u64)unord_i64(m->tmin_ord);
    const u32 tsh = m->t_sh, tp5 = m->t_p5;
    const ulonglong2* t2 = (const ulonglong2*)table;
    const u64 tiles = ((u64)n + PT - 1) / PT;
    const u64 per = (tiles + gridDim.x - 1) / gridDim.x;
    const u64 tb0 = (u64)blockIdx.x * per;
    const u64 tb1 = tb0 + per < tiles ? tb0 + per : tiles;
    u32 shw = (SHARDS && tb0 < tb1) ? shard_of(soff, S, tb0 * PT) : 0u;
    for (u64 tile = tb0; tile < tb1; ++tile) {
        const u64 base = tile * PT + (u64)w * (PT_I * WAVE);  // this wave's records
        for (int i = l; i < RADIX; i += WAVE) s_whist[w][i] = 0;
        __syncthreads();
        u64 jv[PT_I], tv[PT_I];
        double la[PT_I], lo[PT_I];
        float sp[PT_I];
#pragma unroll
        for (int k = 0; k < PT_I; ++k) {
            u64 i = base + (u64)k * WAVE + l;
            i = i < n ? i : (u64)n - 1;  // past the end: a valid record, not used
            jv[k] = (u64)jid[i];
            tv[k] = (u64)ts[i];
            if (group) {
                la[k] = lat[i];
                lo[k] = lon[i];
                sp[k] = spd[i];
            }
        }
        // ranks: the wave's cache, else the first probe of every miss issued together
        u32 rk[PT_I];
        bool miss[PT_I];
        u64 ph[PT_I];
        ulonglong2 pe[PT_I];
#pragma unroll
        for (int k = 0; k < PT_I; ++k) {
            const u64 i = base + (u64)k * WAVE + l;
            const u64 j = jv[k];
            const bool look = i < n && j != EMPTY;  // the INT64_MIN id has rank 0
            const u32 cs = dict_cache_slot<DCP>(j);
            rk[k] = 0;
            miss[k] = false;
            if (look) {
                if (c_key[w][cs] == j) rk[k] = c_rank[w][cs];
                else miss[k] = true;
            }
            ph[k] = mix64(j) & mask;
            if (miss[k]) pe[k] = t2[ph[k]];
        }
#pragma unroll
        for (int k = 0; k < PT_I; ++k) {
            const u64 j = jv[k];
            const u32 cs = dict_cache_slot<DCP>(j);
            if (miss[k]) {
                rk[k] = dict_rank_from(table, mask, j, ph[k], pe[k]);
                c_own[w][cs] = (u32)l;
            }
            __builtin_amdgcn_wave_barrier();
            if (miss[k] && c_own[w][cs] == (u32)l) {
                c_key[w][cs] = j;
                c_rank[w][cs] = rk[k];
            }
            __builtin_amdgcn_wave_barrier();
        }
        // keys, histograms and the local multisplit by the rank's low byte
        u64 key[PT_I];
        u32 rnk[PT_I];
#pragma unroll
        for (int k = 0; k < PT_I; ++k) {
            const u64 i = base + (u64)k * WAVE + l;
            const bool valid = i < n;
            key[k] = 0;
            if (valid && !bad) {
                key[k] = tdrop ? (u64)rk[k] : ((tb >= 64 ? 0ull : ((u64)rk[k] << tb)) | time_offset(tv[k] - tmin, tsh, tp5));
                if (SHARDS && sbits) {
                    shw = __builtin_amdgcn_readfirstlane(shard_from(soff, S, shw, base + (u64)k * WAVE));
                    const u32 sh = shard_from(soff, S, shw, i);
                    key[k] |= (u64)sh << (rbits + tb);
                }
            }
            const u64 vm = __ballot(valid);
            const int lead = vm ? __ffsll((long long)vm) - 1 : 0;
            for (u32 p = p_first; p < np; ++p) {
                const u32 dlo = p ? fdb + (p - 1) * RADIX_BITS : 0u;
                const u32 d = (u32)(key[k] >> dlo) & ((p ? RADIX : 1u << fdb) - 1u);
                u32* hp = s_h + hist_wide_off((int)p);
                const u32 d0 = __shfl(d, lead, WAVE);
                if (__ballot(valid && d != d0) == 0) {
                    if (l == lead && vm) atomicAdd(&hp[d0], (u32)__popcll(vm));
                } else if (valid) {
                    atomicAdd(&hp[d], 1u);
                }
            }
            rnk[k] = 0;
            if (group) {
                const u32 d = rk[k] & (RADIX - 1);
                const u64 peers = wave_peers<RADIX_BITS>(d, vm);
                const u32 below = popc_below(peers);
                const u32 cnt = (u32)__popcll(peers);
                const u32 before = valid ? (u32)s_whist[w][d] : 0u;
                rnk[k] = before + below;
                __builtin_amdgcn_wave_barrier();
                if (valid && below == cnt - 1) s_whist[w][d] = (uint16_t)(before + cnt);
                __builtin_amdgcn_wave_barrier();
            }
        }
        if (group) {
            __syncthreads();
            // per digit: offsets of the waves, and the tile's digit starts
            u32 tcount = 0;
            if (threadIdx.x < RADIX) {
                const int d = threadIdx.x;
#pragma unroll
                for (int ww = 0; ww < NW; ++ww) {
                    const u32 c = s_whist[ww][d];
                    s_whist[ww][d] = (uint16_t)tcount;
                    tcount += c;
                }
            }
            if (p_first && threadIdx.x < RADIX && tcount) s_h[threadIdx.x] += tcount;
            u32 total;
            const u32 st = block_exclusive_sum<PT_B>(threadIdx.x < RADIX ? tcount : 0u, s_tmp, total);
            if (threadIdx.x < RADIX) s_start[threadIdx.x] = st;
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < PT_I; ++k) {
            const u64 i = base + (u64)k * WAVE + l;
            if (i >= n) continue;
            u64 at = i;
            if (group) {
                const u32 d = rk[k] & (RADIX - 1);
                at = tile * PT + s_start[d] + s_whist[w][d] + rnk[k];
                ulonglong2* q = (ulonglong2*)(pay + at);
                q[0] = make_ulonglong2(tv[k], (u64)__double_as_longlong(la[k]));
                q[1] = make_ulonglong2((u64)__double_as_longlong(lo[k]), (u64)__float_as_uint(sp[k]) | (i << 32));
            }
            keys[at] = packed ? ((key[k] << ib) | at) : key[k];
        }
        __syncthreads();
    }
    __syncthreads();
    for (u32 i = threadIdx.x; i < (u32)HIST_WIDE_WORDS; i += blockDim.x)
        if (s_h[i]) atomicAdd(&hist[i], s_h[i]);
}

// The final words are packed: (key >> 8 p0) << ib | source index.  Every
// thread takes GU records a grid stride apart per round, their loads issued
// together.  SHARDS = false compiles the plain form without the shard search;
// FULL = true is the form for callers that want every sorted column; of
// interleaved input it reads the packed payloads, one line per record instead of
// one per column (the whole sort of 2 M records in time order: 292 -> 208 us, of
// 20 M 2355 -> 1622, of 50 000 46 -> 46).
constexpr int GU = 4;
template <bool SHARDS, bool FULL>
__global__ void __launch_bounds__(256) k_gather(u32 n, const SortMeta* m, const u64* __restrict__ K0,
                                                const u64* __restrict__ K1, const u64* __restrict__ dict_sorted,
                                                const i64* __restrict__ jid, const i64* __restrict__ ts,
                                                const double* __restrict__ lat, const double* __restrict__ lon,
                                                const float* __restrict__ spd, u32* __restrict__ perm,
                                                i64* __restrict__ o_jid, i64* __restrict__ o_ts,
                                                double* __restrict__ o_lat, double* __restrict__ o_lon,
                                                float* __restrict__ o_spd, const u64* __restrict__ soff, u32 S,
                                                const PayRec* __restrict__ pay)
{
    const u32 np = m->passes;
    const u32 tb = m->t_bits;
    const u32 rb = m->rank_bits;
    const u32 ib = m->ib;
    const u32 drop = m->p0 * RADIX_BITS;
    const u64 rmask = rb >= 64 ? ~0ull : ((1ull << rb) - 1);
    const u64 imask = (1ull << ib) - 1;
    const u32 dn = m->dict_n;
    const bool exact = (m->range_err == 0) && (m->overflow == 0);
    // the journey rank survives packing when its bits lie above the dropped digits
    const bool rank_in_key = exact && drop <= tb;
    const u32 rshift = ib + tb - drop;
    // the time offset survives only when nothing was dropped (and the key had it)
    const bool ts_in_key = exact && drop == 0 && !m->ts_dropped;
    const u64 tmin = (u64)unord_i64(m->tmin_ord);
    const u64 tmask = tb >= 64 ? ~0ull : ((1ull << tb) - 1);
    const u64 tdiv = ((u64)m->t_p5) << m->t_sh;  // the time offset's unit
    const u64* K = (np & 1) ? K1 : K0;
    const bool packed = FULL && pay_packed(m, n);  // the sort's index is a payload's place
    const u32 stride = gridDim.x * blockDim.x;
    for (u32 k0 = blockIdx.x * blockDim.x + threadIdx.x; k0 < n; k0 += GU * stride) {
        u64 wv[GU];
        u32 vv[GU];
#pragma unroll
        for (int u = 0; u < GU; ++u) {
            const u32 k = k0 + u * stride;
            wv[u] = K[k < n ? k : n - 1];  // past the end: a valid word, not stored
        }
#pragma unroll
        for (int u = 0; u < GU; ++u) {
            // (input that changes under the call may leave a word of grouped input unwritten)
            const u32 v = (u32)(wv[u] & imask);
            vv[u] = v < n ? v : n - 1;
        }
        if constexpr (FULL) {
            // every column requested: all gathers issued before the first store
            double ola[GU], olo[GU];
            float osp[GU];
            i64 oj[GU], ot[GU], pts[GU];
            if (packed) {
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    const ulonglong2* q = (const ulonglong2*)(pay + vv[u]);
                    const ulonglong2 a = q[0], b = q[1];
                    pts[u] = (i64)a.x;
                    ola[u] = __longlong_as_double((long long)a.y);
                    olo[u] = __longlong_as_double((long long)b.x);
                    osp[u] = __uint_as_float((u32)b.y);
                    vv[u] = (u32)(b.y >> 32);
                }
            } else {
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    ola[u] = lat[vv[u]];
                    olo[u] = lon[vv[u]];
                    osp[u] = spd[vv[u]];
                }
            }
            if (rank_in_key) {
#pragma unroll
                for (int u = 0; u < GU; ++u) {
                    u64 r = rshift >= 64 ? 0ull : ((wv[u] >> rshift) & rmask);
                    r = r < dn ? r : dn - 1;
                    oj[u] = (i64)(dict_sorted[r] ^ SIGN);
                }
            } else {
#pragma unroll
                for (int u = 0; u < GU; ++u) oj[u] = jid[vv[u]];
            }
            if (ts_in_key) {
#pragma unroll
                for (int u = 0; u < GU; ++u) ot[u] = (i64)(tmin + ((wv[u] >> ib) & tmask) * tdiv);
            } else if (packed) {
#pragma unroll
                for (int u = 0; u < GU; ++u) ot[u] = pts[u];
            } else {
#pragma unroll
                for (int u = 0; u < GU; ++u) ot[u] = ts[vv[u]];
            }
#pragma unroll
            for (int u = 0; u < GU; ++u) {
                const u32 k = k0 + u * stride;
                if (k >= n) break;
                u32 pv = vv[u];
                if (SHARDS) {
                    // a shard keeps its records: the output position and its source share the shard
                    u32 sh = shard_of(soff, S, k - threadIdx.x);  // the block row's first shard, then forward
                    while (sh + 1 < S && soff[sh + 1] <= k) ++sh;
                    pv -= (u32)soff[sh];
                }
                perm[k] = pv;
                o_jid[k] = oj[u];
                o_ts[k] = ot[u];
                o_lat[k] = ola[u];
                o_lon[k] = olo[u];
                o_spd[k] = osp[u];
            }
        } else {
#pragma unroll
            for (int u = 0; u < GU; ++u) {
                const u32 k = k0 + u * stride;
                if (k >= n) break;
                const u64 w = wv[u];
                const u32 v = vv[u];
                u32 pv = v;
                if (SHARDS) {
                    u32 sh = shard_of(soff, S, k - threadIdx.x);
                    while (sh + 1 < S && soff[sh + 1] <= k) ++sh;
                    pv = v - (u32)soff[sh];
                }
                perm[k] = pv;
                if (o_jid) {
                    const u64 r = rshift >= 64 ? 0ull : ((w >> rshift) & rmask);
                    o_jid[k] = (rank_in_key && r < dn) ? (i64)(dict_sorted[r] ^ SIGN) : jid[v];
                }
                if (o_ts) o_ts[k] = ts_in_key ? (i64)(tmin + ((w >> ib) & tmask) * tdiv) : ts[v];
                if (o_lat) o_lat[k] = lat[v];
                if (o_lon) o_lon[k] = lon[v];
                if (o_spd) o_spd[k] = spd[v];
            }
        }
    }
}

__global__ void k_passes(const SortMeta* m, u32* passes)
{
    if (threadIdx.x == 0) *passes = m->passes;
}

__global__ void k_empty_result(cv_result* res)
{
    if (threadIdx.x == 0) {
        cv_result r = {};
        *res = r;
    }
}

struct SortLayout {
    SortMeta* meta;
    u64* table;  // slots x {id, rank}
    u64* dl0;
    u64* dl1;
    u32* dv0;
    u32* dv1;
    u64* dsk0;  // batched: shard keys of the sorted distinct ids (ping-pong)
    u64* dsk1;
    u64* dlf;   // batched: the distinct ids in (shard, id) order
    u32* shist;
    u64* sstatus;
    u32* zero_begin;  // start of the region cleared to zero
    u32* hist;
    u32* dhist;
    u64* status;
    u64* dstatus;
    size_t zero_bytes;
    u64* K0;
    u64* K1;
    PayRec* pay;  // packed payload (interleaved input, fused gather)
    u32* V0;
    u32* V1;
    u64 slots;
    u64 tiles, dtiles;
    size_t bytes;

    SortLayout(void* ws, u64 n, u64 max_j)
    {
        cvh::Carver c(ws);
        slots = cvh::next_pow2(2 * max_j < 1024 ? 1024 : 2 * max_j);
        tiles = (n + sort_min_tile() - 1) / sort_min_tile();
        dtiles = (max_j + sort_min_tile() - 1) / sort_min_tile();
        meta = c.take<SortMeta>(1);
        table = c.take<u64>(2 * slots);
        dl0 = c.take<u64>(max_j);
        dl1 = c.take<u64>(max_j);
        dv0 = c.take<u32>(max_j);
        dv1 = c.take<u32>(max_j);
        dsk0 = c.take<u64>(max_j);
        dsk1 = c.take<u64>(max_j);
        dlf = c.take<u64>(max_j);
        size_t z0 = cvh::align_up(c.off);
        hist = c.take<u32>(HIST_WIDE_WORDS);  // record sort: wide layout
        dhist = c.take<u32>(MAX_PASSES * RADIX);
        shist = c.take<u32>(MAX_PASSES * RADIX);
        dstatus = c.take<u64>(dtiles * RADIX + 1);
        sstatus = c.take<u64>(dtiles * RADIX + 1);
        // last in the cleared range: room for 512 words per tile of the
        // smallest tile (a 9-bit first digit); a call clears what its shape uses
        status = c.take<u64>(tiles * 2 * RADIX + 1);
        size_t z1 = cvh::align_up(c.off);
        zero_begin = (u32*)(c.base ? c.base + z0 : nullptr);
        zero_bytes = z1 - z0;
        if (c.base) {
            const size_t zu =
                cvh::align_up((size_t)((char*)(status + sort_status_words(n, RadixCount::exact, true)) - (char*)c.base));
            zero_bytes = (zu < z1 ? zu : z1) - z0;
        }
        K0 = c.take<u64>(n);
        K1 = c.take<u64>(n);
        pay = c.take<PayRec>(n);
        V0 = c.take<u32>(n);
        V1 = c.take<u32>(n);
        bytes = c.size();
    }
};

bool valid_ptr8(const void* p) { return p == nullptr || cvh::aligned(p, 8); }

u32 bit_width_host(u64 x)
{
    u32 b = 0;
    while (x) {
        ++b;
        x >>= 1;
    }
    return b;
}

}  // namespace

namespace {

// The gather fused with the per-point kinematics of the sorted records: every
// block writes a contiguous tile of GFT sorted records and evaluates the same
// stencil as the features kernel (cv_kin.h) on them, so that the sorted
// columns are not read back from memory.  Record t0 + 64 g + l of the tile is
// lane l of group g = u * 4 + wave (u = 0, 1): its predecessor is lane l - 1
// of the same group (a lane move), or for lane 0 the last lane of group
// g - 1, which leaves it in a small LDS edge array.  Edge slot 0 holds record
// t0 - 2 and slot 1 record t0 - 1 (the tile's predecessor, whose own step
// thread 0 evaluates); group g's last record goes to slot g + 2.
constexpr int GFT = 512;
template <bool SHARDS>
__global__ void __launch_bounds__(256) k_gather_feat(u32 n, const SortMeta* m, const u64* __restrict__ K0,
                                                     const u64* __restrict__ K1, const u64* __restrict__ dict_sorted,
                                                     const i64* __restrict__ jid, const i64* __restrict__ ts,
                                                     const double* __restrict__ lat, const double* __restrict__ lon,
                                                     const float* __restrict__ spd, u32* __restrict__ perm,
                                                     cv_records_out so, cv_features fo, const u64* __restrict__ soff,
                                                     u32 S, const PayRec* __restrict__ pay)
{
    constexpr int GFI = GFT / 256;
    constexpr int NWB = 256 / WAVE;
    constexpr int NE = GFI * NWB + 2;
    __shared__ i64 e_jid[NE], e_ts[NE];
    __shared__ double e_lat[NE], e_lon[NE], e_sphi[NE], e_cphi[NE], e_v[NE], e_b[NE];
    __shared__ u32 e_f[NE];
    __shared__ u32 s_sh0;  // shard of record t0 - 2 (batched form)
    const u32 tb = m->t_bits;
    const u32 rb = m->rank_bits;
    const u32 ib = m->ib;
    const u32 drop = m->p0 * RADIX_BITS;
    const u64 rmask = rb >= 64 ? ~0ull : ((1ull << rb) - 1);
    const u64 imask = (1ull << ib) - 1;
    const u32 dn = m->dict_n;
    const bool exact = (m->range_err == 0) && (m->overflow == 0);
    const bool rank_in_key = exact && drop <= tb;
    const u32 rshift = ib + tb - drop;
    const bool ts_in_key = exact && drop == 0 && !m->ts_dropped;
    const u64 tmin = (u64)unord_i64(m->tmin_ord);
    const u64 tmask = tb >= 64 ? ~0ull : ((1ull << tb) - 1);
    const u64 tdiv = ((u64)m->t_p5) << m->t_sh;  // the time offset's unit
    const u64* K = (m->passes & 1) ? K1 : K0;
    const int t = threadIdx.x;
    const int w = t / WAVE;
    const int l = lane_id();
    const long t0 = (long)blockIdx.x * GFT;
    // slots 0 .. GFI - 1: the tile's records; slot GFI: threads 0 and 1 fetch
    // records t0 - 2 and t0 - 1 (the others repeat their first record)
    constexpr int NS = GFI + 1;
    long kk[NS];
#pragma unroll
    for (int u = 0; u < GFI; ++u) kk[u] = t0 + (long)(u * NWB + w) * WAVE + l;
    kk[GFI] = t < 2 ? t0 - 2 + t : kk[0];
    if (SHARDS && t == 0) s_sh0 = shard_of(soff, S, (u64)(t0 >= 2 ? t0 - 2 : 0));
    // the sorted words, their source indices and columns; every load from a
    // clamped index, all issued before any is used
    u64 wv[NS];
    u32 vv[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        const long k = kk[u] < 0 ? 0 : (kk[u] < (long)n ? kk[u] : (long)n - 1);
        wv[u] = K[k];
    }
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        // (input that changes under the call may leave a word of grouped input unwritten)
        const u32 v = (u32)(wv[u] & imask);
        vv[u] = v < n ? v : n - 1;
    }
    double ola[NS], olo[NS];
    float osp[NS];
    i64 oj[NS], ot[NS];
    i64 pts[NS];  // time stamps read with the packed payload
    // the input index of each sorted record: the sort's value, or, with the
    // packed payload (whose positions the key packing regrouped), the index
    // the payload carries
    u32 src[NS];
    const bool packed = pay_packed(m, n);
    if (packed) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const ulonglong2* q = (const ulonglong2*)(pay + vv[u]);
            const ulonglong2 a = q[0], b = q[1];
            pts[u] = (i64)a.x;
            ola[u] = __longlong_as_double((long long)a.y);
            olo[u] = __longlong_as_double((long long)b.x);
            osp[u] = __uint_as_float((u32)b.y);
            src[u] = (u32)(b.y >> 32);
        }
    } else {
#pragma unroll
        for (int u = 0; u < NS; ++u) src[u] = vv[u];
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            ola[u] = lat[vv[u]];
            olo[u] = lon[vv[u]];
            osp[u] = spd[vv[u]];
        }
    }
    if (rank_in_key) {
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            u64 r = rshift >= 64 ? 0ull : ((wv[u] >> rshift) & rmask);
            r = r < dn ? r : dn - 1;
            oj[u] = (i64)(dict_sorted[r] ^ SIGN);
        }
    } else {
#pragma unroll
        for (int u = 0; u < NS; ++u) oj[u] = jid[src[u]];
    }
    if (ts_in_key) {
#pragma unroll
        for (int u = 0; u < NS; ++u) ot[u] = (i64)(tmin + ((wv[u] >> ib) & tmask) * tdiv);
    } else if (packed) {
#pragma unroll
        for (int u = 0; u < NS; ++u) ot[u] = pts[u];
    } else {
#pragma unroll
        for (int u = 0; u < NS; ++u) ot[u] = ts[vv[u]];
    }
    // sin and cos of each latitude, once per point
    double osph[NS], ocph[NS];
#pragma unroll
    for (int u = 0; u < NS; ++u) {
        osph[u] = 0.0;
        ocph[u] = 0.0;
        if (isfinite(ola[u]) && isfinite(olo[u])) sincos(ola[u] * KIN_DEG2RAD, &osph[u], &ocph[u]);
    }
#pragma unroll
    for (int u = 0; u < GFI; ++u) {
        const long k = kk[u];
        if (k < (long)n) {
            if (!SHARDS) perm[k] = src[u];
            so.journey_id[k] = oj[u];
            so.ts_ms[k] = ot[u];
            so.lat_deg[k] = ola[u];
            so.lon_deg[k] = olo[u];
            so.speed_mps[k] = osp[u];
        }
        if (l == WAVE - 1) {
            const int e = u * NWB + w + 2;
            e_jid[e] = oj[u];
            e_ts[e] = ot[u];
            e_lat[e] = ola[u];
            e_lon[e] = olo[u];
            e_sphi[e] = osph[u];
            e_cphi[e] = ocph[u];
        }
    }
    if (t < 2) {
        e_jid[t] = oj[GFI];
        e_ts[t] = ot[GFI];
        e_lat[t] = ola[GFI];
        e_lon[t] = olo[GFI];
        e_sphi[t] = osph[GFI];
        e_cphi[t] = ocph[GFI];
    }
    __syncthreads();
    // shard of each record (batched form), walked forward from the tile's
    // first one: journey heads at shard starts, shard-relative source indices
    // (records before the next shard's start need no load: the block's first
    // shard and the start of the shard after it are read once)
    u32 shs[GFI];
    u64 sst[GFI];  // start of each record's shard
    {
        const u32 sh0 = SHARDS ? s_sh0 : 0u;
        const u64 st0 = SHARDS ? soff[sh0] : 0ull;
        const u64 nx0 = (SHARDS && sh0 + 1 < S) ? soff[sh0 + 1] : ~0ull;
#pragma unroll
        for (int u = 0; u < GFI; ++u) {
            shs[u] = 0;
            sst[u] = 0;
            if (SHARDS && kk[u] < (long)n) {
                const bool same = (u64)kk[u] < nx0;
                shs[u] = same ? sh0 : shard_from(soff, S, sh0, (u64)kk[u]);
                sst[u] = same ? st0 : soff[shs[u]];
                perm[kk[u]] = src[u] - (u32)sst[u];
            }
        }
    }
    // steps (k - 1 -> k) of the tile's records; thread 0 also takes the step
    // of record t0 - 1 (the first record's predecessor)
    KinStep ks[GFI];
#pragma unroll
    for (int u = 0; u < GFI; ++u) {
        const long k = kk[u];
        const int g = u * NWB + w;
        i64 pj = lane_below(oj[u]), pt = lane_below(ot[u]);
        double pla = lane_below(ola[u]), plo = lane_below(olo[u]);
        double psph = lane_below(osph[u]), pcph = lane_below(ocph[u]);
        if (l == 0) {
            pj = e_jid[g + 1];
            pt = e_ts[g + 1];
            pla = e_lat[g + 1];
            plo = e_lon[g + 1];
            psph = e_sphi[g + 1];
            pcph = e_cphi[g + 1];
        }
        bool head = k == 0 || pj != oj[u];
        if (SHARDS && !head && k < (long)n) head = sst[u] == (u64)k;
        ks[u] = kin_step(head, isfinite(ola[u]) && isfinite(olo[u]), ot[u], ola[u], olo[u], ocph[u],
                         isfinite(pla) && isfinite(plo), pt, pla, plo, pcph, psph);
        if (l == WAVE - 1) {
            const int e = g + 2;
            e_f[e] = ks[u].f;
            e_v[e] = ks[u].v;
            e_b[e] = ks[u].b;
        }
    }
    if (t == 0) {
        const long kr = t0 - 1;
        KinStep hs = KinStep{0.0, 0.0, 0.0, 0.0, 0u};
        if (kr >= 0) {
            bool head = kr == 0 || e_jid[0] != e_jid[1];
            if (SHARDS && !head) head = soff[shard_from(soff, S, s_sh0, (u64)kr)] == (u64)kr;
            const double la = e_lat[1], lo = e_lon[1], lap = e_lat[0], lop = e_lon[0];
            hs = kin_step(head, isfinite(la) && isfinite(lo), e_ts[1], la, lo, e_cphi[1], isfinite(lap) && isfinite(lop),
                          e_ts[0], lap, lop, e_cphi[0], e_sphi[0]);
        }
        e_f[1] = hs.f;
        e_v[1] = hs.v;
        e_b[1] = hs.b;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < GFI; ++u) {
        const long k = kk[u];
        const int g = u * NWB + w;
        u32 pf = lane_below(ks[u].f);
        double pv = lane_below(ks[u].v), pb = lane_below(ks[u].b);
        if (l == 0) {
            pf = e_f[g + 1];
            pv = e_v[g + 1];
            pb = e_b[g + 1];
        }
        if (k >= (long)n) continue;
        u32 f = ks[u].f;
        double acc, dh;
        kin_final(f, ks[u].v, ks[u].b, ks[u].dts, pf, pv, pb, acc, dh);
        fo.step_m[k] = ks[u].step;
        fo.dt_s[k] = ks[u].dts;
        fo.speed_mps[k] = ks[u].v;
        fo.accel_mps2[k] = acc;
        fo.bearing_deg[k] = ks[u].b;
        fo.dheading_deg[k] = dh;
        fo.flags[k] = (uint8_t)f;
    }
}

// The distinct ids in order (with several shards: by shard, then id) and their
// ranks in the table.  See cv_dictsort.h for where the lines between the three
// ways lie; the ids' count is known on the device alone, so a kernel of a way
// that it does not choose leaves at once.
template <bool SH>
void launch_dict_order_as(const SortLayout& L, u32 mj, u32 n, u32 S, u64 mask, const InsPart* parts, u32 nparts,
                          const u32* used, cv_result* res, hipStream_t s)
{
    // the counted ids may not be written over the list they are counted in
    u64* out = SH ? L.dlf : L.dl1;
    u64* words = L.dsk0;  // the slots' second words with the list
    u64* tag = SH ? words : nullptr;
    u64* runs = SH ? nullptr : L.dsk1;        // the journeys' runs by rank
    u32* delta = SH ? nullptr : (u32*)L.dlf;  // see k_dict_count
    hipLaunchKernelGGL(k_dict_compact, dim3(cvh::grid_for(L.slots, 256 * compact_slots(L.slots), 2048)), dim3(256), 0, s, L.table,
                       L.slots, mj, L.meta, L.dl0, words, parts, nparts, n, S, sort_wide_first() ? 1u : 0u, res,
                       used);
    hipLaunchKernelGGL(k_dict_count<SH>, dim3(cvh::grid_for(mj < DS_COUNT ? mj : DS_COUNT, WAVE)), dim3(DS_B), 0, s,
                       L.meta, L.table, mask, L.dl0, words, out, delta);
    if (mj <= DS_COUNT) return;
    auto offsets = [&] {
        if (!SH)
            hipLaunchKernelGGL(k_run_offsets, dim3(OFF_BLOCKS), dim3(256), 0, s, L.meta, runs, L.sstatus, delta);
    };
    const u32* big = &L.meta->big_n;
    if (mj <= DS_MERGE) {
        const dim3 jg((unsigned)cvh::grid_for(mj, 256, 2048));
        const u32 group = DS_CHUNK * DS_FAN;
        // sorted in place; the last step writes `out`, so the first of two steps of ids alone starts from there
        u64* chunks = (!SH && mj > group) ? L.dl1 : L.dl0;
        hipLaunchKernelGGL(k_ds_chunks<SH>, dim3((mj + DS_CHUNK - 1) / DS_CHUNK), dim3(DS_B), 0, s, L.dl0, chunks, tag,
                           big, &L.meta->multi_shard);
        static_assert(DS_MERGE <= (u64)DS_CHUNK * DS_FAN * DS_FAN, "two steps join every chunk");
        if (mj <= group) {
            hipLaunchKernelGGL((k_dict_join<SH, true>), jg, dim3(256), 0, s, L.meta, L.table, mask, chunks, tag,
                               DS_CHUNK, out, (u64*)nullptr, runs);
            offsets();
            return;
        }
        hipLaunchKernelGGL((k_dict_join<SH, false>), jg, dim3(256), 0, s, L.meta, L.table, mask, chunks, tag, DS_CHUNK,
                           SH ? L.dl1 : L.dl0, SH ? L.dsk1 : nullptr, (u64*)nullptr);
        hipLaunchKernelGGL((k_dict_join<SH, true>), jg, dim3(256), 0, s, L.meta, L.table, mask, SH ? L.dl1 : L.dl0,
                           SH ? L.dsk1 : nullptr, group, out, (u64*)nullptr, runs);
        offsets();
        return;
    }
    // radix passes over the ids (64-bit, signed order via the flipped sign bit)
    radix_hist(L.dl0, mj, big, MAX_PASSES, nullptr, L.dhist, cvh::grid_for(mj, 256, 512), s);
    radix_passes(L.dl0, L.dl1, nullptr, L.dv0, L.dv1, mj, big, nullptr, MAX_PASSES, L.dhist, L.dstatus,
                 L.meta->tickets + MAX_PASSES, s);
    const int dg = cvh::grid_for(mj, 256, 1024);
    if (SH) {
        // the id-sorted list, stably by shard: (shard, id) order, and ranks in it
        const int sp = (int)((bit_width_host((u64)S - 1) + RADIX_BITS - 1) / RADIX_BITS);
        hipLaunchKernelGGL(k_dict_shardkey, dim3(dg), dim3(256), 0, s, L.dl0, L.meta, L.table, mask, L.dsk0);
        radix_hist(L.dsk0, mj, big, sp, nullptr, L.shist, cvh::grid_for(mj, 256, 512), s);
        radix_passes(L.dsk0, L.dsk1, nullptr, L.dv0, L.dv1, mj, big, nullptr, sp, L.shist, L.sstatus,
                     L.meta->tickets + 2 * MAX_PASSES, s);
        hipLaunchKernelGGL(k_dict_final, dim3(dg), dim3(256), 0, s, L.dl0, (sp & 1) ? L.dv1 : L.dv0, L.meta, L.table,
                           mask, L.dlf);
    } else {
        hipLaunchKernelGGL(k_dict_rank, dim3(dg), dim3(256), 0, s, L.dl0, L.meta, L.table, mask, out, runs);
        offsets();
    }
}

void launch_dict_order(const SortLayout& L, u32 mj, u32 n, u32 S, u64 mask, const InsPart* parts, u32 nparts,
                       const u32* used, cv_result* res, hipStream_t s)
{
    if (S > 1) launch_dict_order_as<true>(L, mj, n, S, mask, parts, nparts, used, res, s);
    else launch_dict_order_as<false>(L, mj, n, S, mask, parts, nparts, used, res, s);
}

}  // namespace

static cv_status sort_impl(const cv_records* in, const uint64_t* soff, uint32_t S, uint64_t max_journeys, uint32_t* perm,
                           const cv_records_out* sorted, cv_result* res, void* ws, size_t ws_bytes, void* stream,
                           const cv_features* feat = nullptr)
{
    if (!in || in->n >= (1ull << 32) || max_journeys >= (1ull << 31)) return CV_ERR_INVALID_ARGUMENT;
    const u64 n = in->n;
    if (max_journeys == 0) max_journeys = 1;
    hipStream_t s = (hipStream_t)stream;
    cv_records_out so = {};
    if (sorted) so = *sorted;
    if (n > 0) {
        if (!in->journey_id || !in->ts_ms || !perm) return CV_ERR_INVALID_ARGUMENT;
        if ((so.lat_deg && !in->lat_deg) || (so.lon_deg && !in->lon_deg) || (so.speed_mps && !in->speed_mps))
            return CV_ERR_INVALID_ARGUMENT;
        if (!valid_ptr8(in->journey_id) || !valid_ptr8(in->ts_ms) || !valid_ptr8(in->lat_deg) ||
            !valid_ptr8(in->lon_deg) || !valid_ptr8(so.journey_id) || !valid_ptr8(so.ts_ms) ||
            !valid_ptr8(so.lat_deg) || !valid_ptr8(so.lon_deg) || !cvh::aligned(perm, 4))
            return CV_ERR_INVALID_ARGUMENT;
    }
    SortLayout need(nullptr, n, max_journeys);
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < need.bytes) return CV_ERR_WORKSPACE;
    if (n == 0) {
        if (res) hipLaunchKernelGGL(k_empty_result, dim3(1), dim3(64), 0, s, res);
        return cvh::last_launch_status();
    }
    SortLayout L(ws, n, max_journeys);
    const u32 nn = (u32)n;
    const u32 mj = (u32)max_journeys;
    const u64 mask = L.slots - 1;
    const int gs = cvh::grid_for(n, 256, 2048);
    const bool full = so.journey_id && so.ts_ms && so.lat_deg && so.lon_deg && so.speed_mps;
    {
        cvh::TimedScope ts_("sort_prep", s);
        // the insert's per-block parts lie in the second key buffer, which the
        // passes write later (a block for at least 256 of its 8-byte words, and
        // every buffer holds at least 256 bytes)
        InsPart* parts = (InsPart*)L.K1;
        static_assert(sizeof(InsPart) <= 256, "one part fits the smallest buffer");
        // the occupied slots' bits lie in the second list of ids, which is written once
        // the first is complete (fewer than four slots, of a bit each, per id allowed)
        u32* used = L.slots >= USED_MIN ? (u32*)L.dl1 : nullptr;
        const u64 fill_words = L.slots > L.zero_bytes / 4 ? L.slots : L.zero_bytes / 4;
        hipLaunchKernelGGL(k_sort_begin, dim3(cvh::grid_for(fill_words, 256, 4096)), dim3(256), 0, s, L.meta, L.table,
                           2 * L.slots, L.zero_begin, (u64)(L.zero_bytes / 4), used);
        // at least 8 windows per wave, so that a wave meets ids in its cache
        // (insert of 1 M shuffled records of 2 000 journeys 383 -> 55 us, of a
        // 2 M batch 242 -> 24, of a 437 k push 75 -> 27, of a 200 M batch 1 760 -> 1 430;
        // with the slots read again and one insert per id and window, below)
        const int gi = cvh::grid_for(n, 256 * 8, 2048);
        auto* ins = S > 1 ? (used ? k_dict_insert<true, true> : k_dict_insert<true, false>)
                          : (used ? k_dict_insert<false, true> : k_dict_insert<false, false>);
        hipLaunchKernelGGL(ins, dim3(gi), dim3(256), 0, s, in->journey_id, in->ts_ms, nn, L.table, mask,
                           L.meta, parts, soff, S, used);
        launch_dict_order(L, mj, nn, S, mask, parts, (u32)gi, used, res, s);
        // interleaved input (short runs of equal ids): the payload packed per
        // record for a gather of every column, in the same pass
        hipLaunchKernelGGL(S > 1 ? k_pack_hist<true> : k_pack_hist<false>, dim3(gs), dim3(256), 0, s, in->journey_id,
                           in->ts_ms, nn, L.table, mask, L.meta, L.K0, L.hist, soff, S,
                           (const u32*)L.dlf);
        const int pi = pack_items(n);
        auto* il = S > 1 ? (pi == 1 ? k_pack_il<true, 1> : pi == 2 ? k_pack_il<true, 2> : k_pack_il<true, 4>)
                         : (pi == 1 ? k_pack_il<false, 1> : pi == 2 ? k_pack_il<false, 2> : k_pack_il<false, 4>);
        hipLaunchKernelGGL(il, dim3(cvh::grid_for(n, PT_B * pi, 2048)), dim3(PT_B), 0, s, in->journey_id, in->ts_ms,
                           in->lat_deg, in->lon_deg, in->speed_mps, feat || full ? L.pay : nullptr, nn, L.table, mask,
                           L.meta, L.K0, L.hist, soff, S);
    }
    radix_passes(L.K0, L.K1, nullptr, L.V0, L.V1, nn, nullptr, &L.meta->sort_bits, MAX_PASSES, L.hist, L.status,
                 L.meta->tickets, s, /*timed=*/true, &L.meta->ib, &L.meta->w0);
    const u64* dict_ids = S > 1 ? L.dlf : L.dl1;  // journey ids by rank
    if (feat) {
        cvh::TimedScope ts_("gather_features", s);
        auto gk = S > 1 ? k_gather_feat<true> : k_gather_feat<false>;
        hipLaunchKernelGGL(gk, dim3((unsigned)((n + GFT - 1) / GFT)), dim3(256), 0, s, nn, L.meta, L.K0, L.K1, dict_ids,
                           in->journey_id, in->ts_ms, in->lat_deg, in->lon_deg, in->speed_mps, perm, so, *feat, soff,
                           S, L.pay);
    } else {
        cvh::TimedScope ts_("gather", s);
        auto gk = S > 1 ? (full ? k_gather<true, true> : k_gather<true, false>)
                        : (full ? k_gather<false, true> : k_gather<false, false>);
        hipLaunchKernelGGL(gk, dim3(cvh::grid_for(n, 256, 8192)), dim3(256), 0, s, nn, L.meta, L.K0, L.K1, dict_ids,
                           in->journey_id, in->ts_ms, in->lat_deg, in->lon_deg, in->speed_mps, perm,
                           so.journey_id, so.ts_ms, so.lat_deg, so.lon_deg, so.speed_mps, soff, S, L.pay);
    }
    cvh::debug_sort(L.K0, L.K1, &L.meta->passes, &L.meta->range_err, &L.meta->overflow, n, perm, soff, S, s);
    return cvh::last_launch_status();
}


namespace cv {
// the record sort for other translation units of the library (no shards)
cv_status sort_records_into(const cv_records* in, uint64_t max_journeys, uint32_t* perm, const cv_records_out* sorted,
                            cv_result* res, void* ws, size_t ws_bytes, hipStream_t stream)
{
    return sort_impl(in, nullptr, 0, max_journeys, perm, sorted, res, ws, ws_bytes, (void*)stream);
}
}  // namespace cv

extern "C" {

cv_status cv_sort_workspace_size(uint64_t n, uint64_t max_journeys, size_t* bytes)
{
    if (!bytes || n >= (1ull << 32) || max_journeys >= (1ull << 31)) return CV_ERR_INVALID_ARGUMENT;
    if (max_journeys == 0) max_journeys = 1;
    SortLayout L(nullptr, n, max_journeys);
    *bytes = L.bytes;
    return CV_OK;
}

cv_status cv_sort_passes(const void* ws, uint32_t* passes, void* stream)
{
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || !passes || !cvh::aligned(passes, 4)) return CV_ERR_INVALID_ARGUMENT;
    hipLaunchKernelGGL(k_passes, dim3(1), dim3(64), 0, (hipStream_t)stream, (const SortMeta*)ws, passes);
    return cvh::last_launch_status();
}

cv_status cv_sort_records(const cv_records* in, uint64_t max_journeys, uint32_t* perm, const cv_records_out* sorted,
                          cv_result* res, void* ws, size_t ws_bytes, void* stream)
{
    return sort_impl(in, nullptr, 0, max_journeys, perm, sorted, res, ws, ws_bytes, stream);
}

cv_status cv_batch_sort_records(const cv_records* in, const uint64_t* shard_offsets, uint32_t n_shards,
                                uint64_t max_journeys, uint32_t* perm, const cv_records_out* sorted, cv_result* res,
                                void* ws, size_t ws_bytes, void* stream)
{
    if (n_shards == 0 || !shard_offsets || !cvh::aligned(shard_offsets, 8)) return CV_ERR_INVALID_ARGUMENT;
    return sort_impl(in, shard_offsets, n_shards, max_journeys, perm, sorted, res, ws, ws_bytes, stream);
}

static bool feat_complete(const cv_records_out* so, const cv_features* f)
{
    return so && f && so->journey_id && so->ts_ms && so->lat_deg && so->lon_deg && so->speed_mps && f->step_m &&
           f->dt_s && f->speed_mps && f->accel_mps2 && f->bearing_deg && f->dheading_deg && f->flags;
}

cv_status cv_sort_records_features(const cv_records* in, uint64_t max_journeys, uint32_t* perm,
                                   const cv_records_out* sorted, const cv_features* feat, cv_result* res, void* ws,
                                   size_t ws_bytes, void* stream)
{
    if (in && in->n && !feat_complete(sorted, feat)) return CV_ERR_INVALID_ARGUMENT;
    return sort_impl(in, nullptr, 0, max_journeys, perm, sorted, res, ws, ws_bytes, stream, feat);
}

cv_status cv_batch_sort_records_features(const cv_records* in, const uint64_t* shard_offsets, uint32_t n_shards,
                                         uint64_t max_journeys, uint32_t* perm, const cv_records_out* sorted,
                                         const cv_features* feat, cv_result* res, void* ws, size_t ws_bytes,
                                         void* stream)
{
    if (n_shards == 0 || !shard_offsets || !cvh::aligned(shard_offsets, 8)) return CV_ERR_INVALID_ARGUMENT;
    if (in && in->n && !feat_complete(sorted, feat)) return CV_ERR_INVALID_ARGUMENT;
    return sort_impl(in, shard_offsets, n_shards, max_journeys, perm, sorted, res, ws, ws_bytes, stream, feat);
}

}  // extern "C"
