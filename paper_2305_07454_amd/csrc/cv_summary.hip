// cv_summary.hip -- cv_journey_summary: one row per journey of sorted records.
//
// Journeys are maximal runs of equal journey id.  Tiles of NW waves' chunks:
//   k_sum_count   journey starts per wave chunk (k_sum_count_flags: from the
//                 features' flags);
//   k_tile_scan   exclusive scan of the tile totals (one block) -> journey index
//                 of each tile's first start, J (calls of more than N_S records; in
//                 shorter ones every block sums the counts that it needs);
//   k_sum_init    identity values in the accumulator rows of the J journeys;
//   k_sum_reduce  (up to N_S records k_sum_both: box and sums in one launch)
//                 segmented reduction over journey boundaries: every wave walks
//                 its records in coalesced windows of 64, folding them in exact
//                 fixed point; a journey that starts and ends inside one wave's
//                 records is written out directly, the pieces of one that
//                 crosses a wave edge meet in its accumulator row through
//                 integer atomics (order-independent, hence deterministic);
//   k_sum_finalize accumulator rows -> output rows (exact sums rounded once).
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "cv_device.h"
#include "cv_host.h"
#include "cv_sumtab.h"

using namespace cv;

namespace {

constexpr int SB = 256;
// Windows of 64 records that a wave walks, by the record count.  A wave goes
// through its windows one after the other, so a small call is bound by one
// wave's walk unless the records are split finer; a large one pays for finer
// chunks with more journeys that cross a chunk edge (merged by atomics).
//   SI_S  up to N_S records: 2 048 per block; every block sums the (at most
//         2 048) journey counts before its own itself, and both reductions
//         run in one launch, which saves two launches as well;
//   SI_M  up to N_M records;
//   SI_L  above.
// Whole summary, SI_S / SI_M / SI_L: 33 k records 26 / 48 / 105 us, 1 M 34 / 56 /
// 124, 4 M 82 / 80 / 140, 8 M 162 / 143 / 162, a 30 M batch of shards 639 / 366 /
// 393; 100 M records 948 / 931 / 933 and a 200 M batch - / 2 238 / 1 960.  Where
// SI_M ends follows journeys of thousands of records (SI_M / SI_L, 24 M: 260 / 266,
// 26 M 280 / 284, 28 M 301 / 293, 33 M 351 / 326; of 150 records 453 / 502, 489 / 552,
// 521 / 556, 613 / 617).
constexpr int SI_S = 8, SI_M = 16, SI_L = 64;
constexpr u64 N_S = 4ull << 20, N_M = 25ull << 20;
constexpr int FX_DIST = SUM_FX_DIST;  // distance: 2^-128 m resolution (exact for steps >= 2^-75 m)
constexpr int FX_SPD = SUM_FX_SPD;    // speed: exact for every float32

struct SumMeta {
    u32 J;
};

constexpr int NW = SB / WAVE;  // waves per block
// a tile is NW wave chunks of WAVE * SI records
constexpr u64 sum_tiles(u64 n, int si) { return (n + (u64)SB * si - 1) / ((u64)SB * si); }

// Journey starts among the records of window [a, a + 64) of a wave that walks
// consecutive windows, from this lane's id jv (already loaded): jprev is the
// id before the window (carried), sk the shard cursor.  Returns the lane mask
// of starts.
__device__ __forceinline__ u64 heads_of(i64 jv, u64 a, u64 end, i64& jprev, const u64* __restrict__ soff, u32 S,
                                        u32& sk, u64& smask, bool& s_end)
{
    const int l = lane_id();
    const u64 r = a + l;
    const bool valid = r < end;
    i64 jp = lane_below(jv);
    if (l == 0) jp = jprev;
    jprev = __shfl(jv, WAVE - 1, WAVE);
    smask = 0;
    s_end = false;
    if (S > 1) smask = shard_starts_in(soff, S, sk, a, s_end);
    return __ballot(valid && (r == 0 || jv != jp || ((smask >> l) & 1ull)));
}

// journey starts per wave chunk of WCH records: wcnt[tile * NW + wave], and
// per tile: tcnt[tile]
template <int SI>
__global__ void __launch_bounds__(SB) k_sum_count(const i64* __restrict__ jid, u32 n, u32* __restrict__ wcnt,
                                                  u32* __restrict__ tcnt, const u64* __restrict__ soff, u32 S)
{
    constexpr int WCH = WAVE * SI, ST = SB * SI;
    __shared__ u32 s_w[NW];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);  // wave-uniform
    const u64 cs = (u64)blockIdx.x * ST + (u64)w * WCH;
    const u64 ce = cs + WCH < n ? cs + WCH : (u64)n;
    u32 c = 0;
    if (cs < ce) {
        i64 jprev = cs > 0 ? jid[cs - 1] : 0;
        u32 sk = S > 1 ? shard_lower_bound(soff, S, cs) : 0u;
        i64 jn = cs + lane_id() < ce ? jid[cs + lane_id()] : 0;
        for (u64 a = cs; a < ce; a += WAVE) {
            const i64 jv = jn;
            if (a + WAVE + lane_id() < ce) jn = jid[a + WAVE + lane_id()];  // next window, loaded ahead
            u64 sm;
            bool se;
            c += (u32)__popcll(heads_of(jv, a, ce, jprev, soff, S, sk, sm, se));
        }
    }
    if (lane_id() == 0) {
        wcnt[(u64)blockIdx.x * NW + w] = c;
        s_w[w] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        u32 t = 0;
        for (int k = 0; k < NW; ++k) t += s_w[k];
        tcnt[blockIdx.x] = t;
    }
}

// The same counts from the features' FIRST flags (set exactly at journey and
// shard starts): one byte per record instead of an id and its predecessor.
template <int SI>
__global__ void __launch_bounds__(SB) k_sum_count_flags(const uint8_t* __restrict__ flags, u32 n,
                                                        u32* __restrict__ wcnt, u32* __restrict__ tcnt)
{
    constexpr int WCH = WAVE * SI, ST = SB * SI;
    __shared__ u32 s_w[NW];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const u64 cs = (u64)blockIdx.x * ST + (u64)w * WCH;
    const u64 ce = cs + WCH < n ? cs + WCH : (u64)n;
    constexpr int FB = WCH / WAVE;  // flag bytes per lane
    static_assert((FB == 8 || FB % 16 == 0) && CV_FLAG_FIRST == 1u, "whole 8- or 16-byte loads per lane; FIRST is bit 0");
    u32 c = 0;
    if (cs < ce) {
        // lane l counts the chunk's bytes [FB l, FB l + FB): 16-byte (8-byte)
        // loads when the chunk is whole and the column 16-byte aligned
        const u64 b0 = cs + (u64)lane_id() * FB;
        if (ce - cs == (u64)WCH && ((uintptr_t)flags & 15u) == 0) {
            if (FB == 8) c = (u32)__popcll(*reinterpret_cast<const u64*>(flags + b0) & 0x0101010101010101ull);
#pragma unroll
            for (int q = 0; q < FB / 16; ++q) {
                const uint4 v = *reinterpret_cast<const uint4*>(flags + b0 + 16 * q);
                c += (u32)(__popc(v.x & 0x01010101u) + __popc(v.y & 0x01010101u) + __popc(v.z & 0x01010101u) +
                           __popc(v.w & 0x01010101u));
            }
        } else {
            for (int k = 0; k < FB; ++k)
                if (b0 + k < ce) c += flags[b0 + k] & CV_FLAG_FIRST;
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) c += (u32)__shfl_xor((int)c, d, WAVE);
    }
    if (lane_id() == 0) {
        wcnt[(u64)blockIdx.x * NW + w] = c;
        s_w[w] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        u32 t = 0;
        for (int k = 0; k < NW; ++k) t += s_w[k];
        tcnt[blockIdx.x] = t;
    }
}

// single block: tile_prefix[i] = journey starts before tile i; meta->J = total.
// Each thread sums a contiguous run of tiles, one block scan joins the runs.
constexpr int SCAN_B = 1024;
__global__ void __launch_bounds__(SCAN_B) k_tile_scan(const u32* __restrict__ tcnt, u32* __restrict__ tile_prefix,
                                                      u32 tiles, SumMeta* meta)
{
    __shared__ u32 tmp[SCAN_B / WAVE];
    const u32 per = (tiles + SCAN_B - 1) / SCAN_B;
    const u32 a = threadIdx.x * per;
    const u32 b = a + per < tiles ? a + per : tiles;
    u32 sum = 0;
#pragma unroll 8
    for (u32 i = a; i < b; ++i) sum += tcnt[i];
    u32 total;
    u32 e = block_exclusive_sum<SCAN_B>(sum, tmp, total);
    for (u32 i = a; i < b; ++i) {
        tile_prefix[i] = e;
        e += tcnt[i];
    }
    if (threadIdx.x == 0) meta->J = total;
}

__device__ __forceinline__ void jacc_identity(JAcc& a)
{
    a.dist[0] = a.dist[1] = a.dist[2] = 0;
    a.spd[0] = a.spd[1] = a.spd[2] = 0;
    a.maxd = ord_f64(0.0);
    a.latmin = ord_f64(__builtin_inf());
    a.latmax = ord_f64(-__builtin_inf());
    a.lonmin = ord_f64(__builtin_inf());
    a.lonmax = ord_f64(-__builtin_inf());
    a.count = 0;
    a.ndtz = 0;
    a.maxs = 0;
    a.gfirst = 0;
}

// sum of c[0, tiles) over the block (SB threads), in every thread
__device__ __forceinline__ u32 block_count_sum(const u32* __restrict__ c, u32 tiles, u32* s_t)
{
    u32 v = 0;
    for (u32 i = threadIdx.x; i < tiles; i += SB) v += c[i];
    u32 total;
    block_exclusive_sum<SB>(v, s_t, total);
    return total;
}

// tcnt (nullable): the tiles' journey counts, whose sum is J (the small form);
// else meta holds it
__global__ void __launch_bounds__(SB) k_sum_init(JAcc* __restrict__ acc, AccX* __restrict__ accx, SumMeta* meta,
                                                u32 cap, const u32* __restrict__ tcnt, u32 tiles)
{
    __shared__ u32 s_t[NW];
    u32 J;
    if (tcnt) {
        J = block_count_sum(tcnt, tiles, s_t);
        if (blockIdx.x == 0 && threadIdx.x == 0) meta->J = J;
    } else {
        J = meta->J;
    }
    u32 m = J < cap ? J : cap;
    for (u32 j = blockIdx.x * blockDim.x + threadIdx.x; j < m; j += gridDim.x * blockDim.x) {
        JAcc a;
        jacc_identity(a);
        acc[j] = a;
        AccX x = {};
        accx[j] = x;
    }
}

// Partial aggregates of one journey (a lane's records, a wave's, or a tile's),
// in two field groups reduced by two launches of the same kernel: the record
// count with the bounding box, and the exact sums with the zero-dt count and
// the maxima.  Each launch keeps only its group live, which keeps its
// register use (and so the waves in flight per SIMD) in bounds.
struct PartBox {
    u64 latmin, latmax, lonmin, lonmax;
    u32 count;
};
// The sums are 128-bit two's-complement integers: distance in units of 2^-72
// m, exact for steps of at least 2^-20 m (and zero); speed in units of 2^-53,
// exact for float32 speeds v with 2^-30 <= |v| < 2^10 (and zeros).  Any other
// value is added on its own, in the full 192-bit format, to the journey's
// side row (AccX).
struct PartSum {
    u64 dlo, dhi, slo, shi;
    u64 maxd;
    u32 ndtz, maxs, n;  // n: records folded in (empty partials are not flushed)
};

__device__ __forceinline__ void add128(u64& lo, u64& hi, u64 blo, u64 bhi)
{
    const u64 s = lo + blo;
    hi += bhi + (s < lo ? 1ull : 0ull);
    lo = s;
}

// v * 2^72 as a 128-bit integer when 2^-20 <= |v| < 2^40 or v = +-0
__device__ __forceinline__ bool dist_fix72(double v, u64& lo, u64& hi)
{
    const u64 b = (u64)__double_as_longlong(v);
    const u32 e = (u32)((b >> 52) & 0x7FFu);
    const u64 m = b & ((1ull << 52) - 1);
    lo = 0;
    hi = 0;
    if (e == 0) return m == 0;
    if (e < 1003 || e > 1062) return false;
    const u64 M = m | (1ull << 52);
    const u32 sft = e - 1003;  // 0 .. 59
    lo = M << sft;
    hi = sft ? (M >> (64 - sft)) : 0ull;
    if (b >> 63) {
        lo = ~lo + 1;
        hi = ~hi + (lo == 0 ? 1ull : 0ull);
    }
    return true;
}

// v * 2^53 as a signed integer when 2^-30 <= |v| < 2^10 or v = +-0
__device__ __forceinline__ bool spd_fix53(float v, i64& x)
{
    const u32 b = __float_as_uint(v);
    const u32 e = (b >> 23) & 0xFFu;
    const u32 m = b & 0x7FFFFFu;
    x = 0;
    if (e == 0) return m == 0;
    if (e < 97 || e > 136) return false;
    const i64 mag = (i64)((u64)(m | 0x800000u) << (e - 97));
    x = (b >> 31) ? -mag : mag;
    return true;
}

// the 128-bit sums in the 192-bit formats of the rows (2^-128 m, 2^-149)
__device__ __forceinline__ Fx192 dist192(u64 lo, u64 hi)
{
    Fx192 r;
    r.w[0] = lo << 56;
    r.w[1] = (lo >> 8) | (hi << 56);
    r.w[2] = (u64)((i64)hi >> 8);
    return r;
}
__device__ __forceinline__ Fx192 spd192(u64 lo, u64 hi)
{
    Fx192 r;
    r.w[0] = 0;
    r.w[1] = lo << 32;
    r.w[2] = (lo >> 32) | (hi << 32);
    return r;
}

__device__ __forceinline__ void part_reset(PartBox& p)
{
    p.latmin = ord_f64(__builtin_inf());
    p.latmax = ord_f64(-__builtin_inf());
    p.lonmin = ord_f64(__builtin_inf());
    p.lonmax = ord_f64(-__builtin_inf());
    p.count = 0;
}
__device__ __forceinline__ void part_reset(PartSum& p)
{
    p.dlo = p.dhi = p.slo = p.shi = 0;
    p.maxd = ord_f64(0.0);
    p.ndtz = 0;
    p.maxs = 0;
    p.n = 0;
}

__device__ __forceinline__ void part_combine(PartBox& a, const PartBox& b)
{
    a.latmin = b.latmin < a.latmin ? b.latmin : a.latmin;
    a.latmax = b.latmax > a.latmax ? b.latmax : a.latmax;
    a.lonmin = b.lonmin < a.lonmin ? b.lonmin : a.lonmin;
    a.lonmax = b.lonmax > a.lonmax ? b.lonmax : a.lonmax;
    a.count += b.count;
}
__device__ __forceinline__ void part_combine(PartSum& a, const PartSum& b)
{
    add128(a.dlo, a.dhi, b.dlo, b.dhi);
    add128(a.slo, a.shi, b.slo, b.shi);
    a.maxd = b.maxd > a.maxd ? b.maxd : a.maxd;
    a.ndtz += b.ndtz;
    a.maxs = b.maxs > a.maxs ? b.maxs : a.maxs;
    a.n += b.n;
}

// Cross-lane steps work one field at a time, so that only that field's moved
// copy is live next to the partial.  Step K of the segmented scan folds in the
// lane that scan_move brings (where scan_takes' bit K says so); a step of the
// full reduction the lane 2^K away by xor.
template <int K, bool SCAN, class T>
__device__ __forceinline__ T part_move(T v, typename std::common_type<T>::type none)
{
    if constexpr (SCAN) return scan_move<K>(v, none);
    else return (T)__shfl_xor(v, 1 << K, WAVE);
}

template <int K, bool SCAN>
__device__ __forceinline__ void part_step(PartBox& p, u32 takes)
{
    const bool take = !SCAN || ((takes >> K) & 1u);
    u64 v;
    v = part_move<K, SCAN>(p.latmin, ~0ull);
    if (take && v < p.latmin) p.latmin = v;
    v = part_move<K, SCAN>(p.latmax, 0ull);
    if (take && v > p.latmax) p.latmax = v;
    v = part_move<K, SCAN>(p.lonmin, ~0ull);
    if (take && v < p.lonmin) p.lonmin = v;
    v = part_move<K, SCAN>(p.lonmax, 0ull);
    if (take && v > p.lonmax) p.lonmax = v;
    const u32 x = part_move<K, SCAN>(p.count, 0u);
    if (take) p.count += x;
}
template <int K, bool SCAN>
__device__ __forceinline__ void part_step(PartSum& p, u32 takes)
{
    const bool take = !SCAN || ((takes >> K) & 1u);
    const u64 dlo = part_move<K, SCAN>(p.dlo, 0ull), dhi = part_move<K, SCAN>(p.dhi, 0ull);
    if (take) add128(p.dlo, p.dhi, dlo, dhi);
    const u64 slo = part_move<K, SCAN>(p.slo, 0ull), shi = part_move<K, SCAN>(p.shi, 0ull);
    if (take) add128(p.slo, p.shi, slo, shi);
    const u64 v = part_move<K, SCAN>(p.maxd, 0ull);
    if (take && v > p.maxd) p.maxd = v;
    u32 x;
    x = part_move<K, SCAN>(p.ndtz, 0u);
    if (take) p.ndtz += x;
    x = part_move<K, SCAN>(p.maxs, 0u);
    if (take && x > p.maxs) p.maxs = x;
    x = part_move<K, SCAN>(p.n, 0u);
    if (take) p.n += x;
}

template <bool SCAN, class P>
__device__ __forceinline__ void part_steps(P& p, u32 takes)
{
    part_step<0, SCAN>(p, takes);
    part_step<1, SCAN>(p, takes);
    part_step<2, SCAN>(p, takes);
    part_step<3, SCAN>(p, takes);
    part_step<4, SCAN>(p, takes);
    part_step<5, SCAN>(p, takes);
}

// full wave reduction; every lane ends with the total
template <class P>
__device__ __forceinline__ void part_wave_reduce(P& p)
{
    part_steps<false>(p, 0u);
}

// segmented inclusive scan across lanes; `head` starts a segment
template <class P>
__device__ __forceinline__ void part_seg_scan(P& p, bool head)
{
    part_steps<true>(p, scan_takes(__ballot(head)));
}

struct Out {
    int64_t* jid;
    uint32_t* first;
    uint32_t* npts;
    int64_t* tstart;
    int64_t* tend;
    double* dist;
    double* sumspd;
    float* maxspd;
    double* maxdspd;
    uint32_t* ndtz;
    double *latmin, *latmax, *lonmin, *lonmax;
};

__device__ __forceinline__ void write_final(const Out& o, u32 j, u32 count, u32 ndtz, const Fx192& dist,
                                            const Fx192& spd, u32 maxs, u64 maxd, u64 la0, u64 la1, u64 lo0, u64 lo1)
{
    o.npts[j] = count;
    o.ndtz[j] = ndtz;
    o.dist[j] = fx_to_double<FX_DIST>(dist);
    o.sumspd[j] = fx_to_double<FX_SPD>(spd);
    o.maxspd[j] = unord_f32(maxs);
    o.maxdspd[j] = unord_f64(maxd);
    o.latmin[j] = unord_f64(la0);
    o.latmax[j] = unord_f64(la1);
    o.lonmin[j] = unord_f64(lo0);
    o.lonmax[j] = unord_f64(lo1);
}

// A journey's partial into its accumulator row: a whole journey (all its
// records are in the partial) is stored, a piece is merged with integer atomics.
// The rows are turned into output rows by k_sum_finalize.
__device__ __forceinline__ void flush_part(JAcc* acc, u32 cap, u32 j, const PartBox& p, bool whole)
{
    if (j >= cap || p.count == 0) return;
    JAcc& a = acc[j];
    if (whole) {
        a.latmin = p.latmin;
        a.latmax = p.latmax;
        a.lonmin = p.lonmin;
        a.lonmax = p.lonmax;
        a.count = p.count;
        return;
    }
    atomicMin((unsigned long long*)&a.latmin, (unsigned long long)p.latmin);
    atomicMax((unsigned long long*)&a.latmax, (unsigned long long)p.latmax);
    atomicMin((unsigned long long*)&a.lonmin, (unsigned long long)p.lonmin);
    atomicMax((unsigned long long*)&a.lonmax, (unsigned long long)p.lonmax);
    atomicAdd(&a.count, p.count);
}
__device__ __forceinline__ void flush_part(JAcc* acc, u32 cap, u32 j, const PartSum& p, bool whole)
{
    if (j >= cap || p.n == 0) return;
    JAcc& a = acc[j];
    const Fx192 d = dist192(p.dlo, p.dhi), sp = spd192(p.slo, p.shi);
    if (whole) {
        for (int i = 0; i < 3; ++i) {
            a.dist[i] = d.w[i];
            a.spd[i] = sp.w[i];
        }
        a.maxd = p.maxd;
        a.ndtz = p.ndtz;
        a.maxs = p.maxs;
        return;
    }
    atomic_add_fx(a.dist, d);
    atomic_add_fx(a.spd, sp);
    atomicMax((unsigned long long*)&a.maxd, (unsigned long long)p.maxd);
    atomicAdd(&a.ndtz, p.ndtz);
    atomicMax(&a.maxs, p.maxs);
}

// Each wave owns WCH consecutive records and walks them in coalesced windows of
// 64, loaded a group of windows at a time.  Lanes fold their records into a private partial while the window holds
// no journey start; a window with starts closes the open journey (wave
// reduction), runs a segmented scan for journeys that begin in it, and hands
// the last one on as the new open journey.  A journey that begins and ends in
// the wave's records is stored directly; otherwise its pieces meet in the
// accumulator row through integer atomics.  Neighbouring ids come from lane
// shuffles.  BOX = true reduces PartBox and also writes each journey's id,
// first record; BOX = false reduces PartSum.  SHARDS = false compiles the
// plain form without the shard branches, whose loads would otherwise make
// every window wait for all loads in flight, prefetch included.
// FL = true: journey starts are read from the features' FIRST flags instead
// of comparing ids (the box pass then loads an id only at a journey start,
// to write it out).
// seen: journey starts before the block's tile.
template <bool BOX, bool SHARDS, bool FL, int SI>
__device__ __forceinline__ void sum_reduce(u32 n, const i64* __restrict__ jid, const double* __restrict__ lat,
                                           const double* __restrict__ lon, const float* __restrict__ spd,
                                           const double* __restrict__ step, const double* __restrict__ dspd,
                                           const uint8_t* __restrict__ flags, u32 seen, const u32* __restrict__ wcnt,
                                           u32 cap, Out o, JAcc* __restrict__ acc, AccX* __restrict__ accx,
                                           const u64* __restrict__ soff, u32 S, u64* __restrict__ jo)
{
    using P = typename std::conditional<BOX, PartBox, PartSum>::type;
    constexpr int WI = SI, WCH = WAVE * SI, ST = SB * SI;
    if (!SHARDS) S = 0;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);  // wave-uniform
    const int l = lane_id();
    const u64 cs = (u64)blockIdx.x * ST + (u64)w * WCH;  // wave chunk start
    const u64 ce = cs + WCH < n ? cs + WCH : (u64)n;      // wave chunk end (may be <= cs)
    if (cs >= ce) return;
    // (from here on: journey starts before the current window)
    for (int k = 0; k < w; ++k) seen += wcnt[(u64)blockIdx.x * NW + k];

    P p;
    part_reset(p);
    // open journey: the one containing the record before the next window
    u32 open_j = seen - 1;   // valid when the chunk starts mid-journey
    bool open_here = false;  // its first record lies in this chunk
    i64 jprev = (!FL && cs > 0) ? jid[cs - 1] : 0;
    u32 sk = (SHARDS && !FL) ? shard_lower_bound(soff, S, cs) : 0u;
    // the shard holding the chunk's first record: a journey head's shard is
    // walked forward from it (a chunk spans few shards) instead of searched
    const u32 shc = (SHARDS && FL && S > 1) ? shard_of(soff, S, cs) : 0u;
    // the id after the chunk (its last record may end a journey)
    const i64 jend = (!FL && ce < n) ? jid[ce] : 0;
    // Windows are taken in groups of WG: the columns of a group (ids included)
    // are loaded together, from addresses clamped into the chunk, so that all
    // of a group's loads are in flight at once.
    constexpr int WG = 4;
    static_assert(WI % WG == 0, "whole groups");
    for (int g0 = 0; g0 < WI; g0 += WG) {
        if (cs + (u64)g0 * WAVE >= ce) break;
        i64 gj[WG];
        double gx0[WG], gx1[WG];
        float gsp[WG];
        uint8_t gf[WG];
#pragma unroll
        for (int k = 0; k < WG; ++k) {
            u64 r = cs + (u64)(g0 + k) * WAVE + l;
            r = r < ce ? r : ce - 1;
            gj[k] = FL ? 0 : jid[r];
            if constexpr (BOX) {
                gx0[k] = lat[r];
                gx1[k] = lon[r];
                if (FL) gf[k] = flags[r];
            } else {
                gx0[k] = step[r];
                gx1[k] = dspd[r];
                gsp[k] = spd[r];
                gf[k] = flags[r];
            }
        }
#pragma unroll
        for (int k = 0; k < WG; ++k) {
            const u64 a = cs + (u64)(g0 + k) * WAVE;
            if (a >= ce) break;
            const u64 r = a + l;
            const bool valid = r < ce;
            const i64 jv = gj[k];
            u64 smask;
            bool s_end;
            u64 H;
            if constexpr (FL) {
                H = __ballot(valid && (gf[k] & CV_FLAG_FIRST) != 0);
                smask = 0;
                s_end = false;
            } else {
                H = heads_of(jv, a, ce, jprev, soff, S, sk, smask, s_end);
            }
            const bool h = (H >> l) & 1ull;
            // journey index of this lane's record
            const u32 jl = seen + popc_below(H) + (h ? 1u : 0u) - 1u;
            P c;
            part_reset(c);
            if (valid) {
                if constexpr (BOX) {
                    c.count = 1;
                    if (isfinite(gx0[k]) && isfinite(gx1[k])) {
                        c.latmin = c.latmax = ord_f64(gx0[k]);
                        c.lonmin = c.lonmax = ord_f64(gx1[k]);
                    }
                } else {
                    c.n = 1;
                    c.ndtz = (gf[k] & CV_FLAG_DT_ZERO) ? 1u : 0u;
                    if (!dist_fix72(gx0[k], c.dlo, c.dhi) && jl < cap)
                        atomic_add_fx(accx[jl].dist, fx_from_double<FX_DIST>(gx0[k]));
                    i64 x;
                    if (spd_fix53(gsp[k], x)) {
                        c.slo = (u64)x;
                        c.shi = (u64)(x >> 63);
                    } else if (jl < cap) {
                        atomic_add_fx(accx[jl].spd, fx_from_double<FX_SPD>((double)gsp[k]));
                    }
                    c.maxs = ord_f32(gsp[k]);
                    if (gf[k] & CV_FLAG_SPEED_OK) c.maxd = ord_f64(gx1[k]);
                }
            }
            if constexpr (BOX) {
                const u32 sh = (h && S > 1) ? (FL ? shard_from(soff, S, shc, r) : shard_of(soff, S, r)) : 0u;
                if (h && jl < cap) {
                    // a journey's first record is indexed within its shard
                    if (o.jid) o.jid[jl] = FL ? jid[r] : jv;
                    if (o.first) o.first[jl] = (u32)(S > 1 ? r - soff[sh] : r);
                    acc[jl].gfirst = (u32)r;
                }
                if (h && S > 1 && jo) {
                    // this record opens its shard's first journey: every shard
                    // starting here (empty ones included) begins at journey jl
                    if (soff[sh] == r)
                        for (int z = (int)sh; z >= 0 && soff[z] == r; --z) jo[z] = jl;
                }
            }
            if (H != 0) {
                const int f0 = __ffsll((long long)H) - 1;
                if (l < f0) part_combine(p, c);
                // close the journey that was open before the first start in this window
                part_wave_reduce(p);
                if (l == 0) flush_part(acc, cap, open_j, p, open_here);
                // journeys starting in this window
                P sc = c;
                part_seg_scan(sc, h);
                // a segment that ends before lane 63 (next lane starts a journey)
                // is a whole journey: it began and ended inside this window
                const bool next_head = (l < WAVE - 1) && ((H >> (l + 1)) & 1ull);
                if (l >= f0 && next_head) flush_part(acc, cap, jl, sc, true);
                // the last segment stays open; lane 63 holds its partial
                part_reset(p);
                if (l == WAVE - 1) p = sc;
                seen += (u32)__popcll(H);
                open_j = seen - 1;
                open_here = true;
            } else {
                part_combine(p, c);
            }
        }
    }
    part_wave_reduce(p);
    if (l == 0) {
        const bool ends = FL ? ((ce >= n) || (flags[ce] & CV_FLAG_FIRST) != 0)
                             : ((ce >= n) || (jend != jprev) || (S > 1 && shard_start(soff, S, ce)));
        flush_part(acc, cap, open_j, p, open_here && ends);
    }
}

template <bool BOX, bool SHARDS, bool FL, int SI>
__global__ void __launch_bounds__(SB) k_sum_reduce(u32 n, const i64* __restrict__ jid, const double* __restrict__ lat,
                                                   const double* __restrict__ lon, const float* __restrict__ spd,
                                                   const double* __restrict__ step, const double* __restrict__ dspd,
                                                   const uint8_t* __restrict__ flags,
                                                   const u32* __restrict__ tile_prefix, const u32* __restrict__ wcnt,
                                                   u32 cap, Out o, JAcc* __restrict__ acc, AccX* __restrict__ accx,
                                                   const u64* __restrict__ soff, u32 S, u64* __restrict__ jo)
{
    sum_reduce<BOX, SHARDS, FL, SI>(n, jid, lat, lon, spd, step, dspd, flags, tile_prefix[blockIdx.x], wcnt, cap, o, acc,
                                    accx, soff, S, jo);
}

// The small form: both reductions in one launch (grid row 0 the box, row 1 the
// sums), the journeys before the tile counted here.
template <bool SHARDS, bool FL>
__global__ void __launch_bounds__(SB) k_sum_both(u32 n, const i64* __restrict__ jid, const double* __restrict__ lat,
                                                 const double* __restrict__ lon, const float* __restrict__ spd,
                                                 const double* __restrict__ step, const double* __restrict__ dspd,
                                                 const uint8_t* __restrict__ flags, const u32* __restrict__ tcnt,
                                                 const u32* __restrict__ wcnt, u32 cap, Out o, JAcc* __restrict__ acc,
                                                 AccX* __restrict__ accx, const u64* __restrict__ soff, u32 S,
                                                 u64* __restrict__ jo)
{
    __shared__ u32 s_t[NW];
    const u32 seen = block_count_sum(tcnt, blockIdx.x, s_t);
    if (blockIdx.y == 0)
        sum_reduce<true, SHARDS, FL, SI_S>(n, jid, lat, lon, spd, step, dspd, flags, seen, wcnt, cap, o, acc, accx,
                                           soff, S, jo);
    else
        sum_reduce<false, SHARDS, FL, SI_S>(n, jid, lat, lon, spd, step, dspd, flags, seen, wcnt, cap, o, acc, accx,
                                            soff, S, jo);
}

__global__ void __launch_bounds__(256) k_sum_finalize(const JAcc* __restrict__ acc, const AccX* __restrict__ accx,
                                                      const SumMeta* meta, u32 cap,
                                                      Out o, const i64* __restrict__ ts, cv_result* res,
                                                      const u64* __restrict__ soff, u32 S, u64* __restrict__ jo,
                                                      u32 n)
{
    u32 J = meta->J;
    u32 m = J < cap ? J : cap;
    for (u32 j = blockIdx.x * blockDim.x + threadIdx.x; j < m; j += gridDim.x * blockDim.x) {
        const JAcc& a = acc[j];
        Fx192 d, s;
        d.w[0] = a.dist[0];
        d.w[1] = a.dist[1];
        d.w[2] = a.dist[2];
        s.w[0] = a.spd[0];
        s.w[1] = a.spd[1];
        s.w[2] = a.spd[2];
        // values outside the 128-bit formats, added on their own
        const AccX& x = accx[j];
        Fx192 xd, xs;
        for (int i = 0; i < 3; ++i) {
            xd.w[i] = x.dist[i];
            xs.w[i] = x.spd[i];
        }
        fx_add(d, xd);
        fx_add(s, xs);
        write_final(o, j, a.count, a.ndtz, d, s, a.maxs, a.maxd, a.latmin, a.latmax, a.lonmin, a.lonmax);
        // a journey's records are consecutive: its time span is read at both ends
        o.tstart[j] = ts[a.gfirst];
        o.tend[j] = ts[a.gfirst + a.count - 1];
    }
    if (jo && blockIdx.x == 0 && threadIdx.x == 0) {
        // shards that start at the end of the records hold no journey
        jo[S] = J;
        for (int z = (int)S - 1; z >= 0 && soff[z] >= n; --z) jo[z] = J;
        if (S == 1) jo[0] = 0;
    }
    if (res && blockIdx.x == 0 && threadIdx.x == 0) {
        cv_result r = {};
        r.status = J > cap ? CV_ERR_CAPACITY : CV_OK;
        r.count = J;
        r.required = J > cap ? J : 0;
        *res = r;
    }
}

__global__ void k_sum_empty(cv_result* res)
{
    if (threadIdx.x == 0) {
        cv_result r = {};
        *res = r;
    }
}

struct SumLayout {
    SumMeta* meta;
    u32* wcnt;
    u32* tcnt;
    u32* tile_prefix;
    JAcc* acc;
    AccX* accx;
    u64 tiles;
    size_t bytes;
    SumLayout(void* ws, u64 n, u64 cap, int si = SI_L)
    {
        cvh::Carver c(ws);
        tiles = sum_tiles(n, si);
        meta = c.take<SumMeta>(1);
        wcnt = c.take<u32>(tiles * NW);
        tcnt = c.take<u32>(tiles + 1);
        tile_prefix = c.take<u32>(tiles + 1);
        acc = c.take<JAcc>(cap < n ? cap : n);
        accx = c.take<AccX>(cap < n ? cap : n);
        bytes = c.size();
    }
};

// windows per wave for n records (see SI_S); a workspace that holds only the
// coarsest form's tile counts gets that form
int sum_windows(u64 n, u64 cap, size_t ws_bytes)
{
    const int si = n <= N_S ? SI_S : (n <= N_M ? SI_M : SI_L);
    return SumLayout(nullptr, n, cap, si).bytes <= ws_bytes ? si : SI_L;
}

// bytes that hold every form for every record count up to n
size_t sum_bytes(u64 n, u64 cap)
{
    const size_t l = SumLayout(nullptr, n, cap).bytes;
    const size_t small = SumLayout(nullptr, n < N_S ? n : N_S, 0, SI_S).bytes;
    const size_t mid = SumLayout(nullptr, n < N_M ? n : N_M, 0, SI_M).bytes;
    return l + (small > mid ? small : mid);
}

struct SumArgs {
    const cv_records* r;
    const cv_features* f;
    const SumLayout* L;
    u32 cap;
    Out o;
    JAcc* acc;
    AccX* accx;
    const u64* soff;
    u32 S;
    u64* jo;
    hipStream_t s;
};

// tile counts, J, the rows' identities and both reductions, SI windows per wave.
// FL: journey starts from the FIRST flags, else from the ids.
template <bool SHARDS, bool FL, int SI>
void sum_launch_as(const SumArgs& a)
{
    const u32 n = (u32)a.r->n, tiles = (u32)a.L->tiles;
    const SumLayout& L = *a.L;
    if (FL)
        hipLaunchKernelGGL((k_sum_count_flags<SI>), dim3(tiles), dim3(SB), 0, a.s, a.f->flags, n, L.wcnt, L.tcnt);
    else
        hipLaunchKernelGGL((k_sum_count<SI>), dim3(tiles), dim3(SB), 0, a.s, a.r->journey_id, n, L.wcnt, L.tcnt, a.soff,
                           a.S);
    constexpr bool small = SI == SI_S;
    if (!small)
        hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(SCAN_B), 0, a.s, L.tcnt, L.tile_prefix, tiles, L.meta);
    hipLaunchKernelGGL(k_sum_init, dim3(cvh::grid_for(a.cap, SB, small ? 256 : 2048)), dim3(SB), 0, a.s, a.acc, a.accx,
                       L.meta, a.cap, small ? L.tcnt : (const u32*)nullptr, tiles);
    if (small) {
        hipLaunchKernelGGL((k_sum_both<SHARDS, FL>), dim3(tiles, 2), dim3(SB), 0, a.s, n, a.r->journey_id, a.r->lat_deg,
                           a.r->lon_deg, a.r->speed_mps, a.f->step_m, a.f->speed_mps, a.f->flags, L.tcnt, L.wcnt, a.cap,
                           a.o, a.acc, a.accx, a.soff, a.S, a.jo);
        return;
    }
    hipLaunchKernelGGL((k_sum_reduce<true, SHARDS, FL, SI>), dim3(tiles), dim3(SB), 0, a.s, n, a.r->journey_id,
                       a.r->lat_deg, a.r->lon_deg, a.r->speed_mps, a.f->step_m, a.f->speed_mps, a.f->flags,
                       L.tile_prefix, L.wcnt, a.cap, a.o, a.acc, a.accx, a.soff, a.S, a.jo);
    hipLaunchKernelGGL((k_sum_reduce<false, SHARDS, FL, SI>), dim3(tiles), dim3(SB), 0, a.s, n, a.r->journey_id,
                       a.r->lat_deg, a.r->lon_deg, a.r->speed_mps, a.f->step_m, a.f->speed_mps, a.f->flags,
                       L.tile_prefix, L.wcnt, a.cap, a.o, a.acc, a.accx, a.soff, a.S, a.jo);
}

template <bool SHARDS, bool FL>
void sum_launch(const SumArgs& a, int si)
{
    if (si == SI_S) sum_launch_as<SHARDS, FL, SI_S>(a);
    else if (si == SI_M) sum_launch_as<SHARDS, FL, SI_M>(a);
    else sum_launch_as<SHARDS, FL, SI_L>(a);
}

}  // namespace

static cv_status summary_impl(const cv_records* sorted, const cv_features* feat, const u64* soff, u32 S,
                              const cv_journeys* out, uint64_t capacity, u64* jo, cv_result* res, void* ws,
                              size_t ws_bytes, void* stream)
{
    if (!sorted || !feat || !out || sorted->n >= (1ull << 32) || capacity >= (1ull << 32))
        return CV_ERR_INVALID_ARGUMENT;
    const u64 n = sorted->n;
    hipStream_t s = (hipStream_t)stream;
    SumLayout need(nullptr, n, capacity);
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < need.bytes) return CV_ERR_WORKSPACE;
    if (n == 0) {
        if (res) hipLaunchKernelGGL(k_sum_empty, dim3(1), dim3(64), 0, s, res);
        if (jo) cvh::fill_u64(jo, 0, (u64)S + 1, s);
        return cvh::last_launch_status();
    }
    if (!sorted->journey_id || !sorted->ts_ms || !sorted->lat_deg || !sorted->lon_deg || !sorted->speed_mps ||
        !feat->step_m || !feat->speed_mps || !feat->flags)
        return CV_ERR_INVALID_ARGUMENT;
    if (capacity > 0 && (!out->journey_id || !out->first || !out->n_points || !out->t_start_ms || !out->t_end_ms ||
                         !out->distance_m || !out->sum_speed || !out->max_speed || !out->max_derived_speed ||
                         !out->n_dt_zero || !out->lat_min || !out->lat_max || !out->lon_min || !out->lon_max))
        return CV_ERR_INVALID_ARGUMENT;
    const int si = sum_windows(n, capacity, ws_bytes);
    SumLayout L(ws, n, capacity, si);
    Out o{out->journey_id, out->first, out->n_points, out->t_start_ms, out->t_end_ms, out->distance_m,
          out->sum_speed, out->max_speed, out->max_derived_speed, out->n_dt_zero, out->lat_min, out->lat_max,
          out->lon_min, out->lon_max};
    const u32 cap = (u32)(capacity < n ? capacity : n);
    const u32 nn = (u32)n;
    cvh::TimedScope ts_("summary", s);
    // journey starts come from the features' FIRST flags here (the features
    // of these records mark exactly the journey and shard starts)
    const SumArgs a{sorted, feat, &L, cap, o, L.acc, L.accx, soff, S, jo, s};
    if (S > 1) sum_launch<true, true>(a, si);
    else sum_launch<false, true>(a, si);
    hipLaunchKernelGGL(k_sum_finalize, dim3(cvh::grid_for(cap, 256, 2048)), dim3(256), 0, s, L.acc, L.accx, L.meta, cap, o,
                       sorted->ts_ms, res, soff, S, jo, nn);
    cvh::debug_rows(out->journey_id, nullptr, nullptr, res, cap, jo, S, CV_DEBUG_JOURNEY_ORDER, s);
    return cvh::last_launch_status();
}

// Workspace of the allocation-free entry point: one copy of this array per GPU
// (the code object's static device data), held until the process ends.  Host
// code reaches it only through the device address taken below; the array's
// name is not a device address on the host.
static __device__ __align__(256) unsigned char scratch[CV_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {};

// the array's address on the current device, taken once per device
void* noalloc_scratch()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return nullptr;
        }
        if (!cvh::aligned(p, cvh::WS_ALIGN)) return nullptr;
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

}  // namespace

namespace cv {

size_t sum_partials_bytes(u64 n) { return sum_bytes(n, 0); }

cv_status sum_partials(const cv_records* sorted, const cv_features* feat, u32 rows, JAcc* acc, AccX* accx, void* ws,
                       hipStream_t s)
{
    const u64 n = sorted->n;
    if (n == 0) return CV_OK;
    const int si = sum_windows(n, 0, ~(size_t)0);
    SumLayout L(ws, n, 0, si);
    sum_launch<false, false>(SumArgs{sorted, feat, &L, rows, Out{}, acc, accx, nullptr, 0u, nullptr, s}, si);
    return cvh::last_launch_status();
}

}  // namespace cv

extern "C" {

cv_status cv_summary_workspace_size(uint64_t n, uint64_t capacity, size_t* bytes)
{
    if (!bytes || n >= (1ull << 32)) return CV_ERR_INVALID_ARGUMENT;
    *bytes = sum_bytes(n, capacity);
    return CV_OK;
}

cv_status cv_journey_summary(const cv_records* sorted, const cv_features* feat, const cv_journeys* out,
                             uint64_t capacity, cv_result* res, void* ws, size_t ws_bytes, void* stream)
{
    return summary_impl(sorted, feat, nullptr, 0, out, capacity, nullptr, res, ws, ws_bytes, stream);
}

cv_status cv_journey_summary_noalloc(const cv_records* sorted, const cv_features* feat, const cv_journeys* out,
                                     uint64_t capacity, cv_result* res, void* stream)
{
    if (!sorted || sorted->n >= (1ull << 32) || capacity >= (1ull << 32)) return CV_ERR_INVALID_ARGUMENT;
    SumLayout need(nullptr, sorted->n, capacity);
    if (need.bytes > (size_t)CV_NOALLOC_SCRATCH_BYTES) return CV_ERR_WORKSPACE;
    void* ws = noalloc_scratch();
    if (!ws) return CV_ERR_DEVICE;
    return summary_impl(sorted, feat, nullptr, 0, out, capacity, nullptr, res, ws, (size_t)CV_NOALLOC_SCRATCH_BYTES,
                        stream);
}

cv_status cv_batch_journey_summary(const cv_records* sorted, const cv_features* feat, const uint64_t* shard_offsets,
                                   uint32_t n_shards, const cv_journeys* out, uint64_t capacity,
                                   uint64_t* journey_offsets, cv_result* res, void* ws, size_t ws_bytes, void* stream)
{
    if (n_shards == 0 || !shard_offsets || !journey_offsets || !cvh::aligned(shard_offsets, 8) ||
        !cvh::aligned(journey_offsets, 8))
        return CV_ERR_INVALID_ARGUMENT;
    return summary_impl(sorted, feat, shard_offsets, n_shards, out, capacity, journey_offsets, res, ws, ws_bytes,
                        stream);
}

}  // extern "C"
