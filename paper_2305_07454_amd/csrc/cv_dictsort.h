// cv_dictsort.h -- order of the record sort's distinct ids, and each id's rank.
//
// The distinct ids are few (a full day has 50 000) and their order is needed
// before any record's key, so what it costs is launches and latency, not
// bytes: eight radix passes with their histogram and scan took 11 launches and
// about 110 us of every sort.  Here:
//   up to DS_COUNT ids   an id's rank is the count of smaller ids, each id
//                        compared with all: one launch without a barrier
//                        chain (a block's bitonic network over 2 048 ids took
//                        35 us, this takes 10, and 18 with shards or 5 000 ids);
//   more, when the caller's capacity allows at most DS_MERGE ids
//                        every chunk of DS_CHUNK ids is sorted by a block, then
//                        each id's rank among DS_FAN sorted chunks is its place
//                        in its own plus a binary search in every other one;
//                        a second such step joins the groups of chunks.
// The counts grow with the square of the ids (16 384: 20 us; at 32 768 they
// would take as long as the chunks, 80 us), the searches with their number:
// above DS_MERGE ids they (DS_FAN x 12 reads per id and step) cost more than the
// radix passes, which keep that range (the caller launches them for such
// capacities; they leave at once when the ids turn out to be few).
// Ids are ordered by (shard, id image); without shards the shard words are
// absent.
#pragma once
#include "cv_device.h"

namespace cv {
namespace {

constexpr int DS_B = 1024;             // threads of a sorting block
constexpr u32 DS_COUNT = 16384;        // ids ranked by counting
constexpr u32 DS_CHUNK = 4096;         // ids per sorted chunk (48 KB of LDS with shards)
constexpr u32 DS_FAN = 16;             // sorted chunks joined by one step
constexpr u64 DS_MERGE = 512 * 1024;   // capacity up to which chunks are sorted and joined

// Sorts n <= DS_CHUNK (shard, id) pairs of LDS in place (all DS_B threads).
template <bool SH>
__device__ __forceinline__ void ds_block_sort(u64* k, u32* sh, u32 n)
{
    u32 m = 2;
    while (m < n) m <<= 1;
    for (u32 i = n + threadIdx.x; i < m; i += DS_B) {
        k[i] = ~0ull;
        if (SH) sh[i] = ~0u;
    }
    __syncthreads();
    for (u32 size = 2; size <= m; size <<= 1) {
        for (u32 d = size >> 1; d > 0; d >>= 1) {
            for (u32 t = threadIdx.x; t < m / 2; t += DS_B) {
                const u32 a = 2 * t - (t & (d - 1)), b = a + d;  // the pair's places
                const bool up = (a & size) == 0;
                const u64 x = k[a], y = k[b];
                bool gt = x > y;
                u32 p = 0, q = 0;
                if (SH) {
                    p = sh[a];
                    q = sh[b];
                    gt = p > q || (p == q && gt);
                }
                if (gt == up) {
                    k[a] = y;
                    k[b] = x;
                    if (SH) {
                        sh[a] = q;
                        sh[b] = p;
                    }
                }
            }
            __syncthreads();
        }
    }
}

// Chunk blockIdx.x of the list (DS_CHUNK ids), sorted into out (which may be the
// list); tag: the ids' shards (SH), sorted in place, all taken as 0 when *multi.
template <bool SH>
__global__ void __launch_bounds__(DS_B) k_ds_chunks(const u64* list, u64* out, u64* __restrict__ tag,
                                                    const u32* __restrict__ n_dev, const u32* __restrict__ multi)
{
    __shared__ u64 s_k[DS_CHUNK];
    __shared__ u32 s_s[SH ? DS_CHUNK : 1];
    const u32 n = *n_dev, a = blockIdx.x * DS_CHUNK;
    if (a >= n) return;
    const u32 c = n - a < DS_CHUNK ? n - a : DS_CHUNK;
    const bool one = SH && *multi;
    for (u32 i = threadIdx.x; i < c; i += DS_B) {
        s_k[i] = list[a + i];
        if (SH) s_s[i] = one ? 0u : (u32)tag[a + i];
    }
    __syncthreads();
    ds_block_sort<SH>(s_k, s_s, c);
    for (u32 i = threadIdx.x; i < c; i += DS_B) {
        out[a + i] = s_k[i];
        if (SH) tag[a + i] = s_s[i];
    }
}

// Ranks by counting, for the WAVE ids from blockIdx.x * WAVE on: lane l of every
// wave holds id l, each wave goes through its share of the list with uniform
// (scalar) reads, and wave 0 adds the waves' counts and calls done(r, id).
template <bool SH, class Done>
__device__ __forceinline__ void ds_count(const u64* __restrict__ list, const u64* __restrict__ tag, u32 n, bool multi,
                                         Done done)
{
    constexpr int NWD = DS_B / WAVE;
    __shared__ u32 s_c[NWD][WAVE];
    const u32 i0 = blockIdx.x * WAVE;
    if (i0 >= n) return;
    const int l = lane_id();
    const u32 w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const u32 i = i0 + l < n ? i0 + l : n - 1;
    const bool sh = SH && !multi;  // (one id in several shards: the order is by id alone)
    const u64 key = list[i], own = sh ? tag[i] : 0ull;
    const u32 per = (n + NWD - 1) / NWD;
    const u32 a = w * per, b = a + per < n ? a + per : n;
    u32 c = 0;
    if (sh) {
#pragma unroll 8
        for (u32 j = a; j < b; ++j) {
            const u64 t = tag[j];
            c += (t < own || (t == own && list[j] < key)) ? 1u : 0u;
        }
    } else {
#pragma unroll 8
        for (u32 j = a; j < b; ++j) c += list[j] < key ? 1u : 0u;
    }
    s_c[w][l] = c;
    __syncthreads();
    if (w != 0 || i0 + l >= n) return;
    u32 r = 0;
#pragma unroll
    for (int k = 0; k < NWD; ++k) r += s_c[k][l];
    done(r, key);
}

// The same for (id, run) pairs without shards, with the records of the smaller
// ids' runs (high half: start, low half: end) added up: done(r, id, before, run).
template <class Done>
__device__ __forceinline__ void ds_count_runs(const u64* __restrict__ list, const u64* __restrict__ runs, u32 n,
                                              Done done)
{
    constexpr int NWD = DS_B / WAVE;
    __shared__ u32 s_n[NWD][WAVE], s_r[NWD][WAVE];
    const u32 i0 = blockIdx.x * WAVE;
    if (i0 >= n) return;
    const int l = lane_id();
    const u32 w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const u32 i = i0 + l < n ? i0 + l : n - 1;
    const u64 key = list[i];
    const u32 per = (n + NWD - 1) / NWD;
    const u32 a = w * per, b = a + per < n ? a + per : n;
    u32 c = 0, rec = 0;
#pragma unroll 8
    for (u32 j = a; j < b; ++j) {
        const u64 run = runs[j];
        const bool less = list[j] < key;
        c += less ? 1u : 0u;
        rec += less ? (u32)run - (u32)(run >> 32) : 0u;
    }
    s_n[w][l] = c;
    s_r[w][l] = rec;
    __syncthreads();
    if (w != 0 || i0 + l >= n) return;
    u32 r = 0, before = 0;
#pragma unroll
    for (int k = 0; k < NWD; ++k) {
        r += s_n[k][l];
        before += s_r[k][l];
    }
    done(r, key, before, runs[i]);
}

// One step of the join: runs of `run` sorted ids, DS_FAN of them to a group.
// Id i goes to its group's start plus its place in its own run plus the count
// of smaller ids in each other run of the group (ids are distinct).  The
// searches of four runs go on together, since each is a chain of dependent
// reads.  done(r, id) is called for the id at final place r.
template <bool SH, class Done>
__device__ __forceinline__ void ds_join(const u64* __restrict__ in, const u64* __restrict__ tin, u32 n, u32 run,
                                        u64* __restrict__ out, u64* __restrict__ tout, Done done)
{
    for (u32 i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const u64 key = in[i];
        const u64 sh = SH ? tin[i] : 0ull;
        const u32 own = i / run, g0 = own / DS_FAN * DS_FAN;
        u32 r = g0 * run + (i - own * run);
        for (u32 q = g0; q < g0 + DS_FAN && (u64)q * run < n; q += 4) {
            u32 lo[4], hi[4];
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                const u64 b = (u64)(q + z) * run;
                const bool on = q + z != own && b < n;
                lo[z] = on ? (u32)b : 0u;
                hi[z] = on ? (u32)(b + run < n ? b + run : n) : 0u;
                r -= lo[z];
            }
            bool more = true;
            while (more) {
                more = false;
#pragma unroll
                for (int z = 0; z < 4; ++z) {
                    if (lo[z] >= hi[z]) continue;
                    const u32 mid = (lo[z] + hi[z]) >> 1;
                    bool less;
                    if (SH) {
                        const u64 t = tin[mid];
                        less = t < sh || (t == sh && in[mid] < key);
                    } else {
                        less = in[mid] < key;
                    }
                    if (less) lo[z] = mid + 1;
                    else hi[z] = mid;
                    more |= lo[z] < hi[z];
                }
            }
#pragma unroll
            for (int z = 0; z < 4; ++z) r += lo[z];
        }
        out[r] = key;
        if (SH && tout) tout[r] = sh;
        done(r, key);
    }
}

}  // namespace
}  // namespace cv
