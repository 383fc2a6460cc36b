// cv_dictsort.h -- order of the record sort's distinct ids, and each id's rank.
//
// The distinct ids are few (a full day has 50 000) and their order is needed
// before any record's key, so what it costs is launches and latency, not
// bytes: eight radix passes with their histogram and scan took 11 launches and
// about 110 us of every sort.  Here:
//   up to DS_ONE ids     one block sorts them in LDS (a bitonic network over the
//                        next power of two) and writes their ranks;
//   more, when the caller's capacity allows at most DS_MERGE ids
//                        every chunk of DS_ONE ids is sorted by a block, then
//                        each id's rank among DS_FAN sorted chunks is its place
//                        in its own plus a binary search in every other one;
//                        a second such step joins the groups of chunks.
// With 400 to 50 000 ids a sort takes 60 to 110 us less than with the radix
// passes (1 M shuffled records of 2 000 journeys 685 -> 614 us per pass of the
// whole path, 12.3 M records of 5 000 journeys 1 283 -> 1 214 us, a batch of
// 2 M records 963 -> 775 us).
// Above DS_MERGE ids the searches (DS_FAN x 12 reads per id and step) cost more
// than the radix passes, which keep that range (the caller launches them for
// such capacities; they leave at once when the ids turn out to be few).
// Ids are ordered by (shard, id image); without shards the shard words are
// absent.
#pragma once
#include "cv_device.h"

namespace cv {
namespace {

constexpr int DS_B = 1024;             // threads of a sorting block
constexpr u32 DS_ONE = 4096;           // ids per block (48 KB of LDS with shards)
constexpr u32 DS_FAN = 16;             // sorted chunks joined by one step
constexpr u64 DS_MERGE = 512 * 1024;   // capacity up to which chunks are sorted and joined

// Sorts n <= DS_ONE (shard, id) pairs of LDS in place (all DS_B threads).
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

// Chunk blockIdx.x of the list (DS_ONE ids), sorted into out (which may be the
// list); tag: the ids' shards (SH), sorted in place, all taken as 0 when *multi.
template <bool SH>
__global__ void __launch_bounds__(DS_B) k_ds_chunks(const u64* list, u64* out, u64* __restrict__ tag,
                                                    const u32* __restrict__ n_dev, const u32* __restrict__ multi)
{
    __shared__ u64 s_k[DS_ONE];
    __shared__ u32 s_s[SH ? DS_ONE : 1];
    const u32 n = *n_dev, a = blockIdx.x * DS_ONE;
    if (a >= n) return;
    const u32 c = n - a < DS_ONE ? n - a : DS_ONE;
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
