// cv_radix.hip -- kernels and host launchers of the stable LSD radix sort
// described in cv_radix.h.
#include <hip/hip_runtime.h>

#include <string>
#include <type_traits>

#include "cv_host.h"
#include "cv_radix.h"

namespace cv {

namespace {

// status word: [flag:2 | tag:6 | value:56]; the tag (pass + 1) lets all passes
// of one sort share one status array cleared once per sort.
__device__ __forceinline__ u64 rs_word(u64 flag, u32 tag, u64 v) { return (flag << 62) | ((u64)tag << 56) | v; }

// Histogram of all digits of all passes.  hist[p * RADIX + d].
__global__ void __launch_bounds__(256) k_radix_hist(const u64* __restrict__ keys, u32 n_max,
                                                    const u32* __restrict__ n_dev, int passes,
                                                    const u32* __restrict__ bits_dev, u32* __restrict__ hist)
{
    __shared__ u32 s_h[MAX_PASSES * RADIX];
    for (int i = threadIdx.x; i < MAX_PASSES * RADIX; i += blockDim.x) s_h[i] = 0;
    __syncthreads();
    u32 n = n_dev ? *n_dev : n_max;
    int np = passes;
    if (bits_dev) {
        int b = (int)*bits_dev;
        int need = (b + RADIX_BITS - 1) / RADIX_BITS;
        np = need < np ? need : np;
    }
    // the loop runs the same trips in every lane of a wave (whole waves per
    // stride); a digit shared by every valid lane adds once
    const u32 stride = gridDim.x * blockDim.x;
    const u32 first = blockIdx.x * blockDim.x + (threadIdx.x & ~(u32)(WAVE - 1));
    for (u32 b = first; b < n; b += stride) {
        const u32 i = b + (u32)lane_id();
        const bool ok = i < n;
        const u64 k = ok ? keys[i] : 0ull;
        const u64 vm = __ballot(ok);
        const int lead = __ffsll((long long)vm) - 1;
        for (int p = 0; p < np; ++p) {
            const u32 d = (u32)(k >> (p * RADIX_BITS)) & (RADIX - 1);
            const u32 d0 = __shfl(d, lead, WAVE);
            if (__ballot(ok && d != d0) == 0) {
                if (lane_id() == lead) atomicAdd(&s_h[p * RADIX + d0], (u32)__popcll(vm));
            } else if (ok) {
                atomicAdd(&s_h[p * RADIX + d], 1u);
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < np * RADIX; i += blockDim.x)
        if (s_h[i]) atomicAdd(&hist[i], s_h[i]);
}

// LDS of a pass over tiles of B x I keys with digits of DB bits at most.
template <int B, int I, int DB>
struct RadixLds {
    // staging: keys in digit order; then, in passes that carry index values,
    // the values in the same order (the buffer reused as 32-bit words)
    u64 keys[B * I];
    u64 tmp[B / WAVE];
    u32 start[1 << DB], gshift[1 << DB];
    uint16_t whist[(B / WAVE) << DB];  // per-wave digit counts, then in-tile offsets (< tile, so 16 bits)
};

// What a pass needs besides its tile.
struct RadixPass {
    const u64* keys_in;
    const u32* vals_in;  // nullptr: the identity (input index)
    u64* keys_out;
    u32* vals_out;
    u64* status;
    u32 n, tag, ib;
    u32 dcnt;   // the pass's global count of digit threadIdx.x
    int shift;  // the digit's lowest bit in the input words
    int drop;   // key bits dropped by the pass that starts packing
    bool pin, pout;  // input / output words are packed
    bool tin, tout;  // words loaded / stored past the L2
};

// Key and value words of a pass.  THROUGH: the pass before (loads) or after it
// (stores) runs in the same launch, on any XCD: the words go past the XCD's L2.
template <bool THROUGH, class T>
__device__ __forceinline__ T word_load(const T* p)
{
    return THROUGH ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
template <bool THROUGH, class T>
__device__ __forceinline__ void word_store(T* p, T v)
{
    if (THROUGH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = v;
}

// One tile of a stable scatter pass on a digit of DB bits.  whist is clear and
// every thread of the block has seen it so.
template <int SORT_BLOCK, int SORT_ITEMS, int DB, class Lds>
__device__ __forceinline__ void radix_tile(Lds& s, const RadixPass& a, u32 tile)
{
    constexpr int NW = SORT_BLOCK / WAVE;
    constexpr int SORT_TILE = SORT_BLOCK * SORT_ITEMS;
    constexpr int RK = 1 << DB;  // digit values
    static_assert(SORT_BLOCK >= RK, "one thread per digit");
    static_assert(SORT_TILE <= 65535, "16-bit in-tile offsets");
    const u64 n = a.n;
    const u64 tile_base = (u64)tile * SORT_TILE;
    const int shift = a.shift;
    const int w = threadIdx.x / WAVE;
    const int l = lane_id();
    uint16_t* whist = s.whist + w * RK;
    u64 key[SORT_ITEMS];
    u32 val[SORT_ITEMS];
    u32 rnk[SORT_ITEMS];
    const u64 wbase = tile_base + (u64)w * (SORT_ITEMS * WAVE);
    auto load = [&](auto through) {
#pragma unroll
        for (int i = 0; i < SORT_ITEMS; ++i) {
            u64 idx = wbase + (u64)i * WAVE + l;
            bool ok = idx < n;
            key[i] = ok ? word_load<through()>(a.keys_in + idx) : ~0ull;
            val[i] = (ok && !a.pin) ? (a.vals_in ? word_load<through()>(a.vals_in + idx) : (u32)idx) : 0u;
        }
    };
    if (a.tin) load(std::true_type());
    else load(std::false_type());
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) {
        u64 idx = wbase + (u64)i * WAVE + l;
        bool ok = idx < n;
        u32 d = (u32)(key[i] >> shift) & (RK - 1);
        const u64 peers = wave_peers<DB>(d, __ballot(ok));
        u32 below = popc_below(peers);
        u32 cnt = __popcll(peers);
        u32 before = ok ? (u32)whist[d] : 0u;
        rnk[i] = before + below;
        __builtin_amdgcn_wave_barrier();
        if (ok && below == cnt - 1) whist[d] = (uint16_t)(before + cnt);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // per digit: exclusive offsets across waves, tile count
    u32 tcount = 0;
    if (threadIdx.x < RK) {
        const int d = threadIdx.x;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            u32 c = s.whist[ww * RK + d];
            s.whist[ww * RK + d] = (uint16_t)tcount;
            tcount += c;
        }
    }
    // one scan for the tile's digit starts and (high word) the pass's global
    // ones: a scan kernel between the histogram and the passes cost a launch
    u64 total;
    const u64 ex =
        block_exclusive_sum<SORT_BLOCK>(((u64)a.dcnt << 32) | (threadIdx.x < RK ? tcount : 0u), s.tmp, total);
    const u32 start = (u32)ex, doff = (u32)(ex >> 32);
    if (threadIdx.x < RK) {
        s.start[threadIdx.x] = start;
        // this tile's digit count, for the look-back of later tiles
        lb_publish(a.status + (u64)tile * RK + threadIdx.x, rs_word(tile == 0 ? 2 : 1, a.tag, tcount));
    }
    __syncthreads();

    // keys to LDS in digit order (stable); the look-back below overlaps with
    // the other threads' staging
    u32 pos[SORT_ITEMS];
#pragma unroll
    for (int i = 0; i < SORT_ITEMS; ++i) {
        u64 idx = wbase + (u64)i * WAVE + l;
        pos[i] = ~0u;
        if (idx < n) {
            u32 d = (u32)(key[i] >> shift) & (RK - 1);
            pos[i] = s.start[d] + whist[d] + rnk[i];
            s.keys[pos[i]] = key[i];
        }
    }
    if (threadIdx.x < RK) {
        const int d = threadIdx.x;
        // look-back for digit d over earlier tiles of this pass
        u64 excl = 0;
        if (tile != 0) {
            // LBW tiles at a time (their status words read together): take
            // aggregates in order up to the first inclusive prefix; stop early
            // at a tile that has not published yet and read again from it
            constexpr int LBW = 4;
            long t = (long)tile - 1;
            bool done = false;
            while (!done) {
                u64 wv[LBW];
#pragma unroll
                for (int j = 0; j < LBW; ++j)
                    wv[j] = t - j >= 0 ? lb_peek(a.status + (u64)(t - j) * RK + d) : 0ull;
                int used = 0;
#pragma unroll
                for (int j = 0; j < LBW; ++j) {
                    if (done || used < j) break;  // stopped earlier in this batch
                    const u32 hdr = (u32)(wv[j] >> 56);
                    if (t - j < 0 || (hdr & 63u) != a.tag) break;
                    excl += wv[j] & ((1ull << 56) - 1);
                    used = j + 1;
                    if ((hdr >> 6) == 2u) done = true;
                }
                t -= used;
                if (!done && used < LBW) __builtin_amdgcn_s_sleep(1);
            }
            lb_publish(a.status + (u64)tile * RK + d, rs_word(2, a.tag, excl + tcount));
        }
        s.gshift[d] = doff + (u32)excl - start;
    }
    __syncthreads();
    const u32 tvalid = (u32)((n - tile_base) < (u64)SORT_TILE ? (n - tile_base) : (u64)SORT_TILE);
    // read back the staged keys this thread writes out: positions t + k * SORT_BLOCK
    u64 kk[SORT_ITEMS];
#pragma unroll
    for (int k = 0; k < SORT_ITEMS; ++k) {
        const u32 j = threadIdx.x + (u32)k * SORT_BLOCK;
        kk[k] = j < tvalid ? s.keys[j] : 0ull;
    }
    auto store = [&](auto through) {
        constexpr bool TH = through();
        if (a.pin) {
#pragma unroll
            for (int k = 0; k < SORT_ITEMS; ++k) {
                const u32 j = threadIdx.x + (u32)k * SORT_BLOCK;
                if (j < tvalid) word_store<TH>(a.keys_out + s.gshift[(u32)(kk[k] >> shift) & (RK - 1)] + j, kk[k]);
            }
            return;
        }
        // the index values follow the keys through the same staging buffer
        __syncthreads();
        u32* s_vals = (u32*)s.keys;
#pragma unroll
        for (int i = 0; i < SORT_ITEMS; ++i)
            if (pos[i] != ~0u) s_vals[pos[i]] = val[i];
        __syncthreads();
        // the pass that starts packing packs on the way out
#pragma unroll
        for (int k = 0; k < SORT_ITEMS; ++k) {
            const u32 j = threadIdx.x + (u32)k * SORT_BLOCK;
            if (j < tvalid) {
                const u32 g = s.gshift[(u32)(kk[k] >> shift) & (RK - 1)] + j;
                const u32 v = s_vals[j];
                if (a.pout) {
                    const u64 top = a.drop >= 64 ? 0ull : (kk[k] >> a.drop);
                    word_store<TH, u64>(a.keys_out + g, (top << a.ib) | (u64)v);
                } else {
                    word_store<TH, u64>(a.keys_out + g, kk[k]);
                    word_store<TH, u32>(a.vals_out + g, v);
                }
            }
        }
    };
    if (a.tout) store(std::true_type());
    else store(std::false_type());
}

// Packing and first digit of a sort, read from device memory.  From pass p0 on, a
// key word holds (key >> 8 p0) << ib | index (a wide first digit only with p0 = 0).
struct RadixForm {
    u32 ib, w0;
    int p0;
    __device__ __forceinline__ explicit RadixForm(const u32* pack) : ib(0), w0(RADIX_BITS), p0(1 << 20)
    {
        if (!pack) return;
        ib = pack[0];
        p0 = (int)pack[1];
        w0 = pack[2] == RADIX_BITS + 1 ? RADIX_BITS + 1 : RADIX_BITS;
    }
    // the lowest key bit of a pass's digit
    __device__ __forceinline__ int low(int pass) const { return pass == 0 ? 0 : (int)w0 + (pass - 1) * RADIX_BITS; }
    __device__ __forceinline__ void set(RadixPass& a, int pass) const
    {
        a.tag = (u32)pass + 1;
        a.ib = ib;
        a.pin = pass >= p0;
        a.pout = pass + 1 >= p0;
        a.drop = p0 * RADIX_BITS;
        a.shift = a.pin ? (int)ib + low(pass) - a.drop : low(pass);
    }
};

// One stable scatter pass on digit `pass`: bits [8*pass, 8*pass+8), or, with
// a first digit of w0 = pack[2] bits (9): [0, w0) for pass 0 and
// [w0 + 8 (pass - 1), w0 + 8 pass) after it.  DB: bits of the digit this
// instantiation handles (8, or 9 for a wide first digit; a launch whose
// width is not the pass's leaves at once).
// vals_in == nullptr means the identity (input index).  LOOP: a block goes on
// taking tiles (a grid smaller than the tile count); otherwise it takes one.
template <int SORT_BLOCK, int SORT_ITEMS, bool LOOP, int DB = RADIX_BITS>
__global__ void __launch_bounds__(SORT_BLOCK)
k_radix_pass(const u64* __restrict__ keys_in, const u32* __restrict__ vals_in, u64* __restrict__ keys_out,
             u32* __restrict__ vals_out, u32 n_max, const u32* __restrict__ n_dev, int pass,
             const u32* __restrict__ bits_dev, const u32* __restrict__ hist, u64* __restrict__ status,
             u32* __restrict__ ticket, const u32* __restrict__ pack)
{
    constexpr int SORT_TILE = SORT_BLOCK * SORT_ITEMS;
    __shared__ RadixLds<SORT_BLOCK, SORT_ITEMS, DB> s;
    __shared__ u32 s_tile;

    // the launch's scalars from device memory, all loaded before any is used
    const RadixForm form(pack);
    const u32 bits = bits_dev ? *bits_dev : ~0u;
    const u32 n = n_dev ? *n_dev : n_max;
    if ((pass == 0 ? (int)form.w0 : RADIX_BITS) != DB) return;  // the other width's launch takes this pass
    if ((u32)form.low(pass) >= bits) return;
    RadixPass a{keys_in, vals_in, keys_out, vals_out, status, n};
    form.set(a, pass);
    a.tin = a.tout = false;
    a.dcnt = threadIdx.x < (1 << DB) ? hist[threadIdx.x] : 0u;
    // Tiles are taken by ticket (with LOOP, until the tickets pass the last
    // tile, so a grid smaller than the tile count covers every tile); a tile
    // waits only on tiles whose tickets were taken before, by blocks already
    // running.
    // A block of a one-tile-per-block grid sized for n_max whose tile lies past
    // a count read on the device leaves before it takes a ticket: exactly the
    // first ceil(n / tile) blocks take the tickets 0 .. ceil(n / tile) - 1,
    // and the idle ones put no load on the ticket counter.
    if (!LOOP && (u64)blockIdx.x * SORT_TILE >= n) return;
    for (;;) {
        if (threadIdx.x == 0) s_tile = atomicAdd(ticket, 1u);
        for (int i = threadIdx.x; i < (SORT_BLOCK / WAVE) << DB; i += SORT_BLOCK) s.whist[i] = 0;
        __syncthreads();
        const u32 tile = s_tile;
        if ((u64)tile * SORT_TILE >= n) return;
        radix_tile<SORT_BLOCK, SORT_ITEMS, DB>(s, a, tile);
        if constexpr (!LOOP) return;
        __syncthreads();  // LDS free for the next tile
    }
}

// Every pass of a small sort in one launch: its passes are a few tiles each,
// and those of digits that the keys turn out not to have are launches that do
// nothing, each as long on the stream as a working one's start (4.5 us), and as
// long to enqueue for a host that is the slower of the two.
// Tickets run through the tiles of pass after pass.  A tile of a later pass
// waits until the pass before it has counted all its tiles as done (tickets[1 +
// pass]), that is, on earlier tickets only, whose blocks run: no block waits
// for one that has not started.
struct RadixAll {
    u64 *k0, *k1;
    const u32* v_first;
    u32 *v0, *v1;
    u32 n_max;
    const u32* n_dev;
    int max_passes;
    const u32* bits_dev;
    const u32* hist;
    u32 wide;
    u64* status;
    u32* tickets;
    const u32* pack;
};
template <int SORT_BLOCK, int SORT_ITEMS, class Lds>
__device__ __forceinline__ void radix_all(const RadixAll& r, u32 n, Lds& s, u32& s_tile)
{
    constexpr u32 SORT_TILE = SORT_BLOCK * SORT_ITEMS;
    u64 *const k0 = r.k0, *const k1 = r.k1;
    u32 *const v0 = r.v0, *const v1 = r.v1, *const tickets = r.tickets;
    const RadixForm form(r.pack);
    const u32 bits = r.bits_dev ? *r.bits_dev : ~0u;
    const int max_passes = r.max_passes;
    int np = 0;
    while (np < max_passes && (u32)form.low(np) < bits) ++np;
    const u32 tiles = (u32)(((u64)n + SORT_TILE - 1) / SORT_TILE);
    if (np == 0 || blockIdx.x >= tiles) return;
    for (;;) {
        if (threadIdx.x == 0) s_tile = atomicAdd(&tickets[0], 1u);
        for (int i = threadIdx.x; i < (SORT_BLOCK / WAVE) << (RADIX_BITS + 1); i += SORT_BLOCK) s.whist[i] = 0;
        __syncthreads();
        u32 tile = s_tile;
        int pass = 0;
        for (; pass < np && tile >= tiles; ++pass) tile -= tiles;
        if (pass == np) return;
        if (pass > 0) {
            if (threadIdx.x == 0) {
                while (__hip_atomic_load(&tickets[pass], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < tiles)
                    __builtin_amdgcn_s_sleep(4);
            }
            __syncthreads();
        }
        RadixPass a{(pass & 1) ? k1 : k0, pass == 0 ? r.v_first : ((pass & 1) ? v1 : v0), (pass & 1) ? k0 : k1,
                    (pass & 1) ? v0 : v1, r.status, n};
        form.set(a, pass);
        a.tin = pass > 0;
        a.tout = pass + 1 < np;
        const u32* h = r.hist + (r.wide ? hist_wide_off(pass) : pass * RADIX);
        if (pass == 0 && form.w0 == RADIX_BITS + 1) {
            a.dcnt = threadIdx.x < 2 * RADIX ? h[threadIdx.x] : 0u;
            radix_tile<SORT_BLOCK, SORT_ITEMS, RADIX_BITS + 1>(s, a, tile);
        } else {
            a.dcnt = threadIdx.x < RADIX ? h[threadIdx.x] : 0u;
            radix_tile<SORT_BLOCK, SORT_ITEMS, RADIX_BITS>(s, a, tile);
        }
        // Each thread's words have arrived before the tile is counted.  They were
        // written through, so that this wait is enough; a fence at agent scope
        // would write back the XCD's L2 for every tile (1 M keys, four passes:
        // 92 us, 339 with a fence of every wave, 79 written through).
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        __syncthreads();                     // LDS free for the next tile
        if (pass + 1 < np && threadIdx.x == 0)
            __hip_atomic_fetch_add(&tickets[1 + pass], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
template <int B, int I>
__global__ void __launch_bounds__(B) k_radix_all(RadixAll r)
{
    __shared__ RadixLds<B, I, RADIX_BITS + 1> s;
    __shared__ u32 s_tile;
    radix_all<B, I>(r, r.n_dev ? *r.n_dev : r.n_max, s, s_tile);
}
// the tile by a count known on the device alone
constexpr u32 ALL_SMALL = 1u << 19;  // keys up to which tiles of 512 x 8 are the better ones
template <int B>
__global__ void __launch_bounds__(B) k_radix_all_counted(RadixAll r)
{
    __shared__ union {
        RadixLds<B, 8, RADIX_BITS + 1> small;
        RadixLds<B, 16, RADIX_BITS + 1> large;
    } s;
    __shared__ u32 s_tile;
    const u32 n = *r.n_dev;
    if (n <= ALL_SMALL) radix_all<B, 8>(r, n, s.small, s_tile);
    else radix_all<B, 16>(r, n, s.large, s_tile);
}

}  // namespace

void radix_hist(const u64* keys, u32 n_max, const u32* n_dev, int passes, const u32* bits_dev, u32* hist,
                int grid, hipStream_t s)
{
    hipLaunchKernelGGL(k_radix_hist, dim3(grid), dim3(256), 0, s, keys, n_max, n_dev, passes, bits_dev, hist);
}

namespace {

// A pass whose record count is read on the device launches one block per
// tile of n_max (the blocks past the count leave at once) up to
// DEVICE_COUNT_MAX_TILES tiles; beyond that, DEVICE_COUNT_GRID blocks that
// loop over tiles (a form that needs more registers, so fewer blocks per CU).
constexpr u64 DEVICE_COUNT_GRID = 2048;
constexpr u64 DEVICE_COUNT_MAX_TILES = 1ull << 17;

// Sorts of few keys take all passes in one launch, whatever the shape: tiles of 512 x 8
// keys where the chip has idle CUs left (500 000 keys, three passes that work: 84 ->
// 49 us; 30 000: 46 -> 26), of 512 x 16 above (1 M, four passes: 108 -> 82; 2 M, two:
// 88 -> 59).  A pass between others writes its words through, some 8-byte runs
// at a time, and at 2 M keys and four passes that takes what the launches saved
// (126, 128 us; 4 M 157, 211).  A count known on the device alone may be far below
// its bound or come near it, so the kernel picks the tile, and the line lies where
// one launch costs the second little more than launches per pass and the first less:
//   few   distinct ids, a flush's rows (the record sort whole, one launch / per pass):
//         3 M ids allowed, 5 000 there 498 / 508 us, all there 1575 / 1466 (1680 when
//         each pass read its offsets from a scan's launch); 4.1 M 603 / 615, 2008 / 1871
//         (2022);
//   rows  the grid's partial rows (the whole call; every record one of its own: random
//         places): 1.2 M records at 0.001 deg x 1 min 101 / 109, random 306 / 304; 2 M 115 /
//         123, 378 / 369; 3 M 140 / 149, 616 / 584 (567 with the scan); 4.1 M 161 / 169, 749 /
//         712 (722);
//   many  the same with directions: a row for every two or three records.
// Tiles of 512 x 8 alone took 452 us for 2 M random records, 2375 for 4.1 M distinct ids.
constexpr int ALL_B = 512;
constexpr int ALL_GRID = 512;
enum class AllForm { none, small, large, counted };  // none: a launch per pass
AllForm all_form(u64 n_max, RadixCount count)
{
    if (n_max <= ALL_SMALL) return AllForm::small;
    switch (count) {
    case RadixCount::exact: return n_max <= (1u << 21) ? AllForm::large : AllForm::none;
    case RadixCount::few:
    case RadixCount::rows: return n_max <= (1u << 22) ? AllForm::counted : AllForm::none;
    default: return AllForm::none;
    }
}

// tile shapes compiled into the library; the sort uses sort_shape()
struct Shape {
    int block, items;
};
// (every shape has at least one thread per digit)
constexpr Shape SHAPES[] = {{256, 16}, {256, 32}, {512, 8}, {512, 16}, {1024, 8}, {1024, 16}};
constexpr int N_SHAPES = sizeof(SHAPES) / sizeof(SHAPES[0]);
int g_shape = 0;
bool g_wide_first = true;  // tuning "radix_wide_first"

template <int B, int I, int DB = RADIX_BITS>
void launch_pass(u64 tiles, hipStream_t s, const u64* kin, const u32* vin, u64* kout, u32* vout, u32 n_max,
                 const u32* n_dev, int p, const u32* bits_dev, const u32* hist, u64* status, u32* ticket,
                 const u32* pack)
{
    // a count known only on the device and a very large bound: a grid that
    // fills the GPU, whose blocks take tiles until the count is covered
    if (n_dev && tiles > DEVICE_COUNT_MAX_TILES)
        hipLaunchKernelGGL((k_radix_pass<B, I, true, DB>), dim3((unsigned)DEVICE_COUNT_GRID), dim3(B), 0, s, kin,
                           vin, kout, vout, n_max, n_dev, p, bits_dev, hist, status, ticket, pack);
    else
        hipLaunchKernelGGL((k_radix_pass<B, I, false, DB>), dim3((unsigned)(tiles ? tiles : 1)), dim3(B), 0, s, kin,
                           vin, kout, vout, n_max, n_dev, p, bits_dev, hist, status, ticket, pack);
}

}  // namespace

int sort_shape_count() { return N_SHAPES; }
int sort_shape() { return g_shape; }
bool set_sort_shape(int i)
{
    if (i < 0 || i >= N_SHAPES) return false;
    g_shape = i;
    return true;
}
int sort_tile(int i) { return SHAPES[i].block * SHAPES[i].items; }
int sort_block(int i) { return SHAPES[i].block; }
bool sort_wide_first() { return g_wide_first && SHAPES[g_shape].block >= 2 * RADIX; }
u64 sort_status_words(u64 n_max, RadixCount count, bool wide)
{
    const AllForm form = all_form(n_max, count);
    const u64 tile = form == AllForm::none ? (u64)sort_tile(g_shape) : (u64)ALL_B * (form == AllForm::large ? 16 : 8);
    const bool nine = wide && (form != AllForm::none || SHAPES[g_shape].block >= 2 * RADIX);
    return (n_max + tile - 1) / tile * (nine ? 2 * RADIX : RADIX) + 1;
}
int sort_min_tile()
{
    int m = sort_tile(0);
    for (int i = 1; i < N_SHAPES; ++i) m = sort_tile(i) < m ? sort_tile(i) : m;
    return m;
}

void radix_passes(u64* k0, u64* k1, const u32* v_first, u32* v0, u32* v1, u32 n_max, const u32* n_dev,
                  const u32* bits_dev, int passes, const u32* hist, u64* status, u32* tickets, hipStream_t s,
                  bool timed, const u32* pack, const u32* w0_dev, RadixCount count)
{
    static const char* const names[MAX_PASSES] = {"sort_pass0", "sort_pass1", "sort_pass2", "sort_pass3",
                                                  "sort_pass4", "sort_pass5", "sort_pass6", "sort_pass7"};
    const int sh = g_shape;
    const u64 tile = (u64)sort_tile(sh);
    // the kernels read the first digit's width with the packing words
    if (w0_dev && w0_dev != pack + 2) return;  // (the record sort keeps them adjacent)
    const AllForm form = all_form(n_max, n_dev ? count : RadixCount::exact);
    if (form != AllForm::none) {
        cvh::TimedScope ts_(timed ? names[0] : nullptr, s);
        const RadixAll all{k0, k1, v_first, v0, v1, n_max, n_dev, passes, bits_dev, hist, w0_dev ? 1u : 0u, status, tickets,
                           pack};
        auto* kern = form == AllForm::small ? k_radix_all<ALL_B, 8> :
                     form == AllForm::large ? k_radix_all<ALL_B, 16> : k_radix_all_counted<ALL_B>;
        const int at = ALL_B * (form == AllForm::large ? 16 : 8);
        hipLaunchKernelGGL(kern, dim3(cvh::grid_for(n_max, at, ALL_GRID)), dim3(ALL_B), 0, s, all);
        return;
    }
    const u64 tiles = ((u64)n_max + tile - 1) / tile;
    for (int p = 0; p < passes; ++p) {
        const u64* kin = (p & 1) ? k1 : k0;
        const u32* vin = p == 0 ? v_first : ((p & 1) ? v1 : v0);
        u64* kout = (p & 1) ? k0 : k1;
        u32* vout = (p & 1) ? v0 : v1;
        cvh::TimedScope ts_(timed ? names[p] : nullptr, s);
        const u32* h = hist + (w0_dev ? hist_wide_off(p) : p * RADIX);
        auto go = [&](auto launch) {
            launch(tiles, s, kin, vin, kout, vout, n_max, n_dev, p, bits_dev, h, status, tickets + p, pack);
        };
        // the first pass of a sort that may take a 9-bit first digit: both
        // widths are launched, and the one that is not the pass's leaves at once
        // (shapes below 512 threads have no 9-bit form; the sort then keeps 8)
        const bool wide = w0_dev && p == 0;
        switch (sh) {
        case 0: go(launch_pass<256, 16>); break;
        case 1: go(launch_pass<256, 32>); break;
        case 2:
            if (wide) go(launch_pass<512, 8, RADIX_BITS + 1>);
            go(launch_pass<512, 8>);
            break;
        case 3:
            if (wide) go(launch_pass<512, 16, RADIX_BITS + 1>);
            go(launch_pass<512, 16>);
            break;
        case 4:
            if (wide) go(launch_pass<1024, 8, RADIX_BITS + 1>);
            go(launch_pass<1024, 8>);
            break;
        default:
            if (wide) go(launch_pass<1024, 16, RADIX_BITS + 1>);
            go(launch_pass<1024, 16>);
            break;
        }
    }
}

}  // namespace cv

extern "C" {

cv_status cv_tuning_set(const char* name, int64_t value)
{
    if (!name) return CV_ERR_INVALID_ARGUMENT;
    const std::string n(name);
    // range-checked as int64 before the narrowing, so 2^32 + i is not shape i
    if (n == "sort_shape")
        return value >= 0 && value < cv::sort_shape_count() && cv::set_sort_shape((int)value)
                   ? CV_OK
                   : CV_ERR_INVALID_ARGUMENT;
    if (n == "radix_wide_first") {
        if (value != 0 && value != 1) return CV_ERR_INVALID_ARGUMENT;
        cv::g_wide_first = value != 0;
        return CV_OK;
    }
    return CV_ERR_INVALID_ARGUMENT;
}

cv_status cv_tuning_get(const char* name, int64_t* value)
{
    if (!name || !value) return CV_ERR_INVALID_ARGUMENT;
    const std::string n(name);
    if (n == "sort_shape") *value = cv::sort_shape();
    else if (n == "sort_shapes") *value = cv::sort_shape_count();
    else if (n == "sort_tile") *value = cv::sort_tile(cv::sort_shape());
    else if (n == "sort_block") *value = cv::sort_block(cv::sort_shape());
    else if (n == "radix_bits") *value = cv::RADIX_BITS;
    else if (n == "radix_wide_first") *value = cv::g_wide_first ? 1 : 0;
    else return CV_ERR_INVALID_ARGUMENT;
    return CV_OK;
}

}  // extern "C"
