// cv_grid.hip -- cv_grid_aggregate: the spatio-temporal lattice of the paper
// (Methods steps (3)-(5); Algorithm 2's floor((x - x_min) / x_step) bins; the
// count / sum / count-unique / mean reductions of Table 3), as a sparse,
// key-sorted group table over (journey, time)-sorted records.
//
//   k_grid_part  per tile of GT records, read with coalesced loads:
//     * key = (tbin * n_lat + ilat) * n_lon + ilon per record (-1 outside);
//     * runs: maximal stretches of one key inside one (journey, time-bin)
//       segment; each is reduced once (count, exact speed sum, min, max);
//     * the runs of one (journey, key) inside the tile add into one partial
//       row, and the tile writes its partial rows in record order into its
//       own region (at most GT rows: each holds >= 1 record);
//   k_gpart_compact  partials of all tiles -> (key, row) pairs in tile order,
//     with the digit counts of their keys;
//   radix sort of the pairs by key (the same stable LSD sort as the record
//     order), so a key's partials stay in record order;
//   k_gpart_emit: groups are runs of equal key in the sorted
//     pairs; each group's first pair sums its partials exactly (integer adds
//     and min / max, so the order of the partials changes nothing), counts a
//     journey once per run of equal journey ids among them (the partials of
//     one journey are adjacent in record order), and writes the row, in
//     ascending key.
#include <hip/hip_runtime.h>

#include <cmath>

#include "cv_device.h"
#include "cv_host.h"
#include "cv_gridpart.h"
#include "cv_gridtab.h"
#include "cv_radix.h"

using namespace cv;

namespace {

// blocks of the compaction and of the emit at most: a block takes a contiguous
// range of tiles (chunks), so that the look-back between them stays short and
// its tickets few (they are atomics on one word, some 8 ns each)
constexpr u32 CMP_BLOCKS = 512;
constexpr u32 CMP_TILES = 4;     // tiles per block at least (one per wave)
constexpr u32 CMP_FULL = 48;     // tiles per block from which twice as many blocks pay
// (4 096: with 2 048, 50 M records at random places, a row of its own for each, took
// 23.6 ms, now 23.2 and 22.9 with a chunk after the other to 4 096 blocks; 12 M 2.85,
// 2.77 and 2.77; at 0.001 deg x 1 min 50 M walked ones 952 us, 946)
constexpr u32 EMIT_BLOCKS = 4096;
constexpr u32 EMIT_CHUNKS = 2;   // chunks of the bound per block at least
// With directions a tile may have a row for every two or three records, and the
// blocks above are too few for the rows (derived bearings, emit of 100 000
// records 142 us with them, 80 with these; 9 M: 983, 846).
constexpr u32 DIRS_EMIT_BLOCKS = 4096, DIRS_EMIT_CHUNKS = 1;
// sorted partial pairs per chunk of the head count and the emit
constexpr int ECB = 256;
constexpr int ECP = 4;  // (4: 118 VGPRs in the emit, 4 waves per SIMD)
constexpr int ECH = ECB * ECP;

struct PartMeta : GridMeta {
    u32 t_compact, t_emit;  // tickets of the compaction's and the emit's ranges
};

struct GridLayout {
    PartMeta* meta;
    GPart* part;  // [pmax] partial rows, GT per tile
    u64* K0;      // [pmax] compacted keys; the sort's first key buffer
    u64* K1;      // [pmax] the tiles' partial keys; then the sort's second key buffer
    u32* V0;      // [pmax] compacted partial rows (the sort's pass-0 values); then its first value buffer
    u32* V1;      // [pmax]
    u32* tcnt;    // [tiles] partial rows per tile
    u64* tmax;    // [tiles] largest key per tile
    u32* zero_begin;
    size_t zero_bytes;
    u32* hist;
    u64* lb1;     // look-back words of the compaction's ranges
    u64* lb2;     // and of the emit's
    u64* status;
    u64 pmax, stiles, tiles, chunks;
    u32 cblocks, eblocks;
    size_t bytes;
    GridLayout(void* ws, u64 n, bool dirs = false)
    {
        cvh::Carver c(ws);
        tiles = (n + GT - 1) / GT;
        pmax = tiles * GT;
        stiles = (pmax + sort_min_tile() - 1) / sort_min_tile();
        chunks = (pmax + ECH - 1) / ECH;
        cblocks = (u32)cvh::grid_for(tiles, CMP_TILES, tiles > CMP_BLOCKS * CMP_FULL ? 2 * CMP_BLOCKS : CMP_BLOCKS);
        eblocks = dirs ? (u32)cvh::grid_for(chunks, DIRS_EMIT_CHUNKS, DIRS_EMIT_BLOCKS)
                       : (u32)cvh::grid_for(chunks, EMIT_CHUNKS, EMIT_BLOCKS);
        meta = c.take<PartMeta>(1);
        part = c.take<GPart>(pmax);
        K0 = c.take<u64>(pmax);
        K1 = c.take<u64>(pmax);
        V0 = c.take<u32>(pmax);
        V1 = c.take<u32>(pmax);
        tcnt = c.take<u32>(tiles);
        tmax = c.take<u64>(tiles);
        size_t z0 = cvh::align_up(c.off);
        hist = c.take<u32>(MAX_PASSES * RADIX);
        lb1 = c.take<u64>(cblocks);
        lb2 = c.take<u64>((u64)cvh::grid_for(chunks, DIRS_EMIT_CHUNKS, DIRS_EMIT_BLOCKS));
        // last in the cleared range: a call clears what its tile shape uses
        status = c.take<u64>(stiles * RADIX + 1);
        zero_begin = (u32*)(c.base ? c.base + z0 : nullptr);
        const size_t used = c.base ? (size_t)((char*)(status + sort_status_words(pmax, RadixCount::rows, false)) - c.base) : 0;
        zero_bytes = c.base ? cvh::align_up(used) - z0 : 0;
        bytes = c.size();
    }
};

// The call's scratch words in one launch: meta, the cleared region and the
// shards' counts of records outside the grid (sout, nullable).
__global__ void __launch_bounds__(256) k_gpart_begin(PartMeta* meta, u32* __restrict__ zero, u64 words,
                                                     u64* __restrict__ sout, u32 S)
{
    const u64 i0 = (u64)blockIdx.x * 256 + threadIdx.x;
    const u64 stride = (u64)gridDim.x * 256;
    if (i0 == 0) {
        PartMeta z = {};
        *meta = z;
    }
    for (u64 i = i0; i < words; i += stride) zero[i] = 0u;
    if (sout)
        for (u64 i = i0; i < S; i += stride) sout[i] = 0ull;
}

// The tiles' partial rows packed into (key, row) pairs, in tile order, with
// the digit counts of the key sort.  Block `range` (taken by ticket, so that
// every range it looks back on is held by a block already running) sums its
// tiles' row counts, gets its first position by decoupled look-back, and
// copies; one wave per tile.
__global__ void __launch_bounds__(256) k_gpart_compact(const u64* __restrict__ pkey, const u32* __restrict__ tcnt,
                                                       const u64* __restrict__ tmax, u32 tiles, u64* __restrict__ K0,
                                                       u32* __restrict__ V0, PartMeta* meta, u64* __restrict__ lb,
                                                       int passes, u32* __restrict__ hist)
{
    constexpr int NWC = 256 / WAVE, CU = 4;
    __shared__ u32 s_h[MAX_PASSES * RADIX];
    __shared__ u32 s_off[256], s_cnt[256];
    __shared__ u32 s_t[NWC];
    __shared__ u32 s_bits[NWC];
    __shared__ u32 s_range;
    __shared__ u64 s_base;
    const int l = lane_id(), w = threadIdx.x / WAVE;
    const u32 per = (tiles + gridDim.x - 1) / gridDim.x;
    if ((u64)blockIdx.x * per >= tiles) return;  // exactly the blocks before take the tickets
    if (threadIdx.x == 0) s_range = atomicAdd(&meta->t_compact, 1u);
    for (int i = threadIdx.x; i < passes * RADIX; i += 256) s_h[i] = 0;
    __syncthreads();
    const u32 a = s_range * per;
    const u32 b = a + per < tiles ? a + per : tiles;
    u32 c = 0;
    u64 km = 0;
    for (u32 t = a + threadIdx.x; t < b; t += 256) {
        c += tcnt[t];
        km = tmax[t] > km ? tmax[t] : km;
    }
    u32 tot;
    block_exclusive_sum<256>(c, s_t, tot);
    u32 bits = km ? 64u - (u32)__clzll((long long)km) : 0u;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const u32 o = (u32)__shfl_xor((int)bits, d, WAVE);
        bits = o > bits ? o : bits;
    }
    if (l == 0) s_bits[w] = bits;
    if (w == 0) {
        const u64 e = wave_lookback_exclusive(lb, s_range, tot);
        if (l == 0) s_base = e;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < NWC; ++k) bits = s_bits[k] > bits ? s_bits[k] : bits;
        if (bits > meta->key_bits) atomicMax(&meta->key_bits, bits);  // most ranges have keys of one width
        if (b == tiles) meta->compact_n = (u32)(s_base + tot);
    }
    u32 base = (u32)s_base;
    for (u32 t0 = a; t0 < b; t0 += 256) {
        const u32 t = t0 + threadIdx.x;
        u32 sum;
        const u32 ct = t < b ? tcnt[t] : 0u;
        const u32 ex = block_exclusive_sum<256>(ct, s_t, sum);
        s_off[threadIdx.x] = base + ex;
        s_cnt[threadIdx.x] = ct;
        base += sum;
        __syncthreads();
        const u32 m = b - t0 < 256 ? b - t0 : 256;
        // a wave takes CU of its tiles together, so that their reads are in flight at once
        for (u32 k0 = w; k0 < m; k0 += NWC * CU) {
            u32 cn[CU], o[CU], top = 0;
#pragma unroll
            for (int u = 0; u < CU; ++u) {
                const u32 k = k0 + u * NWC;
                cn[u] = k < m ? s_cnt[k] : 0u;
                o[u] = k < m ? s_off[k] : 0u;
                top = cn[u] > top ? cn[u] : top;
            }
            for (u32 j = 0; j < top; j += WAVE) {
                u64 key[CU];
#pragma unroll
                for (int u = 0; u < CU; ++u)
                    key[u] = j + l < cn[u] ? pkey[(u64)(t0 + k0 + u * NWC) * GT + j + l] : 0ull;
#pragma unroll
                for (int u = 0; u < CU; ++u) {
                    if (j >= cn[u]) continue;  // wave-uniform
                    const bool ok = j + l < cn[u];
                    if (ok) {
                        K0[o[u] + j + l] = key[u];
                        V0[o[u] + j + l] = (u32)((u64)(t0 + k0 + u * NWC) * GT + j + l);
                    }
                    const u64 vm = __ballot(ok);
                    for (int p = 0; p < passes; ++p) {
                        // (a digit shared by every row adds once)
                        const u32 d = (u32)(key[u] >> (p * RADIX_BITS)) & (RADIX - 1);
                        const u32 d0 = __builtin_amdgcn_readfirstlane(d);
                        if (__ballot(ok && d != d0) == 0) {
                            if (l == 0) atomicAdd(&s_h[p * RADIX + d0], (u32)__popcll(vm));
                        } else if (ok) {
                            atomicAdd(&s_h[p * RADIX + d], 1u);
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < passes * RADIX; i += 256)
        if (s_h[i]) atomicAdd(&hist[i], s_h[i]);
}

// the passes of the key sort, and the sorted pairs after them (ping-pong buffers)
__device__ __forceinline__ u32 key_passes(const PartMeta* m) { return (m->key_bits + RADIX_BITS - 1) / RADIX_BITS; }

// Rows in ascending key: the first pair of each key sums the partials of its
// group (the pairs that follow with the same key) and writes the row.  In the
// batched form, group_offsets[s] = first row of shard s (keys carry the shard
// above bit kb).  A block takes a contiguous range of chunks by ticket, counts
// their group heads, gets its first row by decoupled look-back and then reads
// its keys again (from cache) for the rows; counts, their scan in three
// launches and the rows apart took 4 launches more.
__global__ void __launch_bounds__(ECB) k_gpart_emit(PartMeta* meta, const u64* __restrict__ K0,
                                                    const u64* __restrict__ K1, const u32* __restrict__ V0,
                                                    const u32* __restrict__ V1, const GPart* __restrict__ part,
                                                    u64* __restrict__ lb, u32 cap, i64* __restrict__ o_key,
                                                    u32* __restrict__ o_cnt, u32* __restrict__ o_nj,
                                                    double* __restrict__ o_sum, float* __restrict__ o_min,
                                                    float* __restrict__ o_max, u64* __restrict__ go, u32 S, u32 kb,
                                                    u64 kmask, cv_result* res)
{
    __shared__ u32 s_rw[ECP][ECB / WAVE];
    __shared__ u32 s_t[ECB / WAVE];
    __shared__ u32 s_range;
    __shared__ u64 s_base;
    const u32 P = meta->compact_n;
    const u32 chunks = (u32)(((u64)P + ECH - 1) / ECH);
    const bool odd = key_passes(meta) & 1;
    const u64* K = odd ? K1 : K0;
    const u32* V = odd ? V1 : V0;
    const bool sharded = go && S > 1;
    const int t = threadIdx.x, lane = lane_id(), w = t / WAVE;
    // exactly the first ceil(chunks / per) blocks take the tickets (one when there are no pairs)
    const u32 per = (chunks + gridDim.x - 1) / gridDim.x;
    if (blockIdx.x > 0 && (u64)blockIdx.x * per >= chunks) return;
    if (t == 0) s_range = atomicAdd(&meta->t_emit, 1u);
    __syncthreads();
    const u32 range = s_range;
    const u32 c0 = range * per;
    const u32 c1 = c0 + per < chunks ? c0 + per : chunks;
    u32 heads = 0;
    for (u32 c = c0; c < c1; c += 2) {  // two chunks' keys in flight
        u64 x[2 * ECP], y[2 * ECP];
#pragma unroll
        for (int k = 0; k < 2 * ECP; ++k) {
            const u64 i = (u64)c * ECH + (u64)k * ECB + t;
            const u64 j = i < P ? i : (u64)P - 1;
            x[k] = K[j];
            y[k] = K[j > 0 ? j - 1 : 0];
        }
        const u64 end = (u64)c1 * ECH < P ? (u64)c1 * ECH : (u64)P;
#pragma unroll
        for (int k = 0; k < 2 * ECP; ++k) {
            const u64 i = (u64)c * ECH + (u64)k * ECB + t;
            heads += (i < end && (i == 0 || x[k] != y[k])) ? 1u : 0u;
        }
    }
    u32 mine;
    block_exclusive_sum<ECB>(heads, s_t, mine);
    if (w == 0) {
        const u64 e = wave_lookback_exclusive(lb, range, mine);
        if (lane == 0) s_base = e;
    }
    __syncthreads();
    u32 rbase = (u32)s_base;
    const u32 G = rbase + mine;  // the groups, in the block of the last range
    if (c1 == chunks && t == 0) {
        if (res) {
            cv_result r = {};
            r.status = meta->overflow ? CV_ERR_DEVICE : (G > cap ? CV_ERR_CAPACITY : CV_OK);
            r.count = G;
            r.required = G > cap ? G : 0;
            r.n_out_of_grid = meta->n_out;
            r.key_bits = meta->key_bits;
            *res = r;
        }
        if (go && (P == 0 || !sharded))  // no groups, or one problem: shard 0 holds every row
            for (u32 s = 0; s <= S; ++s) go[s] = s == 0 ? 0u : G;
    }
    // A chunk's ECH pairs are taken in ECP rows of ECB: thread t has pairs
    // c * ECH + k * ECB + t, so the heads of a row write consecutive output
    // rows (coalesced stores), and each thread still issues its ECP gathers
    // of first partials together.
    for (u32 c = c0; c < c1; ++c) {
        const u64 ic = (u64)c * ECH;
        u64 key[ECP], kprev[ECP];
        u32 hb = 0;
#pragma unroll
        for (int k = 0; k < ECP; ++k) {
            const u64 i = ic + (u64)k * ECB + t;
            key[k] = i < P ? K[i] : 0ull;
            kprev[k] = (i > 0 && i < P) ? K[i - 1] : ~0ull;
        }
#pragma unroll
        for (int k = 0; k < ECP; ++k) {
            const u64 i = ic + (u64)k * ECB + t;
            const bool h = i < P && (i == 0 || key[k] != kprev[k]);
            if (h) hb |= 1u << k;
            const u64 bm = __ballot(h);
            if (lane == 0) s_rw[k][w] = (u32)__popcll(bm);
        }
        // every head's first partial, the gathers issued together
        u32 vv[ECP];
        GPart pf[ECP];
#pragma unroll
        for (int k = 0; k < ECP; ++k) vv[k] = ((hb >> k) & 1u) ? V[ic + (u64)k * ECB + t] : 0u;
#pragma unroll
        for (int k = 0; k < ECP; ++k)
            if ((hb >> k) & 1u) pf[k] = part[vv[k]];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < ECP; ++k) {
            const u64 i = ic + (u64)k * ECB + t;
            u32 before = 0, rowt = 0;
#pragma unroll
            for (int x = 0; x < ECB / WAVE; ++x) {
                const u32 v = s_rw[k][x];
                before += x < w ? v : 0u;
                rowt += v;
            }
            const u32 row = rbase + before + popc_below(__ballot((hb >> k) & 1u));
            rbase += rowt;
            if (!((hb >> k) & 1u)) continue;
            if (sharded) {
                const u32 sh = (u32)(key[k] >> kb);
                const long ps = i == 0 ? -1 : (long)(kprev[k] >> kb);
                for (long s2 = ps + 1; s2 <= (long)sh; ++s2) go[s2] = row;
            }
            if (row < cap) {
                GPart pr = pf[k];
                u64 cnt = 0;
                u32 nj = 0;
                Fx192 sum;
                fx_zero(sum);
                u32 mn = ~0u, mx = 0;
                i64 pj = pr.jid;
                u64 j = i;
                bool more = j + 1 < P && K[j + 1] == key[k];
                for (;;) {
                    cnt += pr.cn & ~PART_ODD;
                    nj += (j == i || pr.jid != pj) ? 1u : 0u;
                    pj = pr.jid;
                    const Fx192 tt = (pr.cn & PART_ODD) ? fx_from_double<FX_SPD>((double)__uint_as_float(pr.s[0]))
                                                        : part_sum192(pr);
                    fx_add(sum, tt);
                    mn = pr.mn < mn ? pr.mn : mn;
                    mx = pr.mx > mx ? pr.mx : mx;
                    if (!more) break;
                    ++j;
                    pr = part[V[j]];
                    more = j + 1 < P && K[j + 1] == key[k];
                }
                o_key[row] = (i64)(key[k] & kmask);
                o_cnt[row] = (u32)cnt;
                o_nj[row] = nj;
                o_sum[row] = fx_to_double<FX_SPD>(sum);
                o_min[row] = unord_f32(mn);
                o_max[row] = unord_f32(mx);
            }
        }
        if (sharded && P > 0 && (u64)P - 1 >= ic && (u64)P - 1 < ic + ECH && ((u64)P - 1 - ic) % ECB == (u64)t) {
            // the last pair: the shards after the last group's shard start at G
            const u32 sh = (u32)(K[P - 1] >> kb);
            for (u32 s2 = sh + 1; s2 <= S; ++s2) go[s2] = G;
        }
        __syncthreads();
    }
}

// out[k] = in[perm[k]]: a payload column in the sort's order (GU per round,
// loads issued together)
template <class T>
__global__ void __launch_bounds__(256) k_gather_col(const T* __restrict__ in, const u32* __restrict__ perm,
                                                    T* __restrict__ out, u32 n)
{
    constexpr int GU = 4;
    const u64 stride = (u64)gridDim.x * blockDim.x;
    for (u64 k0 = (u64)blockIdx.x * blockDim.x + threadIdx.x; k0 < n; k0 += GU * stride) {
        u32 p[GU];
        T v[GU];
#pragma unroll
        for (int u = 0; u < GU; ++u) {
            const u64 k = k0 + u * stride;
            p[u] = perm[k < n ? k : n - 1];
        }
#pragma unroll
        for (int u = 0; u < GU; ++u) v[u] = in[p[u] < n ? p[u] : n - 1];  // a permutation of [0, n)
#pragma unroll
        for (int u = 0; u < GU; ++u) {
            const u64 k = k0 + u * stride;
            if (k < n) out[k] = v[u];
        }
    }
}

bool spec_ok(const cv_grid_spec* g)
{
    if (!g) return false;
    if (!(g->dlat_deg > 0.0) || !(g->dlon_deg > 0.0)) return false;
    if (!std::isfinite(g->lat0_deg) || !std::isfinite(g->lon0_deg) || !std::isfinite(g->dlat_deg) ||
        !std::isfinite(g->dlon_deg))
        return false;
    if (g->n_lat <= 0 || g->n_lon <= 0 || g->bin_ms <= 0) return false;
    if (g->n_lat > (1ll << 31) || g->n_lon > (1ll << 31)) return false;
    __int128 cells = (__int128)g->n_lat * g->n_lon;
    if (g->n_t > 0 && cells * g->n_t >= ((__int128)1 << 63)) return false;
    return true;
}

}  // namespace

// the tile kernel for a direction source (0 none, 1 heading column, 2 bearing)
template <int KD, bool FL = false>
static void launch_parts(dim3 gg, hipStream_t s, u32 nn, const cv_records* sorted, const Spec& g, const PartSink& sk,
                         GridMeta* meta, const uint8_t* first = nullptr)
{
    hipLaunchKernelGGL((k_grid_part<KD, FL>), gg, dim3(GB), 0, s, nn, sorted->journey_id, sorted->ts_ms,
                       sorted->lat_deg, sorted->lon_deg, sorted->speed_mps, g, sk, meta, first);
}

// nd > 0: a direction dimension of nd sectors (plus one for records without a
// direction) from the sorted heading column hdg, else from feat's bearing
static cv_status grid_impl(const cv_records* sorted, const u64* soff, u32 S, const cv_grid_spec* grid,
                           const cv_groups* out, uint64_t capacity, u64* go, cv_result* res, void* ws, size_t ws_bytes,
                           void* stream, u32 nd = 0, double doff = 0.0, const float* hdg = nullptr,
                           const cv_features* feat = nullptr, u64* sout = nullptr, const uint8_t* first = nullptr)
{
    if (!sorted || !out || sorted->n >= (1ull << 32) || capacity >= (1ull << 32) || !spec_ok(grid))
        return CV_ERR_INVALID_ARGUMENT;
    const u64 n = sorted->n;
    hipStream_t s = (hipStream_t)stream;
    GridLayout need(nullptr, n);
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < need.bytes) return CV_ERR_WORKSPACE;
    if (n == 0) {
        if (res) hipLaunchKernelGGL(k_grid_empty, dim3(1), dim3(64), 0, s, res);
        if (go) cvh::fill_u64(go, 0, (u64)S + 1, s);
        if (sout) cvh::fill_u64(sout, 0ull, S ? S : 1, s);
        return cvh::last_launch_status();
    }
    if (!sorted->journey_id || !sorted->ts_ms || !sorted->lat_deg || !sorted->lon_deg || !sorted->speed_mps)
        return CV_ERR_INVALID_ARGUMENT;
    if (capacity > 0 &&
        (!out->key || !out->count || !out->n_journeys || !out->sum_speed || !out->min_speed || !out->max_speed))
        return CV_ERR_INVALID_ARGUMENT;
    GridLayout L(ws, n, nd > 0);
    Spec g;
    g.lat0 = grid->lat0_deg;
    g.lon0 = grid->lon0_deg;
    g.dlat = grid->dlat_deg;
    g.dlon = grid->dlon_deg;
    g.n_lat = grid->n_lat;
    g.n_lon = grid->n_lon;
    g.t0 = grid->t0_ms;
    g.bin_ms = grid->bin_ms;
    g.tinv = 1.0 / (double)grid->bin_ms;
    g.rlat = 1.0 / grid->dlat_deg;
    g.rlon = 1.0 / grid->dlon_deg;
    g.cells = (u64)grid->n_lat * (u64)grid->n_lon;
    const auto inverts = [](double d) { return d > 1e-100 && d < 1e100; };
    g.quick = grid->bin_ms < (1ll << 30) && g.cells < (1ull << 32) && inverts(grid->dlat_deg) && inverts(grid->dlon_deg);
    g.tmax = grid->n_t > 0 ? grid->n_t : (INT64_MAX / (grid->n_lat * grid->n_lon * (i64)(nd + 1)));
    g.soff = soff;
    g.S = S;
    g.kb = 0;
    g.nd = nd;
    g.dstep = nd ? 360.0 / (double)nd : 0.0;
    g.doff = doff;
    g.hdg = hdg;
    g.brg = (nd && !hdg) ? feat->bearing_deg : nullptr;
    g.bfl = (nd && !hdg) ? feat->flags : nullptr;
    g.sout = sout;
    u32 sb = 0;
    if (S > 1) {
        // cell keys < n_t * n_lat * n_lon; the shard index goes above them
        const unsigned __int128 cells = (unsigned __int128)grid->n_t * grid->n_lat * grid->n_lon;
        u32 kb = 0;
        while (kb < 63 && ((unsigned __int128)1 << kb) < cells) ++kb;
        while (((u64)1 << sb) < S) ++sb;
        if (kb + sb > 63) return CV_ERR_RANGE;
        g.kb = kb;
    }
    // passes the merge's key sort can need: every key lies below the grid's
    // count of (time bin, sector, cell) keys, with the shard index above kb
    // when sharded; the device's count of key bits skips the rest
    int mpasses = MAX_PASSES;
    {
        const unsigned __int128 keys = (unsigned __int128)g.tmax * (unsigned __int128)(nd + 1) *
                                       (unsigned __int128)grid->n_lat * (unsigned __int128)grid->n_lon;
        u32 b = 0;
        while (b < 64 && ((unsigned __int128)1 << b) < keys) ++b;
        if (S > 1) b = nd == 0 ? g.kb + sb : 64u;
        const int need = (int)((b + RADIX_BITS - 1) / RADIX_BITS);
        mpasses = need < MAX_PASSES ? need : MAX_PASSES;
    }
    const u64 kmask = S > 1 ? ((1ull << g.kb) - 1) : ~0ull;
    const u32 nn = (u32)n;
    const u32 tiles = (u32)L.tiles;
    const u32 pmax = (u32)(L.pmax - 1 < 0xFFFFFFFFull ? L.pmax : 0xFFFFFFFFull);
    {
        cvh::TimedScope ts_("grid_agg", s);
        const u64 words = L.zero_bytes / 4;
        hipLaunchKernelGGL(k_gpart_begin, dim3(cvh::grid_for(words, 256, 4096)), dim3(256), 0, s, L.meta, L.zero_begin,
                           words, sout, S ? S : 1u);
        PartSink sk{L.K1, L.part, L.tcnt, L.tmax};
        const dim3 gg(tiles);
        if (nd == 0 && first) launch_parts<0, true>(gg, s, nn, sorted, g, sk, L.meta, first);
        else if (nd == 0) launch_parts<0>(gg, s, nn, sorted, g, sk, L.meta);
        else if (hdg) launch_parts<1>(gg, s, nn, sorted, g, sk, L.meta);
        else launch_parts<2>(gg, s, nn, sorted, g, sk, L.meta);
    }
    {
        cvh::TimedScope ts_("grid_tail", s);
        // partial rows -> compacted (key, row) pairs, with the key sort's digit counts
        hipLaunchKernelGGL(k_gpart_compact, dim3(L.cblocks), dim3(256), 0, s, L.K1, L.tcnt, L.tmax, tiles, L.K0, L.V0,
                           L.meta, L.lb1, mpasses, L.hist);
        // key sort of the pairs
        radix_passes(L.K0, L.K1, L.V0, L.V0, L.V1, pmax, &L.meta->compact_n, &L.meta->key_bits, mpasses, L.hist,
                     L.status, L.meta->tickets, s, /*timed=*/false, nullptr, nullptr,
                     nd ? RadixCount::many : RadixCount::rows);
        // groups: runs of equal keys, their rows
        hipLaunchKernelGGL(k_gpart_emit, dim3(L.eblocks), dim3(ECB), 0, s, L.meta, L.K0, L.K1, L.V0, L.V1, L.part,
                           L.lb2, (u32)capacity, out->key, out->count, out->n_journeys, out->sum_speed, out->min_speed,
                           out->max_speed, go, S, g.kb, kmask, res);
        cvh::debug_rows(out->key, out->count, out->n_journeys, res, capacity, go, S, CV_DEBUG_GROUP_ORDER, s);
    }
    return cvh::last_launch_status();
}


extern "C" {

cv_status cv_grid_workspace_size(uint64_t n, const cv_grid_spec* grid, uint64_t capacity, size_t* bytes)
{
    if (!bytes || n >= (1ull << 32) || capacity >= (1ull << 32) || !spec_ok(grid)) return CV_ERR_INVALID_ARGUMENT;
    GridLayout L(nullptr, n);
    *bytes = L.bytes;
    return CV_OK;
}

cv_status cv_grid_aggregate(const cv_records* sorted, const cv_grid_spec* grid, const cv_groups* out,
                            uint64_t capacity, cv_result* res, void* ws, size_t ws_bytes, void* stream)
{
    return grid_impl(sorted, nullptr, 0, grid, out, capacity, nullptr, res, ws, ws_bytes, stream);
}

cv_status cv_grid_aggregate_flags(const cv_records* sorted, const uint8_t* flags, const cv_grid_spec* grid,
                                  const cv_groups* out, uint64_t capacity, cv_result* res, void* ws, size_t ws_bytes,
                                  void* stream)
{
    if (!flags && sorted && sorted->n > 0) return CV_ERR_INVALID_ARGUMENT;
    return grid_impl(sorted, nullptr, 0, grid, out, capacity, nullptr, res, ws, ws_bytes, stream, 0, 0.0, nullptr,
                     nullptr, nullptr, flags);
}

cv_status cv_grid_aggregate_dir(const cv_records* sorted, const float* heading_deg, const cv_features* feat,
                                const cv_grid_spec* grid, uint32_t n_dir, double dir_offset_deg, const cv_groups* out,
                                uint64_t capacity, cv_result* res, void* ws, size_t ws_bytes, void* stream)
{
    if (!grid || n_dir < 1 || n_dir > 64 || !(dir_offset_deg >= 0.0 && dir_offset_deg < 360.0))
        return CV_ERR_INVALID_ARGUMENT;
    if (!heading_deg && (!feat || !feat->bearing_deg || !feat->flags)) return CV_ERR_INVALID_ARGUMENT;
    if (grid->n_t > 0 && (__int128)grid->n_t * grid->n_lat * grid->n_lon * (n_dir + 1) >= ((__int128)1 << 63))
        return CV_ERR_RANGE;
    return grid_impl(sorted, nullptr, 0, grid, out, capacity, nullptr, res, ws, ws_bytes, stream, n_dir,
                     dir_offset_deg, heading_deg, feat);
}

cv_status cv_gather_column(const void* in, const uint32_t* perm, void* out, uint64_t n, uint32_t elem_bytes,
                           void* stream)
{
    if (n >= (1ull << 32) || (elem_bytes != 4 && elem_bytes != 8)) return CV_ERR_INVALID_ARGUMENT;
    if (n == 0) return CV_OK;
    if (!in || !perm || !out || !cvh::aligned(in, elem_bytes) || !cvh::aligned(out, elem_bytes))
        return CV_ERR_INVALID_ARGUMENT;
    hipStream_t s = (hipStream_t)stream;
    const unsigned blocks = (unsigned)cvh::grid_for(n, 256, 8192);
    if (elem_bytes == 4)
        hipLaunchKernelGGL((k_gather_col<uint32_t>), dim3(blocks), dim3(256), 0, s, (const uint32_t*)in, perm,
                           (uint32_t*)out, (u32)n);
    else
        hipLaunchKernelGGL((k_gather_col<u64>), dim3(blocks), dim3(256), 0, s, (const u64*)in, perm, (u64*)out,
                           (u32)n);
    return cvh::last_launch_status();
}

cv_status cv_batch_grid_aggregate(const cv_records* sorted, const uint64_t* shard_offsets, uint32_t n_shards,
                                  const cv_grid_spec* grid, const cv_groups* out, uint64_t capacity,
                                  uint64_t* group_offsets, cv_result* res, void* ws, size_t ws_bytes, void* stream)
{
    if (n_shards == 0 || !shard_offsets || !group_offsets || !cvh::aligned(shard_offsets, 8) ||
        !cvh::aligned(group_offsets, 8) || !grid || grid->n_t <= 0)
        return CV_ERR_INVALID_ARGUMENT;
    return grid_impl(sorted, shard_offsets, n_shards, grid, out, capacity, group_offsets, res, ws, ws_bytes, stream);
}

cv_status cv_batch_workspace_size(uint64_t n, uint32_t n_shards, uint64_t max_journeys, uint64_t journey_capacity,
                                  const cv_grid_spec* grid, uint64_t group_capacity, size_t* bytes)
{
    if (!bytes || n_shards == 0) return CV_ERR_INVALID_ARGUMENT;
    size_t a = 0, b = 0, c = 0;
    cv_status e = cv_sort_workspace_size(n, max_journeys, &a);
    if (e == CV_OK) e = cv_summary_workspace_size(n, journey_capacity, &b);
    if (e == CV_OK) e = cv_grid_workspace_size(n, grid, group_capacity, &c);
    if (e != CV_OK) return e;
    // the stages run one after the other on one stream: one region serves all three
    size_t m = a > b ? a : b;
    *bytes = m > c ? m : c;
    return CV_OK;
}

cv_status cv_batch_run(const cv_records* in, const uint64_t* shard_offsets, uint32_t n_shards,
                       const cv_grid_spec* grid, uint64_t max_journeys, uint32_t* perm, const cv_records_out* sorted,
                       const cv_features* feat, const cv_journeys* journeys, uint64_t journey_capacity,
                       uint64_t* journey_offsets, const cv_groups* groups, uint64_t group_capacity,
                       uint64_t* group_offsets, uint64_t* shard_n_out, cv_result* res, void* ws, size_t ws_bytes,
                       void* stream)
{
    if (!in || !sorted || !feat || !grid || n_shards == 0 || !shard_offsets || !journey_offsets ||
        !group_offsets || !res || grid->n_t <= 0)
        return CV_ERR_INVALID_ARGUMENT;
    if (!sorted->journey_id || !sorted->ts_ms || !sorted->lat_deg || !sorted->lon_deg || !sorted->speed_mps)
        return CV_ERR_INVALID_ARGUMENT;
    if (shard_n_out && !cvh::aligned(shard_n_out, 8)) return CV_ERR_INVALID_ARGUMENT;
    size_t need = 0;
    cv_status e = cv_batch_workspace_size(in->n, n_shards, max_journeys, journey_capacity, grid, group_capacity,
                                          &need);
    if (e != CV_OK) return e;
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < need) return CV_ERR_WORKSPACE;
    e = cv_batch_sort_records_features(in, shard_offsets, n_shards, max_journeys, perm, sorted, feat, res, ws,
                                       ws_bytes, stream);
    if (e != CV_OK) return e;
    cv_records srt{};
    srt.journey_id = sorted->journey_id;
    srt.ts_ms = sorted->ts_ms;
    srt.lat_deg = sorted->lat_deg;
    srt.lon_deg = sorted->lon_deg;
    srt.speed_mps = sorted->speed_mps;
    srt.n = in->n;
    e = cv_batch_journey_summary(&srt, feat, shard_offsets, n_shards, journeys, journey_capacity, journey_offsets,
                                 res + 1, ws, ws_bytes, stream);
    if (e != CV_OK) return e;
    return grid_impl(&srt, shard_offsets, n_shards, grid, groups, group_capacity, group_offsets, res + 2, ws,
                     ws_bytes, stream, 0, 0.0, nullptr, nullptr, shard_n_out, feat->flags);
}

}  // extern "C"
