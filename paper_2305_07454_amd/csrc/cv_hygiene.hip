// cv_hygiene.hip -- optional record hygiene on (journey, time)-sorted records:
// dropping exact duplicate records (Table 1 shows one) and splitting journeys
// into trips at time gaps.  Both are order-preserving single passes over tiles
// of HT records: a tile's columns are loaded once, its survivors (trip starts)
// counted by ballots, its first position found by decoupled look-back over the
// tiles before, and its rows written.
//
//   k_dup    records kept: not an exact copy of an earlier record of the same
//            (journey, time stamp)
//   k_trip   trip starts: a journey's first record or a gap longer than gap_ms;
//            dense trip numbers
//
// Bound by HBM (80 bytes per record for k_dup, 24 for k_trip).  Counting in one
// kernel and writing in another read every column twice, one record per thread
// and barrier at a time: 40 M records took 1 136 + 318 us of kernels.
#include <hip/hip_runtime.h>

#include "cv_device.h"
#include "cv_host.h"

using namespace cv;

namespace {

constexpr int HB = 1024;
constexpr int HI = 8;         // records per thread, rows of HB striped over the block
constexpr int HT = HB * HI;   // records per tile (40 M records: k_dup 785 us and k_trip 265; with tiles of 4 096
                              // 913 and 300, with 16 records per thread of 512 921 and 280)
constexpr int HNW = HB / WAVE;
constexpr int HT_SIZE = 2048; // records per 4 bytes of the workspace query, whose multiples of 256 bytes hold an
                              // 8-byte ticket counter and an 8-byte look-back word per tile
static_assert(HT >= 4 * HT_SIZE, "two or more tiles: 16 tiles - 8 bytes asked for, 8 tiles + 8 used");

// The ticket counter and the tiles' look-back words cleared; without a tile, the result.
__global__ void __launch_bounds__(256) k_hyg_begin(u64* __restrict__ ws, u64 tiles, cv_result* res)
{
    const u64 i = (u64)blockIdx.x * 256 + threadIdx.x;
    if (tiles == 0) {
        cv_result r = {};
        if (i == 0) *res = r;
    } else if (i <= tiles) {
        ws[i] = 0ull;
    }
}

// The block's tile, by ticket: the tiles a block looks back on are held by
// blocks already running.  (The counter lies in the workspace, which no other call
// uses: in the caller's result, a call on another stream with the same result
// would have given out tiles that do not exist.)
__device__ __forceinline__ u32 take_tile(u64* ticket, u32* s_tile)
{
    if (threadIdx.x == 0) *s_tile = (u32)atomicAdd((unsigned long long*)ticket, 1ull);
    __syncthreads();
    return *s_tile;
}

// Position of each of the thread's marked records among the marked ones of all
// tiles: m[i] are the ballots of the tile's rows, in every lane.  Returns the
// position of row i's lane in pos[i] (the count of marked records before it)
// and the marks up to the tile's end.
__device__ __forceinline__ u64 tile_positions(const u64 (&m)[HI], u64* lb, u32 tile, u32* s_cnt, u64* s_base,
                                              u64 (&pos)[HI])
{
    constexpr int R = HI * HNW / WAVE;  // row counts per lane
    static_assert(R * WAVE == HI * HNW, "whole lanes");
    const int l = lane_id(), w = threadIdx.x / WAVE;
    if (l == 0) {
#pragma unroll
        for (int i = 0; i < HI; ++i) s_cnt[i * HNW + w] = (u32)__popcll(m[i]);
    }
    __syncthreads();
    u32 c[R], sum = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        c[k] = s_cnt[l * R + k];
        sum += c[k];
    }
    const u32 inc = wave_inclusive_sum(sum);
    const u32 tot = (u32)__shfl((int)inc, WAVE - 1, WAVE);
    __syncthreads();
    if (w == 0) {
        u32 e = inc - sum;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            s_cnt[l * R + k] = e;
            e += c[k];
        }
        const u64 x = wave_lookback_exclusive(lb, tile, tot);
        if (l == 0) *s_base = x;
    }
    __syncthreads();
    const u64 base = *s_base;
#pragma unroll
    for (int i = 0; i < HI; ++i) pos[i] = base + s_cnt[i * HNW + w] + popc_below(m[i]);
    return base + tot;
}

__device__ __forceinline__ void write_result(cv_result* res, u64 total, u64 cap)
{
    cv_result r = {};
    r.status = total > cap ? CV_ERR_CAPACITY : CV_OK;
    r.count = total;
    r.required = total > cap ? total : 0;
    *res = r;
}

// true when an earlier record than p of the (journey, time stamp) run j, t that
// p belongs to equals (a, b, c) bit for bit
__device__ bool dup_before(const i64* jid, const i64* ts, const double* lat, const double* lon, const float* spd, u64 p,
                           i64 j, i64 t, u64 a, u64 b, u32 c)
{
    while (p > 0) {
        --p;
        if (jid[p] != j || ts[p] != t) return false;
        if ((u64)__double_as_longlong(lat[p]) == a && (u64)__double_as_longlong(lon[p]) == b &&
            __float_as_uint(spd[p]) == c)
            return true;
    }
    return false;
}

__global__ void __launch_bounds__(HB) k_dup(const i64* __restrict__ jid, const i64* __restrict__ ts,
                                            const double* __restrict__ lat, const double* __restrict__ lon,
                                            const float* __restrict__ spd, const u32* __restrict__ perm, u64 n,
                                            u64* ticket, u64* __restrict__ lb, cv_records_out o,
                                            u32* __restrict__ perm_out,
                                            cv_result* res)
{
    __shared__ u32 s_cnt[HI * HNW];
    __shared__ u32 s_tile;
    __shared__ u64 s_base;
    const u32 tile = take_tile(ticket, &s_tile);
    const u64 t0 = (u64)tile * HT + threadIdx.x;
    const int l = lane_id();
    // every column of the thread's records, and the record before each wave row (lane 0)
    i64 vj[HI], vt[HI];
    u64 va[HI], vb[HI];
    u32 vc[HI], vp[HI];
#pragma unroll
    for (int i = 0; i < HI; ++i) {
        u64 k = t0 + (u64)i * HB;
        k = k < n ? k : n - 1;  // past the end: a valid record, not used
        vj[i] = jid[k];
        vt[i] = ts[k];
        va[i] = (u64)__double_as_longlong(lat[k]);
        vb[i] = (u64)__double_as_longlong(lon[k]);
        vc[i] = __float_as_uint(spd[k]);
        vp[i] = perm_out ? perm[k] : 0u;
    }
    u64 m[HI];
#pragma unroll
    for (int i = 0; i < HI; ++i) {
        const u64 k = t0 + (u64)i * HB;
        i64 pj = lane_below(vj[i]), pt = lane_below(vt[i]);
        u64 pa = lane_below(va[i]), pb = lane_below(vb[i]);
        u32 pc = lane_below(vc[i]);
        if (l == 0 && k > 0 && k < n) {
            pj = jid[k - 1];
            pt = ts[k - 1];
            pa = (u64)__double_as_longlong(lat[k - 1]);
            pb = (u64)__double_as_longlong(lon[k - 1]);
            pc = __float_as_uint(spd[k - 1]);
        }
        bool keep = k < n;
        if (keep && k > 0 && pj == vj[i] && pt == vt[i])
            keep = !((pa == va[i] && pb == vb[i] && pc == vc[i]) ||
                     dup_before(jid, ts, lat, lon, spd, k - 1, vj[i], vt[i], va[i], vb[i], vc[i]));
        m[i] = __ballot(keep);
    }
    u64 pos[HI];
    const u64 total = tile_positions(m, lb, tile, s_cnt, &s_base, pos);
#pragma unroll
    for (int i = 0; i < HI; ++i) {
        if (!((m[i] >> l) & 1ull)) continue;
        o.journey_id[pos[i]] = vj[i];
        o.ts_ms[pos[i]] = vt[i];
        o.lat_deg[pos[i]] = __longlong_as_double((long long)va[i]);
        o.lon_deg[pos[i]] = __longlong_as_double((long long)vb[i]);
        o.speed_mps[pos[i]] = __uint_as_float(vc[i]);
        if (perm_out) perm_out[pos[i]] = vp[i];
    }
    if (tile == gridDim.x - 1 && threadIdx.x == 0) write_result(res, total, n);
}

// trip_id[k] = number of trip starts at or before k, minus one; trip
// journeys[t] = the journey id of trip t's first record (t < cap)
__global__ void __launch_bounds__(HB) k_trip(const i64* __restrict__ jid, const i64* __restrict__ ts, u64 n, i64 gap,
                                             u64* ticket, u64* __restrict__ lb, i64* __restrict__ trip_id,
                                             i64* __restrict__ trip_journey, u64 cap, cv_result* res)
{
    __shared__ u32 s_cnt[HI * HNW];
    __shared__ u32 s_tile;
    __shared__ u64 s_base;
    const u32 tile = take_tile(ticket, &s_tile);
    const u64 t0 = (u64)tile * HT + threadIdx.x;
    const int l = lane_id();
    i64 vj[HI], vt[HI];
#pragma unroll
    for (int i = 0; i < HI; ++i) {
        u64 k = t0 + (u64)i * HB;
        k = k < n ? k : n - 1;
        vj[i] = jid[k];
        vt[i] = ts[k];
    }
    u64 m[HI];
#pragma unroll
    for (int i = 0; i < HI; ++i) {
        const u64 k = t0 + (u64)i * HB;
        i64 pj = lane_below(vj[i]), pt = lane_below(vt[i]);
        if (l == 0 && k > 0 && k < n) {
            pj = jid[k - 1];
            pt = ts[k - 1];
        }
        // ts is non-decreasing inside a journey: the difference is exact in u64
        m[i] = __ballot(k < n && (k == 0 || pj != vj[i] || (u64)vt[i] - (u64)pt > (u64)gap));
    }
    u64 pos[HI];
    const u64 total = tile_positions(m, lb, tile, s_cnt, &s_base, pos);
#pragma unroll
    for (int i = 0; i < HI; ++i) {
        const u64 k = t0 + (u64)i * HB;
        if (k >= n) continue;
        const bool st = (m[i] >> l) & 1ull;
        trip_id[k] = (i64)(pos[i] + (st ? 1 : 0)) - 1;
        if (st && pos[i] < cap && trip_journey) trip_journey[pos[i]] = vj[i];
    }
    if (tile == gridDim.x - 1 && threadIdx.x == 0) write_result(res, total, cap);
}

bool records_ok(const cv_records* r)
{
    return r && (r->n == 0 || (r->journey_id && r->ts_ms && r->lat_deg && r->lon_deg && r->speed_mps));
}

}  // namespace

extern "C" {

cv_status cv_hygiene_workspace_size(uint64_t n, size_t* bytes)
{
    if (!bytes || n >= (1ull << 32)) return CV_ERR_INVALID_ARGUMENT;
    *bytes = cvh::align_up(((n + HT_SIZE - 1) / HT_SIZE + 1) * sizeof(u32));
    return CV_OK;
}

cv_status cv_drop_duplicates(const cv_records* sorted, const uint32_t* perm, const cv_records_out* out,
                             uint32_t* perm_out, cv_result* res, void* ws, size_t ws_bytes, void* stream)
{
    if (!records_ok(sorted) || sorted->n >= (1ull << 32) || !out || !res) return CV_ERR_INVALID_ARGUMENT;
    const u64 n = sorted->n;
    if (n && (!out->journey_id || !out->ts_ms || !out->lat_deg || !out->lon_deg || !out->speed_mps))
        return CV_ERR_INVALID_ARGUMENT;
    if (perm_out && !perm) return CV_ERR_INVALID_ARGUMENT;
    size_t need = 0;
    cv_hygiene_workspace_size(n, &need);
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < need) return CV_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    cvh::TimedScope ts_("drop_duplicates", s);
    const u64 tiles = (n + HT - 1) / HT;
    u64 *ticket = (u64*)ws, *lb = ticket + 1;
    hipLaunchKernelGGL(k_hyg_begin, dim3(cvh::grid_for(tiles + 1, 256)), dim3(256), 0, s, ticket, tiles, res);
    if (tiles)
        hipLaunchKernelGGL(k_dup, dim3((unsigned)tiles), dim3(HB), 0, s, sorted->journey_id, sorted->ts_ms,
                           sorted->lat_deg, sorted->lon_deg, sorted->speed_mps, perm, n, ticket, lb, *out, perm_out, res);
    return cvh::last_launch_status();
}

cv_status cv_split_trips(const cv_records* sorted, int64_t gap_ms, int64_t* trip_id, int64_t* trip_journey,
                         uint64_t capacity, cv_result* res, void* ws, size_t ws_bytes, void* stream)
{
    if (!sorted || sorted->n >= (1ull << 32) || gap_ms < 0 || !res) return CV_ERR_INVALID_ARGUMENT;
    const u64 n = sorted->n;
    if (n && (!sorted->journey_id || !sorted->ts_ms || !trip_id)) return CV_ERR_INVALID_ARGUMENT;
    if (capacity && !trip_journey) return CV_ERR_INVALID_ARGUMENT;
    size_t need = 0;
    cv_hygiene_workspace_size(n, &need);
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < need) return CV_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    cvh::TimedScope ts_("split_trips", s);
    const u64 tiles = (n + HT - 1) / HT;
    u64 *ticket = (u64*)ws, *lb = ticket + 1;
    hipLaunchKernelGGL(k_hyg_begin, dim3(cvh::grid_for(tiles + 1, 256)), dim3(256), 0, s, ticket, tiles, res);
    if (tiles)
        hipLaunchKernelGGL(k_trip, dim3((unsigned)tiles), dim3(HB), 0, s, sorted->journey_id, sorted->ts_ms, n,
                           (i64)gap_ms, ticket, lb, trip_id, capacity ? trip_journey : nullptr, (u64)capacity, res);
    return cvh::last_launch_status();
}

}  // extern "C"
