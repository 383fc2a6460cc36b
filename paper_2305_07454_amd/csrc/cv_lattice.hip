// cv_lattice.hip -- the dense spatio-temporal lattice built from a group
// table, its per-channel min-max normalisation, and a filter over groups
// (Methods steps (4)-(6); Table 2's speed / volume normalisation and volume
// filter rows; the transformed-data output's speed and volume channels per
// direction and time bin).
//
//   k_lat_fill     zero the lattice (16-byte stores)
//   k_lat_scatter  one thread per group: mean speed and distinct journeys
//                  into the cell of its time bin and direction
//   k_lat_minmax   per channel, min and max over the occupied cells
//   k_lat_norm     both channels rescaled, in the stretches with occupied cells
//   k_filt_*       order-preserving compaction of group indices
#include <hip/hip_runtime.h>

#include <cmath>

#include "cv_device.h"
#include "cv_host.h"

using namespace cv;

namespace {

constexpr int LB = 256;
constexpr int FT = LB * 8;  // groups per filter tile

// Bound by HBM writes; a block zeroes one contiguous stretch of LB * FU 16-byte
// words (2.84 GB: 464 us, 6.1 TB/s; 541 with 8 192 blocks striding over the
// whole tensor, 473 with FU 16, 555 with stores that bypass the caches).
constexpr int FU = 4;
__global__ void __launch_bounds__(LB) k_lat_fill(float4* __restrict__ p, u64 n4)
{
    const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
    const u64 i0 = (u64)blockIdx.x * (LB * FU) + threadIdx.x;
#pragma unroll
    for (int k = 0; k < FU; ++k)
        if (i0 + k * LB < n4) p[i0 + k * LB] = z;
}

__global__ void __launch_bounds__(LB) k_lat_fill_tail(float* __restrict__ p, u64 from, u64 n)
{
    const u64 i = from + threadIdx.x;
    if (i < n) p[i] = 0.f;
}

// Group g's key = (td * n_lat + ilat) * n_lon + ilon with td = tbin, or
// tbin * D + sector when the lattice has D = n_dir + 1 direction sectors.
// Channels of a time bin: 2 d (mean speed of sector d) and 2 d + 1 (its
// distinct journeys).
__global__ void __launch_bounds__(LB) k_lat_scatter(const i64* __restrict__ key, const u32* __restrict__ count,
                                                     const u32* __restrict__ nj, const double* __restrict__ sum,
                                                     u64 G, i64 cells, u32 D, i64 t_first, i64 n_t,
                                                     float* __restrict__ out)
{
    for (u64 g = (u64)blockIdx.x * LB + threadIdx.x; g < G; g += (u64)gridDim.x * LB) {
        const i64 k = key[g];
        if (k < 0) continue;
        const i64 td = k / cells, cell = k % cells;
        const i64 tb = td / (i64)D, d = td % (i64)D;
        const i64 t = tb - t_first;
        if (t < 0 || t >= n_t) continue;
        const u32 c = count[g];
        const u64 base = ((u64)t * 2 * D + 2 * (u64)d) * (u64)cells + (u64)cell;
        out[base] = c ? (float)(sum[g] / (double)c) : 0.f;
        out[base + (u64)cells] = (float)nj[g];
    }
}

// Per channel, min and max over occupied cells (volume > 0), as ordered
// integer images.  Block b takes cells [CH * (b % cpi), +CH) of (time bin,
// sector) image b / cpi and writes its four partials (speed min / max, volume
// min / max) to part[4 b ..]; k_lat_mm_reduce joins them (no atomics on shared
// addresses).  occ (nullable): one bit per 64 cells of the chunk, set where one
// is occupied, so that the rescaling reads those cells only.
// The volumes are read whole, CH / LB of them per thread before any is used
// (16 bytes a load when the image lies on 16 bytes): 1.42 GB of a full day's in
// 343 us, 4.1 TB/s; one load of 4 bytes at a time took 584.
constexpr int CH = LB * 16;
constexpr int SUB = CH / WAVE;  // stretches of 64 cells per chunk: the bits of a word
static_assert(SUB == 64, "one word per chunk");

__global__ void __launch_bounds__(LB) k_lat_minmax(const float* __restrict__ lat, u32 D, u64 cells, u64 cpi,
                                                    u32* __restrict__ part, u64* __restrict__ occ)
{
    constexpr int NWL = LB / WAVE, PT = CH / LB;
    __shared__ u32 s_mm[NWL][4];
    __shared__ u64 s_occ[NWL];
    const int w = threadIdx.x / WAVE, l = lane_id();
    const u64 img = blockIdx.x / cpi;
    const u64 c0 = (blockIdx.x % cpi) * CH;
    const u32 d = (u32)(img % D);
    const float* sp = lat + (img / D * 2 * D + 2 * d) * cells;
    const float* vo = sp + cells;
    u32 smin = ~0u, smax = 0u, vmin = ~0u, vmax = 0u;
    auto take = [&](float v, u64 i) {
        const u32 a = ord_f32(sp[i]), b = ord_f32(v);
        smin = a < smin ? a : smin;
        smax = a > smax ? a : smax;
        vmin = b < vmin ? b : vmin;
        vmax = b > vmax ? b : vmax;
    };
    u64 oc = 0;
    if (((uintptr_t)vo & 15u) == 0 && c0 + CH <= cells) {
        float4 x[PT / 4];
#pragma unroll
        for (int k = 0; k < PT / 4; ++k) x[k] = *(const float4*)(vo + c0 + 4 * (u64)(k * LB + threadIdx.x));
#pragma unroll
        for (int k = 0; k < PT / 4; ++k) {
            const u64 i = c0 + 4 * (u64)(k * LB + threadIdx.x);
            const bool any = x[k].x > 0.f || x[k].y > 0.f || x[k].z > 0.f || x[k].w > 0.f;
            const u64 m = __ballot(any);
            // the wave's 256 cells are 4 stretches, 16 lanes each
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((m >> (16 * q)) & 0xFFFFull) oc |= 1ull << (4 * (k * NWL + w) + q);
            if (!any) continue;
            if (x[k].x > 0.f) take(x[k].x, i);
            if (x[k].y > 0.f) take(x[k].y, i + 1);
            if (x[k].z > 0.f) take(x[k].z, i + 2);
            if (x[k].w > 0.f) take(x[k].w, i + 3);
        }
    } else {
        float x[PT];
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const u64 i = c0 + (u64)k * LB + threadIdx.x;
            x[k] = vo[i < cells ? i : cells - 1];
        }
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const u64 i = c0 + (u64)k * LB + threadIdx.x;
            const bool on = i < cells && x[k] > 0.f;
            if (__ballot(on)) oc |= 1ull << (k * NWL + w);
            if (on) take(x[k], i);
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const u32 a = __shfl_xor(smin, o, WAVE), b = __shfl_xor(smax, o, WAVE);
        const u32 c = __shfl_xor(vmin, o, WAVE), e = __shfl_xor(vmax, o, WAVE);
        smin = a < smin ? a : smin;
        smax = b > smax ? b : smax;
        vmin = c < vmin ? c : vmin;
        vmax = e > vmax ? e : vmax;
    }
    if (l == 0) {
        s_mm[w][0] = smin;
        s_mm[w][1] = smax;
        s_mm[w][2] = vmin;
        s_mm[w][3] = vmax;
        s_occ[w] = oc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < NWL; ++k) {
            smin = s_mm[k][0] < smin ? s_mm[k][0] : smin;
            smax = s_mm[k][1] > smax ? s_mm[k][1] : smax;
            vmin = s_mm[k][2] < vmin ? s_mm[k][2] : vmin;
            vmax = s_mm[k][3] > vmax ? s_mm[k][3] : vmax;
            oc |= s_occ[k];
        }
        *(uint4*)(part + 4 * (u64)blockIdx.x) = make_uint4(smin, smax, vmin, vmax);
        if (occ) occ[blockIdx.x] = oc;
    }
}

// the join of a wave's four extrema, in every lane
__device__ __forceinline__ void mm_wave(uint4& a)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const u32 x0 = __shfl_xor(a.x, o, WAVE), x1 = __shfl_xor(a.y, o, WAVE);
        const u32 x2 = __shfl_xor(a.z, o, WAVE), x3 = __shfl_xor(a.w, o, WAVE);
        a.x = x0 < a.x ? x0 : a.x;
        a.y = x1 > a.y ? x1 : a.y;
        a.z = x2 < a.z ? x2 : a.z;
        a.w = x3 > a.w ? x3 : a.w;
    }
}

// Block r of sector d (grid MR x D): the partials [r * per, (r + 1) * per) of
// the sector's n_t * cpi, left in the first of them (one block per sector went
// through 87 000 partials of a full day in 167 us).
constexpr u32 MR = WAVE;
__device__ __forceinline__ u64 mm_slot(u64 i, u32 d, u32 D, u64 cpi) { return ((i / cpi) * D + d) * cpi + i % cpi; }
__global__ void __launch_bounds__(LB) k_lat_mm_reduce(u32* __restrict__ part, u64 n_t, u32 D, u64 cpi)
{
    __shared__ uint4 s_a[LB / WAVE];
    const u32 d = blockIdx.y;
    const u64 n = n_t * cpi, per = (n + MR - 1) / MR;
    const u64 i0 = blockIdx.x * per, i1 = i0 + per < n ? i0 + per : n;
    if (i0 >= n) return;
    uint4 a = make_uint4(~0u, 0u, ~0u, 0u);
    for (u64 i = i0 + threadIdx.x; i < i1; i += LB) {
        const uint4 p = *(const uint4*)(part + 4 * mm_slot(i, d, D, cpi));
        a.x = p.x < a.x ? p.x : a.x;
        a.y = p.y > a.y ? p.y : a.y;
        a.z = p.z < a.z ? p.z : a.z;
        a.w = p.w > a.w ? p.w : a.w;
    }
    mm_wave(a);
    if (lane_id() == 0) s_a[threadIdx.x / WAVE] = a;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < LB / WAVE; ++k) {
        const uint4 p = s_a[k];
        a.x = p.x < a.x ? p.x : a.x;
        a.y = p.y > a.y ? p.y : a.y;
        a.z = p.z < a.z ? p.z : a.z;
        a.w = p.w > a.w ? p.w : a.w;
    }
    *(uint4*)(part + 4 * mm_slot(i0, d, D, cpi)) = a;
}

// occupied cell: (x - min) / (max - min) of its channel in double, rounded to
// float (0 when max == min); an empty cell stays 0
__device__ __forceinline__ float rescale(float x, float mn, float mx)
{
    if (!(mx > mn)) return 0.f;
    return (float)(((double)x - (double)mn) / ((double)mx - (double)mn));
}

// Block b rescales chunks [NCH * (b % gpi), +NCH) of image b / gpi: the stretches
// of 64 cells that occ marks (every one without occ), a wave each.  With 8 chunks
// to a block (a full day's 1.55 M occupied cells: 201 us, 542 when every volume was
// read again; 4 or 16 chunks per block 226 and 260) a lattice of fewer than NORM_FEW
// chunks would leave CUs idle, and a wave with one chunk after the other in turn:
// there a block takes one chunk and its waves a quarter of it each (scatter and
// rescaling with 8 and 1: 24 full images of 200 x 200 cells 84 and 30 us, 288 a tenth
// full 132 and 94, 96 full ones of 333 x 333 178 and 144; 320 full ones of 320 x 320,
// 8 000 chunks, 439 and 408; the full day's 21 888 1209 and 1288).  The first
// block of a sector's first image writes the channels' min and max as floats
// (NaN for a channel with no occupied cell).
constexpr u64 NORM_FEW = 8192;
template <u32 NCH>
__global__ void __launch_bounds__(LB) k_lat_norm(float* __restrict__ lat, u32 D, u64 cells, u64 cpi, u64 gpi, u64 n_t,
                                                  const u32* __restrict__ part, const u64* __restrict__ occ,
                                                  float* __restrict__ out)
{
    constexpr u32 NWL = LB / WAVE, NU = 4, SPLIT = NCH < NWL ? NWL / NCH : 1;  // waves per chunk
    const u32 w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int l = lane_id();
    const u64 img = blockIdx.x / gpi;
    const u64 ch0 = (blockIdx.x % gpi) * NCH;
    const u32 d = (u32)(img % D);
    const u64 n = n_t * cpi, per = (n + MR - 1) / MR;
    uint4 a = make_uint4(~0u, 0u, ~0u, 0u);
    if ((u64)l * per < n) a = *(const uint4*)(part + 4 * mm_slot((u64)l * per, d, D, cpi));
    mm_wave(a);
    const float smn = unord_f32(a.x), smx = unord_f32(a.y);
    const float vmn = unord_f32(a.z), vmx = unord_f32(a.w);
    if (img == d && ch0 == 0 && threadIdx.x == 0) {
        const float nan = __builtin_nanf("");
        const bool none = a.x == ~0u;
        out[4 * d + 0] = none ? nan : smn;
        out[4 * d + 1] = none ? nan : smx;
        out[4 * d + 2] = none ? nan : vmn;
        out[4 * d + 3] = none ? nan : vmx;
    }
    float* sp = lat + (img / D * 2 * D + 2 * d) * cells;
    float* vo = sp + cells;
    for (u32 c = w / SPLIT; c < NCH && ch0 + c < cpi; c += NWL / SPLIT) {
        const u64 c0 = (ch0 + c) * CH;
        u64 m = (~0ull >> (SUB - SUB / SPLIT)) << (w % SPLIT * (SUB / SPLIT));  // the wave's stretches
        if (occ) m &= occ[img * cpi + ch0 + c];
        while (m) {
            u64 i[NU];
            float v[NU], x[NU];
#pragma unroll
            for (u32 q = 0; q < NU; ++q) {
                i[q] = cells;
                if (m) i[q] = c0 + 64 * (u64)(__ffsll((long long)m) - 1) + l;
                m &= m - 1;  // (0 stays 0)
            }
#pragma unroll
            for (u32 q = 0; q < NU; ++q) v[q] = i[q] < cells ? vo[i[q]] : 0.f;
#pragma unroll
            for (u32 q = 0; q < NU; ++q) x[q] = v[q] > 0.f ? sp[i[q]] : 0.f;
#pragma unroll
            for (u32 q = 0; q < NU; ++q) {
                if (!(v[q] > 0.f)) continue;
                sp[i[q]] = rescale(x[q], smn, smx);
                vo[i[q]] = rescale(v[q], vmn, vmx);
            }
        }
    }
}

// filter predicate of group g
__device__ __forceinline__ bool keep(const u32* count, const u32* nj, const double* sum, u64 g, double vmin,
                                     double slo, double shi)
{
    const u32 c = count[g];
    if (c == 0 || (double)nj[g] < vmin) return false;
    const double m = sum[g] / (double)c;
    return m >= slo && m <= shi;
}

__global__ void __launch_bounds__(LB) k_filt_count(const u32* __restrict__ count, const u32* __restrict__ nj,
                                                    const double* __restrict__ sum, u64 G, double vmin, double slo,
                                                    double shi, u32* __restrict__ tcnt)
{
    __shared__ u32 s_w[LB / WAVE];
    const u64 t0 = (u64)blockIdx.x * FT;
    u32 c = 0;
    for (int i = 0; i < FT / LB; ++i) {
        const u64 g = t0 + (u64)i * LB + threadIdx.x;
        c += (u32)__popcll(__ballot(g < G && keep(count, nj, sum, g, vmin, slo, shi)));
    }
    if (lane_id() == 0) s_w[threadIdx.x / WAVE] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        u32 t = 0;
        for (int w = 0; w < LB / WAVE; ++w) t += s_w[w];
        tcnt[blockIdx.x] = t;
    }
}

// exclusive prefix of the tile counts (one block); tcnt[tiles] = total
__global__ void __launch_bounds__(1024) k_filt_scan(u32* __restrict__ tcnt, u64 tiles)
{
    __shared__ u32 s_tmp[1024 / WAVE];
    u32 carry = 0;
    for (u64 b = 0; b < tiles; b += 1024) {
        const u64 i = b + threadIdx.x;
        const u32 v = i < tiles ? tcnt[i] : 0u;
        u32 tot;
        const u32 ex = block_exclusive_sum<1024>(v, s_tmp, tot);
        if (i < tiles) tcnt[i] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) tcnt[tiles] = carry;
}

__global__ void __launch_bounds__(LB) k_filt_write(const u32* __restrict__ count, const u32* __restrict__ nj,
                                                    const double* __restrict__ sum, u64 G, double vmin, double slo,
                                                    double shi, const u32* __restrict__ tpre, u32* __restrict__ index,
                                                    u64 cap)
{
    __shared__ u32 s_w[LB / WAVE];
    __shared__ u32 s_base;
    const u64 t0 = (u64)blockIdx.x * FT;
    const int w = threadIdx.x / WAVE;
    if (threadIdx.x == 0) s_base = tpre[blockIdx.x];
    for (int i = 0; i < FT / LB; ++i) {
        const u64 g = t0 + (u64)i * LB + threadIdx.x;
        const bool k = g < G && keep(count, nj, sum, g, vmin, slo, shi);
        const u64 m = __ballot(k);
        if (lane_id() == 0) s_w[w] = (u32)__popcll(m);
        __syncthreads();
        u32 before = s_base;
        for (int x = 0; x < w; ++x) before += s_w[x];
        const u32 at = before + popc_below(m);
        if (k && at < cap) index[at] = (u32)g;
        __syncthreads();
        if (threadIdx.x == 0)
            for (int x = 0; x < LB / WAVE; ++x) s_base += s_w[x];
        __syncthreads();
    }
}

__global__ void k_filt_result(const u32* __restrict__ tcnt, u64 tiles, u64 cap, cv_result* res)
{
    if (threadIdx.x != 0) return;
    cv_result r = {};
    const u64 total = tcnt[tiles];
    r.status = total > cap ? CV_ERR_CAPACITY : CV_OK;
    r.count = total;
    r.required = total > cap ? total : 0;
    *res = r;
}

bool lattice_dims(const cv_grid_spec* g, uint32_t n_dir, i64& cells, u32& D)
{
    if (!g || g->n_lat <= 0 || g->n_lon <= 0 || g->n_lat > (1ll << 31) || g->n_lon > (1ll << 31) || n_dir > 64)
        return false;
    cells = g->n_lat * g->n_lon;
    D = n_dir ? n_dir + 1 : 1;
    return true;
}

}  // namespace

extern "C" {

cv_status cv_lattice_dense(const cv_groups* groups, uint64_t n_groups, const cv_grid_spec* grid, uint32_t n_dir,
                           int64_t t_first, uint64_t n_t, float* lattice, void* stream)
{
    i64 cells;
    u32 D;
    if (!lattice_dims(grid, n_dir, cells, D) || n_t == 0 || !lattice) return CV_ERR_INVALID_ARGUMENT;
    if ((unsigned __int128)n_t * 2 * D * (u64)cells >= ((unsigned __int128)1 << 62)) return CV_ERR_RANGE;
    if (n_groups && (!groups || !groups->key || !groups->count || !groups->n_journeys || !groups->sum_speed))
        return CV_ERR_INVALID_ARGUMENT;
    if (!cvh::aligned(lattice, 4)) return CV_ERR_INVALID_ARGUMENT;
    hipStream_t s = (hipStream_t)stream;
    cvh::TimedScope ts_("lattice_dense", s);
    const u64 total = n_t * 2 * D * (u64)cells;
    // 16-byte stores from the first 16-byte boundary; the few floats around it singly
    const u64 head = (u64)((16 - ((uintptr_t)lattice & 15)) & 15) / 4;
    const u64 h = head < total ? head : total;
    if (h) hipLaunchKernelGGL(k_lat_fill_tail, dim3(1), dim3(LB), 0, s, lattice, (u64)0, h);
    const u64 n4 = (total - h) / 4;
    if (n4)
        hipLaunchKernelGGL(k_lat_fill, dim3(cvh::grid_for(n4, LB * FU)), dim3(LB), 0, s, (float4*)(lattice + h), n4);
    const u64 done = h + 4 * n4;
    if (done < total) hipLaunchKernelGGL(k_lat_fill_tail, dim3(1), dim3(LB), 0, s, lattice, done, total);
    if (n_groups)
        hipLaunchKernelGGL(k_lat_scatter, dim3(cvh::grid_for(n_groups, LB, 8192)), dim3(LB), 0, s, groups->key,
                           groups->count, groups->n_journeys, groups->sum_speed, (u64)n_groups, cells, D, t_first,
                           (i64)n_t, lattice);
    return cvh::last_launch_status();
}

cv_status cv_lattice_normalize_workspace_size(uint64_t n_t, const cv_grid_spec* grid, uint32_t n_dir, size_t* bytes)
{
    i64 cells;
    u32 D;
    if (!bytes || !lattice_dims(grid, n_dir, cells, D) || n_t == 0) return CV_ERR_INVALID_ARGUMENT;
    const u64 cpi = ((u64)cells + CH - 1) / CH;
    if ((unsigned __int128)n_t * D * cpi >= ((unsigned __int128)1 << 31)) return CV_ERR_RANGE;
    *bytes = cvh::align_up(n_t * D * cpi * 4 * sizeof(u32)) + cvh::align_up(n_t * D * cpi * sizeof(u64));
    return CV_OK;
}

cv_status cv_lattice_normalize(float* lattice, uint64_t n_t, const cv_grid_spec* grid, uint32_t n_dir,
                               float* channel_min_max, void* ws, size_t ws_bytes, void* stream)
{
    i64 cells;
    u32 D;
    if (!lattice_dims(grid, n_dir, cells, D) || n_t == 0 || !lattice || !channel_min_max ||
        !cvh::aligned(channel_min_max, 4))
        return CV_ERR_INVALID_ARGUMENT;
    if ((unsigned __int128)n_t * 2 * D * (u64)cells >= ((unsigned __int128)1 << 62)) return CV_ERR_RANGE;
    size_t need = 0;
    const cv_status e = cv_lattice_normalize_workspace_size(n_t, grid, n_dir, &need);
    if (e != CV_OK) return e;
    // (a workspace without room for the occupancy words: every cell is read again)
    const u64 blocks = n_t * D * (((u64)cells + CH - 1) / CH);
    const size_t parts = cvh::align_up(blocks * 4 * sizeof(u32));
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < parts) return CV_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    cvh::TimedScope ts_("lattice_norm", s);
    const u64 cpi = ((u64)cells + CH - 1) / CH;  // chunks per image
    const u32 nch = blocks < NORM_FEW ? 1 : 8;
    const u64 gpi = (cpi + nch - 1) / nch;
    u32* part = (u32*)ws;
    u64* occ = ws_bytes >= need ? (u64*)((char*)ws + parts) : nullptr;
    hipLaunchKernelGGL(k_lat_minmax, dim3((unsigned)blocks), dim3(LB), 0, s, lattice, D, (u64)cells, cpi, part, occ);
    hipLaunchKernelGGL(k_lat_mm_reduce, dim3(MR, D), dim3(LB), 0, s, part, (u64)n_t, D, cpi);
    hipLaunchKernelGGL(nch == 1 ? k_lat_norm<1> : k_lat_norm<8>, dim3((unsigned)(n_t * D * gpi)), dim3(LB), 0, s, lattice, D, (u64)cells, cpi, gpi,
                       (u64)n_t, part, occ, channel_min_max);
    return cvh::last_launch_status();
}

cv_status cv_groups_filter_workspace_size(uint64_t n_groups, size_t* bytes)
{
    if (!bytes || n_groups >= (1ull << 32)) return CV_ERR_INVALID_ARGUMENT;
    *bytes = cvh::align_up(((n_groups + FT - 1) / FT + 1) * sizeof(u32));
    return CV_OK;
}

cv_status cv_groups_filter(const cv_groups* groups, uint64_t n_groups, double min_volume, double speed_lo,
                           double speed_hi, uint32_t* index, uint64_t capacity, cv_result* res, void* ws,
                           size_t ws_bytes, void* stream)
{
    if (n_groups >= (1ull << 32) || !res || std::isnan(min_volume) || std::isnan(speed_lo) || std::isnan(speed_hi))
        return CV_ERR_INVALID_ARGUMENT;
    if (n_groups && (!groups || !groups->count || !groups->n_journeys || !groups->sum_speed))
        return CV_ERR_INVALID_ARGUMENT;
    if (capacity && !index) return CV_ERR_INVALID_ARGUMENT;
    size_t need = 0;
    cv_groups_filter_workspace_size(n_groups, &need);
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < need) return CV_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    cvh::TimedScope ts_("groups_filter", s);
    const u64 tiles = (n_groups + FT - 1) / FT;
    u32* tcnt = (u32*)ws;
    if (tiles) {
        hipLaunchKernelGGL(k_filt_count, dim3((unsigned)tiles), dim3(LB), 0, s, groups->count, groups->n_journeys,
                           groups->sum_speed, (u64)n_groups, min_volume, speed_lo, speed_hi, tcnt);
    }
    hipLaunchKernelGGL(k_filt_scan, dim3(1), dim3(1024), 0, s, tcnt, tiles);
    if (tiles) {
        hipLaunchKernelGGL(k_filt_write, dim3((unsigned)tiles), dim3(LB), 0, s, groups->count, groups->n_journeys,
                           groups->sum_speed, (u64)n_groups, min_volume, speed_lo, speed_hi, tcnt, index,
                           (u64)capacity);
    }
    hipLaunchKernelGGL(k_filt_result, dim3(1), dim3(64), 0, s, tcnt, tiles, (u64)capacity, res);
    return cvh::last_launch_status();
}

}  // extern "C"
