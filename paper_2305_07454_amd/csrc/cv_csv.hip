// cv_csv.hip -- extraction of Table-1-shaped text rows (journey id,
// timestamp, latitude, longitude, postal code, speed, heading) into record
// columns on the device: the "E" of the ETL path ahead of the key prep.
//
//   k_csv_count   newlines per tile of CT bytes (16-byte loads)
//   k_csv_scan    exclusive prefix of the tile counts (texts of more than
//                 CSV_SELF tiles; the parse sums the counts itself below that)
//   k_csv_parse   per tile: the text staged in LDS with one bit per byte for
//                 newlines, commas and quotes; then one thread per row that
//                 starts in the tile
//
// A row's commas come from the bits, and a row without six of them, or with a
// quote, is malformed.  Its fields are converted eight characters at a time; one
// of another form goes through the byte-wise parsers, which alone say whether it
// is malformed.  A row that runs past the staged bytes (a tile's last one) is read
// by the whole block.  Bound by vector instructions and, in the count, by HBM: 4 M
// rows, 292 MB, take 65 us to count and 156 to parse; reading the text a third time
// for the row starts and finding the commas byte by byte in each row's thread
// took 537, 404 of them the parse.
#include <hip/hip_runtime.h>

#include "cv_device.h"
#include "cv_host.h"

using namespace cv;

namespace {

constexpr int CB = 256;            // threads per block
constexpr int CT = 16 * 1024;      // bytes per tile (25 KB of LDS, six blocks per CU: with 32 KB tiles the
                                   // parse of 4 M rows took 225 instead of 190 us, or 216 in blocks of 512)
constexpr int CHALO = 1024;        // bytes staged after a tile for the rows that run over its end
constexpr u64 CSV_SELF = 2048;     // tiles whose counts every block of the parse sums itself; in a longer text the
constexpr int CG_L = 4;            // count takes groups of tiles, which one block scans

// bytes of w that equal the byte c4 repeats, as the high bit of each byte
__device__ __forceinline__ u32 eq_bytes(u32 w, u32 c4)
{
    const u32 t = w ^ c4;
    return ~(((t & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | t | 0x7F7F7F7Fu);
}
// the four high bits as the low four bits of a word
__device__ __forceinline__ u32 pack_bytes(u32 z) { return ((z >> 7) * 0x10204080u) >> 28; }

// the 16 bytes at p of the text; bytes past its end are 0
__device__ __forceinline__ uint4 load16(const unsigned char* __restrict__ text, u64 p, u64 nbytes)
{
    if (p + 16 <= nbytes) return *reinterpret_cast<const uint4*>(text + p);
    u32 v[4] = {0, 0, 0, 0};
    for (u32 i = 0; i < 16; ++i)
        if (p + i < nbytes) v[i / 4] |= (u32)text[p + i] << (8 * (i % 4));
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// Newlines per group of CG tiles, and in a group of several per tile as 16 bits
// of a word (one block scans the groups, and what one CU can read is what bounds
// that: 18 000 tiles one by one took 18 us, in groups 6; a short text's few tiles
// are counted each by a block of its own, 5 us less at 2.7 MB); block 0 also
// clears the result (the parse adds the malformed rows to it and sets the rest).
template <int CG>
__global__ void __launch_bounds__(CB) k_csv_count(const unsigned char* __restrict__ text, u64 nbytes,
                                                  u32* __restrict__ gcnt, u64* __restrict__ sub, cv_result* res)
{
    constexpr int Q = CT / 16 / CB;
    static_assert(CG <= 4 && CT <= 32768, "a tile's count in 16 bits");
    __shared__ u64 s_w[CB / WAVE];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        cv_result r = {};
        *res = r;
    }
    const u64 t0 = (u64)blockIdx.x * CG * CT;
    if (t0 >= nbytes) return;
    u64 c = 0;
    uint4 v[CG * Q];
    const u64 p0 = t0 + 16 * (u64)threadIdx.x;
    if (t0 + CG * CT <= nbytes) {  // (no test per load: all in flight together)
#pragma unroll
        for (int k = 0; k < CG * Q; ++k) v[k] = *reinterpret_cast<const uint4*>(text + p0 + 16 * (u64)(k * CB));
    } else {
#pragma unroll
        for (int k = 0; k < CG * Q; ++k) v[k] = load16(text, p0 + 16 * (u64)(k * CB), nbytes);
    }
#pragma unroll
    for (int k = 0; k < CG * Q; ++k)
        c += (u64)(u32)(__popc(eq_bytes(v[k].x, 0x0A0A0A0Au)) + __popc(eq_bytes(v[k].y, 0x0A0A0A0Au)) +
                        __popc(eq_bytes(v[k].z, 0x0A0A0A0Au)) + __popc(eq_bytes(v[k].w, 0x0A0A0A0Au)))
             << (16 * (k / Q));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o, WAVE);
    if (lane_id() == 0) s_w[threadIdx.x / WAVE] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        u64 t = 0;
        for (int w = 0; w < CB / WAVE; ++w) t += s_w[w];
        if (CG > 1) sub[blockIdx.x] = t;
        gcnt[blockIdx.x] = (u32)((t & 0xFFFF) + ((t >> 16) & 0xFFFF) + ((t >> 32) & 0xFFFF) + (t >> 48));
    }
}

// (one block, 8 counts per thread and round, read before any is used)
__global__ void __launch_bounds__(1024) k_csv_scan(u32* __restrict__ tcnt, u64 tiles)
{
    constexpr int P = 8;
    __shared__ u32 s_tmp[1024 / WAVE];
    u32 carry = 0;
    for (u64 b = 0; b < tiles; b += 1024 * P) {
        const u64 i = b + (u64)threadIdx.x * P;
        u32 v[P], sum = 0;
#pragma unroll
        for (int k = 0; k < P; ++k) v[k] = tcnt[i + k < tiles ? i + k : tiles - 1];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            v[k] = i + k < tiles ? v[k] : 0u;
            sum += v[k];
        }
        u32 tot;
        u32 e = carry + block_exclusive_sum<1024>(sum, s_tmp, tot);
#pragma unroll
        for (int k = 0; k < P; ++k) {
            if (i + k < tiles) tcnt[i + k] = e;
            e += v[k];
        }
        carry += tot;
    }
}

// ------------------------------------------------------------------ fields

__device__ __forceinline__ bool is_digit(unsigned char c) { return c >= '0' && c <= '9'; }

// up to 8 bytes, packed big-endian (string order = integer order)
__device__ __forceinline__ bool parse_id(const unsigned char* s, int len, i64& out)
{
    if (len < 1 || len > 8) return false;
    u64 v = 0;
    for (int i = 0; i < 8; ++i) v = (v << 8) | (i < len ? (u64)s[i] : 0ull);
    out = (i64)v;
    return (v >> 63) == 0;  // bytes below 0x80
}

__device__ __forceinline__ int digits(const unsigned char* s, int n)
{
    int v = 0;
    for (int i = 0; i < n; ++i) {
        if (!is_digit(s[i])) return -1;
        v = v * 10 + (s[i] - '0');
    }
    return v;
}

// days since 1970-01-01 of a proleptic Gregorian date (civil-from-days
// inverse: eras of 400 years, March-based years)
__device__ __forceinline__ i64 days_from_civil(i64 y, int m, int d)
{
    y -= m <= 2;
    const i64 era = (y >= 0 ? y : y - 399) / 400;
    const i64 yoe = y - era * 400;
    const i64 doy = (153 * (m + (m > 2 ? -3 : 9)) + 2) / 5 + d - 1;
    const i64 doe = yoe * 365 + yoe / 4 - yoe / 100 + doy;
    return era * 146097 + doe - 719468;
}

// "YYYY-MM-DD HH:MM:SS" with an optional fraction of 1 to 3 digits: UTC ms
__device__ __forceinline__ bool parse_ts(const unsigned char* s, int len, i64& out)
{
    if (len < 19 || s[4] != '-' || s[7] != '-' || s[10] != ' ' || s[13] != ':' || s[16] != ':') return false;
    const int y = digits(s, 4), mo = digits(s + 5, 2), d = digits(s + 8, 2);
    const int h = digits(s + 11, 2), mi = digits(s + 14, 2), se = digits(s + 17, 2);
    if (y < 1 || mo < 1 || mo > 12 || d < 1 || h < 0 || h > 23 || mi < 0 || mi > 59 || se < 0 || se > 59) return false;
    const bool leap = (y % 4 == 0 && y % 100 != 0) || y % 400 == 0;
    const int mdays[12] = {31, 28, 31, 30, 31, 30, 31, 31, 30, 31, 30, 31};
    if (d > mdays[mo - 1] + ((mo == 2 && leap) ? 1 : 0)) return false;
    int ms = 0;
    if (len > 19) {
        const int f = len - 20;
        if (s[19] != '.' || f < 1 || f > 3) return false;
        const int v = digits(s + 20, f);
        if (v < 0) return false;
        ms = f == 1 ? v * 100 : (f == 2 ? v * 10 : v);
    }
    out = ((days_from_civil(y, mo, d) * 24 + h) * 60 + mi) * 60000 + (i64)se * 1000 + ms;
    return true;
}

// A plain decimal ([-+]digits[.digits]): the integer of its significant
// digits (below 2^53) and the count of fraction digits (at most 22) give
// the exact quotient rounded once (one IEEE division by an exact power of
// ten); other forms are refused.
__device__ __forceinline__ bool parse_decimal(const unsigned char* s, int len, double& out)
{
    constexpr double P10[23] = {1e0,  1e1,  1e2,  1e3,  1e4,  1e5,  1e6,  1e7,  1e8,  1e9,  1e10, 1e11,
                                1e12, 1e13, 1e14, 1e15, 1e16, 1e17, 1e18, 1e19, 1e20, 1e21, 1e22};
    int i = 0;
    bool neg = false;
    if (i < len && (s[i] == '-' || s[i] == '+')) neg = s[i++] == '-';
    u64 m = 0;
    int nd = 0, frac = 0;
    bool dot = false;
    for (; i < len; ++i) {
        const unsigned char c = s[i];
        if (c == '.') {
            if (dot) return false;
            dot = true;
            continue;
        }
        if (!is_digit(c)) return false;
        ++nd;
        if (m > (1ull << 53) / 10) return false;  // beyond the exact range
        m = m * 10 + (c - '0');
        if (dot) ++frac;
    }
    if (nd == 0 || m >= (1ull << 53) || frac > 22) return false;
    const double v = frac ? (double)m / P10[frac] : (double)m;
    out = neg ? -v : v;
    return true;
}

struct Row {
    i64 jid, ts;
    double lat, lon, spd, hdg;
    bool ok;
};

__device__ __forceinline__ Row malformed()
{
    Row w;
    w.jid = 0;
    w.ts = 0;
    w.lat = w.lon = w.spd = w.hdg = __builtin_nan("");
    w.ok = false;
    return w;
}

// The fields of a row of len bytes at s (no line end, no quote) whose six commas
// lie at cpos.  Inlined into each caller, so that a row staged in LDS is read with
// LDS loads.
__device__ __forceinline__ Row parse_fields(const unsigned char* s, const u32* cpos, u32 len)
{
    Row w = malformed();
    const u32 hl = len - cpos[5] - 1;
    w.ok = parse_id(s, (int)cpos[0], w.jid) && parse_ts(s + cpos[0] + 1, (int)(cpos[1] - cpos[0] - 1), w.ts) &&
           parse_decimal(s + cpos[1] + 1, (int)(cpos[2] - cpos[1] - 1), w.lat) &&
           parse_decimal(s + cpos[2] + 1, (int)(cpos[3] - cpos[2] - 1), w.lon) &&
           parse_decimal(s + cpos[4] + 1, (int)(cpos[5] - cpos[4] - 1), w.spd) &&
           (hl == 0 || parse_decimal(s + cpos[5] + 1, (int)hl, w.hdg));
    return w.ok ? w : malformed();
}

// ------------------------------------------------------------------ fields,
// eight characters at a time from staged text (dwords of LDS)

// the 4 bytes from byte position p
__device__ __forceinline__ u32 ld4(const u32* s, u32 p)
{
    return __builtin_amdgcn_alignbyte(s[(p >> 2) + 1], s[p >> 2], p & 3);
}
// the 8 bytes that end before position p
__device__ __forceinline__ void ld8_end(const u32* s, u32 p, u32& lo, u32& hi)
{
    const u32 q = p - 8, i = q >> 2;
    const u32 a = s[i], b = s[i + 1], c = s[i + 2];
    lo = __builtin_amdgcn_alignbyte(b, a, q & 3);
    hi = __builtin_amdgcn_alignbyte(c, b, q & 3);
}

// whether a byte of d (characters with '0' taken off by xor) is no digit
__device__ __forceinline__ u32 no_digit(u32 d) { return ((d + 0x76767676u) | d) & 0x80808080u; }

// the number of four digit bytes, the first character lowest
__device__ __forceinline__ u32 num4(u32 d)
{
    return __builtin_amdgcn_udot4(d, 0x0000010Au, 0u, false) * 100u + __builtin_amdgcn_udot4(d, 0x010A0000u, 0u, false);
}

// The number of the last n (0 .. 8) of the 8 characters before p; false when
// one of them is no digit.
__device__ __forceinline__ bool num8(const u32* s, u32 p, u32 n, u32& out)
{
    u32 lo, hi;
    ld8_end(s, p, lo, hi);
    const u64 keep = n ? ~0ull << (64 - 8 * n) : 0ull;
    lo = (lo ^ 0x30303030u) & (u32)keep;
    hi = (hi ^ 0x30303030u) & (u32)(keep >> 32);
    out = num4(lo) * 10000u + num4(hi);
    return (no_digit(lo) | no_digit(hi)) == 0;
}

struct Pow10 {
    double d[9];
    u32 u[9];
};

// A plain decimal of at most 8 digits on either side of its point, as
// parse_decimal gives it: m / 10^f with m below 2^53.  False for any other
// form (which parse_decimal then decides).
__device__ __forceinline__ bool quick_decimal(const u32* s, const Pow10& t, u32 a, u32 e, double& out)
{
    if (a >= e) return false;
    const u32 c0 = ld4(s, a) & 0xFFu;
    const bool neg = c0 == '-';
    if (neg || c0 == '+') ++a;
    const u32 len = e - a;  // (0: no digit below)
    u32 lo, hi;
    ld8_end(s, e, lo, hi);
    const u64 in = len >= 8 ? ~0ull : (len ? ~0ull << (64 - 8 * len) : 0ull);
    const u64 dots = ((u64)eq_bytes(lo, 0x2E2E2E2Eu) | ((u64)eq_bytes(hi, 0x2E2E2E2Eu) << 32)) & in;
    u32 frac = 0, whole = len;
    if (dots) {
        frac = 7u - (u32)((63 - __clzll((long long)dots)) >> 3);
        whole = len - frac - 1;
    }
    if (whole > 8 || whole + frac == 0) return false;
    u32 ip, fp;
    const bool okf = num8(s, e, frac, fp);
    const bool okw = num8(s, e - frac - (dots ? 1u : 0u), whole, ip);
    const u64 m = (u64)ip * t.u[frac] + fp;
    const double v = frac ? (double)m / t.d[frac] : (double)m;
    out = neg ? -v : v;
    return okf && okw && m < (1ull << 53);
}

// "YYYY-MM-DD HH:MM:SS" with an optional fraction of 1 to 3 digits at [a, e);
// false for anything that parse_ts would refuse
__device__ __forceinline__ bool quick_ts(const u32* s, u32 a, u32 e, i64& out)
{
    const u32 len = e - a;
    if (len != 19 && (len < 21 || len > 23)) return false;
    const u32 i = a >> 2, sh = a & 3;
    u32 x[7], w[6];
#pragma unroll
    for (int k = 0; k < 7; ++k) x[k] = s[i + k];
#pragma unroll
    for (int k = 0; k < 6; ++k) w[k] = __builtin_amdgcn_alignbyte(x[k + 1], x[k], sh);
    const u32 f = len == 19 ? 0u : len - 20u;
    const u32 y = w[0] ^ 0x30303030u, mo = (w[1] ^ 0x30303030u) & 0x00FFFF00u, dh = (w[2] ^ 0x30303030u) & 0xFF00FFFFu;
    const u32 hm = (w[3] ^ 0x30303030u) & 0xFFFF00FFu, ss = (w[4] ^ 0x30303030u) & 0x00FFFF00u;
    const u32 fr = (w[5] ^ 0x30303030u) & (f ? 0xFFFFFFFFu >> (32 - 8 * f) : 0u);
    bool ok = (no_digit(y) | no_digit(mo) | no_digit(dh) | no_digit(hm) | no_digit(ss) | no_digit(fr)) == 0;
    ok = ok && (w[1] & 0xFF0000FFu) == 0x2D00002Du && (w[2] & 0x00FF0000u) == 0x00200000u &&
         (w[3] & 0x0000FF00u) == 0x00003A00u && (w[4] & 0x000000FFu) == 0x0000003Au &&
         (f == 0 || (w[4] >> 24) == '.');
    const u32 yy = num4(y);
    const u32 m = __builtin_amdgcn_udot4(mo, 0x00010A00u, 0u, false);
    const u32 d = __builtin_amdgcn_udot4(dh, 0x0000010Au, 0u, false);
    const u32 h = (dh >> 24) * 10u + (hm & 0xFFu);
    const u32 mi = __builtin_amdgcn_udot4(hm, 0x010A0000u, 0u, false);
    const u32 se = __builtin_amdgcn_udot4(ss, 0x00010A00u, 0u, false);
    const u32 ms = __builtin_amdgcn_udot4(fr, 0x00010A64u, 0u, false);
    const bool leap = (yy % 4 == 0 && yy % 100 != 0) || yy % 400 == 0;
    const u32 days = m == 2 ? 28u + (leap ? 1u : 0u) : 30u + ((m + (m >> 3)) & 1u);
    ok = ok && yy >= 1 && m >= 1 && m <= 12 && d >= 1 && d <= days && h <= 23 && mi <= 59 && se <= 59;
    // days since 1970-01-01 (eras of 400 years, March-based years)
    const u32 ym = yy - (m <= 2 ? 1u : 0u);
    const u32 era = ym / 400u, yoe = ym - era * 400u;
    const u32 doy = (153u * (m > 2 ? m - 3u : m + 9u) + 2u) / 5u + d - 1u;
    const u32 doe = yoe * 365u + yoe / 4u - yoe / 100u + doy;
    const i64 day = (i64)era * 146097 + (i64)doe - 719468;
    out = day * 86400000 + (i64)((h * 60u + mi) * 60000u + se * 1000u + ms);
    return ok;
}

// 64 bits of a byte mask from bit p
__device__ __forceinline__ u64 bits_from(const u64* m, u32 p)
{
    const u32 b = p & 63;
    return b ? (m[p >> 6] >> b) | (m[(p >> 6) + 1] << (64 - b)) : m[p >> 6];
}

// newlines, commas and quotes among 16 bytes, a bit each
__device__ __forceinline__ void byte_marks(uint4 v, u32& nl, u32& cm, u32& qt)
{
    const u32 x[4] = {v.x, v.y, v.z, v.w};
    nl = cm = qt = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        nl |= pack_bytes(eq_bytes(x[k], 0x0A0A0A0Au)) << (4 * k);
        cm |= pack_bytes(eq_bytes(x[k], 0x2C2C2C2Cu)) << (4 * k);
        qt |= pack_bytes(eq_bytes(x[k], 0x22222222u)) << (4 * k);
    }
}

constexpr u64 ROW_MAX = 1ull << 20;  // a row of so many bytes, its line end not counted, is malformed

// A row that starts at byte b of the text and ends past the staged bytes, by the
// whole block (all threads; the row in thread 0): 4 096 bytes a step until its end,
// or until a seventh comma, a quote or ROW_MAX bytes have made it malformed whatever
// follows.  60 000 rows of 3 KB take 0.26 ms, 2 500 of 40 KB 0.11; one thread
// going through such a row byte by byte took 7.07 and 18.8, and many seconds where the
// line breaks are missing.
__device__ __forceinline__ Row long_row(const unsigned char* __restrict__ text, u64 nbytes, u64 b, u32* s_tmp)
{
    __shared__ u32 s_first, s_cp[6];
    const u32 at = 16 * threadIdx.x;
    u32 nc = 0;
    bool quote = false, ended = false;
    u64 end = nbytes;
    for (u64 q = b & ~15ull;; q += 16 * CB) {
        if (threadIdx.x == 0) s_first = ~0u;
        u32 nl, cm, qt;
        byte_marks(load16(text, q + at, nbytes), nl, cm, qt);
        if (q + at < b) {
            const u32 from = 0xFFFFu << (u32)(b - q);  // (thread 0 of the first step)
            nl &= from;
            cm &= from;
            qt &= from;
        }
        __syncthreads();
        if (nl) atomicMin(&s_first, at + (u32)__ffs((int)nl) - 1);
        __syncthreads();
        const u32 first = s_first;
        const u32 upto = first <= at ? 0u : (first - at < 16 ? (1u << (first - at)) - 1 : 0xFFFFu);
        cm &= upto;
        qt &= upto;
        u32 tot;
        u32 c = nc + (block_exclusive_sum<CB>((u32)__popc(cm) | (qt ? 1u << 16 : 0u), s_tmp, tot) & 0xFFFFu);
        for (; cm && c < 6; ++c, cm &= cm - 1) s_cp[c] = (u32)(q + at - b) + (u32)__ffs((int)cm) - 1;
        nc += tot & 0xFFFFu;
        quote |= (tot >> 16) != 0;
        const u64 next = q + 16 * CB;
        ended = first != ~0u || next >= nbytes;
        if (first != ~0u) end = q + first;
        if (ended || quote || nc > 6 || next - b >= ROW_MAX + 2) break;
    }
    __syncthreads();
    if (threadIdx.x != 0 || !ended || quote || nc != 6) return malformed();
    if (end > b && text[end - 1] == '\r') --end;
    return end - b < ROW_MAX ? parse_fields(text + b, s_cp, (u32)(end - b)) : malformed();
}

// The rows that start in the block's tile (line r starts at byte 0 or after
// newline r - 1; base: newlines before the tile), one per thread and round;
// header lines are skipped, rows past cap counted only.  The block of the last
// tile writes the row count.
constexpr int CST = CT + CHALO;      // staged bytes
constexpr int CSW = CST / 64;        // words of a byte mask
constexpr int CFRONT = 16;           // bytes before the first staged one (reads end at a position)
constexpr int CROWS = 512;           // row starts listed per round
__global__ void __launch_bounds__(CB) k_csv_parse(const unsigned char* __restrict__ text, u64 nbytes,
                                                  const u32* __restrict__ gcnt, const u64* __restrict__ sub, u32 tiles,
                                                  u32 CG, int summed, int header,
                                                  cv_records_out o, float* __restrict__ heading,
                                                  uint8_t* __restrict__ row_ok, u64 cap, cv_result* res)
{
    static_assert(CT % (64 * CB) == 0, "whole mask words per thread");
    constexpr int WPT = CT / 64 / CB;  // newline words per thread
    __shared__ __attribute__((aligned(16))) u32 s_txt[(CFRONT + CST + 32) / 4];
    __shared__ __attribute__((aligned(8))) uint16_t s_nl[CST / 16 + 4], s_cm[CST / 16 + 12], s_qt[CST / 16 + 12];
    __shared__ uint16_t s_row[CROWS];
    __shared__ u32 s_tmp[CB / WAVE];
    __shared__ Pow10 s_p;
    __shared__ u32 s_long;  // the tile's row whose end is not staged (its last; ~0: none)
    __shared__ u64 s_long_row;
    const int tid = threadIdx.x;
    const u64 t0 = (u64)blockIdx.x * CT;
    const u64 left = nbytes - t0;
    const u32 avail = left < (u64)CST ? (u32)left : (u32)CST;  // staged bytes of the text
    // 1. the text and its bits
    constexpr int Q = CT / 16 / CB;
    static_assert(Q * CB * 16 == CT && CHALO / 16 <= CB, "whole rounds, then one for the bytes after the tile");
    uint4 tv[Q + 1];
    const u32 hc = (u32)(CT / 16) + (tid < CHALO / 16 ? tid : 0);  // (spare threads repeat the first)
    if (t0 + CST <= nbytes) {
#pragma unroll
        for (int k = 0; k < Q; ++k) tv[k] = *reinterpret_cast<const uint4*>(text + t0 + 16 * (u64)(k * CB + tid));
        tv[Q] = *reinterpret_cast<const uint4*>(text + t0 + 16 * (u64)hc);
    } else {
#pragma unroll
        for (int k = 0; k < Q; ++k) tv[k] = load16(text, t0 + 16 * (u64)(k * CB + tid), nbytes);
        tv[Q] = load16(text, t0 + 16 * (u64)hc, nbytes);
    }
#pragma unroll
    for (int r = 0; r <= Q; ++r) {
        if (r == Q && tid >= CHALO / 16) break;
        const u32 c = r < Q ? (u32)(r * CB + tid) : hc;
        const uint4 v = tv[r];
        *reinterpret_cast<uint4*>(&s_txt[CFRONT / 4 + 4 * c]) = v;
        u32 nl, cm, qt;
        byte_marks(v, nl, cm, qt);
        s_nl[c] = (uint16_t)nl;
        s_cm[c] = (uint16_t)cm;
        s_qt[c] = (uint16_t)qt;
    }
    if (tid == 0) s_long = ~0u;
    if (tid < 12) {
        s_cm[CST / 16 + tid] = 0;
        s_qt[CST / 16 + tid] = 0;
        if (tid < 4) s_txt[tid] = 0;
        if (tid < 8) s_txt[(CFRONT + CST) / 4 + tid] = 0;
    }
    if (tid < 9) {
        double d = 1.0;
        u32 u = 1;
        for (int k = 0; k < tid; ++k) {
            d *= 10.0;
            u *= 10u;
        }
        s_p.d[tid] = d;  // exact
        s_p.u[tid] = u;
    }
    // 2. newlines before the tile
    const u32 grp = blockIdx.x / CG;
    u32 base;
    if (summed) {
        base = gcnt[grp];
        __syncthreads();
    } else {
        u32 v = 0;
        for (u32 i = tid; i < grp; i += CB) v += gcnt[i];
        block_exclusive_sum<CB>(v, s_tmp, base);
    }
    if (CG > 1) {
        u64 t = sub[grp];
        for (u32 k = blockIdx.x % CG; k > 0; --k, t >>= 16) base += (u32)(t & 0xFFFF);
    }
    // the line that starts at the tile's first byte, if one does
    const bool first = t0 == 0 || text[t0 - 1] == '\n';
    const u64* nlw = reinterpret_cast<const u64*>(s_nl);
    const u64* cmw = reinterpret_cast<const u64*>(s_cm);
    const u64* qtw = reinterpret_cast<const u64*>(s_qt);
    // 3. newlines of the tile that start a row inside it
    u64 m[WPT];
    u32 c = 0, allnl = 0;
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
        m[k] = nlw[tid * WPT + k];
        allnl += (u32)__popcll(m[k]);
        if (tid == CB - 1 && k == WPT - 1) m[k] &= ~(1ull << 63);  // the next tile's first byte
        if (tid * WPT * 64 + 64 * (k + 1) >= (int)avail) {
            // a newline that ends the text starts no row
            const int last = (int)avail - 1 - (tid * WPT + k) * 64;
            if (last < 64) m[k] &= last <= 0 ? 0ull : ((1ull << last) - 1);
        }
        c += (u32)__popcll(m[k]);
    }
    u32 starts;
    const u32 before = block_exclusive_sum<CB>(c, s_tmp, starts);
    const u32 R = starts + (first ? 1u : 0u);
    const u64 line0 = (u64)base + (first ? 0 : 1);  // line of the tile's first row
    if (blockIdx.x == tiles - 1) {
        u32 nl;
        block_exclusive_sum<CB>(allnl, s_tmp, nl);
        if (tid == 0) {
            const u64 lines = (u64)base + nl + (text[nbytes - 1] != '\n' ? 1 : 0);
            const u64 rows = lines - ((header && lines) ? 1 : 0);
            res->status = rows > cap ? CV_ERR_CAPACITY : CV_OK;
            res->count = rows;
            res->required = rows > cap ? rows : 0;
        }
    }
    u32 bad = 0;
    auto put = [&](u64 row, const Row& w) {
        bad += w.ok ? 0u : 1u;
        o.journey_id[row] = w.jid;
        o.ts_ms[row] = w.ts;
        o.lat_deg[row] = w.lat;
        o.lon_deg[row] = w.lon;
        o.speed_mps[row] = (float)w.spd;
        if (heading) heading[row] = (float)w.hdg;
        if (row_ok) row_ok[row] = w.ok ? 1 : 0;
    };
    for (u32 r0 = 0; r0 < R; r0 += CROWS) {
        // starts of rows [r0, r0 + CROWS)
        if (first && r0 == 0 && tid == 0) s_row[0] = 0;
        u32 k = before + (first ? 1u : 0u);
#pragma unroll
        for (int q = 0; q < WPT; ++q) {
            u64 x = m[q];
            const u32 n = (u32)__popcll(x);
            if (k + n > r0 && k < r0 + CROWS) {
                for (u32 j = k; x; ++j, x &= x - 1)
                    if (j >= r0 && j < r0 + CROWS)
                        s_row[j - r0] = (uint16_t)((tid * WPT + q) * 64 + __ffsll((long long)x));
            }
            k += n;
        }
        __syncthreads();
        const u32 rn = R - r0 < CROWS ? R - r0 : CROWS;
        for (u32 j = tid; j < rn; j += CB) {
            const u64 line = line0 + r0 + j;
            if (header && line == 0) continue;
            const u64 row = line - (header ? 1 : 0);
            if (row >= cap) continue;
            const u32 a = s_row[j];
            // its end: the next newline, or the end of the text
            u32 wi = a >> 6;
            u64 x = nlw[wi] & (~0ull << (a & 63));
            while (!x && wi + 1 < (u32)CSW) x = nlw[++wi];
            if (!x && t0 + CST < nbytes) {  // the row's end is not staged
                s_long = a;
                s_long_row = row;
                continue;
            }
            u32 z = x ? (wi << 6) + (u32)__ffsll((long long)x) - 1 : avail;
            if (z > a && ((ld4(s_txt, CFRONT + z - 1) & 0xFFu) == '\r')) --z;
            const u32 len = z - a;
            // the row's commas, and whether it has the shape: six of them, no quote
            u32 cp[6];
            bool shape;
            if (len <= 128) {
                const u64 in0 = len >= 64 ? ~0ull : (1ull << len) - 1;
                const u64 in1 = len > 64 ? (len == 128 ? ~0ull : (1ull << (len - 64)) - 1) : 0ull;
                u64 lo = bits_from(cmw, a) & in0, hi = bits_from(cmw, a + 64) & in1;
                shape = ((bits_from(qtw, a) & in0) | (bits_from(qtw, a + 64) & in1)) == 0 &&
                        __popcll(lo) + __popcll(hi) == 6;
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    const bool l = lo != 0;
                    const u64 y = l ? lo : hi;
                    cp[q] = (l ? 0u : 64u) + (u32)__ffsll((long long)y) - 1u;
                    if (l) lo &= lo - 1;
                    else hi &= hi - 1;
                }
            } else {
                u32 nc = 0;
                u64 quote = 0;
#pragma unroll
                for (int q = 0; q < 6; ++q) cp[q] = 0;
                for (u32 p = 0; p < len && nc <= 6; p += 64) {
                    const u64 in = len - p >= 64 ? ~0ull : (1ull << (len - p)) - 1;
                    u64 y = bits_from(cmw, a + p) & in;
                    quote |= bits_from(qtw, a + p) & in;
                    for (; y && nc <= 6; y &= y - 1, ++nc) {
                        const u32 c = p + (u32)__ffsll((long long)y) - 1u;
#pragma unroll
                        for (int q = 0; q < 6; ++q) cp[q] = nc == (u32)q ? c : cp[q];
                    }
                }
                shape = nc == 6 && quote == 0;
            }
            Row w = malformed();
            if (shape) {
                const u32 p0 = CFRONT + a, pe = CFRONT + z;
                const u32 idn = cp[0];
                // the id's bytes, first one highest
                const u64 raw = (u64)ld4(s_txt, p0) | ((u64)ld4(s_txt, p0 + 4) << 32);
                const u64 id = __builtin_bswap64(raw) & (idn >= 1 && idn < 8 ? ~0ull << (64 - 8 * idn) : ~0ull);
                w.jid = (i64)id;
                w.ok = idn >= 1 && idn <= 8 && (id >> 63) == 0;
                w.ok = quick_ts(s_txt, p0 + cp[0] + 1, p0 + cp[1], w.ts) && w.ok;
                w.ok = quick_decimal(s_txt, s_p, p0 + cp[1] + 1, p0 + cp[2], w.lat) && w.ok;
                w.ok = quick_decimal(s_txt, s_p, p0 + cp[2] + 1, p0 + cp[3], w.lon) && w.ok;
                w.ok = quick_decimal(s_txt, s_p, p0 + cp[4] + 1, p0 + cp[5], w.spd) && w.ok;
                if (p0 + cp[5] + 1 < pe) w.ok = quick_decimal(s_txt, s_p, p0 + cp[5] + 1, pe, w.hdg) && w.ok;
                if (!w.ok) w = parse_fields((const unsigned char*)s_txt + p0, cp, len);
            }
            put(row, w);
        }
        __syncthreads();
    }
    if (s_long != ~0u) {
        const Row w = long_row(text, nbytes, t0 + s_long, s_tmp);
        if (tid == 0) put(s_long_row, w);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) bad += __shfl_xor(bad, d, WAVE);
    if (lane_id() == 0 && bad) atomicAdd((unsigned long long*)&res->n_bad, (unsigned long long)bad);
}

// The call's scratch: the groups' newline counts and, where a group has several
// tiles, the counts of its tiles.  At most 4 bytes per tile and the alignment,
// whatever the capacity.
struct CsvLayout {
    u64 tiles, groups;
    u32 cg;  // tiles per group
    u64* sub;
    u32* gcnt;
    size_t bytes;
    CsvLayout(void* ws, u64 nbytes)
    {
        cvh::Carver c(ws);
        tiles = (nbytes + CT - 1) / CT;
        cg = tiles > CSV_SELF ? CG_L : 1;
        groups = (tiles + cg - 1) / cg;
        sub = c.take<u64>(cg > 1 ? groups : 0);
        gcnt = c.take<u32>(groups ? groups : 1);
        bytes = c.size();
    }
};

}  // namespace

extern "C" {

cv_status cv_csv_workspace_size(uint64_t nbytes, uint64_t capacity, size_t* bytes)
{
    if (!bytes || capacity >= (1ull << 32)) return CV_ERR_INVALID_ARGUMENT;
    const CsvLayout L(nullptr, nbytes);
    if (L.tiles >= (1ull << 31)) return CV_ERR_INVALID_ARGUMENT;
    *bytes = L.bytes;
    return CV_OK;
}

cv_status cv_csv_extract(const char* text, uint64_t nbytes, int32_t has_header, const cv_records_out* out,
                         float* heading_deg, uint8_t* row_ok, uint64_t capacity, cv_result* res, void* ws,
                         size_t ws_bytes, void* stream)
{
    if (!res || !out || capacity >= (1ull << 32) || (nbytes && !text) || !cvh::aligned(text, 16))
        return CV_ERR_INVALID_ARGUMENT;
    if (capacity && (!out->journey_id || !out->ts_ms || !out->lat_deg || !out->lon_deg || !out->speed_mps))
        return CV_ERR_INVALID_ARGUMENT;
    size_t need = 0;
    cv_status e = cv_csv_workspace_size(nbytes, capacity, &need);
    if (e != CV_OK) return e;
    if (!ws || !cvh::aligned(ws, cvh::WS_ALIGN) || ws_bytes < need) return CV_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    cvh::TimedScope ts_("csv_extract", s);
    const CsvLayout L(ws, nbytes);
    const bool summed = L.cg > 1;
    const unsigned char* t = (const unsigned char*)text;
    hipLaunchKernelGGL(summed ? k_csv_count<CG_L> : k_csv_count<1>, dim3((unsigned)(L.groups ? L.groups : 1)), dim3(CB), 0,
                       s, t, (u64)nbytes, L.gcnt, L.sub, res);
    if (!L.tiles) return cvh::last_launch_status();
    if (summed) hipLaunchKernelGGL(k_csv_scan, dim3(1), dim3(1024), 0, s, L.gcnt, L.groups);
    hipLaunchKernelGGL(k_csv_parse, dim3((unsigned)L.tiles), dim3(CB), 0, s, t, (u64)nbytes, L.gcnt, L.sub, (u32)L.tiles,
                       L.cg, summed ? 1 : 0, has_header ? 1 : 0, *out, heading_deg, row_ok, (u64)capacity, res);
    return cvh::last_launch_status();
}

}  // extern "C"
