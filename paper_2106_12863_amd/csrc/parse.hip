// Session text to columns (section "Dataset Description", Table 1: the
// PA-7080 session record, 24 fields).  One record per line, Table 1's fields
// in order separated by ','; the columns come from field 1 (capture_time,
// "YYYY/MM/DD HH:MM:SS.mmm", as milliseconds since midnight of the origin
// day), fields 5 and 8 (source and destination, dotted quads) and field 21
// (bytes).  Every '\n'-ended segment is a line (an empty one too); a last
// segment without '\n' is a line when it is not empty.  A line with fewer
// than 21 fields, an impossible date, a time outside [0, 2^32 - 1) ms of the
// origin, an octet above 255 or a byte count above 2^64 - 1 gives
// ts = 0xFFFFFFFF, src = dst = bytes = 0 and counts as bad.
//
// k_parse reads the text once.  A workgroup takes a block of kOwn bytes, in
// order (a ticket each), and looks at the kWindow - kOwn bytes after it too: 64
// bytes per lane, classified in registers and staged in LDS.  The positions of
// the delimiters (',' and '\n') are compacted into LDS by rank, so a line, which
// starts after a delimiter that is a newline, finds the ends of its fields by
// index.  A lane per line then parses the four fields with four-byte reads and
// byte dot products.  A window with more delimiters or lines than the lists hold
// (lines of less than 130 bytes) is parsed in rounds, a list at a time; the last
// line, where its fields leave the window, by one wave from device memory.
// The number of newlines before a block comes from the blocks before it: each
// publishes its own count at once, then the count up to its end, and one wave
// adds up its predecessors' counts back to the nearest such sum while the
// others parse.  A block waits only for lower tickets, whose holders publish
// their counts before they wait, so the lowest unfinished block never waits and
// every wait ends.
//
// Bound by vector issue (681 instructions per 4 KB wave, 66 % of its cycles),
// then HBM.  3.9 GB of text, 2e7 lines: 4.22 ms with a counting pass, an index
// of line starts and a pass over staged lines; 2.41 with a counting pass and
// this kernel; 2.29 with the byte-permute classification instead of zero-byte
// arithmetic; 2.10 with the counts found by the kernel itself; 1.84 ms (2.4
// TB/s) with the search for them beside the parsing.  Persistent workgroups
// that fetched their next block early took 4.30 ms: a ticket taken early
// publishes its count late.  4e8 bytes of 79-byte lines, 10,000 delimiters a
// window: 0.87 ms with the lines beyond the lists read from device memory, 0.44 in
// rounds.  2e8 bytes of 5,080-byte lines: 5.83 ms with the lines that leave their
// window read by a lane, byte by byte, 0.22 by a wave.
// The block that holds a newline owns the line after it; the first block owns
// the first line.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pass_common.h"
#include "sinet.h"
#include "sinet_internal.h"

namespace sinet {
namespace {

constexpr int kParseBlock = 512;
constexpr uint32_t kWindow = 64 * kParseBlock;  // text bytes a workgroup looks at
constexpr uint32_t kOwn = kWindow - 1024;       // of which it owns the newlines
constexpr uint32_t kOwnLanes = kOwn / 64;       // lanes whose bytes it owns
static_assert(kOwn % 64 == 0, "a lane's bytes are owned or not");
// state of a block: its newlines (its own, or up to its end) and what they are
constexpr uint64_t kOwnCount = 1ull << 62, kSumCount = 2ull << 62, kCountMask = kOwnCount - 1;
constexpr uint32_t kDelims = 6144;              // delimiters listed (25 per line of 200 bytes: 4,100)
constexpr uint32_t kLines = 1024;               // newlines listed
constexpr uint32_t kBadTs = 0xFFFFFFFFu;

// The text as whole 16-byte groups: position x (from the aligned address at or
// below the text) holds text byte x - skew.
struct Text {
    const uint8_t* base;  // 16-byte aligned; bytes [skew, end) are the text
    uint32_t skew;
    uint64_t end;
};

// The 16 bytes from position x (a multiple of 16); bytes outside the text are
// 0 and are not read.
__device__ __forceinline__ uint4 group16(const Text& t, uint64_t x) {
    if (x >= t.skew && x + 16 <= t.end) {
        const u32x4_t v = *glob(reinterpret_cast<const u32x4_t*>(t.base + x));
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    uint32_t w[4] = {0u, 0u, 0u, 0u};
    for (uint32_t b = 0; b < 16; ++b)
        if (x + b >= t.skew && x + b < t.end) w[b >> 2] |= (uint32_t)*glob(t.base + x + b) << (8 * (b & 3u));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// Per byte of w: 0x00 where it is the character C, else 0xFF.  A byte permute
// takes its selectors from the text: selector 12 gives 0x00, every other one
// 0xFF when all the bytes it may select (and their signs) are ones, and the
// exclusive or moves C to 12.
template <uint32_t C>
__device__ __forceinline__ uint32_t not_char(uint32_t w) {
    return __builtin_amdgcn_perm(0xFFFFFFFFu, 0xFFFFFFFFu, w ^ (0x01010101u * (C ^ 12u)));
}

// Low eight bits: which of the eight bytes of lo and hi are C.  Flags of 0 and
// -1 times the weights 1, 2, .. 64, -128 sum to minus the mask of the other
// bytes (modulo 256); starting from -1 leaves its complement.
template <uint32_t C>
__device__ __forceinline__ uint32_t chars8(uint32_t lo, uint32_t hi) {
    const int m = __builtin_amdgcn_sdot4((int)not_char<C>(lo), 0x08040201, -1, false);
    return (uint32_t)__builtin_amdgcn_sdot4((int)not_char<C>(hi), (int)0x80402010u, m, false);
}

// Bit i: byte i of the 16 bytes v is C.
template <uint32_t C>
__device__ __forceinline__ uint32_t chars16(uint4 v) {
    return __builtin_amdgcn_perm(chars8<C>(v.z, v.w), chars8<C>(v.x, v.y), 0x0C0C0400u);
}

// days since 1970-01-01 of a proleptic Gregorian date (H. Hinnant's
// days_from_civil)
// (years 0..9999 here: 32-bit arithmetic suffices)
__device__ __forceinline__ int32_t days_from_civil(int32_t y, int32_t m, int32_t d) {
    y -= m <= 2 ? 1 : 0;
    const int32_t era = (y >= 0 ? y : y - 399) / 400;
    const int32_t yoe = y - era * 400;
    const int32_t mp = m > 2 ? m - 3 : m + 9;
    const int32_t doy = (153 * mp + 2) / 5 + d - 1;
    const int32_t doe = yoe * 365 + yoe / 4 - yoe / 100 + doy;
    return era * 146097 + doe - 719468;
}

// Byte access to one line staged in LDS.
struct LdsLine {
    const uint8_t* p;  // the line's first byte
    __device__ __forceinline__ uint32_t operator[](uint32_t i) const { return p[i]; }
    // byte i, or 0xFF at or past e; reads up to 3 bytes past a field's end
    // stay inside the staging (it has 16 bytes of slack), so no branch
    __device__ __forceinline__ uint32_t upto(uint32_t i, uint32_t e) const {
        const uint32_t c = p[i];
        return i < e ? c : 0xFFu;
    }
};

// The date and time of day as milliseconds from the origin day's midnight;
// false for an impossible one or one outside [0, 2^32 - 1).
__device__ __forceinline__ bool time_of(int32_t y, int32_t mo, int32_t d, int32_t h, int32_t mi, int32_t se,
                                        int32_t ms, int64_t origin, uint32_t& ts) {
    if (mo < 1 || mo > 12 || d < 1) return false;
    const bool leap = (y % 4 == 0 && y % 100 != 0) || y % 400 == 0;
    // days in month: 31 except April, June, September, November (30) and February
    const int32_t dim = mo == 2 ? (leap ? 29 : 28) : ((mo == 4 || mo == 6 || mo == 9 || mo == 11) ? 30 : 31);
    if (d > dim || h > 23 || mi > 59 || se > 59) return false;
    // a day before the origin's is negative, the 50th after it past 2^32
    const int64_t day = (int64_t)days_from_civil(y, mo, d) - origin;
    if (day < 0 || day > 49) return false;
    const uint64_t t = (uint64_t)(uint32_t)day * 86400000u + (uint32_t)(h * 3600000 + mi * 60000 + se * 1000 + ms);
    if (t >= kBadTs) return false;
    ts = (uint32_t)t;
    return true;
}

// 1 to 20 decimal digits in [s, e), at most 2^64 - 1.
__device__ __forceinline__ bool count_u64(const LdsLine& b, uint32_t s, uint32_t e, uint64_t& out) {
    if (e <= s || e - s > 20) return false;
    // 19 digits stay below 10^19 < 2^64 - 1, so only a 20th digit can
    // overflow; the digits before it are taken four at a time
    const uint32_t last = e - s == 20 ? e - 1 : e;
    uint64_t v = 0;
    for (uint32_t i = s; i < last; i += 4) {
        const uint32_t k = last - i < 4u ? last - i : 4u;  // digits in this group
        const uint32_t d0 = b.upto(i, last) - '0', d1 = b.upto(i + 1, last) - '0';
        const uint32_t d2 = b.upto(i + 2, last) - '0', d3 = b.upto(i + 3, last) - '0';
        if (d0 > 9u || (k > 1u && d1 > 9u) || (k > 2u && d2 > 9u) || (k > 3u && d3 > 9u)) return false;
        const uint32_t g2 = d0 * 10 + d1, g3 = g2 * 10 + d2;
        const uint32_t g = k == 1u ? d0 : k == 2u ? g2 : k == 3u ? g3 : g3 * 10 + d3;
        const uint32_t p10 = k == 1u ? 10u : k == 2u ? 100u : k == 3u ? 1000u : 10000u;
        v = v * p10 + g;
    }
    if (last != e) {
        const uint32_t c = b[last] - '0';
        if (c > 9u) return false;
        // v * 10 + c > 2^64 - 1 = 18446744073709551615 exactly when v exceeds
        // floor((2^64 - 1) / 10), or equals it and c > 5
        if (v > 1844674407370955161ull || (v == 1844674407370955161ull && c > 5u)) return false;
        v = v * 10 + c;
    }
    out = v;
    return true;
}

// One line of the window, parsed from the staged text and its delimiters.
// Reads of up to three bytes before a field stay inside the line, of up to
// three after one inside the staging (16 bytes of slack).
struct Staged {
    const uint8_t* text;
    __device__ __forceinline__ uint32_t word(uint32_t at) const {  // any alignment
        uint32_t w;
        __builtin_memcpy(&w, text + at, 4);
        return w;
    }
};

// Nonzero when a byte of x (digits less '0' by exclusive or) is above 9.
__device__ __forceinline__ uint32_t not_digits(uint32_t x) { return (x | (x + 0x76767676u)) & 0x80808080u; }

// Field 1 at s, 23 bytes: "YYYY/MM/DD hh:mm:ss.mmm".
__device__ __forceinline__ bool staged_time(const Staged& b, uint32_t s, int64_t origin, uint32_t& ts) {
    constexpr uint32_t z = 0x30303030u;
    const uint32_t w0 = b.word(s), w1 = b.word(s + 4), w2 = b.word(s + 8), w3 = b.word(s + 12),
                   w4 = b.word(s + 16), w5 = b.word(s + 20);
    // "YYYY" "/MM/" "DD h" "h:MM" ":SS." "mmm,"
    const uint32_t seps = ((w1 ^ 0x2F00002Fu) & 0xFF0000FFu) | ((w2 ^ 0x00200000u) & 0x00FF0000u) |
                          ((w3 ^ 0x00003A00u) & 0x0000FF00u) | ((w4 ^ 0x2E00003Au) & 0xFF0000FFu);
    const uint32_t x0 = w0 ^ z, x1 = (w1 ^ z) & 0x00FFFF00u, x2 = (w2 ^ z) & 0xFF00FFFFu,
                   x3 = (w3 ^ z) & 0xFFFF00FFu, x4 = (w4 ^ z) & 0x00FFFF00u, x5 = (w5 ^ z) & 0x00FFFFFFu;
    const uint32_t bad = seps | not_digits(x0) | not_digits(x1) | not_digits(x2) | not_digits(x3) |
                         not_digits(x4) | not_digits(x5);
    if (bad) return false;
    auto dot = [](uint32_t x, uint32_t w, uint32_t c) { return __builtin_amdgcn_udot4(x, w, c, false); };
    const int32_t y = (int32_t)(dot(x0, 0x0000010Au, 0u) * 100u + dot(x0, 0x010A0000u, 0u));
    const int32_t mo = (int32_t)dot(x1, 0x00010A00u, 0u), d = (int32_t)dot(x2, 0x0000010Au, 0u);
    const int32_t h = (int32_t)dot(x2, 0x0A000000u, x3 & 0xFFu), mi = (int32_t)dot(x3, 0x010A0000u, 0u);
    const int32_t se = (int32_t)dot(x4, 0x00010A00u, 0u), ms = (int32_t)dot(x5, 0x00010A64u, 0u);
    return time_of(y, mo, d, h, mi, se, ms, origin, ts);
}

// Four digits or fewer that end before `end`: the last k of them (1 to 4).
__device__ __forceinline__ uint32_t last_digits(const Staged& b, uint32_t end, uint32_t k, uint32_t& bad) {
    const uint32_t x = (b.word(end - 4) ^ 0x30303030u) & (0xFFFFFFFFu << (8u * (4u - k)));
    bad |= not_digits(x);
    return __builtin_amdgcn_udot4(x, 0x0000010Au, 0u, false) * 100u +
           __builtin_amdgcn_udot4(x, 0x010A0000u, 0u, false);
}

// A dotted quad in [s, e): four octets of one to three digits, 0 to 255.
__device__ __forceinline__ bool staged_ipv4(const Staged& b, uint32_t s, uint32_t e, uint32_t& a) {
    const uint32_t n = e - s;
    if (n < 7u || n > 15u) return false;
    // bit i: byte i of the field is '.'
    uint32_t m = chars16<'.'>(make_uint4(b.word(s), b.word(s + 4), b.word(s + 8), b.word(s + 12)));
    m &= (1u << n) - 1u;
    if (__popc(m) != 3) return false;
    uint32_t bad = 0, v = 0, at = 0;  // at: the octet's first byte
#pragma unroll
    for (int part = 0; part < 4; ++part) {
        const uint32_t end = part < 3 ? (uint32_t)__builtin_ctz(m) : n, k = end - at;
        bad |= k - 1u > 2u ? 1u : 0u;
        const uint32_t o = last_digits(b, s + end, min(max(k, 1u), 4u), bad);
        bad |= o > 255u ? 1u : 0u;
        v = (v << 8) | (o & 255u);
        at = end + 1;
        m &= m - 1u;
    }
    a = v;
    return bad == 0u;
}

// The same as count_u64, four digits at a time where none can overflow.
__device__ __forceinline__ bool staged_count(const Staged& b, uint32_t s, uint32_t e, uint64_t& out) {
    const uint32_t n = e - s;
    if (n < 1u || n > 20u) return false;
    if (n == 20u) return count_u64(LdsLine{b.text}, s, e, out);
    uint32_t bad = 0;
    uint64_t v = 0, p10 = 1;
    for (uint32_t k = 0; k < n; k += 4) {  // from the last four digits on
        v += p10 * last_digits(b, e - k, min(n - k, 4u), bad);
        p10 *= 10000u;
    }
    out = v;
    return bad == 0u;
}

struct ParseArgs {
    Text t;
    unsigned long long* state;  // [blocks], zero at first
    unsigned long long* total;  // newlines
    unsigned long long* bad;    // bad lines
    uint32_t* ticket;
    uint32_t n_blocks;
    uint64_t cap;               // lines the columns hold
    int64_t origin;
    uint32_t* ts;
    uint32_t* src;
    uint32_t* dst;
    uint64_t* bytes;
};

// Newlines before block b, by one wave: lanes read 64 blocks' states at a time,
// from b - 1 down, until every block after the nearest sum has its count.
__device__ __forceinline__ uint64_t newlines_before(const ParseArgs& a, uint32_t b, uint32_t lane) {
    uint64_t sum = 0;
    for (int64_t top = (int64_t)b - 1; top >= 0; top -= 64) {
        const int64_t i = top - (int64_t)lane;
        uint64_t x, sums;
        for (;;) {
            x = i >= 0 ? __hip_atomic_load(a.state + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kSumCount;
            sums = __ballot(x >= kSumCount);
            const uint64_t none = __ballot(x < kOwnCount);
            // ready when no lane before the nearest sum (or none at all) is empty
            if ((none & (sums ? (sums & -sums) - 1 : ~0ull)) == 0) break;
            __builtin_amdgcn_s_sleep(1);
        }
        const uint32_t last = sums ? (uint32_t)__builtin_ctzll(sums) : 63u;
        uint64_t v = lane <= last ? x & kCountMask : 0ull;
#pragma unroll
        for (int o = 32; o; o >>= 1) v += __shfl_xor(v, o);
        sum += v;
        if (sums) break;
    }
    return sum;
}

// A line that leaves its window, from position s on, by one wave: 1,024 bytes a
// step, the next ones loaded meanwhile.  A lane ranks its 16 bytes' delimiters and
// notes the ends of the fields that are needed; then the fields are copied to LDS
// (buf, 96 bytes) and every lane parses them.
__device__ __forceinline__ bool line_far(const ParseArgs& a, uint64_t s, uint32_t lane, uint64_t* ends,
                                         uint8_t* buf, uint32_t& ts, uint32_t& src, uint32_t& dst,
                                         uint64_t& nb) {
    constexpr uint32_t kEnds[7] = {1, 4, 5, 7, 8, 20, 21};  // delimiters of the line, by number
    uint64_t x = (s & ~15ull) + 16u * lane;
    uint4 v = group16(a.t, x);
    uint32_t seen = 0;  // delimiters before this step
    for (;; x += 1024) {
        const uint4 next = group16(a.t, x + 1024);
        uint32_t nl = chars16<10>(v), dl = nl | chars16<','>(v);
        if (x < s) {  // the first step's first group: bytes before the line
            nl &= 0xFFFFu << (uint32_t)(s - x);
            dl &= 0xFFFFu << (uint32_t)(s - x);
        }
        const uint32_t c = (uint32_t)__popc(dl);
        uint32_t before = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = (uint32_t)__shfl_up((int)before, o);
            if (lane >= (uint32_t)o) before += y;
        }
        uint32_t upto = (uint32_t)__builtin_amdgcn_readlane((int)before, 63);  // of the line
        before -= c;
        const uint64_t has = __ballot(nl != 0u);
        if (has)  // up to the line's own newline
            upto = (uint32_t)__builtin_amdgcn_readlane((int)(before + (uint32_t)__popc(dl & ((nl & (0u - nl)) * 2u - 1u))),
                                                       __builtin_ctzll(has));
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            uint32_t j = kEnds[k] - seen - before;  // the lane's j-th delimiter, wrapped when below
            if (j - 1u >= c || kEnds[k] - seen > upto) continue;
            uint32_t m = dl;
            for (; j > 1; --j) m &= m - 1u;
            ends[k] = x + (uint32_t)__builtin_ctz(m);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        const bool start = seen == 0;
        seen += upto;
        // a first field of other than 23 bytes: bad, however long the line is
        if (start && (seen == 0 || ends[0] - s != 23u)) return false;
        if (has || seen >= 21u) break;
        if (x - 16u * lane + 1024 >= a.t.end) {  // the text ends with this line
            if (seen == 20u && lane == 0) ends[6] = a.t.end;
            ++seen;  // as a newline would
            break;
        }
        v = next;
    }
    if (seen < 21u) return false;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    const uint64_t f[4] = {s, ends[1] + 1, ends[3] + 1, ends[5] + 1};
    const uint64_t n1 = ends[2] - f[1], n2 = ends[4] - f[2], n3 = ends[6] - f[3];
    if (n1 > 15u || n2 > 15u || n3 > 20u) return false;
    // each field with three bytes before it and three behind in its own part
    constexpr uint32_t kAt[4] = {4, 32, 52, 72};
    const uint32_t n[4] = {23u, (uint32_t)n1, (uint32_t)n2, (uint32_t)n3};
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (lane < n[k]) buf[kAt[k] + lane] = *glob(a.t.base + f[k] + lane);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    const Staged b{buf};
    return staged_time(b, kAt[0], a.origin, ts) && staged_ipv4(b, kAt[1], kAt[1] + n[1], src) &&
           staged_ipv4(b, kAt[2], kAt[2] + n[2], dst) && staged_count(b, kAt[3], kAt[3] + n[3], nb);
}

__device__ __forceinline__ uint32_t put_line(const ParseArgs& a, uint64_t l, bool ok, uint32_t ts,
                                             uint32_t src, uint32_t dst, uint64_t nb) {
    if (l >= a.cap) return 0u;  // the call is refused then
    a.ts[l] = ok ? ts : kBadTs;
    a.src[l] = ok ? src : 0u;
    a.dst[l] = ok ? dst : 0u;
    a.bytes[l] = ok ? nb : 0ull;
    return ok ? 0u : 1u;
}

__global__ void __launch_bounds__(kParseBlock, 6) k_parse(ParseArgs a) {
    __shared__ __attribute__((aligned(16))) uint8_t s_text[kWindow + 16];
    __shared__ __attribute__((aligned(16))) uint16_t s_delim[kDelims];  // positions in the window, ascending
    __shared__ uint16_t s_start[kLines], s_rank[kLines];  // per newline: position + 1, its delimiter rank
    __shared__ uint32_t s_wave[kParseBlock / 64];
    __shared__ uint32_t s_blk, s_own, s_bad, s_end, s_far;
    __shared__ uint64_t s_base, s_ends[7];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    if (tid == 0) {
        s_bad = s_far = 0;
        s_blk = atomicAdd(a.ticket, 1u);
    }
    __syncthreads();
    const uint32_t blk = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_blk);  // below n_blocks, the grid
    const uint64_t b0 = (uint64_t)blk * kOwn;
    uint32_t bad = 0;
    uint4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = group16(a.t, b0 + 64u * tid + 16 * k);
    // 64 bytes: delimiter and newline masks, the bytes to LDS
    uint64_t dm = 0, nm = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        reinterpret_cast<uint4*>(s_text)[4 * tid + k] = v[k];
        const uint32_t n = chars16<10>(v[k]), d = n | chars16<','>(v[k]);
        dm |= (uint64_t)d << (16 * k);
        nm |= (uint64_t)n << (16 * k);
    }
    // ranks: delimiters in the low half, newlines in the high half
    const uint32_t mine = (uint32_t)__popcll(dm) | (uint32_t)__popcll(nm) << 16;
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, o);
        if (lane >= (uint32_t)o) incl += y;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t before = incl - mine, total = 0;
#pragma unroll
    for (uint32_t w = 0; w < kParseBlock / 64; ++w) {
        const uint32_t x = s_wave[w];
        if (w < wave) before += x;
        total += x;
    }
    const uint32_t n_delim = total & 0xFFFFu, n_nl = total >> 16;
    const bool at_end = b0 + kWindow >= a.t.end;  // nothing follows the window
    if (tid == kOwnLanes - 1) {  // the block's own newlines, known to its successors from here on
        s_own = (before + mine) >> 16;
        __hip_atomic_store(a.state + blk, kOwnCount | s_own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the last wave finds the newlines before the block
    auto place = [&]() {
        if (wave != kParseBlock / 64 - 1) return;
        const uint64_t sum = newlines_before(a, blk, lane);
        if (lane == 0) {
            const uint64_t upto = sum + s_own;
            s_base = sum;
            __hip_atomic_store(a.state + blk, kSumCount | upto, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (blk + 1 == a.n_blocks) *a.total = upto;
        }
    };
    // The lines, in rounds: each lists delimiters from rank d_lo and newlines from
    // number k_lo on and parses the lines whose own are all listed.  Lines of 130
    // bytes and more take one round.
    uint32_t line = 0, d_lo = 0, k_lo = 0;  // the round's first line of the block
    for (bool first = true;; first = false) {
        const bool more = n_delim - d_lo > kDelims || n_nl - k_lo > kLines;
        if (!more && first) {
            uint32_t r = before & 0xFFFFu;
#pragma unroll
            for (int h = 0; h < 2; ++h)
                for (uint32_t m = (uint32_t)(dm >> (32 * h)); m; m &= m - 1u, ++r)
                    s_delim[r] = (uint16_t)(64u * tid + 32u * h + (uint32_t)__builtin_ctz(m));
            uint32_t k = before >> 16;
            for (uint64_t m = nm; m; m &= m - 1, ++k) {
                const uint32_t q = (uint32_t)__builtin_ctzll(m);
                s_start[k] = (uint16_t)(64u * tid + q + 1u);
                s_rank[k] = (uint16_t)((before & 0xFFFFu) + (uint32_t)__popcll(dm & ((1ull << q) - 1ull)));
            }
        } else {
            // places in the lists (those before it wrap around and are above any)
            uint32_t r = (before & 0xFFFFu) - d_lo, k = (before >> 16) - k_lo;
            const bool none = (int)r >= (int)kDelims || (int)(r + (mine & 0xFFFFu)) <= 0;
            for (uint64_t m = none ? 0ull : dm; m; m &= m - 1, ++r)
                if (r < kDelims) s_delim[r] = (uint16_t)(64u * tid + (uint32_t)__builtin_ctzll(m));
            for (uint64_t m = nm; m; m &= m - 1, ++k) {
                const uint32_t q = (uint32_t)__builtin_ctzll(m);
                if (k >= kLines) continue;
                s_start[k] = (uint16_t)(64u * tid + q + 1u);
                s_rank[k] = (uint16_t)((before & 0xFFFFu) + (uint32_t)__popcll(dm & ((1ull << q) - 1ull)));
            }
        }
        __syncthreads();
        const uint32_t lead = blk == 0 ? 1u : 0u, n_lines = s_own + lead;
        // line r0 of the block follows newline r0 - lead of the window, whose delimiter
        // rank is d0 - 1; its own newline is number nx, of rank dn (n_delim: none)
        auto rank_of = [&](uint32_t nx) { return nx < n_nl ? (uint32_t)s_rank[nx - k_lo] : n_delim; };
        uint32_t end = n_lines;  // the round's end: the first line that is not all listed
        if (more) {
            if (tid == 0) s_end = n_lines;
            __syncthreads();
            for (uint32_t r0 = line + tid; r0 < n_lines; r0 += kParseBlock) {
                const bool top = r0 < lead;
                const uint32_t i = r0 - lead, nx = top ? 0u : i + 1u;
                bool listed = (top || i - k_lo < kLines) && (nx >= n_nl || nx - k_lo < kLines);
                if (listed) {
                    const uint32_t d0 = top ? 0u : (uint32_t)s_rank[i - k_lo] + 1u;
                    const uint32_t last = min(min(d0 + 20u, rank_of(nx)), n_delim - 1u);
                    listed = d0 >= n_delim || (d0 >= d_lo && last - d_lo < kDelims);
                }
                if (!listed) {
                    atomicMin(&s_end, r0);
                    break;
                }
            }
            __syncthreads();
            end = s_end;
        }
        uint32_t ts = 0, src = 0, dst = 0;
        uint64_t nb = 0;
        bool ok = false;
        // line r0 into ts .. ok; false when there is none
        auto one = [&](uint32_t r0) -> bool {
            if (r0 >= end) return false;
            const uint32_t i = r0 - lead;
            const bool top = r0 < lead;
            const uint32_t s = top ? a.t.skew : (uint32_t)s_start[i - k_lo];
            if (b0 + s >= a.t.end) return false;  // nothing after the text's last newline
            const uint32_t d0 = top ? 0u : (uint32_t)s_rank[i - k_lo] + 1u;
            const uint32_t nx = top ? 0u : i + 1u, dn = rank_of(nx);
            if (d0 + 20u < n_delim || nx < n_nl || at_end) {
                // the line's delimiters are in the window, 21 or to its end
                ok = dn - d0 >= 20u;  // 20 commas before its newline
                if (ok) {
                    const uint16_t* dl = s_delim + (d0 - d_lo);
                    const uint32_t c1 = dl[0], c4 = dl[3], c5 = dl[4], c7 = dl[6], c8 = dl[7], c20 = dl[19];
                    const uint32_t c21 = d0 + 20u < n_delim ? (uint32_t)dl[20] : (uint32_t)(a.t.end - b0);
                    const Staged b{s_text};
                    ok = c1 - s == 23u && staged_time(b, s, a.origin, ts) &&
                         staged_ipv4(b, c4 + 1, c5, src) && staged_ipv4(b, c7 + 1, c8, dst) &&
                         staged_count(b, c20 + 1, c21, nb);
                }
            } else {  // the block's last line leaves the window: below
                s_far = s + 1u;
                return false;
            }
            return true;
        };
        uint32_t r0 = line + tid;
        if (first) {
            // the first kParseBlock lines are parsed while the last wave still finds
            // the block's line number
            place();
            const bool has = one(r0);
            __syncthreads();
            if (has) bad += put_line(a, s_base + 1u - lead + r0, ok, ts, src, dst, nb);
            r0 += kParseBlock;
        }
        for (; one(r0); r0 += kParseBlock) bad += put_line(a, s_base + 1u - lead + r0, ok, ts, src, dst, nb);
        if (end >= n_lines) break;
        // the next round starts with the line after (whose newline is listed: the line
        // before it was)
        line = end;
        const uint32_t k = end - lead, d = (uint32_t)s_rank[k - k_lo] + 1u;
        __syncthreads();  // the lists are written again
        k_lo = k;
        d_lo = d;
    }
    if (!at_end && n_nl == s_own) {  // no newline behind the block's own in the window
        __syncthreads();
        if (wave == 0 && s_far) {
            uint32_t ts = 0, src = 0, dst = 0;
            uint64_t nb = 0;
            const bool ok = line_far(a, b0 + s_far - 1u, lane, s_ends, reinterpret_cast<uint8_t*>(s_delim), ts, src, dst, nb);
            // (the block's last line)
            if (lane == 0) bad += put_line(a, s_base + s_own, ok, ts, src, dst, nb);
        }
    }
    // one counter for all blocks: a block adds its own once (by waves, text without
    // a good line was bound by it: 2e8 bytes of 40-byte lines 0.77 -> 0.25 ms)
    if (bad) atomicAdd(&s_bad, bad);
    __syncthreads();
    if (tid == 0 && s_bad) atomicAdd(a.bad, (unsigned long long)s_bad);
}

}  // namespace

sinet_status parse_sessions(const uint8_t* text, uint64_t len, int64_t origin, const sinet_columns* out,
                            uint64_t* n_lines, uint64_t* n_bad, hipStream_t s) {
    *n_lines = 0;
    *n_bad = 0;
    if (len == 0) return SINET_OK;
    const uint32_t skew = (uint32_t)((uintptr_t)text & 15u);
    const Text t{text - skew, skew, skew + len};
    const uint64_t n_blocks = (t.end + kOwn - 1) / kOwn;
    if (n_blocks >= (1ull << 31)) return fail(SINET_ERR_UNSUPPORTED, "text above 2^46 bytes");
    // block states, newlines, bad lines, ticket
    unsigned long long* ws = nullptr;
    sinet_status st = check_hip(hipMallocAsync((void**)&ws, 8 * (n_blocks + 3), s), "parse workspace");
    if (st != SINET_OK) return st;
    st = launch_zero(ws, n_blocks + 3, s);
    uint64_t out2[2] = {0, 0};
    uint8_t last = 0;
    if (st == SINET_OK) {
        const ParseArgs a{t, ws, ws + n_blocks, ws + n_blocks + 1, (uint32_t*)(ws + n_blocks + 2),
                          (uint32_t)n_blocks, out->n, origin,
                          const_cast<uint32_t*>(out->ts), const_cast<uint32_t*>(out->src),
                          const_cast<uint32_t*>(out->dst), const_cast<uint64_t*>(out->bytes)};
        hipLaunchKernelGGL(k_parse, dim3((unsigned)n_blocks), dim3(kParseBlock), 0, s, a);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = hipMemcpyAsync(out2, ws + n_blocks, 16, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipMemcpyAsync(&last, text + len - 1, 1, hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        st = check_hip(e, "parse");
    }
    (void)hipFreeAsync(ws, s);
    if (st != SINET_OK) return st;
    *n_lines = out2[0] + (last != 10 ? 1 : 0);
    if (*n_lines > out->n)
        return fail(SINET_ERR_INVALID_ARG, "output columns hold fewer sessions than the text has lines");
    *n_bad = out2[1];
    return SINET_OK;
}

}  // namespace sinet

extern "C" sinet_status sinet_parse_sessions(const uint8_t* text, uint64_t len, int32_t origin_days,
                                             sinet_columns* out, uint64_t* n_lines, uint64_t* n_bad,
                                             hipStream_t stream) {
    using namespace sinet;
    if (!out || !n_lines || !n_bad) return fail(SINET_ERR_INVALID_ARG, "NULL argument");
    if (len && !text) return fail(SINET_ERR_INVALID_ARG, "text is NULL");
    if (!out->ts || !out->src || !out->dst || !out->bytes)
        return fail(SINET_ERR_INVALID_ARG, "output column is NULL");
    return parse_sessions(text, len, origin_days, out, n_lines, n_bad, stream);
}
