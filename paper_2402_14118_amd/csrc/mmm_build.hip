// Map builder: evaluates the masks M and N on the device, writes the sparsity maps (paper, section 3
// "Preprocessing": a single sequential, aligned pass per matrix) and lays both operands out for the
// matrix kernel.  Everything here is integer work on bit patterns, bound by HBM bandwidth.
//
// A side (section 3 "Optimizations", Fig. "Blocked sparse row preprocessing"): the non-zero bitmap, its
// column-any summary, and an image of A: blocks of 64 rows x 128 columns with the masked-out elements
// replaced by zero, in exactly the byte order the matrix kernel keeps a block in LDS, so that the
// kernel's copy is one asynchronous load per 1 KiB and needs no registers, no conversion and no
// per-element work.  (Lists of {offset, value} per block, scattered with LDS atomics by every one of
// the N/256 workgroups that need the block, cost the kernel about 0.4 us per step of 128 k.)
// B side (section 3 "Block-Random Sparsity in B", Fig. "Preprocessing patterns"): one bit per block,
// 1 = some non-zero value; the same map transposed to one bit-row per block column; and B packed: for
// every group of 16 columns and segment of 128 k the occupied pieces of rows one after another, with
// the list of their k.  A wave of the matrix kernel owns one group and reads both linearly.
//
// One launch covers both matrices.  Every output word in device memory has exactly one producer, so no
// global atomics are used and nothing needs clearing beforehand.
#include "mmm_internal.h"
#include <cstring>
#include <type_traits>

namespace {

constexpr int BUILD_WAVES = 16;
constexpr int BUILD_THREADS = BUILD_WAVES * 64;
constexpr int SEG = MMM_AB_COLS;                      // rows of B (values of k) per workgroup = k per step of the matrix kernel
constexpr int B_ROWS = SEG / BUILD_WAVES;             // 8 rows per wave
constexpr int A_ROWS = MMM_AB_ROWS / BUILD_WAVES;     // 4 rows of A per wave

template <typename T> struct Tile {   // what a workgroup takes at a time, by element size
    static constexpr int ESZ = (int)sizeof(T);
    static constexpr int A_WORDS = ESZ == 8 ? 1 : 2;             // A: 64 rows x 64 A_WORDS columns
    static constexpr int LANE_COLS = ESZ == 8 ? 2 : 4;           // B: 128 rows x 64 LANE_COLS columns, so many per lane
    static constexpr int B_COLS = 64 * LANE_COLS;
    static constexpr int B_GROUPS = B_COLS / MMM_GROUP_COLS;
};

// Element predicate of M, decided on the bit pattern so that no denormal mode of the float pipeline can
// change a map bit.  Every predicate, the non-zero test included, is membership of the pattern (or of the
// pattern without its sign) in one or two ranges that the host works out (see element_test): two or three
// integer instructions per element, where comparing order-preserving keys took about ten and made the scan
// of X bound by the vector ALUs (2048 x 16384 ReLU: 276 of them per wave and block, 38 us).
enum { TEST_MAGNITUDE = 0, TEST_ONE_RANGE = 1, TEST_TWO_RANGES = 2 };
struct ElementTest {
    int32_t mode;
    uint64_t lo1, len1, lo2, len2;   // lo <= pattern < lo + len
};

struct BuildParams {
    const void *X;
    int64_t ldx;
    const uint64_t *keep_a;
    uint64_t *a_bits;
    uint64_t *a_colany;
    char *a_img;
    const void *Y;
    int64_t ldy;
    const uint64_t *keep_blocks;
    const uint64_t *keep_rows;   // doubles only
    uint64_t *b_bits;
    uint64_t *bt_bits;
    char *bp_val;         // packed B: [group][segment][128 slots][16 columns]
    uint16_t *bp_list;    // [group][segment][128]
    uint32_t *bp_cnt;     // [group][segment]
    int64_t M, K, N, NB, WA, WB, MT, MBA, KBA, NG;
    ElementTest test;
    int32_t pack;         // write packed B
    int32_t y_unaligned;  // 16-bit Y whose rows do not start on 4-byte boundaries
    uint32_t n_b;               // segments x column tiles of B
    uint32_t n_a_wg, n_b_wg;    // workgroups for them
    uint32_t a_per_wg;          // blocks of A per workgroup
    uint32_t ctiles;      // column tiles per segment of B
    int64_t a_units;      // blocks of A side by side
    // row-compacted mode (whole rows of B switched off): k' = 0 .. K' - 1 numbers the rows `rows` leaves on
    const uint64_t *rows;    // keep_rows, or the copy of it a cached B side was built with; else null
    uint64_t *rows_copy;     // where that copy goes (B side built in this call)
    uint32_t *kinfo;         // [0] = K'
    uint32_t *kmap;          // k' -> k
    uint64_t *btc_bits;      // transposed B map over k'
};

template <typename T> __device__ __forceinline__ uint32_t f32_bits(T v);
template <> __device__ __forceinline__ uint32_t f32_bits<float>(float v) { return __float_as_uint(v); }
template <> __device__ __forceinline__ uint32_t f32_bits<uint16_t>(uint16_t v) { return (uint32_t)v << 16; }   // bf16
template <> __device__ __forceinline__ uint32_t f32_bits<_Float16>(_Float16 v) { return __float_as_uint((float)v); }

// bit patterns of the 4- and 8-byte types
template <int ESZ> struct Pattern { typedef uint32_t type; static constexpr type magnitude = 0x7fffffffu; };
template <> struct Pattern<8> { typedef uint64_t type; static constexpr type magnitude = 0x7fffffffffffffffull; };

__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }

__device__ __forceinline__ uint32_t mbcnt64(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(v >> 32), l) << 32) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)v, l);
}

// Bits of two wave-uniform 32-bit masks interleaved: bit 2i = bit i of e, bit 2i + 1 = bit i of o.
__device__ __forceinline__ uint64_t interleave(uint32_t e, uint32_t o)
{
    uint64_t a, b;   // s_bitreplicate writes every bit twice
    asm("s_bitreplicate_b64_b32 %0, %1" : "=s"(a) : "s"(e));
    asm("s_bitreplicate_b64_b32 %0, %1" : "=s"(b) : "s"(o));
    return (a & 0x5555555555555555ull) | (b & 0xaaaaaaaaaaaaaaaaull);
}

// the first `left` (at least 1) bits of a word
__device__ __forceinline__ uint64_t bits_below(uint64_t m, int64_t left) { return left >= 64 ? m : m & ((1ull << left) - 1ull); }
// word w of a bitmap row of K bits with the bits past K cleared
__device__ __forceinline__ uint64_t row_word(const uint64_t *row, int64_t w, int64_t K) { return bits_below(row[w], K - w * 64); }

// ---- A side: one workgroup = a few blocks of 64 rows x 128 columns, one below the other ---------
// A wave takes the four rows that are neighbours in an LDS column: w, w+16, w+32, w+48 for 4- and 8-byte
// elements (one or two 16-byte reads of the matrix kernel yield one element for each of its four 16-row
// tiles), 4w .. 4w+3 for 16-bit ones (natural order: the transposing LDS read wants contiguous rows).
// Blocks of doubles are 64 columns wide.
// The block is turned around in LDS (16-byte or 8-byte pieces whose position is rotated with k, so that
// the 64 lanes of a write do not fall on the same banks) and leaves as whole cache lines.  The loads of
// the next block are issued before the barrier of the current one and two stages alternate, so that the
// memory system always has work of a workgroup although only two of this size fit on a compute unit.
struct AShared {
    char stage[2][MMM_AB_COLS * MMM_AB_ROWS * 4];
    uint64_t any[2][BUILD_WAVES][2][2];         // [stage][wave][32-row half of the block][word]
    uint8_t live[MMM_AB_COLS];                  // row-compacted mode: live columns of the blocks
    uint32_t before[BUILD_WAVES];               // row-compacted mode: live rows before them, by wave
};

template <typename T> struct ABlock {   // one block in a wave's registers
    typename Pattern<sizeof(T)>::type x[A_ROWS][sizeof(T) == 4 ? 2 : 1];   // lane <-> k; 16-bit: two neighbouring k per lane
    uint32_t kb[A_ROWS];   // 16-bit: the byte that holds the lane's keep bits
    uint64_t kw;           // otherwise: keep word of (row t, half h), in lane t * A_WORDS + h
};

template <typename T, int TEST, bool ROWS>
__device__ __forceinline__ void scan_a(const BuildParams &p, int64_t bj, int64_t bi0, int64_t bi1, int lane, int wave, AShared &sh)
{
    typedef typename Pattern<sizeof(T)>::type pattern;
    constexpr int ESZ = (int)sizeof(T);
    constexpr bool WIDE = ESZ >= 4;
    constexpr int A_WORDS = Tile<T>::A_WORDS, A_COLS = 64 * A_WORDS;
    constexpr int UNITS = MMM_AB_ROWS * ESZ / 16;   // 16-byte units per column
    const bool has_keep = p.keep_a != nullptr;
    constexpr bool compact = ROWS;
    auto row_of = [&](int64_t bi, int t) -> int64_t { return bi * MMM_AB_ROWS + (WIDE ? wave + 16 * t : wave * 4 + t); };

    // Every load below is unconditional (indices are clamped, results masked afterwards): a load inside a
    // branch is waited for before the next one is issued.
    // Addresses are a wave-uniform row base plus one 32-bit lane offset that all rows share.
    const int64_t k_lo = bj * A_COLS, w_lo = bj * A_WORDS;
    const int tail = (int)min(p.K - k_lo, (int64_t)A_COLS);   // columns of these blocks that exist
    auto load = [&](int64_t bi, ABlock<T> &r) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            r.kw = ~0ull;
            if (has_keep)
                r.kw = p.keep_a[min(row_of(bi, (lane / A_WORDS) & 3), p.M - 1) * p.WA + min(w_lo + lane % A_WORDS, p.WA - 1)];
            uint32_t off[A_WORDS];
#pragma unroll
            for (int h = 0; h < A_WORDS; ++h) off[h] = (uint32_t)min(lane + 64 * h, tail - 1) * (uint32_t)ESZ;
#pragma unroll
            for (int t = 0; t < A_ROWS; ++t) {
                const char *xr = reinterpret_cast<const char *>(static_cast<const T *>(p.X) + min(row_of(bi, t), p.M - 1) * p.ldx + k_lo);
#pragma unroll
                for (int h = 0; h < A_WORDS; ++h) r.x[t][h] = *reinterpret_cast<const pattern *>(xr + off[h]);
            }
        } else {
            // two neighbouring k per lane and load, at any 2-byte alignment; the last column of an odd K is read
            // together with the one before it, so that nothing past the row is touched
            typedef uint32_t u32_any __attribute__((aligned(2), may_alias));
            typedef uint16_t u16_any __attribute__((may_alias));
            const uint32_t off = (uint32_t)min(2 * lane + 2, tail) * 2u;   // from two elements before the block
            const uint32_t koff = (uint32_t)min(2 * lane, tail - 1) >> 3;
#pragma unroll
            for (int t = 0; t < A_ROWS; ++t) {
                const int64_t row = min(row_of(bi, t), p.M - 1);
                const char *xr = reinterpret_cast<const char *>(static_cast<const T *>(p.X) + row * p.ldx + k_lo);
                r.x[t][0] = p.K > 1 ? *reinterpret_cast<const u32_any *>(xr - 4 + off) : (uint32_t)*reinterpret_cast<const u16_any *>(xr);
                r.kb[t] = 0xffu;
                if (has_keep) r.kb[t] = (reinterpret_cast<const uint8_t *>(p.keep_a + row * p.WA + w_lo))[koff];
            }
        }
    };

    ABlock<T> cur;
    load(bi0, cur);
    uint32_t base = (uint32_t)k_lo;   // image column of the blocks' first
    int cols = A_COLS;                // and how many there are
    if (compact) {   // the blocks' live columns, and how many live rows come before them
        uint32_t n = 0;
        for (int64_t w = threadIdx.x; w < w_lo; w += BUILD_THREADS) n += (uint32_t)__popcll(p.rows[w]);
        const uint64_t m0 = row_word(p.rows, w_lo, p.K), m1 = w_lo + 1 < p.WA ? row_word(p.rows, w_lo + 1, p.K) : 0ull;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) n += (uint32_t)__shfl_xor((int)n, d, 64);
        if (lane == 0) sh.before[wave] = n;
        const uint32_t n0 = (uint32_t)__popcll(m0);
        cols = (int)(n0 + (uint32_t)__popcll(m1));
        if (wave == 0) {
            if ((m0 >> lane) & 1ull) sh.live[mbcnt64(m0)] = (uint8_t)lane;
            if ((m1 >> lane) & 1ull) sh.live[n0 + mbcnt64(m1)] = (uint8_t)(64 + lane);
        }
    }
    for (int64_t bi = bi0; bi < bi1; ++bi) {
        const int st = (int)(bi - bi0) & 1;
        char *const stage = sh.stage[st];
        uint64_t word[A_ROWS][A_WORDS];   // bitmap words (wave-uniform)
        // elements past the edge of X become +0, which is never kept
        const bool edge = tail < A_COLS || (bi + 1) * MMM_AB_ROWS > p.M;   // wave-uniform
        if constexpr (WIDE) {
            if (edge) {
#pragma unroll
                for (int t = 0; t < A_ROWS; ++t)
#pragma unroll
                    for (int h = 0; h < A_WORDS; ++h)
                        if (row_of(bi, t) >= p.M || 64 * h + lane >= tail) cur.x[t][h] = 0;
            }
            pattern u[A_ROWS][A_WORDS];
            const pattern lo1 = (pattern)p.test.lo1, len1 = (pattern)p.test.len1, lo2 = (pattern)p.test.lo2, len2 = (pattern)p.test.len2;
#pragma unroll
            for (int t = 0; t < A_ROWS; ++t)
#pragma unroll
                for (int h = 0; h < A_WORDS; ++h) {
                    const pattern x = cur.x[t][h], v = TEST == TEST_MAGNITUDE ? x & Pattern<ESZ>::magnitude : x;
                    uint64_t m = ballot64(v - lo1 < len1);
                    if (TEST == TEST_TWO_RANGES) m |= ballot64(v - lo2 < len2);
                    if (has_keep) m &= readlane64(cur.kw, t * A_WORDS + h);   // wave-uniform branch
                    word[t][h] = m;
                    u[t][h] = __builtin_amdgcn_inverse_ballot_w64(m) ? x : (pattern)0;   // the word is the lane mask of what stays
                }
#pragma unroll
            for (int h = 0; h < A_WORDS; ++h) {
                const int k = 64 * h + lane;
                char *at = stage + k * (UNITS * 16) + ((wave ^ (k & 15)) << 4);
                if constexpr (ESZ == 4) {
                    *reinterpret_cast<uint4 *>(at) = make_uint4(u[0][h], u[1][h], u[2][h], u[3][h]);
                } else {
                    *reinterpret_cast<ulong2 *>(at) = make_ulong2(u[0][h], u[1][h]);
                    *reinterpret_cast<ulong2 *>(at + 256) = make_ulong2(u[2][h], u[3][h]);
                }
            }
        } else {
            typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
            if (edge) {
#pragma unroll
                for (int t = 0; t < A_ROWS; ++t) {
                    if (2 * lane == tail - 1 && p.K > 1) cur.x[t][0] >>= 16;
                    if (row_of(bi, t) >= p.M || 2 * lane >= tail) cur.x[t][0] = 0;
                    if (2 * lane + 1 >= tail) cur.x[t][0] &= 0xffffu;
                }
            }
            uint32_t d[A_ROWS];
#pragma unroll
            for (int t = 0; t < A_ROWS; ++t) {
                d[t] = cur.x[t][0];
                if (has_keep) {   // wave-uniform branch; dropped elements become +0, which fails every test
                    const uint32_t kbit = cur.kb[t] >> ((2 * lane) & 7);
                    d[t] &= (uint32_t)((int)(kbit << 31) >> 31) & 0xffffu | (uint32_t)((int)(kbit << 30) >> 31) & 0xffff0000u;
                }
                const uint32_t v = TEST == TEST_MAGNITUDE ? d[t] & 0x7fff7fffu : d[t];
                const u16x2 lo1 = {(uint16_t)p.test.lo1, (uint16_t)p.test.lo1}, lo2 = {(uint16_t)p.test.lo2, (uint16_t)p.test.lo2};
                const u16x2 y = __builtin_bit_cast(u16x2, v) - lo1;
                uint64_t me = ballot64(y.x < (uint16_t)p.test.len1), mo = ballot64(y.y < (uint16_t)p.test.len1);
                if (TEST == TEST_TWO_RANGES) {
                    const u16x2 z = __builtin_bit_cast(u16x2, v) - lo2;
                    me |= ballot64(z.x < (uint16_t)p.test.len2);
                    mo |= ballot64(z.y < (uint16_t)p.test.len2);
                }
                word[t][0] = interleave((uint32_t)me, (uint32_t)mo);
                word[t][1] = interleave((uint32_t)(me >> 32), (uint32_t)(mo >> 32));
                d[t] &= (__builtin_amdgcn_inverse_ballot_w64(me) ? 0xffffu : 0u) | (__builtin_amdgcn_inverse_ballot_w64(mo) ? 0xffff0000u : 0u);
            }
            // rows 4w .. 4w+3 of columns 2 lane and 2 lane + 1
            char *at = stage + (2 * lane) * 128 + ((wave ^ ((lane & 7) << 1)) << 3);
            *reinterpret_cast<uint2 *>(at) = make_uint2(__builtin_amdgcn_perm(d[1], d[0], 0x05040100u), __builtin_amdgcn_perm(d[3], d[2], 0x05040100u));
            *reinterpret_cast<uint2 *>(at + 128) = make_uint2(__builtin_amdgcn_perm(d[1], d[0], 0x07060302u), __builtin_amdgcn_perm(d[3], d[2], 0x07060302u));
        }
        // bitmap words: lane t * A_WORDS + h stores the word of (row t, half h)
        uint64_t mine = 0;
#pragma unroll
        for (int t = 0; t < A_ROWS; ++t)
#pragma unroll
            for (int h = 0; h < A_WORDS; ++h) mine = __builtin_amdgcn_inverse_ballot_w64(1ull << (t * A_WORDS + h)) ? word[t][h] : mine;
        if (lane < 4) {   // column-any words of this wave's rows, by 32-row half of the block
            const int t32 = lane >> 1, h = lane & 1;
            constexpr int H = A_WORDS - 1;   // h = 1 with one word: repeats it, not read
            uint64_t any;
            if (WIDE)
                any = t32 ? (h ? word[2][H] | word[3][H] : word[2][0] | word[3][0]) : (h ? word[0][H] | word[1][H] : word[0][0] | word[1][0]);
            else
                any = t32 != wave / (BUILD_WAVES / 2) ? 0ull
                    : h ? word[0][H] | word[1][H] | word[2][H] | word[3][H] : word[0][0] | word[1][0] | word[2][0] | word[3][0];
            sh.any[st][wave][t32][h] = any;
        }
        if (bi + 1 < bi1) load(bi + 1, cur);
        if (lane < A_ROWS * A_WORDS && row_of(bi, lane / A_WORDS) < p.M && w_lo + lane % A_WORDS < p.WA)
            p.a_bits[row_of(bi, lane / A_WORDS) * p.WA + w_lo + lane % A_WORDS] = mine;
        __syncthreads();
        if (wave == 0) {   // lane (t32, h, wave): OR over the sixteen waves
            const int t32 = lane >> 5, h = (lane >> 4) & 1;
            const uint64_t any = sh.any[st][lane & 15][t32][h];
            uint32_t lo = (uint32_t)any, hi = (uint32_t)(any >> 32);
#pragma unroll
            for (int d = 1; d < 16; d <<= 1) {
                lo |= (uint32_t)__shfl_xor((int)lo, d, 64);
                hi |= (uint32_t)__shfl_xor((int)hi, d, 64);
            }
            const int64_t tile = bi * (MMM_AB_ROWS / MMM_COLANY_ROWS) + t32;
            if ((lane & 15) == 0 && tile < p.MT && h < A_WORDS && w_lo + h < p.WA) p.a_colany[tile * p.WA + w_lo + h] = ((uint64_t)hi << 32) | lo;
        }
        // the image: column k (or k') of block row bi is one run of 64 elements
        if (compact && bi == bi0) {
            base = 0;
            for (int w = 0; w < BUILD_WAVES; ++w) base += sh.before[w];
        }
        char *img = p.a_img + ((size_t)bi * p.KBA * MMM_AB_COLS + base) * (UNITS * 16);
        auto stage_of = [&](int k, int unit, uint32_t col) -> int {   // where unit `unit` of image column `col` waits in the stage
            // (16-bit: undo the rotation of the stage, apply that of the image, see mmm_img_swizzle)
            return WIDE ? k * (UNITS * 16) + ((unit ^ (k & 15)) << 4) : k * 128 + ((unit ^ (int)mmm_img_swizzle(col) ^ ((k >> 1) & 7)) << 4);
        };
        if (compact) {
            for (int q = threadIdx.x; q < cols * UNITS; q += BUILD_THREADS) {
                const int j = q / UNITS, k = (int)sh.live[j];
                *reinterpret_cast<uint4 *>(img + (uint32_t)q * 16u) = *reinterpret_cast<const uint4 *>(stage + stage_of(k, q % UNITS, base + j));
            }
        } else {   // two (16-bit: one) units per thread
            const int j = threadIdx.x / UNITS;
            const int at = stage_of(j, threadIdx.x % UNITS, (uint32_t)j);
#pragma unroll
            for (int i = 0; i < A_COLS * UNITS / BUILD_THREADS; ++i)
                *reinterpret_cast<uint4 *>(img + (threadIdx.x * 16u + (uint32_t)(i * BUILD_THREADS * 16))) =
                    *reinterpret_cast<const uint4 *>(stage + at + i * (BUILD_THREADS * 16));
        }
    }
}

// ---- B side: one workgroup = 128 rows (values of k) x 256 columns (doubles: twice 128) --------
// A wave takes 8 rows; a lane owns four (two) neighbouring columns of each, so that 4 (8) lanes are one
// 16-column group.  The 8 loads of a lane are in flight together; blocks the keep bitmaps switch off are given an
// offset past the buffer's end, for which the hardware returns zero without touching memory.  The 128
// occupancy bits of every lane's block are gathered in LDS, one byte per wave; from them follow the map
// words, the transposed map words and the rank of every row within its group's segment, which is its
// slot in the packed operand.
struct BShared {
    uint8_t gbits[64][BUILD_WAVES];   // [lane][wave]: rows in which the lane's 16-column group is occupied
    uint8_t bbits[64][BUILD_WAVES];   // the same for the lane's block, where that is another set (8-wide blocks)
    uint16_t list[16][SEG];
    char pack[16 * (SEG * MMM_GROUP_COLS * 2 + 16)];   // 16-bit types: the packed groups
    int32_t kk[SEG];                  // row-compacted mode: the rows behind the segment's k' (-1: none)
    uint32_t sums[BUILD_WAVES];
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Rows k' = seg*128 .. of the numbering given by `rows`, into sh.kk; returns K'.
__device__ __forceinline__ uint32_t number_rows(const BuildParams &p, int64_t seg, int lane, int wave, BShared &sh)
{
    const int tid = threadIdx.x;
    if (tid < SEG) sh.kk[tid] = -1;
    const int64_t per = (p.WA + BUILD_THREADS - 1) / BUILD_THREADS;   // every thread counts a run of words
    const int64_t w0 = tid * per, w1 = min(p.WA, w0 + per);
    uint32_t cnt = 0;
    for (int64_t w = w0; w < w1; ++w) cnt += (uint32_t)__popcll(row_word(p.rows, w, p.K));
    uint32_t incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)incl, d, 64);
        if (lane >= d) incl += o;
    }
    if (lane == 63) sh.sums[wave] = incl;
    __syncthreads();
    uint32_t pos = incl - cnt, total = 0;
#pragma unroll
    for (int w = 0; w < BUILD_WAVES; ++w) {
        const uint32_t s = sh.sums[w];
        if (w < wave) pos += s;
        total += s;
    }
    const uint32_t lo = (uint32_t)seg * SEG;
    if (pos < lo + SEG && pos + cnt > lo) {
        for (int64_t w = w0; w < w1; ++w)
            for (uint64_t m = row_word(p.rows, w, p.K); m != 0; m &= m - 1, ++pos)
                if (pos >= lo && pos < lo + SEG) sh.kk[pos - lo] = (int32_t)(w * 64 + __builtin_ctzll(m));
    }
    __syncthreads();
    return total;
}

// bits of x at multiples of LPB, moved together
template <int LPB> __device__ __forceinline__ uint32_t squeeze(uint64_t x)
{
    if (LPB == 2) {
        x &= 0x5555555555555555ull;
        x = (x | x >> 1) & 0x3333333333333333ull;
        x = (x | x >> 2) & 0x0f0f0f0f0f0f0f0full;
        x = (x | x >> 4) & 0x00ff00ff00ff00ffull;
        x = (x | x >> 8) & 0x0000ffff0000ffffull;
        return (uint32_t)(x | x >> 16);
    }
    if (LPB == 4) {
        x &= 0x1111111111111111ull;
        x = (x | x >> 3) & 0x0303030303030303ull;
        x = (x | x >> 6) & 0x000f000f000f000full;
        x = (x | x >> 12) & 0x000000ff000000ffull;
        return (uint32_t)((x | x >> 24) & 0xffffull);
    }
    if (LPB == 8) return (uint32_t)(((x & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56);
    return (uint32_t)((x & 1u) | (x >> 15 & 2u) | (x >> 30 & 4u) | (x >> 45 & 8u));   // 16
}

// ROWS (row-compacted mode): the rows are the live rows k' = 128 seg .., and the transposed map is over k'.
// Returns false where ROWS finds no live row in the segment.  carry: doubles in 32-wide blocks fill half a
// byte of a map row per column tile, so the map bits of an even tile are handed to the odd one after it.
template <typename T, int BW, bool ROWS>
__device__ __forceinline__ bool scan_b(const BuildParams &p, int64_t seg, int64_t ct, int lane, int wave, BShared &sh, uint32_t &carry)
{
    constexpr int ESZ = (int)sizeof(T);
    constexpr int LANE_COLS = Tile<T>::LANE_COLS, B_COLS = Tile<T>::B_COLS, B_GROUPS = Tile<T>::B_GROUPS;
    constexpr int LPB = BW / LANE_COLS;               // lanes per block
    constexpr int LPG = MMM_GROUP_COLS / LANE_COLS;   // lanes per group
    constexpr int BPW = B_COLS / BW;                  // blocks per column tile
    constexpr bool WIDE = ESZ >= 4;
    constexpr bool SPLIT = BW < MMM_GROUP_COLS;       // a group holds two blocks
    constexpr uint64_t REP = LPB == 2 ? 0x5555555555555555ull : LPB == 4 ? 0x1111111111111111ull : LPB == 8 ? 0x0101010101010101ull : 0x0001000100010001ull;
    constexpr uint64_t GREP = LPG == 4 ? 0x1111111111111111ull : 0x0101010101010101ull;
    const int64_t col0 = ct * B_COLS, blk0 = ct * BPW;
    if (ROWS) {
        const uint32_t live = number_rows(p, seg, lane, wave, sh);
        if (ct == 0) {   // publish the numbering
            if (threadIdx.x < SEG && sh.kk[threadIdx.x] >= 0) p.kmap[seg * SEG + threadIdx.x] = (uint32_t)sh.kk[threadIdx.x];
            if (seg == 0) {
                if (threadIdx.x == 0) p.kinfo[0] = live;
                for (int64_t w = threadIdx.x; w < p.WA; w += BUILD_THREADS) p.rows_copy[w] = row_word(p.rows, w, p.K);
            }
        }
        if (seg * SEG >= (int64_t)live) return false;   // the whole workgroup
    }
    // lane j < 8: row j of the wave and which of its blocks are switched on
    int64_t krow = -1;
    uint32_t piece = 0;
    {
        const int j = lane & (B_ROWS - 1);
        const int64_t k = ROWS ? (int64_t)sh.kk[wave * B_ROWS + j] : seg * SEG + wave * B_ROWS + j;
        krow = k >= 0 && k < p.K ? k : -1;
        const int64_t kc = max(krow, (int64_t)0);
        uint64_t w = ~0ull;
        if (p.keep_blocks != nullptr) w = p.keep_blocks[kc * p.WB + (blk0 >> 6)];   // wave-uniform branches
        if (ESZ == 8 && p.keep_rows != nullptr && !((p.keep_rows[kc >> 6] >> (kc & 63)) & 1ull)) w = 0;   // (not numbered)
        piece = krow >= 0 ? (uint32_t)(w >> (blk0 & 63)) : 0u;
    }
    u32x4 raw[B_ROWS];
    const uint32_t nrec = (uint32_t)min((int64_t)B_COLS, p.N - col0) * ESZ;
#pragma unroll
    for (int j = 0; j < B_ROWS; ++j) {
        const int64_t k = max((int64_t)readlane64((uint64_t)krow, j), (int64_t)0);
        const uint32_t pj = (uint32_t)__builtin_amdgcn_readlane((int)piece, j);
        const char *row = static_cast<const char *>(p.Y) + (k * p.ldy + col0) * ESZ;
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(row), 0, (int)nrec, 0x00020000);
        const int off = (pj >> (lane / LPB)) & 1u ? lane * (LANE_COLS * ESZ) : 0x40000000;
        if constexpr (WIDE) {
            raw[j] = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        } else if (!p.y_unaligned) {
            const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
            raw[j] = u32x4{v.x, v.y, 0, 0};
        } else {
            uint32_t e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) e[i] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off + 2 * i, 0, 0);
            raw[j] = u32x4{e[0] | e[1] << 16, e[2] | e[3] << 16, 0, 0};
        }
    }
    uint32_t gb = 0, bbm = 0;   // rows (bit j) in which this lane's group / block is occupied
    uint64_t mine = 0;          // lane j: the occupied blocks of row j, at multiples of LPB
#pragma unroll
    for (int j = 0; j < B_ROWS; ++j) {
        const uint32_t nz = ESZ == 8   ? raw[j].x | raw[j].z | ((raw[j].y | raw[j].w) & 0x7fffffffu)
                          : ESZ == 4 ? (raw[j].x | raw[j].y | raw[j].z | raw[j].w) & 0x7fffffffu
                                     : (raw[j].x | raw[j].y) & 0x7fff7fffu;
        uint64_t m = ballot64(nz != 0);
        m |= m >> 1;
        if (LPB >= 4) m |= m >> 2;
        if (LPB >= 8) m |= m >> 4;
        if (LPB >= 16) m |= m >> 8;
        m &= REP;
        const uint64_t blocks = m * ((1u << LPB) - 1u);   // spread over the block's lanes
        uint64_t groups = blocks;
        if (SPLIT) groups = ((m | m >> LPB) & GREP) * ((1u << LPG) - 1u);
        gb |= __builtin_amdgcn_inverse_ballot_w64(groups) ? 1u << j : 0u;
        if (SPLIT) bbm |= __builtin_amdgcn_inverse_ballot_w64(blocks) ? 1u << j : 0u;
        mine = __builtin_amdgcn_inverse_ballot_w64(1ull << j) ? m : mine;
    }
    sh.gbits[lane][wave] = (uint8_t)gb;
    if (SPLIT) sh.bbits[lane][wave] = (uint8_t)bbm;
    if (lane < B_ROWS && krow >= 0) {   // this tile's piece of the map row: 4, 2, 1 or half a byte
        uint32_t v = squeeze<LPB>(mine);
        char *dst = reinterpret_cast<char *>(p.b_bits + krow * p.WB) + blk0 / 8;
        if (BPW == 32)
            *reinterpret_cast<uint32_t *>(dst) = v;
        else if (BPW == 16)
            *reinterpret_cast<uint16_t *>(dst) = (uint16_t)v;
        else if (BPW == 8)
            *reinterpret_cast<uint8_t *>(dst) = (uint8_t)v;
        else {
            if (ct & 1) v = v << 4 | carry;
            carry = v;
            if ((ct & 1) != 0 || ct == p.ctiles - 1) *reinterpret_cast<uint8_t *>(dst) = (uint8_t)v;
        }
        if (ct == p.ctiles - 1)   // pad bits of the row
            for (int64_t q = (blk0 + BPW + 7) / 8; q < p.WB * 8; ++q) reinterpret_cast<uint8_t *>(p.b_bits + krow * p.WB)[q] = 0;
    }
    constexpr int RING = mmm_ring(sizeof(T));
    constexpr uint32_t ZERO_ENTRY = mmm_list_entry(sizeof(T), mmm_zero_col(RING));
    static_assert(B_GROUPS * SEG * 2 <= BUILD_THREADS * 4, "at most one list word per thread");
    if (threadIdx.x < B_GROUPS * SEG / 2) reinterpret_cast<uint32_t *>(sh.list)[threadIdx.x] = ZERO_ENTRY | ZERO_ENTRY << 16;
    __syncthreads();
    if (wave == 0 && (lane % LPB) == 0) {   // transposed map words of this lane's block
        const uint64_t *t = reinterpret_cast<const uint64_t *>(SPLIT ? sh.bbits[lane] : sh.gbits[lane]);
        const int64_t blk = blk0 + lane / LPB;
        if (blk < p.NB) {
            uint64_t *dst = (ROWS ? p.btc_bits : p.bt_bits) + blk * p.WA + seg * 2;
            dst[0] = t[0];
            if (seg * 2 + 1 < p.WA) dst[1] = t[1];
        }
    }
    if (ESZ == 8 && !p.pack) return true;
    const uint64_t *gt = reinterpret_cast<const uint64_t *>(sh.gbits[lane]);
    const uint64_t glo = gt[0], ghi = gt[1];
    const uint32_t n = (uint32_t)__popcll(glo) + (uint32_t)__popcll(ghi);   // rows of this lane's group
    const uint64_t below = (1ull << (8 * (wave & 7))) - 1ull;
    const uint32_t slot0 = wave < 8 ? (uint32_t)__popcll(glo & below) : (uint32_t)__popcll(glo) + (uint32_t)__popcll(ghi & below);
    const int64_t G = ct * B_GROUPS + lane / LPG;   // this lane's group
    const bool group_ok = G < p.NG;
    uint32_t slots[B_ROWS];
    {
        uint32_t s = slot0;
#pragma unroll
        for (int j = 0; j < B_ROWS; ++j) {
            slots[j] = s;
            s += (gb >> j) & 1u;
        }
    }
    if (lane % LPG == 0) {
#pragma unroll
        for (int j = 0; j < B_ROWS; ++j)
            if ((gb >> j) & 1u)
                sh.list[lane / LPG][mmm_list_pos(sizeof(T), slots[j])] =
                    (uint16_t)mmm_list_entry(sizeof(T), ((uint32_t)seg & (RING - 1u)) * SEG + (uint32_t)(wave * B_ROWS + j));
        if (wave == 0 && group_ok) p.bp_cnt[G * p.KBA + seg] = n;
    }
    char *val = p.bp_val + (size_t)(G * p.KBA + seg) * (SEG * MMM_GROUP_COLS * ESZ);   // this lane's group
    if constexpr (WIDE) {
        // slot-major rows of 64 or 128 bytes; the slots that fill up the last quad are zero
        constexpr int ROWB = MMM_GROUP_COLS * ESZ;
        if (group_ok) {
#pragma unroll
            for (int j = 0; j < B_ROWS; ++j)
                if ((gb >> j) & 1u) *reinterpret_cast<u32x4 *>(val + slots[j] * ROWB + (lane % LPG) * 16) = raw[j];
            if (wave < 3 && n + wave < ((n + 3u) & ~3u)) *reinterpret_cast<u32x4 *>(val + (n + wave) * ROWB + (lane % LPG) * 16) = u32x4{0, 0, 0, 0};
        }
        __syncthreads();
    } else {
        // Composed in LDS in the order of mmm_value_pos; the slots that fill up the last batch are zero.  Whole batches are
        // copied out, 1 KiB each.
        constexpr int GROUPB = SEG * MMM_GROUP_COLS * ESZ + 16;   // bytes per group (4 banks apart)
        constexpr uint32_t SLOTS = 32;                            // per batch
        static_assert(B_GROUPS * GROUPB <= (int)sizeof(sh.pack), "room for the groups");
        uint16_t *g = reinterpret_cast<uint16_t *>(sh.pack + (lane / LPG) * GROUPB);
        auto put = [&](uint32_t slot, const u32x4 &v) {
            uint16_t *at = g + mmm_value_pos(ESZ, slot, (uint32_t)(lane & 3) * 4u);
            at[0] = (uint16_t)v.x;
            at[8] = (uint16_t)(v.x >> 16);
            at[16] = (uint16_t)v.y;
            at[24] = (uint16_t)(v.y >> 16);
        };
#pragma unroll
        for (int j = 0; j < B_ROWS; ++j)
            if ((gb >> j) & 1u) put(slots[j], raw[j]);
#pragma unroll
        for (uint32_t i = 0; i < SLOTS; i += BUILD_WAVES)
            if (n + i + wave < ((n + SLOTS - 1) & ~(SLOTS - 1))) put(n + i + wave, u32x4{0, 0, 0, 0});
        __syncthreads();
        constexpr int TPG = BUILD_THREADS / B_GROUPS;   // threads per group
        const int cg = threadIdx.x / TPG;
        const int64_t CG = ct * B_GROUPS + cg;
        if (CG < p.NG) {
            const uint64_t *bits = reinterpret_cast<const uint64_t *>(sh.gbits[cg * LPG]);
            const uint32_t batches = ((uint32_t)(__popcll(bits[0]) + __popcll(bits[1])) + SLOTS - 1u) / SLOTS;
            char *cval = p.bp_val + (size_t)(CG * p.KBA + seg) * (SEG * MMM_GROUP_COLS * ESZ);
            for (uint32_t q = threadIdx.x % TPG; q < batches * 64; q += TPG)
                *reinterpret_cast<uint4 *>(cval + q * 16) = *reinterpret_cast<const uint4 *>(sh.pack + cg * GROUPB + q * 16);
        }
    }
    {   // the lists, one word per thread
        const int64_t LG = ct * B_GROUPS + (threadIdx.x >> 6);
        if ((int)(threadIdx.x >> 6) < B_GROUPS && LG < p.NG)
            reinterpret_cast<uint32_t *>(p.bp_list + (LG * p.KBA + seg) * SEG)[lane] = reinterpret_cast<const uint32_t *>(sh.list)[threadIdx.x];
    }
    if (ROWS) __syncthreads();   // the shared arrays may be reused
    return true;
}

// ROWS: row-compacted mode (A laid out over the live rows of B; B built over them).
template <typename T, int TEST, int BW, bool ROWS>
__global__ __launch_bounds__(BUILD_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) void mmm_build_kernel(const BuildParams p)
{
    __shared__ __align__(16) union { AShared a; BShared b; } sh;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t b = blockIdx.x;
    // Workgroups of B come first: they are bound by latency (keep bits, then scattered rows), and what is left of them
    // when the first finish runs beside the streaming of A.  (Alternating them with those of A, or putting them last,
    // measured the same or slower: 36.8 and 35.6 against 35.3 us for both sides of 4096^2 at p = .05.)
    const bool is_b = b < p.n_b_wg;
    const uint32_t i = is_b ? b : b - p.n_b_wg;
    if (is_b) {
        uint32_t carry = 0;
        if (ROWS) {
            for (int64_t w = i; w < p.WA; w += p.n_b_wg) {   // zero map rows for the rows that are off
                const uint64_t live = row_word(p.rows, w, p.K);
                const uint32_t words = (uint32_t)(min((int64_t)64, p.K - w * 64) * p.WB);
                for (uint32_t q = threadIdx.x; q < words; q += BUILD_THREADS)
                    if (!((live >> (q / (uint32_t)p.WB)) & 1ull)) p.b_bits[w * 64 * p.WB + q] = 0;
            }
            for (uint32_t bb = i; bb < p.n_b; bb += p.n_b_wg) {   // ends at the first segment without a live row
                int l = lane;
                asm volatile("" : "+v"(l));   // keeps what depends on the lane from being carried around the loop (it would spill)
                if (!scan_b<T, BW, true>(p, bb / p.ctiles, bb % p.ctiles, l, wave, sh.b, carry)) break;
            }
        } else if (sizeof(T) < 8) {
            scan_b<T, BW, false>(p, i / p.ctiles, i % p.ctiles, lane, wave, sh.b, carry);
        } else {   // two column tiles
            const uint32_t pairs = (p.ctiles + 1) / 2;
            const int64_t seg = i / pairs, ct = (int64_t)(i % pairs) * 2;
            scan_b<T, BW, false>(p, seg, ct, lane, wave, sh.b, carry);
            if (ct + 1 < p.ctiles) {
                __syncthreads();
                int l = lane;
                asm volatile("" : "+v"(l));
                scan_b<T, BW, false>(p, seg, ct + 1, l, wave, sh.b, carry);
            }
        }
    } else {
        const int64_t bi0 = (int64_t)(i / (uint32_t)p.a_units) * p.a_per_wg;
        scan_a<T, TEST, ROWS>(p, i % (uint32_t)p.a_units, bi0, min(bi0 + p.a_per_wg, p.MBA), lane, wave, sh.a);
    }
}

// Row-compacted mode: bt_bits (over k) by spreading the bits of btc_bits to the places rows_copy names.  One wave per
// word of 64 k.
__global__ __launch_bounds__(256) void mmm_expand_rows_kernel(const uint64_t *rows, const uint64_t *btc_bits, uint64_t *bt_bits,
                                                              int64_t K, int64_t NB, int64_t WA)
{
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= WA) return;
    uint32_t before = 0;
    for (int64_t q = lane; q < w; q += 64) before += (uint32_t)__popcll(rows[q]);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) before += (uint32_t)__shfl_xor((int)before, d, 64);
    const uint64_t live = readlane64(rows[w], 0);
    const int64_t at = (int64_t)(before >> 6);
    const int sh = (int)(before & 63u);
    for (int64_t blk = lane; blk < NB; blk += 64) {
        uint64_t bits = btc_bits[blk * WA + min(at, WA - 1)] >> sh;
        if (sh != 0) bits |= btc_bits[blk * WA + min(at + 1, WA - 1)] << (64 - sh);
        uint64_t out = 0;
        for (uint64_t m = live; m != 0; m &= m - 1) {   // wave-uniform
            out |= (bits & 1ull) << __builtin_ctzll(m);
            bits >>= 1;
        }
        bt_bits[blk * WA + w] = out;
    }
}

// ---- forms that only inspection reads, made when they are asked for ---------------------------
// Column-any words of A over k': bit k' of a row is bit kmap[k'] of the row over k.
__global__ __launch_bounds__(256) void mmm_colany_compact_kernel(const uint64_t *a_colany, const uint32_t *kinfo, const uint32_t *kmap,
                                                                 uint64_t *a_colany_c, int64_t MT, int64_t WA)
{
    const int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // one wave per word
    if (idx >= MT * WA) return;
    const int64_t t = idx / WA, w = idx % WA, kc = w * 64 + (threadIdx.x & 63);
    bool any = false;
    if (kc < (int64_t)*kinfo) {
        const uint32_t k = kmap[kc];
        any = (a_colany[t * WA + (k >> 6)] >> (k & 63)) & 1ull;
    }
    const uint64_t m = ballot64(any);
    if ((threadIdx.x & 63) == 0) a_colany_c[idx] = m;
}

// Counts and lists of the non-zero elements of every block of A, from its image: one workgroup per
// block, a thread per column.  The order is by column, then by place in the column.
template <typename T>
__global__ __launch_bounds__(MMM_AB_COLS) void mmm_lists_kernel(const char *a_img, const uint64_t *a_bits, const uint32_t *kinfo,
                                                                const uint32_t *kmap, uint32_t *a_cnt, uint2 *a_ent, int64_t M,
                                                                int64_t K, int64_t WA, int64_t KBA)
{
    __shared__ uint32_t off[MMM_AB_COLS];
    const int64_t b = blockIdx.x, bi = b / KBA, bj = b % KBA;
    const int c = threadIdx.x;
    const int64_t kc = bj * MMM_AB_COLS + c, klim = kinfo ? (int64_t)*kinfo : K;
    if (kinfo && bj * MMM_AB_COLS >= klim) return;
    const int64_t k = kc < klim ? (kinfo ? (int64_t)kmap[kc] : kc) : -1;
    uint64_t rows = 0;
    if (k >= 0)
        for (int r = 0; r < MMM_AB_ROWS; ++r) {
            const int64_t row = bi * MMM_AB_ROWS + r;
            if (row < M && ((a_bits[row * WA + (k >> 6)] >> (k & 63)) & 1ull)) rows |= 1ull << r;
        }
    off[c] = (uint32_t)__popcll(rows);
    __syncthreads();
    uint32_t at = 0, total = 0;
    for (int q = 0; q < MMM_AB_COLS; ++q) {
        if (q < c) at += off[q];
        total += off[q];
    }
    uint2 *ent = a_ent + (size_t)b * MMM_AB_CAP;
    const char *col = a_img + ((size_t)bi * KBA * MMM_AB_COLS + kc) * (MMM_AB_ROWS * sizeof(T));
    for (uint64_t m = rows; m != 0; m &= m - 1) {
        const int r = __builtin_ctzll(m);
        const T v = *reinterpret_cast<const T *>(col + mmm_img_row(sizeof(T), (uint32_t)kc, (uint32_t)r));
        ent[at++] = make_uint2(mmm_slab_pos((uint32_t)r, (uint32_t)c), f32_bits<T>(v));
    }
    if (c == 0) a_cnt[b] = total;
    if (total + c < ((total + 63u) & ~63u)) ent[total + c] = make_uint2(MMM_SLAB_SPARE, 0u);
}

// ---- statistics (off the hot path) -----------------------------------------------------------
__global__ void mmm_stats_clear_kernel(uint64_t *stats)
{
    if (threadIdx.x < 4) stats[threadIdx.x] = 0;
}

// One workgroup per 64 values of k: lane kb of every wave counts column k of A
// over a slice of rows and row k of B over its words.
__global__ __launch_bounds__(256) void mmm_stats_kernel(const uint64_t *a_bits, const uint64_t *b_bits,
                                                        int64_t M, int64_t K, int64_t WA, int64_t WB,
                                                        int64_t bw, uint64_t *stats)
{
    __shared__ uint32_t col[4 * 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t w = blockIdx.x;
    uint32_t cnt = 0;
    for (int64_t r = wave; r < M; r += 4) cnt += (uint32_t)((a_bits[r * WA + w] >> lane) & 1ull);
    col[wave * 64 + lane] = cnt;
    __syncthreads();
    if (wave == 0) {
        const uint64_t colcount = (uint64_t)col[lane] + col[64 + lane] + col[128 + lane] + col[192 + lane];
        const int64_t k = w * 64 + lane;
        uint64_t rowcount = 0;
        if (k < K)
            for (int64_t j = 0; j < WB; ++j) rowcount += (uint64_t)__popcll(b_bits[k * WB + j]);
        uint64_t v[4] = {colcount, rowcount, colcount * rowcount * (uint64_t)bw, rowcount != 0 ? 1u : 0u};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint64_t x = v[q];
            for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
            if (lane == 0 && x != 0) atomicAdd((unsigned long long *)&stats[q], (unsigned long long)x);
        }
    }
}

}   // namespace

// The ranges of bit patterns a predicate accepts.  `value` maps a magnitude pattern 0 .. inf of the element type to its
// value, rising with the pattern.
template <typename F> static ElementTest element_test(int32_t pred, float threshold, uint64_t inf, uint64_t sign, F value)
{
    auto first = [&](auto &&is) -> uint64_t {   // smallest magnitude pattern for which `is` holds, inf + 1 if none
        uint64_t lo = 0, hi = inf + 1;
        while (lo < hi) {
            const uint64_t mid = lo + (hi - lo) / 2;
            if (is(value(mid)))
                hi = mid;
            else
                lo = mid + 1;
        }
        return lo;
    };
    const double t = (double)threshold;
    ElementTest e{TEST_MAGNITUDE, 1, sign - 1, 0, 0};   // non-zero, NaN included
    if (pred == MMM_PRED_NONZERO) return e;
    e.mode = pred == MMM_PRED_GT ? TEST_ONE_RANGE : TEST_MAGNITUDE;
    e.len1 = 0;
    if (t != t) return e;   // NaN threshold: nothing passes
    if (t >= 0.0) {         // -0 included
        e.lo1 = first([&](double v) { return v > t; });
        e.len1 = inf + 1 - e.lo1;
    } else {                // every non-negative number; of the negative ones those smaller in magnitude
        e.lo1 = 1;
        e.len1 = inf;
        if (pred == MMM_PRED_GT) {
            e.mode = TEST_TWO_RANGES;
            e.lo2 = sign + 1;
            e.len2 = first([&](double v) { return v >= -t; }) - 1;
        }
    }
    return e;
}

static ElementTest element_test(int32_t dtype, int32_t pred, float threshold)
{
    auto single = [](uint64_t v) {
        const uint32_t u = (uint32_t)v;
        float f;
        std::memcpy(&f, &u, 4);
        return (double)f;
    };
    if (dtype == MMM_BF16) return element_test(pred, threshold, 0x7f80u, 0x8000u, [&](uint64_t v) { return single(v << 16); });
    if (dtype == MMM_F16)
        return element_test(pred, threshold, 0x7c00u, 0x8000u, [](uint64_t v) { return (double)__builtin_bit_cast(_Float16, (uint16_t)v); });
    if (dtype == MMM_F64)
        return element_test(pred, threshold, 0x7ff0000000000000ull, 0x8000000000000000ull, [](uint64_t v) {
            double d;
            std::memcpy(&d, &v, 8);
            return d;
        });
    return element_test(pred, threshold, 0x7f800000u, 0x80000000u, single);
}

typedef void (*build_kernel_fn)(const BuildParams);

template <typename T, int TEST, bool ROWS> static build_kernel_fn build_kernel_width(int32_t bw)
{
    return bw == 8 ? mmm_build_kernel<T, TEST, 8, ROWS> : bw == 16 ? mmm_build_kernel<T, TEST, 16, ROWS> : mmm_build_kernel<T, TEST, 32, ROWS>;
}
template <typename T, bool ROWS> static build_kernel_fn build_kernel_test(int32_t mode, int32_t bw)
{
    return mode == TEST_MAGNITUDE ? build_kernel_width<T, TEST_MAGNITUDE, ROWS>(bw)
         : mode == TEST_ONE_RANGE ? build_kernel_width<T, TEST_ONE_RANGE, ROWS>(bw)
                                  : build_kernel_width<T, TEST_TWO_RANGES, ROWS>(bw);
}
template <typename T> static build_kernel_fn build_kernel_rows(int32_t mode, int32_t bw, bool rows)
{
    return rows ? build_kernel_test<T, true>(mode, bw) : build_kernel_test<T, false>(mode, bw);
}
static build_kernel_fn build_kernel(int32_t dtype, int32_t mode, int32_t bw, bool rows)
{
    return dtype == MMM_F64  ? build_kernel_test<double, false>(mode, bw)   // no row-compacted mode
         : dtype == MMM_BF16 ? build_kernel_rows<uint16_t>(mode, bw, rows)
         : dtype == MMM_F16  ? build_kernel_rows<_Float16>(mode, bw, rows)
                             : build_kernel_rows<float>(mode, bw, rows);
}

hipError_t mmm_launch_build(const mmm_maps *m, const mmm_build_args &a, hipStream_t s)
{
    BuildParams p{};
    p.X = a.X;
    p.ldx = a.ldx;
    p.keep_a = a.keep_a;
    p.a_bits = m->a_bits;
    p.a_colany = m->a_colany;
    p.a_img = a.dtype == MMM_F64 ? m->a_img64 : m->a_img;
    p.Y = a.Y;
    p.ldy = a.ldy;
    p.keep_blocks = a.keep_blocks;
    p.keep_rows = a.keep_rows;
    p.b_bits = m->b_bits;
    p.bt_bits = m->bt_bits;
    p.bp_val = m->bp_val;
    p.bp_list = m->bp_list;
    p.bp_cnt = m->bp_cnt;
    p.M = m->M;
    p.K = m->K;
    p.N = m->N;
    p.NB = m->NB;
    p.WA = m->WA;
    p.WB = m->WB;
    p.MT = m->MT;
    p.MBA = m->MBA;
    p.KBA = m->KBA;
    p.NG = m->NG;
    p.pack = mmm_packs(m->M, a.dtype) ? 1 : 0;
    p.test = element_test(a.dtype, a.pred, a.threshold);
    p.y_unaligned = a.dtype != MMM_F32 && a.dtype != MMM_F64 && ((reinterpret_cast<uintptr_t>(a.Y) & 3u) != 0 || (a.ldy & 1) != 0);
    p.kinfo = m->kinfo;
    p.kmap = m->kmap;
    p.btc_bits = m->btc_bits;
    p.rows_copy = m->rows_copy;
    // the numbering the A side follows: that of the B side built in this call, or of the cached one
    p.rows = a.b_compact ? a.keep_rows : a.a_compact ? m->rows_copy : nullptr;
    const bool f64 = a.dtype == MMM_F64;
    const int64_t b_cols = f64 ? Tile<double>::B_COLS : Tile<float>::B_COLS;
    p.ctiles = (uint32_t)((m->N + b_cols - 1) / b_cols);
    p.a_units = f64 ? m->WA : m->KBA;
    const int64_t n_a = a.X ? m->MBA * p.a_units : 0;
    const int64_t n_b = a.Y ? m->KBA * (f64 ? (p.ctiles + 1) / 2 : p.ctiles) : 0;
    // Row-compacted B: how many segments have a live row is known on the device only; at most one workgroup per CU loops
    // over them.
    const int64_t n_b_wg = a.b_compact && n_b > 256 ? 256 : n_b;
    // Blocks of A per workgroup: as many as leave every CU the two workgroups that fit, up to eight, so that one load
    // phase stands in front of several blocks and the others hide behind the stores of the block before (2048 x 16384
    // ReLU: 50.7, 42.1, 38.2 us with one, two, four; a 2048^2 matrix, 512 blocks, wants one: 10.0 against 13.4 with four).
    int64_t per_wg = n_a / 512;
    per_wg = per_wg < 1 ? 1 : per_wg > 8 ? 8 : per_wg;
    if (per_wg > m->MBA) per_wg = m->MBA;
    const int64_t n_a_wg = a.X ? (m->MBA + per_wg - 1) / per_wg * p.a_units : 0;
    const int64_t n_all = n_a_wg + n_b_wg;
    if (n_all <= 0 || n_a > 0x7fffffffLL || n_b > 0x7fffffffLL || n_all > 0x7fffffffLL) return hipErrorInvalidValue;
    p.n_b = (uint32_t)n_b;
    p.n_a_wg = (uint32_t)n_a_wg;
    p.n_b_wg = (uint32_t)n_b_wg;
    p.a_per_wg = (uint32_t)per_wg;
    const dim3 grid((uint32_t)n_all), block(BUILD_THREADS);
    (void)hipGetLastError();   // drop any stale error another library left on this thread
    hipLaunchKernelGGL(build_kernel(a.dtype, p.test.mode, m->bw, p.rows != nullptr), grid, block, 0, s, p);
    return hipGetLastError();
}

hipError_t mmm_launch_expand_rows(const mmm_maps *m, hipStream_t s)
{
    (void)hipGetLastError();
    hipLaunchKernelGGL(mmm_expand_rows_kernel, dim3((uint32_t)((m->WA + 3) / 4)), dim3(256), 0, s, m->rows_copy, m->btc_bits, m->bt_bits,
                       m->K, m->NB, m->WA);
    return hipGetLastError();
}

hipError_t mmm_launch_colany_compact(const mmm_maps *m, hipStream_t s)
{
    (void)hipGetLastError();
    hipLaunchKernelGGL(mmm_colany_compact_kernel, dim3((uint32_t)((m->MT * m->WA + 3) / 4)), dim3(256), 0, s, m->a_colany, m->kinfo,
                       m->kmap, m->a_colany_c, m->MT, m->WA);
    return hipGetLastError();
}

hipError_t mmm_launch_lists(const mmm_maps *m, hipStream_t s)
{
    (void)hipGetLastError();
    const dim3 grid((uint32_t)(m->MBA * m->KBA)), block(MMM_AB_COLS);
    const uint32_t *kinfo = m->a_compact ? m->kinfo : nullptr;
    uint2 *ent = reinterpret_cast<uint2 *>(m->a_ent);
    if (m->a_dtype == MMM_BF16)
        hipLaunchKernelGGL(mmm_lists_kernel<uint16_t>, grid, block, 0, s, m->a_img, m->a_bits, kinfo, m->kmap, m->a_cnt, ent, m->M, m->K, m->WA, m->KBA);
    else if (m->a_dtype == MMM_F16)
        hipLaunchKernelGGL(mmm_lists_kernel<_Float16>, grid, block, 0, s, m->a_img, m->a_bits, kinfo, m->kmap, m->a_cnt, ent, m->M, m->K, m->WA, m->KBA);
    else
        hipLaunchKernelGGL(mmm_lists_kernel<float>, grid, block, 0, s, m->a_img, m->a_bits, kinfo, m->kmap, m->a_cnt, ent, m->M, m->K, m->WA, m->KBA);
    return hipGetLastError();
}

// Per-tile active-k lists (see mmm_debug_k_lists): one wave per (row tile of 64, 16-column group,
// step of 128 k).
__global__ __launch_bounds__(64) void mmm_k_lists_kernel(const uint64_t *a_colany, const uint64_t *bt_bits, const uint32_t *kinfo,
                                                         uint8_t *out, int64_t K, int64_t NB, int64_t WA, int64_t MT, int64_t bw,
                                                         int64_t groups, int64_t steps)
{
    const int lane = threadIdx.x;
    const int64_t c = blockIdx.x % steps, G = (blockIdx.x / steps) % groups, t = blockIdx.x / (steps * groups);
    if (kinfo && c * MMM_AB_COLS >= (int64_t)*kinfo) return;
    uint8_t *rec = out + ((t * groups + G) * steps + c) * 132;
    uint32_t n = 0;
    for (int h = 0; h < 2; ++h) {
        const int64_t w = 2 * c + h;
        uint64_t m = 0;
        if (w < WA) {
            const int64_t b0 = G * MMM_GROUP_COLS / bw, b1 = (G * MMM_GROUP_COLS + MMM_GROUP_COLS - 1) / bw;
            for (int64_t b = b0; b <= b1 && b < NB; ++b) m |= bt_bits[b * WA + w];
            uint64_t any = 0;
            for (int64_t tt = 2 * t; tt < 2 * t + 2 && tt < MT; ++tt) any |= a_colany[tt * WA + w];
            m &= any;
        }
        if ((m >> lane) & 1ull) rec[4 + n + mbcnt64(m)] = (uint8_t)(64 * h + lane);
        n += (uint32_t)__popcll(m);
    }
    if (lane == 0) *reinterpret_cast<uint32_t *>(rec) = n;
}

hipError_t mmm_launch_dump_lists(const mmm_maps *m, uint8_t *out, size_t out_bytes, size_t *need, hipStream_t s)
{
    const int64_t groups = 16 * ((m->N + 255) / 256);
    const int64_t wgs = m->MBA * groups * m->KBA;
    const size_t bytes = (size_t)wgs * 132;
    if (need) *need = bytes;
    if (out == nullptr || out_bytes < bytes || wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    if (m->b_compact)
        if (hipError_t e = mmm_launch_colany_compact(m, s); e != hipSuccess) return e;
    (void)hipGetLastError();
    hipLaunchKernelGGL(mmm_k_lists_kernel, dim3((uint32_t)wgs), dim3(64), 0, s, m->b_compact ? m->a_colany_c : m->a_colany,
                       m->b_compact ? m->btc_bits : m->bt_bits, m->b_compact ? m->kinfo : nullptr, out, m->K, m->NB, m->WA, m->MT,
                       (int64_t)m->bw, groups, m->KBA);
    return hipGetLastError();
}

hipError_t mmm_launch_stats(const mmm_maps *m, hipStream_t s)
{
    (void)hipGetLastError();
    hipLaunchKernelGGL(mmm_stats_clear_kernel, dim3(1), dim3(64), 0, s, m->stats);
    hipLaunchKernelGGL(mmm_stats_kernel, dim3((uint32_t)m->WA), dim3(256), 0, s, m->a_bits, m->b_bits, m->M,
                       m->K, m->WA, m->WB, (int64_t)m->bw, m->stats);
    return hipGetLastError();
}
