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

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct PartedFloat { float v; };   // float elements that are laid out in three parts (see mmm_internal.h)
template <typename T> struct Layout {   // of the operands
    static constexpr size_t ESZ = sizeof(T);
    static constexpr bool PARTED = false;
};
template <> struct Layout<PartedFloat> {
    static constexpr size_t ESZ = MMM_PARTS_ESZ;
    static constexpr bool PARTED = true;
};

template <typename T> struct Tile {   // what a workgroup takes at a time, by element size
    static constexpr int ESZ = (int)sizeof(T);
    static constexpr int A_WORDS = ESZ == 8 ? 1 : 2;             // A: 64 rows x 64 A_WORDS columns
    static constexpr int LANE_COLS = ESZ == 8 ? 2 : 4;           // B: 128 rows x 64 LANE_COLS columns, so many per lane
    static constexpr int B_COLS = 64 * LANE_COLS;
    static constexpr int B_GROUPS = B_COLS / MMM_GROUP_COLS;
};

struct BuildParams {
    const void *X;
    int64_t ldx;
    const uint64_t *keep_a;
    uint64_t *a_bits;
    uint64_t *a_colany;
    char *a_img;
    uint8_t *a_wild;      // floats in parts
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
    mmm_divisor by_units, by_ctiles, by_wb;   // of a_units; of ctiles (doubles: of half of them); of WB
};
// The kernel reads its arguments where it needs them: as a by-value struct they were all loaded at its start, and bringing
// them back from where the compiler had spilled them took a third of the vector instructions.
typedef const __attribute__((address_space(4))) BuildParams ConstParams;
__device__ __forceinline__ ConstParams &reread(ConstParams &p)   // what is used of the result is loaded after this point
{
    ConstParams *q = &p;
    asm volatile("" : "+s"(q));
    return *q;
}

template <typename T> __device__ __forceinline__ uint32_t f32_bits(T v);
template <> __device__ __forceinline__ uint32_t f32_bits<float>(float v) { return __float_as_uint(v); }
template <> __device__ __forceinline__ uint32_t f32_bits<uint16_t>(uint16_t v) { return (uint32_t)v << 16; }   // bf16
template <> __device__ __forceinline__ uint32_t f32_bits<_Float16>(_Float16 v) { return __float_as_uint((float)v); }

// bit patterns of the 4- and 8-byte types
template <int ESZ> struct Pattern { typedef uint32_t type; static constexpr type magnitude = 0x7fffffffu; };
template <> struct Pattern<8> { typedef uint64_t type; static constexpr type magnitude = 0x7fffffffffffffffull; };

__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }

// `old` with the wave-uniform v in one lane (v_writelane_b32, for which clang has the intrinsic but no builtin)
extern "C" __device__ uint32_t mmm_writelane(uint32_t v, uint32_t lane, uint32_t old) __asm("llvm.amdgcn.writelane.i32");

__device__ __forceinline__ uint32_t mbcnt64(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, int l)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(v >> 32), l) << 32) |
           (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)v, l);
}

// Two floats to bf16, rounded to nearest: one instruction.
__device__ __forceinline__ uint32_t round2(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
}
// The next part of two floats; they become the rests.
__device__ __forceinline__ uint32_t take_part(uint32_t &a, uint32_t &b)
{
    const uint32_t part = round2(__uint_as_float(a), __uint_as_float(b));
    a = __float_as_uint(__uint_as_float(a) - __uint_as_float(part << 16));
    b = __float_as_uint(__uint_as_float(b) - __uint_as_float(part & 0xffff0000u));
    return part;
}
// Whether an element that is not zero lies outside the range that three parts hold.
struct OutOfRange {
    uint32_t most = 0, least = ~0u;   // of the magnitudes, and of those less 1 (zero is no magnitude)
    __device__ __forceinline__ void see(uint32_t bits)
    {
        const uint32_t m = bits & 0x7fffffffu;
        most = max(most, m);
        least = min(least, m - 1u);
    }
    __device__ __forceinline__ void add(const OutOfRange &o)
    {
        most = max(most, o.most);
        least = min(least, o.least);
    }
    __device__ __forceinline__ bool any() const { return most >= MMM_PARTS_HI || least < MMM_PARTS_LO - 1u; }
};
__device__ __forceinline__ bool out_of_range(uint32_t bits)
{
    OutOfRange o;
    o.see(bits);
    return o.any();
}

// OR of a value over aligned runs of LANES lanes (2 .. 16), in all of them, without leaving the vector registers
template <int LANES> __device__ __forceinline__ uint32_t or_lanes(uint32_t x)
{
    auto with = [](uint32_t v, auto ctrl) { return v | (uint32_t)__builtin_amdgcn_mov_dpp((int)v, decltype(ctrl)::value, 0xf, 0xf, true); };
    if (LANES >= 2) x = with(x, std::integral_constant<int, 0xb1>{});    // quad_perm 1 0 3 2
    if (LANES >= 4) x = with(x, std::integral_constant<int, 0x4e>{});    // quad_perm 2 3 0 1
    if (LANES >= 8) x = with(x, std::integral_constant<int, 0x141>{});   // row_half_mirror
    if (LANES >= 16) x = with(x, std::integral_constant<int, 0x140>{});  // row_mirror
    return x;
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
    uint8_t wild[2][BUILD_WAVES];               // floats in parts: [stage][wave]
    uint8_t live[MMM_AB_COLS];                  // row-compacted mode: live columns of the blocks
    uint8_t on[MMM_AB_COLS];                    // and floats in parts: whether a column is one (what is switched off marks nothing)
    uint32_t before[BUILD_WAVES];               // row-compacted mode: live rows before them, by wave
};

template <typename T> struct ABlock {   // one block in a wave's registers: lane <-> k (and k + 64)
    typename std::conditional<sizeof(T) == 8, uint64_t, uint32_t>::type x[A_ROWS][Tile<T>::A_WORDS];
    uint64_t kw;   // keep word of (row t, half h), in lane t * A_WORDS + h
};

// Numbers of blocks, words and columns.  Of some 125 scalar instructions per block, which each of sixteen waves takes, 64-bit products were six
// each where 32 by 32 bits are two, and comparisons of 64 bits leave the scalar unit (2048 x 16384, columns, bf16: A 25.3 -> 22.2 us; 2048^2
// floats 7.8 -> 7.5).  Doubles, whose blocks are half as many elements and which wait for memory, are no faster for it (2048^3, p = .1, the whole
// pass: 63.6 with 32 bits, 63.3 with 64).
template <typename T> using block_no = typename std::conditional<sizeof(T) == 8, int64_t, int32_t>::type;

// v_writelane_b32 and DPP instead of selects, wave-uniform words only where a lane mask is wanted, no branch per row and
// one base per block: the sixteen waves of a block share one scalar unit, and the scan of half-precision matrices was
// bound by it (2048 x 16384, one column in ten: 36.5 us with pairs of k per lane, whose masks had to be interleaved there).
// DEEP: two blocks ahead in registers instead of one, for 16-bit types, whose blocks are half as large, where a workgroup has
// several (columns 2048 x 16384: 28 -> 26 us for A, 41 -> 35.4 with B; with one or two blocks per workgroup the loads past
// the last one cost more than they gain, 6.6 -> 9 us for 512 x 8192, and so do more bytes in flight for the wider types).
template <typename T, int TEST, bool ROWS, bool DEEP>
__device__ __forceinline__ void scan_a(ConstParams &p0, block_no<T> bj, block_no<T> bi0, block_no<T> bi1, int lane, int wave, AShared &sh)
{
    ConstParams &p = reread(p0);
    asm volatile("" ::"s"(p.keep_a), "s"(p.M), "s"(p.K), "s"(p.WA), "s"(p.X), "s"(p.ldx));   // (in one go: what stands in front of the first loads)
    typedef typename Pattern<sizeof(T)>::type pattern;
    typedef block_no<T> no_t;
    constexpr int ESZ = (int)sizeof(T);
    constexpr bool WIDE = ESZ >= 4;
    constexpr int A_WORDS = Tile<T>::A_WORDS, A_COLS = 64 * A_WORDS;
    constexpr bool PARTED = Layout<T>::PARTED;
    constexpr bool WIDE_IMG = Layout<T>::ESZ % 4 == 0;   // rows w, w + 16, w + 32, w + 48 in the image, else in natural order
    constexpr int UNITS = MMM_AB_ROWS * (PARTED ? 2 : ESZ) / 16;   // 16-byte units per column (and part)
    constexpr uint32_t COPIES = PARTED ? MMM_PARTS : 1;
    constexpr uint32_t OUTSIDE = 0x80000000u;       // past the end of every buffer resource below, whatever row offset is added
    const bool has_keep = p.keep_a != nullptr;
    constexpr bool compact = ROWS;
    // Buffer resources that end with the last row: what lies past it, and lanes past the last column, reads as +0, which
    // is never kept, and is not stored.  64 rows are at most 2^31 bytes (leading dimensions are below 2^22).
    const no_t k_lo = bj * A_COLS, w_lo = bj * A_WORDS;   // (K < 2^22)
    const int tail = (int)min(p.K - k_lo, (int64_t)A_COLS);   // columns of these blocks that exist
    const uint32_t row_bytes = (uint32_t)p.ldx * ESZ, map_bytes = (uint32_t)p.WA * 8u;
    const uint32_t row0 = WIDE_IMG ? (uint32_t)wave : (uint32_t)wave * A_ROWS;
    constexpr uint32_t ROW_STEP = WIDE_IMG ? BUILD_WAVES : 1;
    uint32_t off[A_WORDS];
#pragma unroll
    for (int h = 0; h < A_WORDS; ++h) off[h] = 64 * h + lane < tail ? (uint32_t)(64 * h + lane) * ESZ : OUTSIDE;
    const uint32_t map_at = lane < A_ROWS * A_WORDS && w_lo + lane % A_WORDS < p.WA
                                ? (row0 + ROW_STEP * (uint32_t)(lane / A_WORDS)) * map_bytes + (uint32_t)(lane % A_WORDS) * 8u
                                : OUTSIDE;
    auto rows_at = [&](no_t bi) -> uint32_t { return (uint32_t)min((no_t)p.M - bi * MMM_AB_ROWS, (no_t)MMM_AB_ROWS); };   // (M is at most 2^30)
    auto block_rows = [](no_t bi, uint32_t row) -> uint64_t {   // bytes up to block row bi
        return ESZ == 8 ? (uint64_t)bi * ((uint64_t)row * MMM_AB_ROWS) : (uint64_t)(uint32_t)bi * (row * MMM_AB_ROWS);
    };
    auto map_rsrc = [&](const uint64_t *map, no_t bi, bool any) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(reinterpret_cast<const char *>(map) + block_rows(bi, map_bytes) + w_lo * 8), 0,
                                                 any ? (int)(rows_at(bi) * map_bytes - (uint32_t)w_lo * 8u) : 0, 0x00020000);
    };
    // Always the same number of loads, so that waiting for one block's does not mean waiting for the next one's: where
    // there is no block or no keep bitmap the buffer is empty.  (With the bitmap's load on one side of a branch the elements were asked for when it
    // had arrived.)
    auto load = [&](no_t bi, ABlock<T> &r) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
        const bool there = bi < bi1;
        const u32x2 k = __builtin_amdgcn_raw_buffer_load_b64(map_rsrc(p.keep_a, bi, there && has_keep), (int)map_at, 0, 0);
        r.kw = (uint64_t)k.y << 32 | k.x;
        const __amdgpu_buffer_rsrc_t x = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char *>(static_cast<const char *>(p.X) + block_rows(bi, row_bytes) + k_lo * ESZ), 0,
            there ? (int)((rows_at(bi) - 1u) * row_bytes + (uint32_t)(tail * ESZ)) : 0, 0x00020000);
#pragma unroll
        for (int t = 0; t < A_ROWS; ++t) {
            const uint32_t row = (row0 + ROW_STEP * (uint32_t)t) * row_bytes;
#pragma unroll
            for (int h = 0; h < A_WORDS; ++h) {
                const int at = (int)(off[h] + row);
                if constexpr (ESZ == 8) {
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(x, at, 0, 0);
                    r.x[t][h] = (uint64_t)v.y << 32 | v.x;
                } else if constexpr (ESZ == 4) {
                    r.x[t][h] = __builtin_amdgcn_raw_buffer_load_b32(x, at, 0, 0);
                } else {
                    r.x[t][h] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(x, at, 0, 0);
                }
            }
        }
        asm volatile("" ::: "memory");
    };

    ABlock<T> even, odd;
    load(bi0, even);
    if (DEEP) load(bi0 + 1, odd);
    uint32_t base = (uint32_t)k_lo;   // image column of the blocks' first
    int cols = A_COLS;                // and how many there are
    if (compact) {   // the blocks' live columns, and how many live rows come before them
        uint32_t n = 0;
        for (int64_t w = threadIdx.x; w < w_lo; w += BUILD_THREADS) n += (uint32_t)__popcll(p.rows[w]);
        const uint64_t m0 = row_word(p.rows, w_lo, p.K), m1 = w_lo + 1 < p.WA ? row_word(p.rows, w_lo + 1, p.K) : 0ull;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) n += (uint32_t)__shfl_xor((int)n, d, 64);
        if (lane == 0) sh.before[wave] = n;
        if (PARTED) {   // (every wave the same: it reads them before a barrier)
            sh.on[lane] = (uint8_t)((m0 >> lane) & 1ull);
            sh.on[64 + lane] = (uint8_t)((m1 >> lane) & 1ull);
        }
        const uint32_t n0 = (uint32_t)__popcll(m0);
        cols = (int)(n0 + (uint32_t)__popcll(m1));
        if (wave == 0) {
            if ((m0 >> lane) & 1ull) sh.live[mbcnt64(m0)] = (uint8_t)lane;
            if ((m1 >> lane) & 1ull) sh.live[n0 + mbcnt64(m1)] = (uint8_t)(64 + lane);
        }
    }
    // 16-bit elements and parts: the rotation of column k's eight 16-byte units in the stage.  Pieces of 8 bytes are written column by column and two
    // units of a plane read column by column: neither finds two of sixteen columns' in the same banks.
    auto turned = [](int k) { return (k >> 1 & 3) << 1 | (k >> 3 & 1); };
    auto block = [&](no_t bi, ABlock<T> &cur, int st, auto ahead) __attribute__((always_inline)) {
        ConstParams &p = reread(p0);
        constexpr int AHEAD = decltype(ahead)::value;   // the block whose loads take this one's place
        char *const stage = sh.stage[PARTED ? 0 : st];
        uint64_t word[A_ROWS][A_WORDS];   // bitmap words: wave-uniform, the lane masks of what stays
        uint32_t pair[2][A_WORDS];        // 16-bit: rows 2t and 2t + 1
        if constexpr (!WIDE)
#pragma unroll
            for (int h = 0; h < A_WORDS; ++h)
#pragma unroll
                for (int t = 0; t < 2; ++t) pair[t][h] = __builtin_amdgcn_perm(cur.x[2 * t + 1][h], cur.x[2 * t][h], 0x05040100u);
        auto words = [&](auto keep) __attribute__((always_inline)) {
            constexpr bool KEEP = decltype(keep)::value;
#pragma unroll
            for (int h = 0; h < A_WORDS; ++h)
#pragma unroll
                for (int t = 0; t < A_ROWS; ++t) {
                    uint64_t m;
                    if constexpr (WIDE) {
                        const pattern v = TEST == TEST_MAGNITUDE ? cur.x[t][h] & Pattern<ESZ>::magnitude : cur.x[t][h];
                        m = ballot64(v - (pattern)p.test.lo1 < (pattern)p.test.len1);
                        if (TEST == TEST_TWO_RANGES) m |= ballot64(v - (pattern)p.test.lo2 < (pattern)p.test.len2);
                    } else {
                        typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
                        const uint32_t v = TEST == TEST_MAGNITUDE ? pair[t / 2][h] & 0x7fff7fffu : pair[t / 2][h];
                        const u16x2 lo1 = {(uint16_t)p.test.lo1, (uint16_t)p.test.lo1}, lo2 = {(uint16_t)p.test.lo2, (uint16_t)p.test.lo2};
                        const u16x2 y = __builtin_bit_cast(u16x2, v) - lo1;
                        m = ballot64(y[t & 1] < (uint16_t)p.test.len1);
                        if (TEST == TEST_TWO_RANGES) {
                            const u16x2 z = __builtin_bit_cast(u16x2, v) - lo2;
                            m |= ballot64(z[t & 1] < (uint16_t)p.test.len2);
                        }
                    }
                    if (KEEP) m &= readlane64(cur.kw, t * A_WORDS + h);
                    word[t][h] = m;
                }
        };
        if (has_keep)
            words(std::true_type{});
        else
            words(std::false_type{});
        if (PARTED && bi > bi0) __syncthreads();   // one stage (48 KiB; two would leave a compute unit one workgroup): the block before has left it
        OutOfRange range;   // of the elements in columns that are on
#pragma unroll
        for (int h = 0; h < A_WORDS; ++h) {
            const int k = 64 * h + lane;
            if constexpr (WIDE) {
                pattern u[A_ROWS];
#pragma unroll
                for (int t = 0; t < A_ROWS; ++t) u[t] = __builtin_amdgcn_inverse_ballot_w64(word[t][h]) ? cur.x[t][h] : (pattern)0;
                if constexpr (PARTED) {
                    OutOfRange here;
#pragma unroll
                    for (int t = 0; t < A_ROWS; ++t) here.see(u[t]);
                    u32x2 part[MMM_PARTS];
                    uint32_t rest[A_ROWS] = {u[0], u[1], u[2], u[3]};
#pragma unroll
                    for (int q = 0; q < MMM_PARTS; ++q) part[q] = u32x2{take_part(rest[0], rest[1]), take_part(rest[2], rest[3])};
                    if (!ROWS) range.add(here);
                    if (ballot64(here.any()) != 0) {   // seldom: such elements as they are
                        if (ROWS && sh.on[k] != 0) range.add(here);   // (no others matter)
#pragma unroll
                        for (int t = 0; t < A_ROWS; ++t)
                            if (out_of_range(u[t])) {
                                auto put = [&](uint32_t &to, uint32_t v) { to = t & 1 ? (to & 0xffffu) | v << 16 : (to & 0xffff0000u) | v; };
                                uint32_t v0 = part[0][t / 2], v1 = part[1][t / 2], v2 = part[2][t / 2];
                                put(v0, u[t] >> 16);
                                put(v1, u[t] & 0xffffu);
                                put(v2, MMM_PARTS_RAW);
                                part[0][t / 2] = v0;
                                part[1][t / 2] = v1;
                                part[2][t / 2] = v2;
                            }
                    }
#pragma unroll
                    for (int q = 0; q < MMM_PARTS; ++q)
                        *reinterpret_cast<u32x2 *>(stage + q * MMM_PART_BYTES + k * 128 + ((wave ^ (turned(k) << 1)) << 3)) = part[q];
                    continue;
                }
                char *at = stage + k * (UNITS * 16) + ((wave ^ (k & 15)) << 4);
                if constexpr (ESZ == 4) {
                    *reinterpret_cast<uint4 *>(at) = make_uint4(u[0], u[1], u[2], u[3]);
                } else {
                    *reinterpret_cast<ulong2 *>(at) = make_ulong2(u[0], u[1]);
                    *reinterpret_cast<ulong2 *>(at + 256) = make_ulong2(u[2], u[3]);
                }
            } else {   // rows 4w .. 4w+3
                uint32_t d[2];
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    d[t] = pair[t][h] & ((__builtin_amdgcn_inverse_ballot_w64(word[2 * t][h]) ? 0xffffu : 0u) |
                                          (__builtin_amdgcn_inverse_ballot_w64(word[2 * t + 1][h]) ? 0xffff0000u : 0u));
                *reinterpret_cast<uint2 *>(stage + k * 128 + ((wave ^ (turned(k) << 1)) << 3)) = make_uint2(d[0], d[1]);
            }
        }
        // lane t * A_WORDS + h takes the word of (row t, half h)
        uint32_t mine_lo = 0, mine_hi = 0;
#pragma unroll
        for (int t = 0; t < A_ROWS; ++t)
#pragma unroll
            for (int h = 0; h < A_WORDS; ++h) {
                mine_lo = mmm_writelane((uint32_t)word[t][h], (uint32_t)(t * A_WORDS + h), mine_lo);
                mine_hi = mmm_writelane((uint32_t)(word[t][h] >> 32), (uint32_t)(t * A_WORDS + h), mine_hi);
            }
        {   // column-any words of this wave's rows, by 32-row half of the block (4- and 8-byte types: rows t < 2 and t >= 2)
            auto other = [](uint32_t v, auto ctrl) { return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, decltype(ctrl)::value, 0xf, 0xf, true); };
            typedef std::integral_constant<int, 0xb1> Swap1;      // quad_perm 1 0 3 2
            typedef std::integral_constant<int, 0x4e> Swap2;      // quad_perm 2 3 0 1
            typedef std::integral_constant<int, 0x141> Mirror8;   // row_half_mirror
            auto any_of = [&](uint32_t v) {
                if constexpr (ESZ == 8) return v | other(v, Swap1{});
                v |= other(v, Swap2{});
                if constexpr (!WIDE_IMG) v |= other(other(v, Mirror8{}), Swap1{});
                return v;
            };
            const uint64_t any = (uint64_t)any_of(mine_hi) << 32 | any_of(mine_lo);
            if (ESZ == 8) {
                if (lane < 4 && (lane & 1) == 0) sh.any[st][wave][lane >> 1][0] = any;
            } else if (WIDE_IMG) {
                if (lane < 8 && (lane & 2) == 0) sh.any[st][wave][lane >> 2][lane & 1] = any;
            } else {
                if (lane < 4) sh.any[st][wave][lane >> 1][lane & 1] = lane >> 1 == wave / (BUILD_WAVES / 2) ? any : 0ull;
            }
        }
        if constexpr (PARTED) {
            const bool wild = ballot64(range.any()) != 0;
            if (lane == 0) sh.wild[st][wave] = wild ? 1 : 0;
        }
        if (AHEAD == 2 || bi + 1 < bi1) load(bi + AHEAD, cur);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{mine_lo, mine_hi}, map_rsrc(p.a_bits, bi, true), (int)map_at, 0, 0);
        __syncthreads();
        if (wave == 0) {   // lane (t32, h, wave): OR over the sixteen waves
            const int t32 = lane >> 5, h = (lane >> 4) & 1;
            const uint64_t any = sh.any[st][lane & 15][t32][h];
            uint32_t lo = (uint32_t)any, hi = (uint32_t)(any >> 32);
            lo = or_lanes<16>(lo);
            hi = or_lanes<16>(hi);
            const int64_t tile = (int64_t)bi * (MMM_AB_ROWS / MMM_COLANY_ROWS) + t32;
            if ((lane & 15) == 0 && tile < p.MT && h < A_WORDS && w_lo + h < p.WA) p.a_colany[tile * p.WA + w_lo + h] = ((uint64_t)hi << 32) | lo;
            if constexpr (PARTED) {
                const uint64_t wild = ballot64(sh.wild[st][lane & 15] != 0);
                if (lane == 0) p.a_wild[bi * p.KBA + bj] = wild != 0 ? 1 : 0;
            }
        }
        // the image: 4- and 8-byte elements: column k (or k') of block row bi is one run of 64; else four planes of 16 rows
        if (compact && bi == bi0) {
            base = 0;
            for (int w = 0; w < BUILD_WAVES; ++w) base += sh.before[w];
        }
        constexpr uint32_t COL_BYTES = MMM_AB_ROWS * (PARTED ? 2 : ESZ), PLANE_UNITS = 2 * MMM_AB_COLS;   // units of a plane: two per column
        if constexpr (!WIDE_IMG) {   // a unit (of each part) per thread
            static_assert(MMM_AB_COLS * UNITS == BUILD_THREADS, "");
            char *const blocks = p.a_img + (uint64_t)(uint32_t)bi * ((uint32_t)p.KBA * (MMM_PART_BYTES * COPIES));
            auto put = [&](char *to, int k, int unit) __attribute__((always_inline)) {
                const char *const from = stage + k * 128 + ((unit ^ turned(k)) << 4);
#pragma unroll
                for (int i = 0; i < (int)COPIES; ++i)
                    *reinterpret_cast<uint4 *>(to + i * MMM_PART_BYTES) = *reinterpret_cast<const uint4 *>(from + i * MMM_PART_BYTES);
            };
            if (compact) {   // the eight units of a column side by side: few waves have any (as above, 31.3 -> 28.2; floats in parts, 45.0 -> 42.3)
                if ((int)threadIdx.x < cols * UNITS) {
                    const uint32_t col = base + threadIdx.x / UNITS, unit = threadIdx.x % UNITS;
                    put(blocks + (col / MMM_AB_COLS * (MMM_PART_BYTES * COPIES) + unit / 2u * MMM_PLANE_BYTES + col % MMM_AB_COLS * MMM_PLANE_COL_BYTES + unit % 2u * 16u),
                        (int)sh.live[threadIdx.x / UNITS], (int)unit);
                }
            } else {   // plane by plane
                put(blocks + ((uint32_t)bj * (MMM_PART_BYTES * COPIES) + threadIdx.x * 16u), (int)(threadIdx.x % PLANE_UNITS / 2u),
                    (int)(threadIdx.x / PLANE_UNITS * 2u + threadIdx.x % 2u));
            }
        } else {
            char *img = p.a_img + (uint64_t)(uint32_t)bi * ((uint32_t)p.KBA * (MMM_AB_COLS * COL_BYTES)) + (uint64_t)base * COL_BYTES;
            auto stage_of = [&](int k, int unit) -> int { return k * (int)COL_BYTES + ((unit ^ (k & 15)) << 4); };   // where it waits in the stage
            if (compact) {
                for (int q = threadIdx.x; q < cols * UNITS; q += BUILD_THREADS) {
                    const int j = q / UNITS, k = (int)sh.live[j];
                    *reinterpret_cast<uint4 *>(img + (uint32_t)q * 16u) = *reinterpret_cast<const uint4 *>(stage + stage_of(k, q % UNITS));
                }
            } else {   // two units per thread
                const int at = stage_of(threadIdx.x / UNITS, threadIdx.x % UNITS);
#pragma unroll
                for (int i = 0; i < A_COLS * UNITS / BUILD_THREADS; ++i)
                    *reinterpret_cast<uint4 *>(img + (threadIdx.x * 16u + (uint32_t)(i * BUILD_THREADS * 16))) =
                        *reinterpret_cast<const uint4 *>(stage + at + i * (BUILD_THREADS * 16));
            }
        }
    };
    if constexpr (DEEP) {
        for (no_t bi = bi0; bi < bi1; bi += 2) {
            block(bi, even, 0, std::integral_constant<int, 2>{});
            if (bi + 1 < bi1) block(bi + 1, odd, 1, std::integral_constant<int, 2>{});
        }
    } else {
        for (no_t bi = bi0; bi < bi1; ++bi) block(bi, even, (int)(bi - bi0) & 1, std::integral_constant<int, 1>{});
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
    __align__(16) uint16_t list[16][SEG];
    __align__(16) char pack[16 * (SEG * MMM_GROUP_COLS * 2 + 16)];   // 16-bit types: the packed groups
    int32_t kk[SEG];                  // row-compacted mode: the rows behind the segment's k' (-1: none)
    uint32_t sums[BUILD_WAVES];
};

// Rows k' = seg*128 .. of the numbering given by `rows`, into sh.kk; returns K'.
// It stands in front of everything else that a workgroup of B does: one round trip, and sums over the lanes in the vector registers (with the words
// read again for their positions, sums by LDS moves, the numbering made once more to find that no segment is left, and the zero rows of the map written
// first: B of 161 x 13627 x 2024 bf16 9.9 -> 8.2 us, of 755 x 5790 x 2560 9.7 -> 7.9, of 2048 x 16384 x 4096 floats 14.5 -> 13.1).
__device__ __forceinline__ uint32_t number_rows(ConstParams &p, uint32_t seg, int lane, int wave, BShared &sh)
{
    const uint32_t tid = threadIdx.x, WA = (uint32_t)p.WA;
    // every thread counts a run of words (a word, but for K above 65536)
    const uint32_t per = (WA + BUILD_THREADS - 1) / BUILD_THREADS, w0 = tid * per, w1 = min(WA, w0 + per);
    const uint64_t word = w0 < w1 ? row_word(p.rows, w0, p.K) : 0ull;   // the first
    if (tid < SEG) sh.kk[tid] = -1;
    uint32_t cnt = (uint32_t)__popcll(word);
    for (uint32_t w = w0 + 1; w < w1; ++w) cnt += (uint32_t)__popcll(row_word(p.rows, w, p.K));
    uint32_t incl = cnt;
    auto add = [&](auto ctrl, auto rows) { incl += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, decltype(ctrl)::value, decltype(rows)::value, 0xf, decltype(rows)::value == 0xf); };
    typedef std::integral_constant<int, 0xf> All;
    add(std::integral_constant<int, 0x111>{}, All{});   // row_shr 1, 2, 4, 8
    add(std::integral_constant<int, 0x112>{}, All{});
    add(std::integral_constant<int, 0x114>{}, All{});
    add(std::integral_constant<int, 0x118>{}, All{});
    add(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});   // row_bcast 15, 31
    add(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
    if (lane == 63) sh.sums[wave] = incl;
    __syncthreads();
    uint32_t pos = incl - cnt, total = 0;
#pragma unroll
    for (int w = 0; w < BUILD_WAVES; ++w) {
        const uint32_t s = sh.sums[w];
        if (w < wave) pos += s;
        total += s;
    }
    const uint32_t lo = seg * SEG;
    if (pos < lo + SEG && pos + cnt > lo)
        for (uint32_t w = w0; w < w1; ++w)
            for (uint64_t m = w == w0 ? word : row_word(p.rows, w, p.K); m != 0; m &= m - 1, ++pos)
                if (pos >= lo && pos < lo + SEG) sh.kk[pos - lo] = (int32_t)(w * 64 + __builtin_ctzll(m));
    __syncthreads();
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)total);
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

// What bounds this for a few workgroups is latency, and of that the scalar unit that the sixteen waves share: per row the
// occupancy stays in the vector registers (one bit per lane, collected with the lane's other rows, then OR'ed over the
// lanes of a block for all rows at once), addresses come from one buffer resource per wave, and lanes with nothing to
// store are given an offset past its end instead of being branched around.
// ROWS (row-compacted mode): the rows are the live rows k' = 128 seg .., and the transposed map is over k'.
// Returns the number of live rows (ROWS; else nothing of use).  carry: doubles in 32-wide blocks fill half a
// byte of a map row per column tile, so the map bits of an even tile are handed to the odd one after it.
// (K and N are below 2^22: numbers of segments, tiles, rows and groups fit in 32 bits, and only what is multiplied by a pitch needs more.)
template <typename T, int BW, bool ROWS>
__device__ __forceinline__ uint32_t scan_b(ConstParams &p0, uint32_t seg, uint32_t ct, int lane, int wave, BShared &sh, uint32_t &carry)
{
    ConstParams &p = reread(p0);
    if (ROWS) asm volatile("" ::"s"(p.rows), "s"(p.WA));
    asm volatile("" ::"s"(p.keep_blocks), "s"(p.K), "s"(p.N), "s"(p.WB), "s"(p.Y), "s"(p.ldy));   // (as in scan_a)
    constexpr int ESZ = (int)sizeof(T);
    constexpr int LANE_COLS = Tile<T>::LANE_COLS, B_COLS = Tile<T>::B_COLS, B_GROUPS = Tile<T>::B_GROUPS;
    constexpr int LPB = BW / LANE_COLS;               // lanes per block
    constexpr int LPG = MMM_GROUP_COLS / LANE_COLS;   // lanes per group
    constexpr int BPW = B_COLS / BW;                  // blocks per column tile
    constexpr bool WIDE = ESZ >= 4;
    constexpr bool SPLIT = BW < MMM_GROUP_COLS;       // a group holds two blocks
    constexpr bool PARTED = Layout<T>::PARTED;
    constexpr size_t LSZ = Layout<T>::ESZ;
    constexpr uint32_t NO_LOAD = 0x80000000u, NO_STORE = 0xfffffff0u;   // offsets past the ends of the buffer resources
    const uint32_t col0 = ct * B_COLS, blk0 = ct * BPW;
    uint32_t live = 0;
    if (ROWS) {
        live = number_rows(p, seg, lane, wave, sh);
        if (ct == 0) {   // publish the numbering
            if (threadIdx.x < SEG && sh.kk[threadIdx.x] >= 0) p.kmap[seg * SEG + threadIdx.x] = (uint32_t)sh.kk[threadIdx.x];
            if (seg == 0) {
                if (threadIdx.x == 0) p.kinfo[0] = live;
                for (int64_t w = threadIdx.x; w < p.WA; w += BUILD_THREADS) p.rows_copy[w] = row_word(p.rows, w, p.K);
            }
        }
        if (seg * SEG >= live) return live;   // the whole workgroup
    }
    // lane j < 8: row j of the wave and which of its blocks are switched on
    int krow = -1;
    uint32_t piece = 0;
    {
        const int j = lane & (B_ROWS - 1);
        const int k = ROWS ? sh.kk[wave * B_ROWS + j] : (int)(seg * SEG) + wave * B_ROWS + j;
        krow = k >= 0 && k < (int)p.K ? k : -1;
        const uint32_t kc = (uint32_t)max(krow, 0);
        uint64_t w = ~0ull;
        if (p.keep_blocks != nullptr) w = p.keep_blocks[(uint64_t)kc * (uint32_t)p.WB + (blk0 >> 6)];   // wave-uniform branches
        if (ESZ == 8 && p.keep_rows != nullptr && !((p.keep_rows[kc >> 6] >> (kc & 63)) & 1ull)) w = 0;   // (not numbered)
        piece = krow >= 0 ? (uint32_t)(w >> (blk0 & 63)) : 0u;
    }
    u32x4 raw[B_ROWS];
    const uint32_t lane_off = (uint32_t)(lane * LANE_COLS) < (uint32_t)p.N - col0 ? (uint32_t)(lane * LANE_COLS * ESZ) : NO_LOAD;   // N is a multiple of LANE_COLS
    const uint32_t row_bytes = (uint32_t)p.ldy * ESZ;
    const char *const ytile = static_cast<const char *>(p.Y) + col0 * ESZ;
    const uint32_t k_first = min(seg * SEG + (uint32_t)(wave * B_ROWS), (uint32_t)p.K - 1u);
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(static_cast<const char *>(p.Y) + ((uint64_t)k_first * (uint32_t)p.ldy + col0) * ESZ), 0,
                                                                 0x7fffffff, 0x00020000);
    auto load_rows = [&](auto any_alignment) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < B_ROWS; ++j) {
            const uint32_t pj = (uint32_t)__builtin_amdgcn_readlane((int)piece, j);   // nothing if there is no such row
            const uint32_t off = (pj >> (lane / LPB)) & 1u ? lane_off : NO_LOAD;
            uint32_t at = (uint32_t)j * row_bytes;
            if (ROWS) {   // rows far from each other
                const uint32_t k = (uint32_t)max(__builtin_amdgcn_readlane(krow, j), 0);
                r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(ytile + (uint64_t)k * row_bytes), 0, 0x7fffffff, 0x00020000);
                at = 0;
            }
            if constexpr (WIDE) {
                raw[j] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)at, 0);
            } else if constexpr (!decltype(any_alignment)::value) {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, (int)at, 0);
                raw[j] = u32x4{v.x, v.y, 0, 0};
            } else {
                uint32_t e[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) e[i] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off, (int)at + 2 * i, 0);
                raw[j] = u32x4{e[0] | e[1] << 16, e[2] | e[3] << 16, 0, 0};
            }
        }
    };
    // (One branch around all loads: one per load made the compiler bring back its spilled scalar registers eight times, 128 of
    // 525 vector instructions per wave, on which half-precision B was bound.)
    if (!WIDE && p.y_unaligned)
        load_rows(std::true_type{});
    else
        load_rows(std::false_type{});
    __builtin_amdgcn_sched_barrier(0);   // all of them are under way before the first is looked at
    uint32_t gb = 0, bbm = 0;   // rows (bit j) in which this lane's group / block is occupied
    uint64_t mine = 0;          // lane j: the lanes with a non-zero element in row j, then at multiples of LPB the occupied blocks
    {
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int j = B_ROWS - 1; j >= 0; --j) {
            const uint32_t nz = ESZ == 8   ? raw[j].x | raw[j].z | ((raw[j].y | raw[j].w) & 0x7fffffffu)
                              : ESZ == 4 ? (raw[j].x | raw[j].y | raw[j].z | raw[j].w) & 0x7fffffffu
                                         : (raw[j].x | raw[j].y) & 0x7fff7fffu;
            const uint64_t m = ballot64(nz != 0);
            gb = gb * 2 + (nz != 0 ? 1u : 0u);
            lo = mmm_writelane((uint32_t)m, (uint32_t)j, lo);
            hi = mmm_writelane((uint32_t)(m >> 32), (uint32_t)j, hi);
        }
        mine = (uint64_t)hi << 32 | lo;
        mine |= mine >> 1;
        if (LPB >= 4) mine |= mine >> 2;
        if (LPB >= 8) mine |= mine >> 4;
        if (LPB >= 16) mine |= mine >> 8;
        gb = or_lanes<LPB>(gb);
        bbm = gb;
        if (SPLIT) gb = or_lanes<LPG>(gb);
    }
    sh.gbits[lane][wave] = (uint8_t)gb;
    if (SPLIT) sh.bbits[lane][wave] = (uint8_t)bbm;
    if (lane < B_ROWS && krow >= 0) {   // this tile's piece of the map row: 4, 2, 1 or half a byte
        uint32_t v = squeeze<LPB>(mine);
        char *const row = reinterpret_cast<char *>(p.b_bits + (uint64_t)(uint32_t)krow * (uint32_t)p.WB), *const dst = row + blk0 / 8;
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
            for (uint32_t q = (blk0 + BPW + 7) / 8; q < (uint32_t)p.WB * 8u; ++q) row[q] = 0;
    }
    constexpr int RING = mmm_ring(LSZ);
    // (floats in parts: their ring has no zero column; the block's first, which exists if there is a list, does as well)
    const uint32_t ZERO_ENTRY = WIDE && !PARTED ? mmm_list_entry(LSZ, mmm_zero_col(RING)) : PARTED ? mmm_list_entry(LSZ, (uint32_t)seg % (uint32_t)RING * SEG) : 0u;
    static_assert(B_GROUPS * SEG * 2 <= BUILD_THREADS * 4, "at most one list word per thread");
    if (threadIdx.x < B_GROUPS * SEG / 2) reinterpret_cast<uint32_t *>(sh.list)[threadIdx.x] = ZERO_ENTRY | ZERO_ENTRY << 16;
    // (Read where all lanes are: a value first read, or made wider, on one side of a branch is taken for one of each lane, and a store through a
    // resource made of it becomes a loop over resources: eight of a dozen instructions each, doubles always had them.)
    const uint32_t KBA = (uint32_t)p.KBA, NG = (uint32_t)p.NG;
    asm volatile("" ::"s"(KBA), "s"(NG));
    __syncthreads();
    if (wave == 0 && (lane % LPB) == 0) {   // transposed map words of this lane's block
        const uint64_t *t = reinterpret_cast<const uint64_t *>(SPLIT ? sh.bbits[lane] : sh.gbits[lane]);
        const uint32_t blk = blk0 + (uint32_t)(lane / LPB);
        if (blk < (uint32_t)p.NB) {
            uint64_t *dst = (ROWS ? p.btc_bits : p.bt_bits) + (uint64_t)blk * (uint32_t)p.WA + seg * 2;
            dst[0] = t[0];
            if (seg * 2 + 1 < (uint32_t)p.WA) dst[1] = t[1];
        }
    }
    if (ESZ == 8 && !p.pack) return 0;
    const uint64_t *gt = reinterpret_cast<const uint64_t *>(sh.gbits[lane]);
    const uint64_t glo = gt[0], ghi = gt[1];
    const uint32_t n = (uint32_t)__popcll(glo) + (uint32_t)__popcll(ghi);   // rows of this lane's group
    const uint64_t below = (1ull << (8 * (wave & 7))) - 1ull;
    const uint32_t slot0 = wave < 8 ? (uint32_t)__popcll(glo & below) : (uint32_t)__popcll(glo) + (uint32_t)__popcll(ghi & below);
    const uint32_t G = ct * B_GROUPS + (uint32_t)(lane / LPG);   // this lane's group
    const bool group_ok = G < NG;
    // the lists: the lanes of a group share the rows out
#pragma unroll
    for (int j0 = 0; j0 < B_ROWS; j0 += LPG) {
        const uint32_t j = (uint32_t)(j0 + lane % LPG);
        if ((gb >> j) & 1u)
            sh.list[lane / LPG][mmm_list_pos(LSZ, slot0 + (uint32_t)__popc(gb & ((1u << j) - 1u)))] =
                (uint16_t)mmm_list_entry(LSZ, (uint32_t)seg % (uint32_t)RING * SEG + (uint32_t)(wave * B_ROWS) + j);
    }
    if (!PARTED && wave == 0 && lane % LPG == 0 && group_ok) {
        uint32_t pitch = KBA, at = seg;
        asm volatile("" : "+s"(pitch), "+s"(at));   // (nor made wider in here for all)
        p.bp_cnt[(uint64_t)G * pitch + at] = n;
    }
    uint32_t slots[B_ROWS];
#pragma unroll
    for (int j = 0; j < B_ROWS; ++j) slots[j] = slot0 + (uint32_t)__popc(gb & ((1u << j) - 1u));
    if constexpr (LSZ % 4 == 0) {
        // slot-major rows of 64 or 128 bytes; the slots that fill up the last quad are zero
        constexpr uint32_t ROWB = MMM_GROUP_COLS * ESZ;
        // the segment of the tile's first group; a group's area is at most 2^28 bytes, 2^29 for doubles (K < 2^22), and a tile
        // has 16 groups, 8 of doubles
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(
            p.bp_val + ((uint64_t)(ct * B_GROUPS) * KBA + seg) * (SEG * ROWB), 0, (int)0xf8000000u, 0x00020000);
        const uint32_t mine_at = group_ok ? (uint32_t)(lane / LPG) * KBA * (SEG * ROWB) + (uint32_t)(lane % LPG) * 16u : NO_STORE;
#pragma unroll
        for (int j = 0; j < B_ROWS; ++j)
            __builtin_amdgcn_raw_buffer_store_b128(raw[j], out, (int)(((gb >> j) & 1u) && group_ok ? mine_at + slots[j] * ROWB : NO_STORE), 0, 0);
        if (wave < 3 && n + wave < ((n + 3u) & ~3u) && group_ok)
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{0, 0, 0, 0}, out, (int)(mine_at + (n + wave) * ROWB), 0, 0);
        __syncthreads();
    } else if constexpr (PARTED) {
        // A wave takes a group, a thread eight slots of a column at a time, in the order of mmm_value_pos.  The values are read
        // again, by the list (they are in the L2): kept in registers and turned round in LDS they took three times as long for B
        // as plain floats do (4096^2, p = .2: 30.8 and 24.5 us, part by part and batch by batch; 9.8 plain).
        __syncthreads();   // the lists
        const uint32_t CG = ct * B_GROUPS + (uint32_t)wave;
        const uint32_t n_out = (uint32_t)__builtin_amdgcn_readlane((int)n, wave * LPG);
        if (CG < NG) {
            const uint32_t c = (uint32_t)lane & 15u, s4 = (uint32_t)lane >> 4, swap = (s4 & 1u) << 2;   // (of odd units the halves)
            const bool col_ok = CG * MMM_GROUP_COLS + c < (uint32_t)p.N;
            const char *const ycol = static_cast<const char *>(p.Y) + (CG * MMM_GROUP_COLS + c) * ESZ;
            char *out = p.bp_val + ((uint64_t)CG * KBA + seg) * (SEG * MMM_GROUP_COLS * LSZ) + s4 * (MMM_PARTS * MMM_UNIT_BYTES) + c * 16;
            const uint8_t *const block_rows = sh.bbits[wave * LPG + (c >= 8u ? LPB : 0)];   // of this lane's half of the group, if it is one
            bool wild = false;
#pragma unroll 1
            for (uint32_t slot = MMM_UNIT * s4; slot < n_out; slot += 4 * MMM_UNIT, out += 4 * MMM_PARTS * MMM_UNIT_BYTES) {   // (units past the last are not read)
                auto value = [&](uint32_t entry, uint32_t at) __attribute__((always_inline)) -> uint32_t {
                    const uint32_t k = entry & (SEG - 1u);   // see mmm_list_entry
                    static_assert(MMM_PARTS_PITCH % SEG == 0, "");
                    bool there = at < n_out && col_ok;
                    if (SPLIT) there = there && ((block_rows[k / 8] >> (k % 8)) & 1u);
                    const uint32_t row = ROWS ? (uint32_t)sh.kk[k] : seg * SEG + k;
                    return there ? *reinterpret_cast<const uint32_t *>(ycol + (uint64_t)row * row_bytes) : 0u;
                };
                const u32x4 entries = *reinterpret_cast<const u32x4 *>(&sh.list[wave][slot]);   // the unit's
                uint32_t v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = value(entries[i % 4] >> (i / 4 * 16), slot + ((uint32_t)i ^ swap));
                OutOfRange here;
#pragma unroll
                for (int i = 0; i < 8; ++i) here.see(v[i]);
                const bool odd = ballot64(here.any()) != 0;
#pragma unroll
                for (int q = 0; q < MMM_PARTS; ++q) {
                    u32x4 part;
#pragma unroll
                    for (int i = 0; i < 4; ++i) part[i] = take_part(v[2 * i], v[2 * i + 1]);
                    *reinterpret_cast<u32x4 *>(out + q * MMM_UNIT_BYTES) = part;
                }
                if (odd) {   // seldom: such elements as they are, read once more
                    wild = true;
#pragma unroll 1
                    for (uint32_t i = 0; i < 8; ++i) {
                        const uint32_t at = slot + (i ^ swap), bits = value(sh.list[wave][mmm_list_pos(LSZ, at)], at);
                        if (!out_of_range(bits)) continue;
                        uint16_t *const to = reinterpret_cast<uint16_t *>(out) + i;
                        to[0] = (uint16_t)(bits >> 16);
                        to[MMM_UNIT_BYTES / 2] = (uint16_t)bits;
                        to[MMM_UNIT_BYTES] = MMM_PARTS_RAW;
                    }
                }
            }
            if (lane == 0) p.bp_cnt[(uint64_t)CG * KBA + seg] = n_out | (wild ? 0x80000000u : 0u);
        }
    } else {
        // The occupied rows go to LDS one after another, zeros behind them up to a whole unit, and come out through the
        // transposing read, which yields four slots of a column to a lane: two of them are a lane's part of a unit in the
        // order of mmm_value_pos.  One LDS write per row; put in place element by element it took four, and a workgroup of B was
        // bound by them (512^3, p = .4, bf16: both sides 5.9 -> 5.0 us, 4096^2, p = .2: 23.2 -> 22.4).
        constexpr uint32_t SLOTS = 4 * MMM_UNIT, ROWB = MMM_GROUP_COLS * ESZ;   // taken out at a time; bytes per row
        constexpr int GROUPB = SEG * ROWB + 16;                       // bytes per group (4 banks apart)
        static_assert(B_GROUPS * GROUPB <= (int)sizeof(sh.pack) && B_GROUPS == BUILD_WAVES, "room for the groups, and a wave for each");
        char *const mine = sh.pack + (lane / LPG) * GROUPB + (lane % LPG) * 8;
#pragma unroll
        for (int j = 0; j < B_ROWS; ++j)
            if ((gb >> j) & 1u) *reinterpret_cast<u32x2 *>(mine + slots[j] * ROWB) = u32x2{raw[j].x, raw[j].y};
        if (wave < MMM_UNIT && n + wave < ((n + MMM_UNIT - 1) & ~(MMM_UNIT - 1u))) *reinterpret_cast<u32x2 *>(mine + (n + wave) * ROWB) = u32x2{0, 0};
        __syncthreads();
        const uint32_t CG = ct * B_GROUPS + (uint32_t)wave;   // the group this wave takes out
        if (CG < NG) {
            typedef short shortx4 __attribute__((ext_vector_type(4)));
            typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
            typedef __attribute__((address_space(3))) char lds_char;
            const uint32_t n_out = (uint32_t)__builtin_amdgcn_readlane((int)n, wave * LPG);
            // (four lanes name a slot and four of its columns each: lane c of sixteen gets column c of their four slots)
            const uint32_t unit = (uint32_t)lane >> 4, half = unit * MMM_UNIT + (unit & 1u) * 4u + (((uint32_t)lane >> 2) & 3u);
            lds_char *const in = (lds_char *)sh.pack + wave * GROUPB + (lane & 3) * 8;
            char *const out = p.bp_val + ((uint64_t)CG * KBA + seg) * (SEG * ROWB) + lane * 16;
            for (uint32_t q = 0; q < n_out; q += SLOTS) {
                const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)(in + (q + half) * ROWB)));
                const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)(in + (q + (half ^ 4u)) * ROWB)));
                if (q + unit * MMM_UNIT < n_out) *reinterpret_cast<u32x4 *>(out + q * ROWB) = u32x4{lo.x, lo.y, hi.x, hi.y};   // (units past the last are not read)
            }
        }
    }
    {   // the lists, one word per thread
        const uint32_t LG = ct * B_GROUPS + (uint32_t)wave;
        if (wave < B_GROUPS && LG < NG)
            reinterpret_cast<uint32_t *>(p.bp_list + ((uint64_t)LG * KBA + seg) * SEG)[lane] = reinterpret_cast<const uint32_t *>(sh.list)[threadIdx.x];
    }
    if (ROWS) __syncthreads();   // the shared arrays may be reused
    return live;
}

// ROWS: row-compacted mode (A laid out over the live rows of B; B built over them).
template <typename T, int TEST, int BW, bool ROWS, bool DEEP>
__global__ __launch_bounds__(BUILD_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) void mmm_build_kernel(const BuildParams)
{
    ConstParams &p = *(ConstParams *)__builtin_amdgcn_kernarg_segment_ptr();
    // A word of every cache line of the arguments, so that where they are read they are there: one round trip in front instead of one
    // after another.  (With this, the keep bitmap's load, the rows of B and the stores as they are: 500^3 floats 5.04 -> 4.58 us, 1000^3 5.50 -> 4.97,
    // A of 512 x 8192 bf16 5.84 -> 5.44, where an empty kernel takes 2.75.)
    asm volatile("" ::"s"(p.n_b_wg), "s"(p.X), "s"(p.Y), "s"(p.M), "s"(p.keep_blocks), "s"(p.test.lo1), "s"(p.by_ctiles.mul));
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
            uint32_t live = ~0u;
            for (uint32_t bb = i; bb < p.n_b; bb += p.n_b_wg) {   // ends at the first segment without a live row
                const uint32_t seg = mmm_divided(bb, mmm_divisor{p.by_ctiles.mul, p.by_ctiles.shift});
                if (seg * SEG >= live) break;
                int l = lane;
                asm volatile("" : "+v"(l));   // keeps what depends on the lane from being carried around the loop (it would spill)
                live = scan_b<T, BW, true>(p, seg, bb - seg * p.ctiles, l, wave, sh.b, carry);
            }
            // Zero map rows for the rows that are off, behind the packing, which they would hold up, and from the last workgroup on: that has
            // nothing to pack where few rows are on.  64 rows at a time, whose words are side by side.  (A row to each lane stored words a row apart: 128 x 4096 x 65536
            // bf16, a tenth of the rows on, blocks of 8, both sides 33.5 us, 30.4 so; 128 x 16384 x 32768 31.4 and 29.5.)
            const uint32_t WA = (uint32_t)p.WA, WB = (uint32_t)p.WB;
            for (uint32_t w = p.n_b_wg - 1u - i; w < WA; w += p.n_b_wg) {
                const uint64_t on = row_word(p.rows, w, p.K);
                const uint32_t words = min(64u, (uint32_t)p.K - w * 64u) * WB;
                for (uint32_t q = threadIdx.x; q < words; q += BUILD_THREADS)
                    if (!((on >> mmm_divided(q, mmm_divisor{p.by_wb.mul, p.by_wb.shift})) & 1ull)) p.b_bits[(uint64_t)(w * 64u) * WB + q] = 0;
            }
        } else if (sizeof(T) < 8) {
            const uint32_t seg = mmm_divided(i, mmm_divisor{p.by_ctiles.mul, p.by_ctiles.shift});
            scan_b<T, BW, false>(p, seg, i - seg * p.ctiles, lane, wave, sh.b, carry);
        } else {   // two column tiles
            const uint32_t pairs = (p.ctiles + 1) / 2;
            const uint32_t segment = mmm_divided(i, mmm_divisor{p.by_ctiles.mul, p.by_ctiles.shift});
            const uint32_t ct = (i - segment * pairs) * 2u;
            scan_b<T, BW, false>(p, segment, ct, lane, wave, sh.b, carry);
            if (ct + 1 < p.ctiles) {
                __syncthreads();
                int l = lane;
                asm volatile("" : "+v"(l));
                scan_b<T, BW, false>(p, segment, ct + 1, l, wave, sh.b, carry);
            }
        }
    } else {
        // Row-compacted planes: the runs of columns of workgroups side by side share cache lines, and neighbours on one XCD put them together in its L2
        // (2048 x 1638 of 16384 bf16, both sides: 33.1 -> 31.3 us).  All rows of workgroups numbered through, where the last one has fewer blocks, gave some
        // XCDs most of those: 1563 x 16083, a tenth of the rows on, one block for six, both sides 21.6 -> 17.6 us with each row by itself; without either 19.3.
        const mmm_a_place at = mmm_place_of_a(i, (uint32_t)p.a_units, mmm_divisor{p.by_units.mul, p.by_units.shift}, ROWS && Layout<T>::ESZ % 4 != 0);
        const int64_t bi0 = (int64_t)at.down * p.a_per_wg;
        scan_a<T, TEST, ROWS, DEEP>(p, at.unit, bi0, min(bi0 + p.a_per_wg, p.MBA), lane, wave, sh.a);
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
// (The numbering of the live rows is held against K: they may be asked for before the build that makes it has run.)
// Column-any words of A over k': bit k' of a row is bit kmap[k'] of the row over k.
__global__ __launch_bounds__(256) void mmm_colany_compact_kernel(const uint64_t *a_colany, const uint32_t *kinfo, const uint32_t *kmap,
                                                                 uint64_t *a_colany_c, int64_t MT, int64_t WA, int64_t K)
{
    const int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);   // one wave per word
    if (idx >= MT * WA) return;
    const int64_t t = idx / WA, w = idx % WA, kc = w * 64 + (threadIdx.x & 63);
    bool any = false;
    if (kc < min((int64_t)*kinfo, K)) {
        const uint32_t k = kmap[kc];
        any = k < K && ((a_colany[t * WA + (k >> 6)] >> (k & 63)) & 1ull);
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
    const int64_t kc = bj * MMM_AB_COLS + c, klim = kinfo ? min((int64_t)*kinfo, K) : K;
    if (kinfo && bj * MMM_AB_COLS >= klim) return;
    const int64_t k = kc < klim ? (kinfo ? (int64_t)kmap[kc] : kc) : K;
    uint64_t rows = 0;
    if (k < K)
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
    const char *block = a_img + (size_t)b * (MMM_AB_CAP * Layout<T>::ESZ);
    for (uint64_t m = rows; m != 0; m &= m - 1) {
        const int r = __builtin_ctzll(m);
        uint32_t bits;
        if constexpr (Layout<T>::PARTED) {
            bits = __float_as_uint(mmm_whole_float(block + mmm_img_pos(2, (uint32_t)c, (uint32_t)r), MMM_PART_BYTES));
        } else {
            bits = f32_bits<T>(*reinterpret_cast<const T *>(block + mmm_img_pos(sizeof(T), (uint32_t)c, (uint32_t)r)));
        }
        ent[at++] = make_uint2(mmm_slab_pos((uint32_t)r, (uint32_t)c), bits);
    }
    if (c == 0) a_cnt[b] = total;
    if (total + c < ((total + 63u) & ~63u)) ent[total + c] = make_uint2(MMM_SLAB_SPARE, 0u);
}

// ---- statistics (off the hot path) -----------------------------------------------------------
__global__ void mmm_stats_clear_kernel(uint64_t *stats)
{
    if (threadIdx.x < MMM_STATS_WORDS) stats[threadIdx.x] = 0;
}

// One workgroup per 64 values of k: lane kb of every wave counts column k of A
// over a slice of rows and row k of B over its words.  Of the k that `rows` leaves on (all, if there is none) the number,
// and in how many 64-row tiles each has a non-zero element.
__global__ __launch_bounds__(256) void mmm_stats_kernel(const uint64_t *a_bits, const uint64_t *b_bits, const uint64_t *a_colany,
                                                        const uint64_t *rows, int64_t M, int64_t K, int64_t WA, int64_t WB,
                                                        int64_t MT, int64_t bw, uint64_t *stats)
{
    __shared__ uint32_t col[4 * 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t w = blockIdx.x;
    auto add = [&](int q, uint64_t x) {
        for (int off = 32; off > 0; off >>= 1) x += __shfl_down(x, off, 64);
        if (lane == 0 && x != 0) atomicAdd((unsigned long long *)&stats[q], (unsigned long long)x);
    };
    const uint64_t live = bits_below(rows != nullptr ? rows[w] : ~0ull, K - w * 64);
    uint64_t active = 0;
    for (int64_t t = 2 * (int64_t)threadIdx.x; t < MT; t += 512)
        active += (uint64_t)__popcll((a_colany[t * WA + w] | a_colany[min(t + 1, MT - 1) * WA + w]) & live);
    add(4, active);
    if (wave == 3) add(5, lane == 0 ? (uint64_t)__popcll(live) : 0ull);
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
        for (int q = 0; q < 4; ++q) add(q, v[q]);
    }
}

// Floats that may come in parts: the steps of row tiles of A (stats[6]) and of groups of B (stats[7]) with an element that parts do
// not hold, a wave for each.  In parts as the matrix kernel finds them marked, else from the elements themselves.
template <bool PARTED>
__global__ __launch_bounds__(256) void mmm_marks_kernel(const char *a_img, const uint8_t *a_wild, const char *bp_val, const uint32_t *bp_cnt,
                                                        const uint32_t *kinfo, const uint32_t *kmap, int64_t K, int64_t KBA, int64_t MBA,
                                                        int64_t NG, uint64_t *stats)
{
    __shared__ uint32_t found[2];   // (one atomic per workgroup: one per wave took 100 us where all are marked)
    const int lane = threadIdx.x & 63;
    const int64_t live = kinfo != nullptr ? (int64_t)*kinfo : K;
    if (threadIdx.x < 2) found[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); item < (MBA + NG) * KBA; item += (int64_t)gridDim.x * 4) {
        const bool of_a = item < MBA * KBA;
        const int64_t at = of_a ? item : item - MBA * KBA, ch = at % KBA;
        if (ch * MMM_AB_COLS >= live) continue;
        OutOfRange range;
        auto scan = [&](const char *from, int64_t quads) {
            for (int64_t q = lane; q < quads; q += 64 * 8) {   // (the last one again past the end)
                uint4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = reinterpret_cast<const uint4 *>(from)[min(q + 64 * u, quads - 1)];
#pragma unroll
                for (int u = 0; u < 8; ++u) range.see(v[u].x), range.see(v[u].y), range.see(v[u].z), range.see(v[u].w);
            }
        };
        bool marked = false;
        if (PARTED && of_a) {
            const int64_t k0 = kinfo != nullptr ? kmap[ch * MMM_AB_COLS] : ch * MMM_AB_COLS;
            const int64_t k1 = kinfo != nullptr ? kmap[min((ch + 1) * MMM_AB_COLS, live) - 1] : k0;
            for (int64_t j = k0 / MMM_AB_COLS + lane; j <= k1 / MMM_AB_COLS; j += 64) marked |= a_wild[at - ch + j] != 0;
        } else if (PARTED) {
            marked = (int32_t)bp_cnt[at] < 0;
        } else if (of_a) {   // (columns past the last live one hold anything)
            scan(a_img + at * (MMM_AB_CAP * 4), min(live - ch * MMM_AB_COLS, (int64_t)MMM_AB_COLS) * (MMM_AB_ROWS / 4));
        } else {
            scan(bp_val + at * (SEG * MMM_GROUP_COLS * 4), (int64_t)bp_cnt[at] * (MMM_GROUP_COLS / 4));
        }
        if (ballot64(marked || range.any()) != 0 && lane == 0) atomicAdd(&found[of_a ? 0 : 1], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 2 && found[threadIdx.x] != 0)
        atomicAdd((unsigned long long *)&stats[6 + threadIdx.x], (unsigned long long)found[threadIdx.x]);
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

ElementTest mmm_element_test(int32_t dtype, int32_t pred, float threshold)
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

template <typename T, int TEST, bool ROWS, bool DEEP> static build_kernel_fn build_kernel_width(int32_t bw)
{
    return bw == 8    ? mmm_build_kernel<T, TEST, 8, ROWS, DEEP>
           : bw == 16 ? mmm_build_kernel<T, TEST, 16, ROWS, DEEP>
                      : mmm_build_kernel<T, TEST, 32, ROWS, DEEP>;
}
template <typename T, bool ROWS, bool DEEP> static build_kernel_fn build_kernel_test(int32_t mode, int32_t bw)
{
    return mode == TEST_MAGNITUDE ? build_kernel_width<T, TEST_MAGNITUDE, ROWS, DEEP>(bw)
         : mode == TEST_ONE_RANGE ? build_kernel_width<T, TEST_ONE_RANGE, ROWS, DEEP>(bw)
                                  : build_kernel_width<T, TEST_TWO_RANGES, ROWS, DEEP>(bw);
}
template <typename T> static build_kernel_fn build_kernel_rows(int32_t mode, int32_t bw, bool rows, bool deep)
{
    constexpr bool HALF = sizeof(T) == 2;
    if (deep && HALF) return rows ? build_kernel_test<T, true, HALF>(mode, bw) : build_kernel_test<T, false, HALF>(mode, bw);
    return rows ? build_kernel_test<T, true, false>(mode, bw) : build_kernel_test<T, false, false>(mode, bw);
}
static build_kernel_fn build_kernel(int32_t dtype, int32_t form, int32_t mode, int32_t bw, bool rows, bool deep)
{
    if (form == MMM_FORM_PARTS) return build_kernel_rows<PartedFloat>(mode, bw, rows, deep);
    return dtype == MMM_F64  ? build_kernel_test<double, false, false>(mode, bw)   // no row-compacted mode
         : dtype == MMM_BF16 ? build_kernel_rows<uint16_t>(mode, bw, rows, deep)
         : dtype == MMM_F16  ? build_kernel_rows<_Float16>(mode, bw, rows, deep)
                             : build_kernel_rows<float>(mode, bw, rows, deep);
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
    p.a_wild = m->a_wild;
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
    p.test = mmm_element_test(a.dtype, a.pred, a.threshold);
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
    p.by_units = mmm_make_divisor((uint32_t)p.a_units);
    p.by_ctiles = mmm_make_divisor(f64 ? (p.ctiles + 1) / 2 : p.ctiles);
    p.by_wb = mmm_make_divisor((uint32_t)m->WB);
    const int64_t n_a = a.X ? m->MBA * p.a_units : 0;
    const int64_t n_b = a.Y ? m->KBA * (f64 ? (p.ctiles + 1) / 2 : p.ctiles) : 0;
    // Row-compacted B: how many segments have a live row is known on the device only; at most one workgroup per CU loops
    // over them.
    const int64_t n_b_wg = a.b_compact && n_b > 256 ? 256 : n_b;
    // Blocks of A per workgroup: as many as leave every CU the two workgroups that fit, up to eight, so that one load
    // phase stands in front of several blocks and the others hide behind the stores of the block before (2048 x 16384
    // ReLU: 50.7, 42.1, 38.2 us with one, two, four; a 2048^2 matrix, 512 blocks, wants one: 10.0 against 13.4 with four).
    // Between 512 and 1024 blocks one each leaves a second round of workgroups that is half empty: two each from 600 of
    // them on, where both sides make 704 workgroups or more (one, then two each, floats and 16-bit: 640 blocks of A beside
    // 80 workgroups of B 10.1 -> 9.8 and 8.7 -> 7.6 us, 784 beside 112 12.1 -> 11.2 and 9.6 -> 7.9, 784 of A alone
    // 11.0 -> 10.3 and 8.7 -> 7.6).  With fewer the short second round costs less than two blocks in turn (640 of A alone
    // 8.9 -> 9.2 and 7.2 -> 7.5, 512 beside 64 8.3 -> 8.7 and 7.2 -> 7.3; whole passes over 528 to 575 .98 to 1.01).  Row-compacted
    // ones gain more (896 blocks beside 224 workgroups of B, 16-bit, 10.3 -> 8.7, floats 840 beside 240 11.5 -> 10.5; 28 problems .94 in the mean, 1.00 at worst).
    // Doubles and floats in parts gain beside some workgroups of B and not beside many (doubles, below 200 of them, .97 in the mean, 1.02 at worst, 200 to
    // 320 1.05 and 1.14; in parts, below 400, .97 and 1.04, more 1.01 and 1.05).  Row-compacted blocks in parts, whose second waits at a barrier for the one
    // stage while the first is read column by column, only where the second round was well filled and beside fewer than the 256 workgroups that B has at most
    // (784 to 992 blocks .94 to 1.02, of A alone .84 to .98; 612 to 720 1.00 to 1.055; beside 256 1.015 in the mean).
    int64_t per_wg = n_a / 512;
    per_wg = per_wg < 1 ? 1 : per_wg > 8 ? 8 : per_wg;
    const bool rows_in_parts = a.form == MMM_FORM_PARTS && p.rows != nullptr;
    const int64_t b_below = f64 ? 200 : rows_in_parts ? 256 : a.form == MMM_FORM_PARTS ? 400 : INT64_MAX;
    const bool two = n_a >= (rows_in_parts ? 768 : 600) && n_a + n_b_wg >= 704 && n_b_wg < b_below;
    if (per_wg == 1 && two) per_wg = 2;
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
    hipLaunchKernelGGL(build_kernel(a.dtype, a.form, p.test.mode, m->bw, p.rows != nullptr, per_wg >= 4), grid, block, 0, s, p);
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
                       m->kmap, m->a_colany_c, m->MT, m->WA, m->K);
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
    else if (m->a_form == MMM_FORM_PARTS)
        hipLaunchKernelGGL(mmm_lists_kernel<PartedFloat>, grid, block, 0, s, m->a_img, m->a_bits, kinfo, m->kmap, m->a_cnt, ent, m->M, m->K, m->WA, m->KBA);
    else
        hipLaunchKernelGGL(mmm_lists_kernel<float>, grid, block, 0, s, m->a_img, m->a_bits, kinfo, m->kmap, m->a_cnt, ent, m->M, m->K, m->WA, m->KBA);
    return hipGetLastError();
}

// Per-tile active-k lists (see mmm_debug_k_lists), read back from what the matrix kernel takes: counts and list entries of
// packed B, held against the column-any words.  One wave per (row tile of 64, 16-column group, step of 128 k).
template <typename T>
__global__ __launch_bounds__(64) void mmm_k_lists_kernel(const uint64_t *a_colany, const uint16_t *bp_list, const uint32_t *bp_cnt,
                                                         const uint32_t *kinfo, uint8_t *out, int64_t NG, int64_t WA, int64_t MT,
                                                         int64_t groups, int64_t steps)
{
    constexpr size_t LSZ = Layout<T>::ESZ;
    constexpr int RING = mmm_ring(LSZ);
    const int lane = threadIdx.x;
    const int64_t c = blockIdx.x % steps, G = (blockIdx.x / steps) % groups, t = blockIdx.x / (steps * groups);
    if (kinfo && c * MMM_AB_COLS >= (int64_t)*kinfo) return;
    uint8_t *rec = out + ((t * groups + G) * steps + c) * 132;
    uint32_t n = 0;
    if (G < NG) {
        const uint32_t slots = bp_cnt[G * steps + c] & 0xffu;   // (without the mark of floats in parts)
        for (int h = 0; h < 2; ++h) {
            const uint32_t slot = (uint32_t)(64 * h + lane);
            const uint32_t entry = bp_list[(G * steps + c) * SEG + mmm_list_pos(LSZ, slot)];
            const uint32_t k = mmm_list_entry_k(LSZ, entry, (uint32_t)c % (uint32_t)RING);
            bool in = false;
            if (slot < slots && k < (uint32_t)SEG) {
                const int64_t w = 2 * c + (k >> 6);
                uint64_t any = 0;
                if (w < WA)
                    for (int64_t tt = 2 * t; tt < 2 * t + 2 && tt < MT; ++tt) any |= a_colany[tt * WA + w];
                in = (any >> (k & 63u)) & 1ull;
            }
            const uint64_t m = ballot64(in);
            if (in) rec[4 + n + mbcnt64(m)] = (uint8_t)k;
            n += (uint32_t)__popcll(m);
        }
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
    const auto kernel = m->b_dtype == MMM_F64 ? mmm_k_lists_kernel<double> : m->b_form == MMM_FORM_PARTS ? mmm_k_lists_kernel<PartedFloat> : m->b_dtype == MMM_F32 ? mmm_k_lists_kernel<float> : mmm_k_lists_kernel<uint16_t>;
    hipLaunchKernelGGL(kernel, dim3((uint32_t)wgs), dim3(64), 0, s, m->b_compact ? m->a_colany_c : m->a_colany, m->bp_list, m->bp_cnt,
                       m->b_compact ? m->kinfo : nullptr, out, m->NG, m->WA, m->MT, groups, m->KBA);
    return hipGetLastError();
}

hipError_t mmm_launch_stats(const mmm_maps *m, hipStream_t s)
{
    (void)hipGetLastError();
    hipLaunchKernelGGL(mmm_stats_clear_kernel, dim3(1), dim3(64), 0, s, m->stats);
    hipLaunchKernelGGL(mmm_stats_kernel, dim3((uint32_t)m->WA), dim3(256), 0, s, m->a_bits, m->b_bits, m->a_colany,
                       m->b_compact ? m->rows_copy : nullptr, m->M, m->K, m->WA, m->WB, m->MT, (int64_t)m->bw, m->stats);
    if (mmm_may_part(m, m->a_dtype) && m->b_dtype == MMM_F32 && m->a_form == m->b_form && m->a_compact == m->b_compact) {
        const int64_t items = (m->MBA + m->NG) * m->KBA;
        hipLaunchKernelGGL(m->b_form == MMM_FORM_PARTS ? mmm_marks_kernel<true> : mmm_marks_kernel<false>, dim3((uint32_t)std::min<int64_t>((items + 3) / 4, 2048)),
                           dim3(256), 0, s, m->a_img, m->a_wild, m->bp_val, m->bp_cnt, m->b_compact ? m->kinfo : nullptr, m->kmap, m->K, m->KBA,
                           m->MBA, m->NG, m->stats);
    }
    return hipGetLastError();
}
