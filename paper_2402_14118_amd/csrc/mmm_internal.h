// Internal declarations shared by the host API and the kernel launchers.
// Not part of the public ABI (that is include/mmm.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "mmm.h"

// Division of numbers below 2^31 by one that the host knows: q = n * mul / 2^(31 + shift) with shift = ceil(log2 d) and
// mul = ceil(2^(31 + shift) / d), at most 2^32 - 1: the product exceeds n / d by less than 1 / d.
struct mmm_divisor { uint32_t mul, shift; };
inline mmm_divisor mmm_make_divisor(uint32_t d)
{
    uint32_t shift = 0;
    while (shift < 31 && (1u << shift) < d) ++shift;
    return {(uint32_t)(((1ull << (31 + shift)) + d - 1) / d), shift};
}
__host__ __device__ inline uint32_t mmm_divided(uint32_t n, const mmm_divisor &d) { return (uint32_t)((uint64_t)(n * 2u) * d.mul >> 32) >> d.shift; }

// Which blocks of A the builder's workgroup i takes: `down` of the rows of workgroups, `unit` across.  xcd: units side by side go to one XCD (workgroups are
// dealt out to the eight in turn), each row by itself, since the last one may have fewer blocks.
struct mmm_a_place { uint32_t down, unit; };
__host__ __device__ inline mmm_a_place mmm_place_of_a(uint32_t i, uint32_t units, const mmm_divisor &by_units, bool xcd)
{
    const uint32_t down = mmm_divided(i, by_units), unit = i - down * units;
    return {down, xcd ? (unit & 7u) * (units >> 3) + ((unit & 7u) < (units & 7u) ? unit & 7u : units & 7u) + (unit >> 3) : unit};
}

// Rows of A summarised by one column-any word.
constexpr int MMM_COLANY_ROWS = 32;
// Geometry of the blocks of A: 64 rows x 128 columns, what one step of the matrix kernel keeps in LDS.
constexpr int MMM_AB_ROWS = 64;
constexpr int MMM_AB_COLS = 128;
constexpr int MMM_AB_CAP = MMM_AB_ROWS * MMM_AB_COLS;   // list capacity per block: the worst case
// Lists of the non-zero elements of a block (inspection only, mmm_maps_view_lists): positions as byte
// offsets in a column-major block with 272-byte columns.
constexpr uint32_t MMM_SLAB_COL_BYTES = 272;
__host__ __device__ constexpr uint32_t mmm_slab_pos(uint32_t row, uint32_t col)   // byte offset of element (row, col)
{
    return col * MMM_SLAB_COL_BYTES + (row & 15u) * 16u + (row >> 4) * 4u;
}
constexpr uint32_t MMM_SLAB_SPARE = mmm_slab_pos(0, MMM_AB_COLS);

// What the builder hands to the matrix kernel.
//
// Image of A: [row block of 64][k, padded to whole blocks][64 rows], element type of X, zeros where the
// mask drops an element.  4-byte elements: the rows r, r+16, r+32, r+48 of a column are neighbours, so that
// one 16-byte LDS read yields the operands of all four 16-row tiles for one k, and the 16 lanes of an
// operand read 256 contiguous bytes.  8-byte elements: the same in two halves of a column, rows r, r+16 at
// 16 r and rows r+32, r+48 at 256 + 16 r.  16-bit elements: a block is four planes of 16 rows, [plane][128 columns][16 rows], so that
// the kernel reads the same place of each plane: one address for all row tiles and immediate offsets.  (With whole columns of 64 rows, their units
// rotated with k against bank conflicts, the addresses took 15 vector instructions per batch instead of four: see `turn`.)
constexpr uint32_t MMM_PLANE_ROWS = 16, MMM_PLANE_COL_BYTES = MMM_PLANE_ROWS * 2, MMM_PLANE_BYTES = MMM_AB_COLS * MMM_PLANE_COL_BYTES;
// byte offset of an element inside its block (floats in parts: esz 2, inside the part's)
__host__ __device__ constexpr uint32_t mmm_img_pos(size_t esz, uint32_t col, uint32_t row)
{
    return esz == 8   ? col * 512u + (row >> 5) * 256u + (row & 15u) * 16u + ((row >> 4) & 1u) * 8u
           : esz == 4 ? col * 256u + (row & 15u) * 16u + (row >> 4) * 4u
                      : row / MMM_PLANE_ROWS * MMM_PLANE_BYTES + col * MMM_PLANE_COL_BYTES + row % MMM_PLANE_ROWS * 2u;
}
// Packed B: per group of 16 columns and segment of 128 k the occupied rows, one after another ("slots"),
// at [group][segment][128 slots][16 columns]; the number of slots; and per slot where its column of A
// sits in the kernel's LDS ring of `ring` blocks: column 128 * (segment mod ring) + k, in units of 256 bytes (4- and
// 8-byte elements) or of 32 bytes in a plane (16-bit elements).  Slots past the
// last name the ring's zero column, which stands behind the blocks (16-bit elements: in front of each plane's columns, so that its entry is 0).
// A vector-memory instruction occupies a compute unit for 8 cycles up to 4 bytes per lane and for 16 above, whether
// it loads 8 or 16.  So the entries, and 16-bit values, are stored in the order in which the kernel's lanes take
// them, one load per batch of slots.  s: lane / 16, c: column.
// 4- and 8-byte elements, batches of 16 slots: slot 4u + s is entry u of [s][4]; values slot by slot.  (Floats in lane
// order save the kernel 1 to 2% - 4096^3, p = .4: 431 against 437 us - and cost the builder more, for putting them
// together in LDS: 2048 x 8192 x 2048 with half of B's blocks: 54 against 46 us.)
// 16-bit elements, batches of 32 in four units of eight (see MMM_UNIT), so that the sixteen lanes of a unit behind a list's last slot need
// not read: 8-byte halves of two units per lane, as it was, 4096^3 bf16, p = .05, .1, .2: multiplication 60.6 -> 52.9, 59.9 -> 54.7, 64.0 -> 62.0 us.
constexpr int MMM_GROUP_COLS = 16;
// Blocks in the ring.  16-bit types take four (64 KiB): a step of the kernel is short then, and a block is requested three
// steps before it is needed.  Floats and doubles take two (64, 128 KiB); four floats deep measured no faster (2048^3,
// p = .1: 28.8 against 29.2 us) and leaves no room for a second ring or workgroup.  Floats in parts take three (144 KiB): a batch of their
// lists reaches into the next block (see MMM_UNIT).
constexpr int mmm_ring(size_t esz) { return esz == 2 ? 4 : esz == 6 ? 3 : 2; }
__host__ __device__ constexpr uint32_t mmm_zero_col(int ring) { return (uint32_t)ring * MMM_AB_COLS; }
// Floats in parts.  The other form of float operands: every element as the sum of three bf16 numbers, each the rounded rest of
// what the ones before leave (8 + 8 + 8 significant bits: nothing is lost), which the 16-bit matrix instructions multiply.  Of the
// nine products of two elements the six that are not below 2^-24 of the whole are summed, those of the two first parts in one set
// of accumulators and the others, 2^-8 of them and less, in another, so that the sums round seldom.  2-norm of the error against 64 bits, in parts and of
// the float instruction: 18 problems of 360 to 3800 rows, .05 to .4 and ReLU layers, 24 to 1200 products per sum, 0.4 to 2.1e-7 and 0.7 to 6.1e-7, .31 to
// .60 of it each; half a product to 10 per sum .91 to .47 of it.  Where every sum is one product 1.02 times as large (at worst 1.6
// instead of 1.0 times 2^-24), and with exponents spread over 2^+-20, where the 16-bit instruction cuts the smaller addends
// off, 1.2 times with 4 products and 1.09 with 32.  32 k of a row tile take 6 instructions of 16.7 cycles instead of 8 of 32.6.
// An element outside [2^-110, 2^55) is not held exactly (or its cross products could overflow where the product does not; infinities and NaN are among
// them): its three parts hold its bits instead (MMM_PARTS_RAW), a block of A and a segment of a group of B that have one are marked,
// and are multiplied as floats, put together again (mmm_whole_float).
// Image: [block of 64 x 128][part], parts as blocks of the 16-bit types.  Packed B: batches of 32 slots as of the
// 16-bit types, [unit of slots][part].  As an "element size": 6.
// Slots come in units of eight, as those of the 16-bit types: slot 8u + 4h + e of a segment is value 4h' + e of [u][c][8], entry h' of [4u + e][2], with h' = h in even units and
// 1 - h in odd ones.  A unit is what sixteen lanes of the kernel take, so that a batch can be put together from the units of two segments.  (The
// columns of A that 32 lanes read at once are half a unit of one and half of the next: of a dense list k .. k + 3 and k + 12 .. k + 15, in different LDS
// banks.  That half of the LDS cycles of sparse ones are conflicts does not bound the kernel: dealt out by k mod 8, or without any, no faster.)
constexpr int MMM_UNIT = 8;
constexpr uint32_t MMM_UNIT_BYTES = 256;   // of one part: [16 columns][8]
constexpr int MMM_PARTS = 3;
constexpr size_t MMM_PARTS_ESZ = 2 * MMM_PARTS;
constexpr uint32_t MMM_PARTS_LO = (127 - 110) << 23, MMM_PARTS_HI = (127 + 55) << 23;   // bit patterns of the bounds
constexpr uint32_t MMM_PART_BYTES = MMM_AB_ROWS * MMM_AB_COLS * 2;                      // of a block of A
constexpr uint32_t MMM_BLOCK_PARTS_BYTES = MMM_PARTS * MMM_PART_BYTES;
constexpr uint16_t MMM_PARTS_RAW = 0xffffu;   // as the third part (no rest is a NaN): the first two are the bits of the element as it is
// the element behind three parts `step` bytes from each other
__device__ inline float mmm_whole_float(const char *at, size_t step)
{
    auto part = [&](int q) -> uint32_t { return *reinterpret_cast<const uint16_t *>(at + q * step); };
    const uint32_t p0 = part(0), p1 = part(1), p2 = part(2);
    return p2 == MMM_PARTS_RAW ? __uint_as_float(p0 << 16 | p1) : __uint_as_float(p0 << 16) + (__uint_as_float(p1 << 16) + __uint_as_float(p2 << 16));
}
enum { MMM_FORM_PLAIN = 0, MMM_FORM_PARTS = 1 };
// col: ring column (4- and 8-byte elements: mmm_zero_col for the zero column; 16-bit: a plane's columns, of all blocks of the ring, begin behind it; parts: blocks
// one after another)
constexpr uint32_t MMM_PARTS_PITCH = MMM_BLOCK_PARTS_BYTES / MMM_PLANE_COL_BYTES;   // from a block to the next, in those units
__host__ __device__ constexpr uint32_t mmm_list_entry(size_t esz, uint32_t col)
{
    return esz == 8 ? col * 2 : esz == 4 ? col : esz == MMM_PARTS_ESZ ? col / MMM_AB_COLS * MMM_PARTS_PITCH + col % MMM_AB_COLS : col + 1;
}
// and back, inside its block
__host__ __device__ constexpr uint32_t mmm_list_entry_k(size_t esz, uint32_t entry, uint32_t block_in_ring)
{
    return (esz == 8 ? entry >> 1 : esz == 4 ? entry : esz == MMM_PARTS_ESZ ? entry - block_in_ring * (MMM_PARTS_PITCH - MMM_AB_COLS) : entry - 1) -
           block_in_ring * MMM_AB_COLS;
}
__host__ __device__ constexpr uint32_t mmm_list_pos(size_t esz, uint32_t slot)
{
    return esz % 4 == 0 ? (slot & ~15u) | (slot & 3u) << 2 | ((slot >> 2) & 3u)
                        : (slot & ~7u) | (slot & 3u) << 1 | ((slot >> 2 ^ slot >> 3) & 1u);
}
__host__ __device__ constexpr uint32_t mmm_value_pos(size_t esz, uint32_t slot, uint32_t col)   // in elements
{
    return esz % 4 == 0 ? slot * 16u + col : col * 8u + ((slot & 7u) ^ (slot >> 1 & 4u));   // (the latter inside a unit)
}
// The groups whose lists a wave walks: its own, or the last ones where it stands past the last column (and multiplies nothing).  All
// `width` of them exist: blocks of 32 columns, which go two groups to a wave, make an even number.
__host__ __device__ constexpr int mmm_walked_group(int group, int groups, int width) { return group < groups - width ? group : groups - width; }
// Floats: per 128 k a group lists `all` k, of which `stay` have a non-zero column of A in the tile.  Whether the kernel is
// faster when it makes the lists without the others (see `filtered` there) than with the lists as packed.  A step then costs
// what about 10 listed k cost (half of that where a list serves two groups), and a listed k a quarter more.  Multiplication, plain
// lists and without dead columns, us: 512 x 8192 x 4096, 12.8 listed: 52 and 52, 58 with a tenth, three tenths of the columns on;
// 64 listed: 165 and 102, 134, 165 with .3, .5, .7; 4096^3, 6.4 listed: 93 and 112 with .02; 12.8: 149 and 134, 155 with
// .1, .3; 128: 968 and 452, 866 with .3, .7; 2048 x 16384 x 4096, blocks of 32, 6.4 listed: 171 and 163, 188 with .1, .3.
__host__ __device__ constexpr bool mmm_filter_pays(float all, float stay, int32_t bw)
{
    return all - stay >= 0.22f * all && all - stay >= (bw == 32 ? 5.5f : 10.f);
}
struct mmm_plan {
    int32_t variant;
    int32_t split_k;
    int32_t tiles_m, tiles_n;
    int32_t panel;             // tile columns that are gone through together (see panel_width)
    int32_t filter;            // workgroups look whether to leave the columns that are zero in their tile out (floats)
    int32_t chunks_total;      // ceil(K / KC)
    int32_t chunks_per_split;
    int64_t workgroups;
};
// what a plan was made for, besides the shape
struct mmm_plan_key {
    int64_t dtype, variant, split, stats_version;
    bool b_compact;
    int32_t form;
    bool operator==(const mmm_plan_key &o) const
    {
        return dtype == o.dtype && variant == o.variant && split == o.split && stats_version == o.stats_version && b_compact == o.b_compact && form == o.form;
    }
};

constexpr int MMM_STATS_WORDS = 8;
enum { BT_MADE = 0, BT_MISSING = 1, BT_LAUNCHED = 2 };

// Graphs that hold a captured call of a handle: counted for as long as they, or what has been instantiated from them, exist, which
// may be longer than the handle.
struct mmm_captures {
    std::atomic<int> owners{1};   // the handle and the graphs
    std::atomic<int> graphs{0};
};

struct mmm_maps {
    int64_t M, K, N;
    int32_t bw;
    int64_t NB;        // N / bw
    int64_t WA;        // ceil(K/64): words per row of a_bits, a_colany and bt_bits
    int64_t WB;        // ceil(NB/64): words per row of b_bits
    int64_t MT;        // ceil(M/32): rows of a_colany
    int64_t MBA, KBA;  // blocks of A: ceil(M/64) x ceil(K/128)
    int64_t NG;        // groups of 16 columns: ceil(N/16)
    // device pointers into the caller's workspace
    uint64_t *a_bits;
    uint64_t *a_colany;
    char *a_img;       // image of A (see above)
    uint8_t *a_wild;   // [MBA][KBA] floats in parts: whether the 64 x 128 elements hold one that is out of range
    uint32_t *a_cnt;   // [MBA][KBA] non-zeros per block            (inspection: written by mmm_launch_lists)
    uint64_t *a_ent;   // [MBA*KBA][MMM_AB_CAP] entries {mmm_slab_pos(row, column), value bits}, padded to a
                       // multiple of 64 with {spare cell, 0}       (inspection)
    char *a_img64;     // image of A for double inputs, which have no lists: takes the place of a_ent
    uint64_t *b_bits;
    uint64_t *bt_bits;
    uint64_t *stats;   // MMM_STATS_WORDS
    // Row-compacted mode (B side built with keep_rows): k' numbers the rows keep_rows leaves on, and the
    // matrix kernel walks k' instead of k.
    uint32_t *kinfo;       // [0] = number of live k (device)
    uint32_t *kmap;        // [K]: k' -> k
    uint64_t *rows_copy;   // [WA]: the keep_rows bitmap the B side was built with
    uint64_t *a_colany_c;  // [MT][WA]: column-any words of A over k'   (inspection)
    uint64_t *btc_bits;    // [NB][WA]: the B map transposed, over k'
    // packed B (see above; over k' in row-compacted mode)
    char *bp_val;
    uint16_t *bp_list;
    uint32_t *bp_cnt;
    float *partials;   // split-K partial sums
    size_t partial_bytes;
    bool parts_room;   // the workspace has room for floats in parts
    void *ws;
    size_t ws_bytes;
    // state
    bool a_built, b_built;
    bool b_compact;   // the B side was built in row-compacted mode
    // bt_bits in row-compacted mode: made with the B side, launched by a call that needed them (bt_event is behind that), or
    // neither yet (see ensure_bt)
    mutable std::atomic<int> bt_state;
    mutable std::mutex bt_mutex;
    mutable hipEvent_t bt_event;
    bool build_captured;   // a build of B in row-compacted mode has been captured into a graph
    bool a_compact;   // the image of A was built over k' (for the numbering of the current B side)
    int32_t a_dtype, b_dtype;
    int32_t a_form, b_form;   // MMM_FORM_*: the same of both where both are built, with floats
    // the form every build keeps to while there is a graph with a captured call, which may run between others
    mmm_captures *captures;
    mutable std::atomic<int32_t> form_captured;
    const void *a_src;   // address and leading dimension of the X the A side was built from (identity only)
    int64_t a_src_ld;
    const void *b_src;   // the same of the Y the B side was built from
    int64_t b_src_ld;
    // launch plan fixed for this handle (-1 / 0: none, follow the process-wide options)
    int32_t plan_variant, plan_split, plan_path;
    // what the most recent mmm_maps_stats call counted: the density estimate behind the choice of kernel
    mutable bool stats_a_valid, stats_b_valid;
    mutable uint64_t stats_nnz_a, stats_occ_b, stats_macs, stats_rows_b;   // non-zeros, blocks, surviving products, rows of B with a block
    mutable double stats_marked_a, stats_marked_b;   // share of the steps of a row tile of A and of a group of B that are marked, or would be, in parts
    mutable double stats_active;   // share of the k that are on whose column of A has a non-zero element in a tile of 64 rows
    mutable int64_t stats_version;
    // the launch plan last made: it is made anew when its key changes
    mutable std::mutex plan_mutex;
    mutable bool plan_valid;
    mutable mmm_plan_key plan_key;
    mutable mmm_plan plan;
    mutable double plan_cost;   // estimated microseconds
    // the form last chosen, and for what
    bool form_valid;
    mmm_plan_key form_key;
    int32_t form_path;
    int32_t form_chosen;
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
ElementTest mmm_element_test(int32_t dtype, int32_t pred, float threshold);

struct mmm_build_args {
    // A side (X == nullptr: skip)
    const void *X;
    int64_t ldx;
    int32_t pred;
    float threshold;
    const uint64_t *keep_a;
    // B side (Y == nullptr: skip)
    const void *Y;
    int64_t ldy;
    const uint64_t *keep_rows;
    const uint64_t *keep_blocks;
    int32_t dtype;
    bool a_compact;   // lay A out over the live k (the numbering exists or is made in this call)
    bool b_compact;   // number the live rows (keep_rows given) and pack those
    int32_t form;     // MMM_FORM_*
};

enum { PARTS_NO = 0, PARTS_FIXED = 1, PARTS_OWN = 2 };   // PARTS_FIXED: only where this tile has been fixed
struct mmm_variant_info {
    const char *name;
    int32_t TM, TN, KC, rows, k_ranges;   // rows: rows of C actually computed (64, or 32 for short matrices); k_ranges: ranges of K inside a workgroup
    bool doubles;                         // takes double inputs
    int32_t parts;                        // PARTS_*: whether it takes floats in parts
};

hipError_t mmm_launch_build(const mmm_maps *m, const mmm_build_args &a, hipStream_t s);
// Whether B is packed (and the matrix kernel can run): always but for double inputs of so few rows that the pair kernel
// is what runs, for which the workspace has no room.
inline bool mmm_may_part(const mmm_maps *m, int32_t dtype) { return dtype == MMM_F32 && m->M > 64 && m->parts_room; }
inline bool mmm_packs(int64_t M, int32_t dtype) { return dtype != MMM_F64 || M > 64; }
hipError_t mmm_launch_stats(const mmm_maps *m, hipStream_t s);
// forms that only inspection reads: column-any words over k'; counts and lists of the blocks of A
hipError_t mmm_launch_colany_compact(const mmm_maps *m, hipStream_t s);
// row-compacted mode: bt_bits (over k) from btc_bits (over k')
hipError_t mmm_launch_expand_rows(const mmm_maps *m, hipStream_t s);
hipError_t mmm_launch_lists(const mmm_maps *m, hipStream_t s);
int32_t mmm_variant_count();
const mmm_variant_info &mmm_variant(int32_t i);
// partials / partial_bytes: where the split-K partial sums go (used only when p.split_k > 1)
hipError_t mmm_launch_matmul(const mmm_maps *m, const mmm_plan &p, int32_t dtype, void *C, int64_t ldc, int32_t accumulate, void *partials,
                             size_t partial_bytes, hipStream_t s);
// The multiplication over exactly the surviving products, on the vector ALUs.  fused: evaluate M
// (pred, threshold, keep_a) on X inside the kernel; otherwise a_bits of the maps are used.
hipError_t mmm_launch_pairs(const mmm_maps *m, int32_t dtype, const void *X, int64_t ldx, const void *Y, int64_t ldy,
                            void *C, int64_t ldc, int32_t accumulate, bool fused, int32_t pred, float threshold,
                            const uint64_t *keep_a, hipStream_t s);
// whether that kernel can address a Y of this leading dimension (it forms 32-bit offsets inside 4096 rows)
bool mmm_pairs_supports(int32_t dtype, int64_t ldy);
// the active-k lists of every row tile and column group, written out (need: bytes required)
hipError_t mmm_launch_dump_lists(const mmm_maps *m, uint8_t *out, size_t out_bytes, size_t *need, hipStream_t s);
// device address of the library's own scratch array on the current device (MMM_STATIC_SCRATCH_BYTES bytes)
hipError_t mmm_static_scratch(float **ptr);
