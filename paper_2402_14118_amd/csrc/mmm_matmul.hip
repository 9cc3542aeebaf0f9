// Masked GEMM:  C[i,j] = sum over k with a_bits[i,k] & b_bits[k, j div bw] of X[i,k] * Y[k,j]
// (paper, section 3 "Matrix Multiplication", Fig. "MMM Pseudocode").
//
// How the skipping is mapped onto a 64-lane wavefront.  The paper's conclusion notes that on a GPU all
// lanes of a wave must work on the same pattern of B rows and A elements.  Here the unit a wave owns is a
// 16-column group of C (one B block for bw = 16; two groups that share their list for bw = 32).  The map
// builder has packed, per group and segment of 128 k, the rows of B that are occupied there, with the list
// of their k.  The wave walks that list: it reads the packed rows linearly, picks the matching columns of
// A out of an LDS copy of the 64 x 128 block of A, and feeds both to matrix instructions.  B's block
// sparsity is skipped exactly: no unoccupied block is ever loaded or multiplied; the zeros of A inside the
// 64 rows of a tile are multiplied (A's element sparsity is what the pair kernel exploits), but for floats
// whose columns are zero in the whole tile often enough (see `filtered`).  The iteration is uniform across
// the wave.
//
// A workgroup owns 64 rows of C and keeps a ring of two to four blocks of A in LDS (see mmm_ring), filled by asynchronous
// global-to-LDS loads of the builder's image, whose byte order is the one the operand reads want: no
// registers, no vector instruction and no LDS atomic is spent on A.  One barrier per step of 128 k.
//
// Why the inner loop looks the way it does: an fp32 matrix instruction and a vector instruction do not run
// side by side on a SIMD of this machine (a loop of v_mfma_f32_16x16x4_f32 on one wave and one of integer
// multiply-adds on another take longer together, 709 us, than the sum of their times alone, 231 + 339 us),
// so every vector instruction costs matrix time.  Per quad of four listed k the loop issues one v_perm_b32
// (LDS address of the A operand), one ds_read_b128 (the operands of all four 16-row tiles), one
// buffer_load_dword with an immediate offset (B) and four matrix instructions.  16-bit inputs use
// v_mfma_f32_16x16x32 on 32 listed k, with ds_read_b64_tr_b16 gathering their A operands, two addresses for all row tiles, and one load of 16 bytes per
// lane for B's.
//
// Floats whose lists are long are multiplied in three bf16 parts (FloatParts; see MMM_PARTS in mmm_internal.h and choose_form):
// six 16-bit matrix instructions for 32 listed k take 100 cycles where the eight float instructions take 261.  A block of A
// is half as large again, so the ring leaves room for one workgroup of 16 waves on a compute unit.  4096^3, p = .4: 426 ->
// 310 to 326 us (matrix cores 55 % and LDS 50 % busy, clock 1.9 GHz), p = .2: 240 -> 185.  There a fifth to a quarter of the slots filled up last
// batches; now batches run from one list into the next (see `joined`).  What is left is the clock, and that operands come from LDS as fast as
// the matrix cores take them: all of them read before the first product 366 -> 389 us for the pass, part by part a part ahead 370 -> 370.  Tried
// before, and no faster: copies two steps ahead (167 -> 181 us at p = .1) or the first operands read before the barrier (175); two
// lists per wave in turns, eight waves (237 and 378).
//
// What bounds it otherwise: dense lists, the matrix cores (4096^3 fp32, p = .4: 437 us, of which 360 are matrix instructions at
// the rate a large product reaches); sparse ones, whose steps are one short batch, the compute unit's scalar unit and vector-memory issue,
// which all waves share.  Hence the schedule of `step` below: 4096^3 p = .05 fp32 118 -> 106 us, 2048^3 p = .1
// 29.3 -> 27.6, 512 x 8192 x 4096 bf16 35.1 -> 32.7, against clamped offsets, one request per quad and a count load per step.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "mmm_internal.h"

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int TM = MMM_AB_ROWS;   // rows of C per workgroup = rows of a block of A
constexpr int KC = MMM_AB_COLS;   // k per step = columns of a block of A

struct MatmulParams {
    void *C;    // float, or double for double inputs
    int64_t ldc;
    void *P;    // split-K partial sums, [split][M][N], of C's type
    const char *a_img;
    const char *bp_val;
    const uint16_t *bp_list;
    const uint32_t *bp_cnt;
    const uint32_t *kinfo;   // row-compacted mode: [0] = number of live k (everything above is then over k'); else null
    int64_t M, N;
    int32_t KBA, NG;   // below 2^15 and 2^19: leading dimensions are below 2^22
    int32_t tiles_m, tiles_n, panel, split_k, chunks_total, chunks_per_split;
    int32_t accumulate;
    mmm_divisor by_tiles, by_in_panel, by_panel, by_last_panel, by_split;   // tiles, those of a panel, its columns, those of the last one
    // for the lists without the columns that are zero in the tile (see `filtered`; behind what every kernel reads)
    int32_t bw;
    const uint64_t *bt_bits;    // transposed B map, over k' in row-compacted mode
    const uint64_t *a_colany;   // column-any words of A, over k
    const uint32_t *kmap;       // row-compacted mode: k' -> k
    int64_t NB, WA, MT;
    const uint8_t *a_wild;      // floats in parts: the marks of the blocks of A
};
struct FloatParts { uint16_t part[MMM_PARTS]; };   // element type of floats in parts

typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));
// accumulators of one 16 x 16 tile, and of C
template <typename T> struct Acc { typedef floatx4 tile; typedef float element; };
template <> struct Acc<double> { typedef doublex4 tile; typedef double element; };

// 16-bit inputs are contracted by the matrix instructions of their own type (fp32 accumulate).
template <typename T> struct Mfma16;
template <> struct Mfma16<uint16_t> {   // bf16
    static __device__ __forceinline__ floatx4 k32(u32x4 a, u32x4 b, floatx4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
};
template <> struct Mfma16<FloatParts> : Mfma16<uint16_t> {};
template <> struct Mfma16<_Float16> {
    static __device__ __forceinline__ floatx4 k32(u32x4 a, u32x4 b, floatx4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
    }
};

// Workgroups are dealt round-robin to the 8 XCDs.  Re-number them so that each
// XCD works on a contiguous range of logical tiles: neighbours in that range
// share block rows of A and column tiles of B, which then stay in that XCD's L2.
__device__ __forceinline__ uint32_t xcd_contiguous_id(uint32_t b, uint32_t n)
{
    const uint32_t x = b & 7u, i = b >> 3, q = n >> 3, rem = n & 7u;
    return x * q + (x < rem ? x : rem) + i;
}

typedef __attribute__((address_space(3))) char lds_char;

// N times 64 lanes x 16 bytes from `base` (wave-uniform) + voff to LDS byte offset `lds` (wave-uniform) + 16 * lane, each
// 1 KiB on (the immediate offset moves both addresses).  Written as assembly because the compiler would wait for every
// outstanding one of these before each LDS read.  Each counts as one vector-memory operation of the wave, in order with
// the others (see wait_vmem).
template <int N> __device__ __forceinline__ void copy_to_lds(const char *base, uint32_t voff, uint32_t lds)
{
    static_assert(N <= 3 || N % 2 == 0, "");
    // (m0 is an operand, so that the compiler sets it and knows what it holds; the nop keeps the distance its write needs.)
    if constexpr (N == 1) {
        asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "{m0}"(lds) : "memory");
    } else if constexpr (N == 2) {
        asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024" ::"v"(voff), "s"(base), "{m0}"(lds) : "memory");
    } else if constexpr (N == 3) {
        asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024\n\t"
                     "global_load_lds_dwordx4 %0, %1 offset:2048" ::"v"(voff), "s"(base), "{m0}"(lds) : "memory");
    } else if constexpr (N % 4 != 0) {
        copy_to_lds<N - 2>(base, voff, lds);
        copy_to_lds<2>(base + (N - 2) * 1024, voff, lds + (N - 2) * 1024);
    } else {
#pragma unroll
        for (int i = 0; i < N / 4; ++i)
            asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024\n\t"
                         "global_load_lds_dwordx4 %0, %1 offset:2048\n\tglobal_load_lds_dwordx4 %0, %1 offset:3072" ::"v"(voff),
                         "s"(base + i * 4096), "{m0}"(lds + i * 4096)
                         : "memory");
    }
}
__device__ __forceinline__ uint32_t mbcnt64(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// wait until at most N of the wave's vector-memory operations are outstanding (they complete in order)
template <int N> __device__ __forceinline__ void wait_vmem()
{
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}

// RT  16-row MFMA sub-tiles computed (4: all 64 rows of the block; 2: matrices of at most 32 rows)
// GW  16-column groups per wave (2: bw = 32, the two groups of a block share their list), NW waves per
//     workgroup: TN = 16*GW*NW columns
// KS  groups of NW waves that share the tile and take consecutive ranges of its K (each with a ring of its own); their
//     sums are added in LDS at the end, in order
// FILTER  floats: look whether to leave the columns of A out that are zero in the whole tile (see `filtered`)
template <int RT, int GW, int NW, int KS, typename T, bool FILTER>
__global__ __launch_bounds__(NW * KS * 64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == MMM_PARTS_ESZ ? (NW + 3) / 4 : sizeof(T) == 8 && GW == 2 ? 2 : FILTER && GW == 1 && NW == 16 ? 8 : 4))) void mmm_matmul_kernel(const MatmulParams p)
{
    constexpr bool F64 = sizeof(T) == 8, WIDE = sizeof(T) == 4 || F64;
    constexpr bool PARTED = sizeof(T) == MMM_PARTS_ESZ;
    constexpr int PARTS = PARTED ? MMM_PARTS : 1;
    constexpr int ESZ = (int)sizeof(T);
    typedef typename Acc<T>::tile tile_t;
    typedef typename Acc<T>::element elem_t;
    constexpr int RING = mmm_ring(sizeof(T));
    constexpr int COLB = TM * ESZ;                  // bytes per LDS column
    constexpr int SLAB = KC * COLB;                 // bytes per block of A
    // 16-bit types: the ring is four planes (two where 32 rows are computed), each a zero column and its columns of all blocks (see mmm_img_pos)
    constexpr bool PLANES = ESZ == 2;
    constexpr int PLANE_PITCH = PLANES ? RING * (int)MMM_PLANE_BYTES + (int)MMM_PLANE_COL_BYTES : (int)MMM_PLANE_BYTES;   // (in parts: inside a block's part)
    constexpr int COPIED = PLANES ? RT * (int)MMM_PLANE_BYTES : SLAB;   // bytes of a block that are copied
    constexpr int PLACE_BYTES = PLANES ? (int)MMM_PLANE_BYTES : SLAB;   // from a place of the ring to the next
    constexpr int DMA = COPIED / 1024 / NW;         // copies per wave and block
    constexpr int DMA_PLANES = PLANES && DMA > 4 ? DMA / 4 : 1;   // in so many planes
    constexpr int BATCH = WIDE ? 16 : 32;           // list slots per batch
    constexpr int OPS = WIDE ? 4 * GW + 1 : PARTS * GW + 1;   // vector-memory operations request() makes
    constexpr int SEGB = KC * MMM_GROUP_COLS * ESZ;       // bytes of a packed segment
    static_assert(DMA * NW * 1024 == COPIED && (!PLANES || DMA <= 4 || DMA % 4 == 0), "whole copies, inside a plane");
    typedef elem_t avec __attribute__((ext_vector_type(RT)));   // 4- and 8-byte types: A operands of the RT row tiles for one k

    constexpr int RING_BYTES = RING * SLAB + (PARTED ? 0 : COLB);
    static_assert(!PLANES || TM / 16 * PLANE_PITCH == RING_BYTES, "");
    static_assert(!PARTED || (RT == TM / 16 && KS == 1 && RING == 3), "");
    __shared__ __align__(1024) char rings[KS * RING_BYTES];
    static_assert(!FILTER || ESZ == 4, "");
    __shared__ uint32_t step_marks[PARTED ? 1024 : 1];   // marked steps of this row tile, if there are any: K is below 2^22
    __shared__ __align__(16) uint16_t lists[FILTER ? KS * NW * 2 * KC : 1];   // of `filtered`: [wave][parity of the step][slot]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = KS == 1 ? wave_all : wave_all % NW, ks = KS == 1 ? 0 : wave_all / NW;   // place in the tile, range of K
    const int c = lane & 15, s = lane >> 4;
    char *const ring = rings + ks * RING_BYTES;
    lds_char *const ring3 = (lds_char *)ring;
    const uint32_t ring_off = (uint32_t)(uintptr_t)ring3;

    // What stands in front of the first load is a chain of round trips for arguments and of scalar arithmetic that sixteen waves share one
    // unit for: 2700 cycles of a kernel's 26000 to 50000 (777 x 3001 x 1992 half, 2048^3 floats, p = .1).  So everything the start needs of
    // the arguments is asked for at once (left to itself the compiler asks where it is used: four round trips), divisors come from the host, and
    // products are 32 bits wide where sizes allow it: first barrier 5400 -> 4970 cycles behind the start with the first two.  Passes 35.30 -> 35.06 and 21.23 -> 21.10 us.
    asm volatile("" ::"s"(p.a_img), "s"(p.bp_val), "s"(p.bp_list), "s"(p.bp_cnt), "s"(p.kinfo), "s"(p.KBA), "s"(p.NG), "s"(p.tiles_m), "s"(p.tiles_n),
                 "s"(p.panel), "s"(p.split_k), "s"(p.chunks_total), "s"(p.chunks_per_split), "s"(p.by_tiles.mul), "s"(p.by_tiles.shift), "s"(p.by_in_panel.mul),
                 "s"(p.by_in_panel.shift), "s"(p.by_panel.mul), "s"(p.by_panel.shift), "s"(p.by_last_panel.mul), "s"(p.by_last_panel.shift));

    // Splits of K one after another, the tiles of each in panels of `panel` tile columns (see panel_width).
    // (The number of workgroups is worked out: the launch's own word for it lies behind all arguments, a cache line on.  512 x 8192 x
    // 4096 bf16, the pass: 27.66 -> 27.34 us.)
    const uint32_t tiles = (uint32_t)p.tiles_m * (uint32_t)p.tiles_n;
    const uint32_t L = xcd_contiguous_id(blockIdx.x, tiles * (uint32_t)p.split_k);
    const int split = (int)mmm_divided(L, p.by_tiles);
    const uint32_t t = L - (uint32_t)split * tiles, n0 = mmm_divided(t, p.by_in_panel) * (uint32_t)p.panel;
    const bool last_panel = n0 + (uint32_t)p.panel >= (uint32_t)p.tiles_n;
    const uint32_t width = last_panel ? (uint32_t)p.tiles_n - n0 : (uint32_t)p.panel, u = t - n0 * (uint32_t)p.tiles_m;
    const uint32_t row = mmm_divided(u, last_panel ? p.by_last_panel : p.by_panel);
    const int tile_m = (int)row;
    const int tile_n = (int)(n0 + u - row * width);
    // steps of this workgroup; in row-compacted mode only the steps that hold a live k exist, shared out anew
    int chunks_live = p.chunks_total, per_split = p.chunks_per_split;
    if (p.kinfo != nullptr) {
        chunks_live = (int)((*p.kinfo + (uint32_t)KC - 1) / (uint32_t)KC);
        per_split = (int)mmm_divided((uint32_t)(chunks_live + p.split_k - 1), p.by_split);
    }
    const int wg_begin = min(split * per_split, chunks_live), wg_end = min(wg_begin + per_split, chunks_live);
    const int steps = (int)((uint32_t)(wg_end - wg_begin + KS - 1) / KS);   // barriers of every wave
    const int chunk_begin = min(wg_begin + ks * steps, wg_end);
    const int chunk_end = min(chunk_begin + steps, wg_end);

    tile_t acc[GW][RT];
#pragma unroll
    for (int g = 0; g < GW; ++g)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[g][r] = tile_t{0, 0, 0, 0};
    tile_t rest[PARTED ? GW : 1][RT];   // floats in parts: the products that are not of two first parts
#pragma unroll
    for (int g = 0; g < (PARTED ? GW : 1); ++g)
#pragma unroll
        for (int r = 0; r < RT; ++r) rest[g][r] = tile_t{0, 0, 0, 0};

    // this wave's groups; a wave past the last column walks the last ones' addresses and multiplies nothing
    const int G0 = (tile_n * NW + wave) * GW;
    const bool active = G0 < p.NG;
    const int Gc = mmm_walked_group(G0, p.NG, GW);
    const uint64_t seg0 = (uint64_t)(uint32_t)Gc * (uint32_t)p.KBA;   // the group's first segment
    // Buffer resources: an operand load is then a register of lane offsets, a scalar step offset and an immediate, with
    // no address arithmetic on the vector ALU.  A group's area is below 2^31 bytes (K < 2^22).
    const __amdgpu_buffer_rsrc_t val_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>(p.bp_val) + seg0 * SEGB, 0, GW * p.KBA * SEGB, 0x00020000);
    const __amdgpu_buffer_rsrc_t list_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t *>(p.bp_list) + seg0 * KC, 0, p.KBA * KC * 2, 0x00020000);
    const int val_next = p.KBA * SEGB;   // second group of a 32-wide block (N is a multiple of 32 then)
    const uint32_t *const cnt0 = p.bp_cnt + seg0;

    // ---- A: block ch of this row tile to place ch mod RING (the builder's list entries assume that place)
    const char *src = p.a_img + ((uint64_t)(uint32_t)tile_m * (uint32_t)p.KBA + (uint32_t)chunk_begin) * SLAB;   // the next block to copy
    int to_copy = chunk_end - chunk_begin;                                       // blocks from there on
    uint32_t dma_v = (uint32_t)(wave * DMA * 1024 + lane * 16);
    const uint32_t dma_plane = (uint32_t)(wave * DMA) * 1024u / MMM_PLANE_BYTES;
    const uint32_t place0 = ring_off + (PLANES ? dma_plane * (uint32_t)PLANE_PITCH + MMM_PLANE_COL_BYTES + (uint32_t)(wave * DMA * 1024) % MMM_PLANE_BYTES
                                               : (uint32_t)(wave * DMA * 1024));
    uint32_t place = (uint32_t)chunk_begin % (uint32_t)RING * PLACE_BYTES;
    // (16-bit types, whose turns are bound by their instructions: the place is the block's number, masked, and the source moves on in the lanes' offset)
    uint32_t copy_at = (uint32_t)chunk_begin * MMM_PLANE_BYTES;
    const uint32_t copy_end = (uint32_t)chunk_end * MMM_PLANE_BYTES;
    auto more_to_copy = [&]() __attribute__((always_inline)) { return PLANES ? copy_at < copy_end : to_copy > 0; };
    auto copy_block = [&]() __attribute__((always_inline)) {
        if constexpr (PLANES) {
            static_assert((RING & (RING - 1)) == 0 || !PLANES, "");
            const uint32_t to = place0 + (copy_at & (uint32_t)((RING - 1) * PLACE_BYTES));
            copy_to_lds<DMA / DMA_PLANES>(src, dma_v, to);
            if constexpr (DMA_PLANES > 1) copy_to_lds<DMA / DMA_PLANES>(src + MMM_PLANE_BYTES, dma_v, to + PLANE_PITCH);
            static_assert(DMA_PLANES <= 2, "");
            dma_v += SLAB;
            copy_at += MMM_PLANE_BYTES;
        } else {
            copy_to_lds<DMA>(src, dma_v, place0 + place);
            src += SLAB;
            place = place == (RING - 1) * SLAB ? 0 : place + SLAB;
            --to_copy;
        }
    };

    // ---- B: one batch of a group's list in registers
    struct Batch {
        elem_t bf[WIDE ? GW : 1][4];    // 4- and 8-byte types: slot 4u + s of column c, u = 0..3
        u32x4 bh[WIDE ? 1 : GW][PARTS]; // 16-bit, and of each part of floats in parts: the eight slots of unit s in column c (see MMM_UNIT for their order)
        u32x2 list;                     // 4- and 8-byte types: ring columns of those four slots (16 bits each)
        uint32_t entry;                 // 16-bit, floats in parts: ring positions of the two slots lane % 16 / 4 of unit s (16 bits each)
        uint32_t what;                  // 16-bit, floats in parts: see `plan`
    };
    Batch B0, B1, B2;
    // The batch whose values and entries lie at these byte offsets of the group's area.  Always OPS loads, so that the waits
    // can count them; past the end of the area they return zeros (and are not used).
    auto request = [&](Batch &b, int off_v, int off_l) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");   // the loads of one call stay together and in their place: the waits count them
        if constexpr (WIDE) {
            b.list = __builtin_amdgcn_raw_buffer_load_b64(list_rsrc, s * 8, off_l, 0);
#pragma unroll
            for (int g = 0; g < GW; ++g) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if constexpr (F64)
                        b.bf[g][u] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(val_rsrc, lane * 8 + u * 512, off_v + g * val_next, 0));
                    else
                        b.bf[g][u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(val_rsrc, lane * 4 + u * 256, off_v + g * val_next, 0));
                }
            }
        }
        asm volatile("" ::: "memory");
    };

    const uint32_t c16 = (uint32_t)c * 16u;
    const uint32_t operand_at = ring_off + (uint32_t)(lane & 3) * 8u;   // this lane's four rows of a plane's column
    // 4- and 8-byte types: the operands of four quads, A's at these ring addresses; left: slots of the list from the batch's
    // first on (at least one)
    struct Quads { avec a[WIDE ? 4 : 1]; };
    auto read_quads = [&](const uint32_t (&at)[4], Quads &o) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            auto &a = o.a;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if constexpr (F64) {
                    typedef const __attribute__((address_space(3))) doublex2 lds_doublex2;
                    const doublex2 lo = *(lds_doublex2 *)(ring3 + at[u]);
                    a[u][0] = lo.x;
                    a[u][1] = lo.y;
                    if constexpr (RT == 4) {
                        const doublex2 hi = *(lds_doublex2 *)(ring3 + at[u] + 256);
                        a[u][2] = hi.x;
                        a[u][3] = hi.y;
                    }
                } else {
                    a[u] = *reinterpret_cast<const __attribute__((address_space(3))) avec *>(ring3 + at[u]);
                }
            }
        }
    };
    auto multiply_quads = [&](Quads &o, const elem_t (&bf)[WIDE ? GW : 1][4], int left) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            auto &a = o.a;
            asm volatile("" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]));   // all four requested before the first is used
            auto quad = [&](int u) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < GW; ++g)
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        if constexpr (F64)
                            acc[g][r] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][r], bf[g][u], acc[g][r], 0, 0, 0);
                        else
                            acc[g][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][r], bf[g][u], acc[g][r], 0, 0, 0);
                    }
            };
            quad(0);
            if (left > 4) {
                quad(1);
                if (left > 8) {
                    quad(2);
                    if (left > 12) quad(3);
                }
            }
        }
    };
    auto read = [&](const Batch &b, Quads &o) __attribute__((always_inline)) {   // 4- and 8-byte types: A's operands of a batch
        // ring address of a column: entry * 256 + 16 c, put together from bytes (doubles: columns are 512 bytes and
        // entries count in 256)
        const uint32_t at[4] = {__builtin_amdgcn_perm(b.list.x, c16, 0x0c050400u), __builtin_amdgcn_perm(b.list.x, c16, 0x0c070600u),
                                __builtin_amdgcn_perm(b.list.y, c16, 0x0c050400u), __builtin_amdgcn_perm(b.list.y, c16, 0x0c070600u)};
        read_quads(at, o);
    };
    auto multiply = [&](const Batch &b, int left) __attribute__((always_inline)) {
        if constexpr (WIDE) {
            Quads o;
            read(b, o);
            multiply_quads(o, b.bf, left);
        } else {
            // columns of 32 bytes; the plane of row tile r, and the part, are immediate offsets
            const uint32_t at[2] = {operand_at + (b.entry & 0xffffu) * MMM_PLANE_COL_BYTES, operand_at + (b.entry >> 16) * MMM_PLANE_COL_BYTES};
            auto operand = [&](int q, int h, int r) __attribute__((always_inline)) -> u32x2 {
                typedef __attribute__((address_space(3))) shortx4 lds_shortx4;
                return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4 *)((lds_char *)(uintptr_t)at[h] + (r * PLANE_PITCH + q * (int)MMM_PART_BYTES))));
            };
            // The whole batch whatever its length: slots past the end name the zero column (floats in parts: the block's
            // first) and hold zeros, units past the end come as zeros.  (A branch to a 16-slot instruction for short lists costs more, in moved accumulators,
            // than it saves in LDS reads, and that instruction takes as long.)
            u32x2 a[PARTS][2][RT];
#pragma unroll
            for (int q = 0; q < PARTS; ++q)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int r = 0; r < RT; ++r) a[q][h][r] = operand(q, h, r);
            auto products = [&](int qa, int qb, auto &sum) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int g = 0; g < GW; ++g)
                        sum[g][r] = Mfma16<T>::k32(u32x4{a[qa][0][r].x, a[qa][0][r].y, a[qa][1][r].x, a[qa][1][r].y}, b.bh[g][qb], sum[g][r]);
            };
            products(0, 0, acc);
            if constexpr (PARTED) {
                products(0, 1, rest);
                products(0, 2, rest);
                products(1, 0, rest);
                products(1, 1, rest);
                products(2, 0, rest);
            }
        }
    };

    // ---- One step (4- and 8-byte types): the block in the ring against the n rows listed for it.  A compute unit has one scalar unit for all of
    // its waves, and steps are short (a sparse one is one batch), so what is done per step is kept to about two dozen scalar
    // instructions: offsets and pointers advance by constants, nothing is clamped, the list lengths sit in a register.
    // (With 55 of them a 512 x 8192 x 4096 half-precision multiplication spent 11 of its 31 us on control alone.)
    //
    // b holds the first batch, requested two steps ago, and receives that of the step after the next; B2 holds the second,
    // if there is one, requested at the end of the step before.  Further batches of a long list alternate between the two.
    //
    // The block must have landed.  The wave's share of it was requested RING - 1 steps ago; since then the wave has made at
    // least OPS loads per step, and operations complete in order, so it is enough that all but that many are done.  After
    // the barrier nobody reads the place of the block before any more, and the next copies may go there.
    constexpr int BATCH_V = BATCH * MMM_GROUP_COLS * ESZ, BATCH_L = BATCH * 2, SEG_L = KC * 2;   // bytes
    int off_v = chunk_begin * SEGB, off_l = chunk_begin * SEG_L;   // the current step's segment
    auto step = [&](int n, int n_next, Batch &b) __attribute__((always_inline)) {
        wait_vmem<(RING - 1) * OPS>();
        asm volatile("s_barrier" ::: "memory");
        // Doubles in the widest tile go through the next copy's instructions while the operands are on their way, where the list is long: 2048^3, p = .1,
        // multiplication, 43.8 -> 42.9 us, 6666 x 5547 x 1864, blocks of 8, 455 -> 446.  With a short one the step waits for that copy, which then went out
        // later: with all lists so 2253 x 1036 x 1152, p = .016, 17.5 -> 17.9, in the narrower tile 2626 x 1899 x 384, p = .05, 20.0 -> 22.1, floats 1317 x 5614 x 1776,
        // p = .018, 34.1 -> 38.6 (2048^3, p = .1, 27.7 -> 27.2).  (Two conditions, no else: with a product on both sides of one, the compiler moves accumulators.)
        constexpr bool EARLY = F64 && KS == 1 && NW * GW == 16;
        constexpr int SHORT = 10;
        Quads o;
        if (EARLY && n > SHORT) read(b, o);
        if (more_to_copy()) copy_block();
        if (n > 0) {
            if (!EARLY || n <= SHORT) read(b, o);
            multiply_quads(o, b.bf, n);
            if (n > BATCH) {
                // (Requests inside are unconditional, the last one repeating the batch in hand: a load on one side of a
                // branch would be waited for as if nothing had been requested after the loads before it.)
                const int end = (n - 1) / BATCH;   // the last batch
                for (int i = 1;;) {
                    const int j = min(i + 1, end);
                    request(b, off_v + j * BATCH_V, off_l + j * BATCH_L);
                    multiply(B2, n - i * BATCH);
                    if (++i > end) break;
                    const int k = min(i + 1, end);
                    request(B2, off_v + k * BATCH_V, off_l + k * BATCH_L);
                    multiply(b, n - i * BATCH);
                    if (++i > end) break;
                }
            }
        }
        if (n_next > BATCH) request(B2, off_v + SEGB + BATCH_V, off_l + SEG_L + BATCH_L);
        request(b, off_v + 2 * SEGB, off_l + 2 * SEG_L);
        off_v += SEGB;
        off_l += SEG_L;
    };

    // ---- 16-bit types: the same with the batches of all steps in one queue, requested three ahead
    // whatever steps they belong to.  Above, second batches are requested a step ahead, further ones only when they are next
    // but one, and a list of several costs a request in vain; here none does.  What a turn has to know about its batch (place,
    // slots, whether a step begins with it) stands ready in a lane of `plan`, made 64 batches at a time on the vector ALU, so
    // that a turn takes some 20 scalar instructions; with the same worked out by scalar selects it took 31, and short lists lost
    // what long ones won.
    // 4096^3, p = .4, bf16 multiplication 111 -> 102 us; 512 x 8192 x 4096, bf16,
    // 24.3 -> 23.6, p = .4 38.0 -> 35.4.  4- and 8-byte types keep the steps above: their batches are half as large and mostly
    // one to a step, and the queue's beginning costs more than it gives (4096^3, p = .05, floats 89.5 -> 93.7, 2048^3, p = .1,
    // doubles 43.3 -> 45.2).
    constexpr int PER_STEP = KC / BATCH;   // batches that fit in a segment
    constexpr uint32_t PAST = 1u << 31, FRESH = 1u, BATCH_BYTES = BATCH * MMM_GROUP_COLS * ESZ, PLACE = PAST - BATCH_BYTES;
    static_assert(WIDE || PARTED || (BATCH_BYTES == 1024 && MMM_UNIT * MMM_GROUP_COLS * ESZ == MMM_UNIT_BYTES), "");
    uint32_t plan = 0;                                       // lane j: the j-th of the next batches: PAST the last, FRESH: first of its step, bytes up to it in
                                                             //   the group's area (below 2^27)
    uint32_t ends = 0;                                       // and where its last unit that holds a slot ends there
    int ahead_j = 0;                                         // the one requested last
    auto request_at = [&](Batch &b, uint32_t what, uint32_t end) __attribute__((always_inline)) {
        b.what = what;
        const uint32_t off_v = what & PLACE;
        constexpr uint32_t PER_ENTRY = BATCH_BYTES / (BATCH * 2);
        // The buffers end behind the last unit that holds a slot: lanes of the others get zeros, which as entries name the zero column, and nothing is fetched
        // for them (hidden by a lane offset of their own, two vector instructions in front of the load: 171 x 2775 x 1904, p = .33, 10.2 instead of 9.7 us, 755 x 544
        // live x 2560 9.15 and 8.95).  So a batch without any, of an empty list or behind the last one, needs no branch either.
        const __amdgpu_buffer_rsrc_t entries = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.bp_list) + seg0 * KC, 0, (int)(end / PER_ENTRY), 0x00020000);
        asm volatile("" ::: "memory");   // (as in `request`)
        b.entry = __builtin_amdgcn_raw_buffer_load_b32(entries, (lane >> 2) * 4, (int)(off_v / PER_ENTRY), 0);
#pragma unroll
        for (int g = 0; g < (WIDE ? 0 : GW); ++g) {
            const __amdgpu_buffer_rsrc_t held = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p.bp_val) + seg0 * SEGB, 0, (int)end + g * val_next, 0x00020000);
            b.bh[g][0] = __builtin_amdgcn_raw_buffer_load_b128(held, lane * 16, (int)off_v + g * val_next, 0);
        }
        asm volatile("" ::: "memory");
    };
    auto request_planned = [&](Batch &b, int j) __attribute__((always_inline)) {
        request_at(b, (uint32_t)__builtin_amdgcn_readlane(plan, j), (uint32_t)__builtin_amdgcn_readlane(ends, j));
    };
    // A turn is bound by its instructions, which are a chain that all waves of a workgroup go through between two barriers: one branch and three scalar
    // instructions more cost 80 cycles of 1000 (512 x 8192 x 4096: 19.8 -> 20.9 us), copies that never wait, batches asked for twice as early, one barrier for two
    // steps nothing or less.  Hence planes (4 instead of 15 vector instructions for addresses), no branch around empty lists, blocks copied by their
    // number.  Multiplication, us: 777 x 3001 x 1992 half, blocks of 8, 13.1 -> 12.1, 256 x 8192 x 4096, blocks of 32, p = .2, 17.55 -> 16.95,
    // 512 x 8192 x 4096 19.8 -> 19.5, columns 2048 x 1638 of 16384 x 4096 32.9 -> 32.2; floats in parts, 4096^3, p = .2, 176 -> 169, .4 295 -> 282.
    // (The last one or two turns stand behind the loop: as turns past the end they multiplied zeros.  1472 x 458 x 4832, p = .04, 11.0 -> 10.2 us,
    // 1472 x 128 8.85 -> 8.1, 4096^3, p = .01, 46.4 -> 45.2.  A branch in each turn instead costs what it gives: 4096 x 4096 x 528, p = .4, 25.2 -> 27.1.)
    auto last_turn = [&](Batch &b) __attribute__((always_inline)) {
        if (b.what & FRESH) {
            wait_vmem<0>();
            asm volatile("s_barrier" ::: "memory");
            if (more_to_copy()) copy_block();
        }
        multiply(b, BATCH);
    };
    auto turn = [&](Batch &b) __attribute__((always_inline)) {
        if (b.what & FRESH) {
            wait_vmem<(RING - 1) * OPS>();
            asm volatile("s_barrier" ::: "memory");
            if (more_to_copy()) copy_block();
        }
        multiply(b, BATCH);
        request_planned(b, ++ahead_j);
    };

    // ---- Floats in parts: lists joined.  A batch takes its four units of eight slots (one for each sixteen lanes) from where the one before
    // stopped, out of the lists of two neighbouring steps if need be, so that only units are padded and not batches.  A step whose list is short
    // or empty counts as three units, those past its end empty, and so a batch never reaches further than the next step.  Before a
    // batch that begins in step t there are the barriers of all steps up to t, two at times; behind that of step t block t + 1 has
    // landed too, and block t + 2 is copied to the place of t - 1.  Whole passes, against a list's batches by themselves and a ring of two: 4096^3,
    // p = .4, 382 -> 366 us, p = .2 237.4 -> 230.2, 2048 x 16384 x 4096 ReLU layer with blocks of 32 129.1 -> 122.6, p = .3 with blocks of 8,
    // multiplication, 380 -> 345.
    // Lane j of `plan` holds the j-th of the next batches: END if there is none | barriers before it << BARRIERS | which of its units are
    // EMPTY | four less its units of the first list << REST | units from there to the next segment << JUMP | place of the first unit (below 2^19).
    // The other units follow the first, with the jump behind the first list's.  A batch that is four units of one list - most are where lists are
    // long - is asked for by scalar offsets alone, as plain lists are.
    // The plan is for the 64 next batches where the lengths in hand (of 64 steps) are known to reach so far or to the end, else for JOINED, and new lengths are
    // fetched only where even those would not.  (With a unit in each lane, fetched from there by the lanes it is for, and
    // sixteen batches to a plan, p = .2 gained 1.5 instead of 3 %.)  46 batches always, steps found by six dependent lane reads, lengths fetched for
    // each plan of more than 64 steps and offsets on the vector ALU, before: multiplication 4096^3, p = .4, 305.4 -> 295 us, 512 x 16384 x 2048, p = .3, 69.3 -> 68.0,
    // 1024 x 16384 x 4096, blocks of 32, 232 -> 226.5.
    // Where every list is full, joining gains nothing and costs: 2048 x 16384 x 4096, a tenth of the columns, all blocks of 32 on, 116.4 (a list's batches by themselves),
    // 119.3 (before), 117.7 now, blocks of 16 123.9, 129.1 and 128.0; three quarters of the blocks of 32 on 103.3, 100.4 and 99.0.
    constexpr uint32_t UNITS = KC / MMM_UNIT, JUMP = 19, REST = 23, EMPTY = 15u << 25, BARRIERS = 29, END = 1u << 31, UNIT_PLACE = (1u << JUMP) - 1u;
    constexpr int JOINED = 46;         // batches that the lengths of 64 steps are always enough for: 3 units a step at least
    uint32_t counts = 0, starts = 0;   // lane i: slots listed for step base + i, and units before it (less those of step `base` that are done)
    int base = 0, unit0 = 0, planned = 0;   // unit0: that lane 0 of `plan` begins with; planned: batches in it
    const uint32_t unit_v = (uint32_t)s * (PARTS * MMM_UNIT_BYTES) + c16, unit_l = (uint32_t)lane & 60u;   // a lane's in its unit of four: [s][..]
    auto request_units = [&](Batch &b, uint32_t what) __attribute__((always_inline)) {
        b.what = what;
        const uint32_t place = what & UNIT_PLACE;
        uint32_t at_v = unit_v, at_l = unit_l;   // from the first unit on
        if ((what & (EMPTY | 3u << REST)) != 0) {   // not four units of one list
            const uint32_t jump = what >> JUMP & (UNITS - 1u), first = 4u - (what >> REST & 3u);
            const uint32_t over = unit_l >= first * (MMM_UNIT * 2u) ? jump : 0u;
            at_v += over * (PARTS * MMM_UNIT_BYTES);
            at_l += over * (MMM_UNIT * 2u);
            if (what & EMPTY) {
                // An empty unit's values: past the end of the buffer, which reads as zero; its columns of A are those of another of its
                // batch, since what an empty step's block holds may be no numbers at all.
                const uint32_t empty = (what & EMPTY) / (EMPTY / 15u);
                uint32_t mine = unit_l;
                asm volatile("" : "+v"(mine));   // (nothing of this is kept in registers over the loop)
                const uint32_t off = empty >> (mine >> 4) & 1u;
                at_v |= off << 31;
                at_l = off ? (empty & 1u ? first + jump : 0u) * (MMM_UNIT * 2u) + (mine & 12u) : at_l;
            }
        }
        const int off_v = (int)(place * (PARTS * MMM_UNIT_BYTES)), off_l = (int)(place * (MMM_UNIT * 2u));
        asm volatile("" ::: "memory");   // (as in `request`)
        b.entry = __builtin_amdgcn_raw_buffer_load_b32(list_rsrc, (int)at_l, off_l, 0);
#pragma unroll
        for (int g = 0; g < (PARTED ? GW : 0); ++g)
#pragma unroll
            for (int q = 0; q < PARTS; ++q) b.bh[g][q] = __builtin_amdgcn_raw_buffer_load_b128(val_rsrc, (int)at_v + q * (int)MMM_UNIT_BYTES, off_v + g * val_next, 0);
        asm volatile("" ::: "memory");
    };
    int passed = 1;   // barriers
    auto joined = [&](Batch &b) __attribute__((always_inline)) {
        if (b.what & 3u << BARRIERS) {
            const uint32_t barriers = b.what >> BARRIERS & 3u;
            wait_vmem<OPS>();   // (a request at least came after the copies behind the barrier before)
            asm volatile("s_barrier" ::: "memory");
            if (more_to_copy()) copy_block();
            if (barriers > 1) {
                wait_vmem<0>();
                asm volatile("s_barrier" ::: "memory");
                if (more_to_copy()) copy_block();
            }
            passed += (int)barriers;
        }
        if (~b.what & EMPTY) multiply(b, BATCH);
        request_units(b, (uint32_t)__builtin_amdgcn_readlane(plan, ++ahead_j));
    };

    const int all_steps = WIDE ? (steps + 1) & ~1 : steps;   // steps of `step` and `filtered` go in pairs; the odd one past the end has no list

    // ---- The same for an A whose columns are zero in all rows of the tile here and there (whole columns switched off, by
    // context, for some rows or for all): the k of such columns are left out of the lists.  The wave makes the list of a step
    // itself, one step ahead, from the occupancy of its group and the column-any words of the tile, and picks the rows of
    // packed B by their slots, where the plain list reads them in order.  Nothing of it can be requested more than a step
    // ahead, so a step takes 0.8 to 1.5 us however short its list is; it pays where the plain lists are long (2048 x 16384 x
    // 4096, blocks of 32 all on, a tenth of the columns on in each tile: 1922 -> 348 us, a third of the blocks on 660 -> 212;
    // 512 x 8192 x 4096 265 -> 70; see mmm_filter_pays).  Launched if the counts call for it (see matrix_problem).  Waves need not agree on it: the barriers and copies are the same.
    // Floats only.  16-bit lists are multiplied in little more time than such steps take (2048 x 16384 x 4096 as above: 284 and
    // 171 us with plain lists), doubles have the pair kernel, whose work is the surviving products.
    const int64_t any_row0 = (int64_t)tile_m * (TM / MMM_COLANY_ROWS), any_row1 = min(any_row0 + 1, p.MT - 1);
    const int64_t blk0 = p.bw == 8 ? (int64_t)Gc * 2 : Gc / GW, blk1 = min(p.bw == 8 ? blk0 + 1 : blk0, p.NB - 1);
    auto filtered = [&]() __attribute__((always_inline)) {
        struct Slots {
            elem_t bf[WIDE ? GW : 1][4];
            u32x2 e;   // slots 4u + s, 16 bits each: ring column | the row's place in the segment << 9
        };
        typedef u32x2 __attribute__((may_alias)) list_quad;
        constexpr uint32_t ZERO = mmm_zero_col(RING);   // of slots past the end; no other column has this bit
        static_assert(!FILTER || ZERO == 256, "nine bits");
        uint16_t *const lst = lists + (FILTER ? wave_all * 2 * KC : 0);
        const char *const vals = p.bp_val + seg0 * SEGB;
        typedef const __attribute__((address_space(4))) uint64_t scalar_words;   // (the same for all lanes)
        scalar_words *const occ_row0 = (scalar_words *)(p.bt_bits + blk0 * p.WA), *const occ_row1 = (scalar_words *)(p.bt_bits + blk1 * p.WA);
        scalar_words *const any_of0 = (scalar_words *)(p.a_colany + any_row0 * p.WA), *const any_of1 = (scalar_words *)(p.a_colany + any_row1 * p.WA);
        struct Words { uint64_t occ[2], any[2]; };   // of a step
        auto words_of = [&](int ch) __attribute__((always_inline)) -> Words {
            Words w{{0, 0}, {0, 0}};
            if (active && ch < chunk_end) {
                const int64_t at = 2 * (int64_t)ch, at1 = min(at + 1, p.WA - 1);
                w.occ[0] = occ_row0[at] | occ_row1[at];
                w.occ[1] = occ_row0[at1] | occ_row1[at1];
                w.any[0] = any_of0[at] | any_of1[at];
                w.any[1] = any_of0[at1] | any_of1[at1];
                if (at1 == at) w.occ[1] = 0;
            }
            return w;
        };
        Words next_words = words_of(chunk_begin);
        // the list of step ch, whose words these are, to its half of the wave's list; its length.  Takes the words of the next.
        auto prepare = [&](int ch) __attribute__((always_inline)) -> int {
            const Words w = next_words;
            next_words = words_of(ch + 1);
            uint64_t m[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                m[h] = w.occ[h] & w.any[h];
                if (p.kinfo != nullptr) {   // the column-any words are over k: the step's bits, one by one
                    const uint32_t kc = (uint32_t)(ch * KC + 64 * h + lane);
                    bool any = false;
                    if (kc < *p.kinfo) {
                        const uint32_t k = p.kmap[kc];
                        any = ((p.a_colany[any_row0 * p.WA + (k >> 6)] | p.a_colany[any_row1 * p.WA + (k >> 6)]) >> (k & 63u)) & 1ull;
                    }
                    m[h] = w.occ[h] & __ballot(any);
                }
            }
            const uint32_t n0 = (uint32_t)__popcll(m[0]), n = n0 + (uint32_t)__popcll(m[1]);
            uint16_t *const out = lst + (ch & 1) * KC;
            const uint32_t col = (uint32_t)(ch & (RING - 1)) * KC + (uint32_t)lane;
            if (__builtin_amdgcn_inverse_ballot_w64(m[0])) out[mmm_list_pos(4, mbcnt64(m[0]))] = (uint16_t)(col | mbcnt64(w.occ[0]) << 9);
            if (__builtin_amdgcn_inverse_ballot_w64(m[1]))
                out[mmm_list_pos(4, n0 + mbcnt64(m[1]))] = (uint16_t)((col + 64u) | ((uint32_t)__popcll(w.occ[0]) + mbcnt64(w.occ[1])) << 9);
            if ((uint32_t)lane < (0u - n) % BATCH) out[mmm_list_pos(4, n + (uint32_t)lane)] = (uint16_t)ZERO;
            return (int)n;
        };
        auto fetch = [&](Slots &b, int ch, int batch) __attribute__((always_inline)) {
            b.e = *reinterpret_cast<const list_quad *>(lst + (ch & 1) * KC + batch * BATCH + s * 4);
            uint32_t at[4];   // slots past the end: past the segment's, which reads as zero
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t e = b.e[u >> 1] >> (16 * (u & 1));
                at[u] = ((e & 0xfe00u) >> 3) + ((e & ZERO) << 8) + (uint32_t)c * 4u;
            }
#pragma unroll
            for (int g = 0; g < (WIDE ? GW : 0); ++g) {
                const __amdgpu_buffer_rsrc_t seg = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<char *>(vals) + (int64_t)ch * SEGB + (int64_t)g * val_next, 0, SEGB, 0x00020000);
#pragma unroll
                for (int u = 0; u < 4; ++u) b.bf[g][u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(seg, (int)at[u], 0, 0));
            }
        };
        auto landed = [&](Slots &b) __attribute__((always_inline)) {   // waited for here
#pragma unroll
            for (int g = 0; g < (WIDE ? GW : 0); ++g) asm volatile("" : "+v"(b.bf[g][0]), "+v"(b.bf[g][1]), "+v"(b.bf[g][2]), "+v"(b.bf[g][3]));
        };
        auto multiply_slots = [&](const Slots &b, int left) __attribute__((always_inline)) {
            const uint32_t e0 = b.e.x & 0x01ff01ffu, e1 = b.e.y & 0x01ff01ffu;
            const uint32_t at[4] = {__builtin_amdgcn_perm(e0, c16, 0x0c050400u), __builtin_amdgcn_perm(e0, c16, 0x0c070600u),
                                    __builtin_amdgcn_perm(e1, c16, 0x0c050400u), __builtin_amdgcn_perm(e1, c16, 0x0c070600u)};
            Quads o;
            read_quads(at, o);
            multiply_quads(o, b.bf, left);
        };
        Slots S0{}, S1{}, S2{};
        // b: the first batch of step ch (n slots), next: that of the step after; S2: the second of either
        auto one = [&](int ch, int n, Slots &b, Slots &next) __attribute__((always_inline)) -> int {
            landed(b);
            landed(S2);
            wait_vmem<0>();   // the block too
            asm volatile("s_barrier" ::: "memory");
            const int n_next = prepare(ch + 1);
            const bool early = n <= BATCH;   // S2 is free
            if (n_next > 0) fetch(next, ch + 1, 0);
            if (early && n_next > BATCH) fetch(S2, ch + 1, 1);
            if (more_to_copy()) copy_block();
            if (n > 0) {
                multiply_slots(b, n);
                if (n > BATCH) {
                    multiply_slots(S2, n - BATCH);
                    for (int j = 2; j * BATCH < n; ++j) {
                        fetch(b, ch, j);
                        multiply_slots(b, n - j * BATCH);
                    }
                }
            }
            if (!early && n_next > BATCH) fetch(S2, ch + 1, 1);
            return n_next;
        };
        int n = prepare(chunk_begin);
        if (n > 0) fetch(S0, chunk_begin, 0);
        if (n > BATCH) fetch(S2, chunk_begin, 1);
        for (int i = 0; i < all_steps; i += 2) {
            n = one(chunk_begin + i, n, S0, S1);
            n = one(chunk_begin + i + 1, n, S1, S0);
        }
    };

    if (chunk_begin < chunk_end) {
        // Lane i: length of the list of step i from there on.
        auto lengths = [&](int from) __attribute__((always_inline)) -> uint32_t {
            // (past the last step, and of a wave without columns: past the end of the buffer, which reads as zero)
            const int bytes = active ? max(chunk_end - from, 0) * 4 : 0;
            auto of_group = [&](int g) { return __builtin_amdgcn_raw_buffer_load_b32(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(cnt0) + g * p.KBA + from, 0, bytes, 0x00020000), lane * 4, 0, 0); };
            uint32_t n = of_group(0);
            if (PARTED && GW > 1) n |= of_group(1) & 0x80000000u;   // (the mark of either group)
            return n;
        };
        // Floats in parts: those of the first steps, and whether a block of this row tile is marked, are asked for ahead of the
        // copies, and the first batch too, so that there is one round trip in front of the first step instead of three (4096^3, p = .4: 359 -> 348 us;
        // where two workgroups share a compute unit it makes no difference).
        uint32_t marks = 0, first_lengths = 0;
        if constexpr (!WIDE) {
            first_lengths = lengths(chunk_begin);
            if constexpr (PARTED)
                request_units(B0, (uint32_t)chunk_begin * UNITS | (UNITS - 4u) << JUMP);   // as if the first list had four units
            else
                request_at(B0, (uint32_t)chunk_begin * (PER_STEP * BATCH_BYTES), ((uint32_t)chunk_begin * PER_STEP + 1u) * BATCH_BYTES);
        }
        if constexpr (PARTED) {
            for (int i = lane; i < p.KBA; i += 64) marks |= p.a_wild[(int64_t)tile_m * p.KBA + i];
            asm volatile("" ::: "memory");
        }
#pragma unroll
        for (int i = 0; i < RING - 1; ++i)
            if (more_to_copy()) copy_block();
        if constexpr (PLANES) {
            for (int i = wave * 64 + lane; i < COLB / 4; i += NW * 64)
                reinterpret_cast<uint32_t *>(ring)[i / (int)(MMM_PLANE_COL_BYTES / 4) * (PLANE_PITCH / 4) + i % (int)(MMM_PLANE_COL_BYTES / 4)] = 0;
        } else if constexpr (!PARTED) {   // the ring's zero column (see mmm_list_entry)
            for (int i = wave * 64 + lane; i < COLB / 4; i += NW * 64) reinterpret_cast<uint32_t *>(ring + RING * SLAB)[i] = 0;
        }
        if constexpr (WIDE) {
            request(B0, off_v, off_l);
            request(B1, off_v + SEGB, off_l + SEG_L);
            wait_vmem<2 * OPS>();   // the blocks so far have landed (the waits of the first steps could not count on enough loads)
        }
        if constexpr (!WIDE) asm volatile("" : "+v"(first_lengths));   // waited for here, not earlier
        bool filter = false;
        if constexpr (FILTER) {   // does it pay here?  slots listed in some steps, and those that would stay
            uint32_t all = 0, stay = 0;
            const int ch = chunk_begin + (int)((int64_t)(chunk_end - chunk_begin) * lane / 64);   // a step per lane, from the whole range
            if (active) {
                const int64_t at = 2 * (int64_t)ch;
                const uint64_t occ = p.bt_bits[blk0 * p.WA + at] | p.bt_bits[blk1 * p.WA + at];
                all = (uint32_t)__popcll(occ);
                stay = (uint32_t)__popcll(occ & (p.a_colany[any_row0 * p.WA + at] | p.a_colany[any_row1 * p.WA + at]));
            }
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) {
                all += (uint32_t)__shfl_xor((int)all, d, 64);
                stay += (uint32_t)__shfl_xor((int)stay, d, 64);
            }
            if (p.kinfo != nullptr) {   // (the words are over k: 64 columns of the range instead)
                const uint32_t from = (uint32_t)chunk_begin * KC, count = min(*p.kinfo, (uint32_t)chunk_end * KC) - from;
                const uint32_t k = p.kmap[from + (uint32_t)((uint64_t)count * (uint32_t)lane / 64u)];
                const uint64_t any = p.a_colany[any_row0 * p.WA + (k >> 6)] | p.a_colany[any_row1 * p.WA + (k >> 6)];
                stay = all * (uint32_t)__popcll(__ballot((any >> (k & 63u)) & 1ull)) / 64u;
            }
            filter = __builtin_amdgcn_readfirstlane(mmm_filter_pays((float)all / 32.f, (float)stay / 32.f, p.bw) ? 1 : 0) != 0;   // 64 times 64 k
        }
        if (filter) {
            if constexpr (FILTER) filtered();
        } else {
        // Floats in parts: a step whose block of A or segment of B is marked has no list in the loop below and is done behind it.
        const bool a_marked = PARTED && __ballot(marks != 0) != 0;
        bool some_marked = false;
        if (a_marked) {   // (the same for all waves)
            for (int w = tid; w * 32 < chunk_end - chunk_begin; w += NW * 64) {
                uint32_t bits = 0;
                for (int i = 0; i < 32 && chunk_begin + w * 32 + i < chunk_end; ++i) {
                    const int ch = chunk_begin + w * 32 + i;
                    int64_t k0 = (int64_t)ch * KC, k1 = k0;
                    if (p.kinfo != nullptr) {   // the marks are over k: all blocks the step's columns come from
                        k0 = p.kmap[(int64_t)ch * KC];
                        k1 = p.kmap[min((uint32_t)(ch + 1) * KC, *p.kinfo) - 1u];
                    }
                    for (int64_t j = k0 / KC; j <= k1 / KC; ++j) bits |= p.a_wild[(int64_t)tile_m * p.KBA + j] != 0 ? 1u << i : 0u;
                }
                step_marks[w] = bits;
            }
            __syncthreads();
        }
        if constexpr (WIDE) {
            bool first = true;
            for (int done = 0; done < all_steps; done += 62) {
                uint32_t counts = lengths(chunk_begin + done);
                asm volatile("" : "+v"(counts));   // waited for here
                if (first && (int)__builtin_amdgcn_readlane(counts, 0) > BATCH) request(B2, off_v + BATCH_V, off_l + BATCH_L);
                first = false;
                const int here = min(62, all_steps - done);
                int n = (int)__builtin_amdgcn_readlane(counts, 0);
                for (int i = 0; i < here; i += 2) {
                    const int n1 = (int)__builtin_amdgcn_readlane(counts, i + 1), n2 = (int)__builtin_amdgcn_readlane(counts, i + 2);
                    step(n, n1, B0);
                    step(n1, n2, B1);
                    n = n2;
                }
            }
        } else {
            // (sums, or ors, over the lanes before, in the vector registers)
            auto across = [](uint32_t v, auto op) __attribute__((always_inline)) {
                v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true));    // row_shr 1, 2, 4, 8
                v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true));
                v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true));
                v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true));
                v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast 15, 31
                return op(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
            };
            const auto sum = [](uint32_t a, uint32_t b) { return a + b; };
            if constexpr (PARTED) {
                // lengths n of the steps from `from` on (lane i: step i), `done` units of the first left out
                auto measure = [&](uint32_t n, int from, int done) __attribute__((always_inline)) {
                    if (a_marked && from + lane < steps) n |= step_marks[(from + lane) >> 5] << (31 - ((from + lane) & 31)) & 0x80000000u;
                    some_marked |= __ballot((int)n < 0) != 0;
                    counts = (int)n < 0 ? 0u : n;
                    const uint32_t units = max((counts + MMM_UNIT - 1) / MMM_UNIT, 3u);
                    starts = across(units, sum) - units - (uint32_t)done;
                    base = from;
                };
                // `plan` from unit u on
                auto join = [&](int u) __attribute__((always_inline)) {
                    bool ends = base + 64 >= steps;   // the lengths in hand are all that are left
                    int reach = (int)__builtin_amdgcn_readlane(starts, 62) - u;
                    int before = __popcll(__ballot((int)starts <= u)) - 1;   // the step of unit u
                    if (!ends && reach < 4 * JOINED) {   // lengths of the steps from that one on
                        const int done = u - (int)__builtin_amdgcn_readlane(starts, before);
                        measure(lengths(chunk_begin + base + before), base + before, done);
                        u = before = 0;
                        ends = base + 64 >= steps;
                        reach = (int)__builtin_amdgcn_readlane(starts, 62);
                    }
                    planned = ends || reach >= 4 * 64 ? 64 : JOINED;
                    unit0 = u;
                    const int unit = u + 4 * lane;
                    // The last step that begins no later.  Bit j: a step begins in front of batch j + 1 and behind j, odd and even steps by
                    // themselves, of which there is one at most.
                    const uint32_t at = (uint32_t)((int)starts - u - 1) >> 2, bit = 1u << (at & 31u);   // (steps up to that of u: past the last bit)
                    const auto either = [](uint32_t a, uint32_t b) { return a | b; };
                    auto begins = [&](bool here) __attribute__((always_inline)) -> uint64_t {
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane(across(here && at < 32u ? bit : 0u, either), 63);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane(across(here && at >= 32u && at < 64u ? bit : 0u, either), 63);
                        return (uint64_t)hi << 32 | lo;
                    };
                    const uint64_t even = begins((lane & 1) == 0), odd = begins((lane & 1) != 0);
                    const int i = before + (int)mbcnt64(even) + (int)mbcnt64(odd);
                    const uint32_t begun = (__builtin_amdgcn_inverse_ballot_w64(even << 1) ? 1u : 0u) + (__builtin_amdgcn_inverse_ballot_w64(odd << 1) ? 1u : 0u);
                    const uint32_t k = (uint32_t)(unit - (int)__shfl(starts, i, 64)), here = ((uint32_t)__shfl(counts, i, 64) + 7u) / MMM_UNIT;
                    const uint32_t then = ((uint32_t)__shfl(counts, min(i + 1, 63), 64) + 7u) / MMM_UNIT;
                    // (past the last step the lists are empty, and the last lane's is as long as it says)
                    const uint32_t length = max(here, 3u), first = min(max(length, k + 1u) - k, 4u);
                    const bool ended = base + i >= steps || k >= length;
                    uint32_t filled = (1u << min(here > k ? here - k : 0u, first)) - 1u;
                    if (i < 63) filled |= ((1u << min(then, 4u - first)) - 1u) << first;
                    const uint32_t jump = UNITS - min(k + first, UNITS);
                    plan = ended ? END | EMPTY
                                 : (uint32_t)(chunk_begin + base + i) * UNITS + k | jump << JUMP | (4u - first) << REST | (15u - filled) * (EMPTY / 15u) | begun << BARRIERS;
                    asm volatile("" : "+v"(plan));   // waited for here
                    ahead_j = 0;
                };
                measure(first_lengths, 0, 0);
                join(0);
                const uint32_t begin = (uint32_t)__builtin_amdgcn_readlane(plan, 0);
                if (begin != B0.what) request_units(B0, begin);
                request_units(B1, (uint32_t)__builtin_amdgcn_readlane(plan, 1));
                request_units(B2, (uint32_t)__builtin_amdgcn_readlane(plan, 2));
                ahead_j = 2;
                wait_vmem<2 * OPS>();   // the blocks so far have landed
                asm volatile("s_barrier" ::: "memory");
                if (more_to_copy()) copy_block();
                do {
                    joined(B0);
                    joined(B1);
                    joined(B2);
                    if (ahead_j > planned - 4) join(unit0 + 4 * ahead_j);
                } while ((int)B0.what >= 0);
                for (; passed < steps; ++passed) asm volatile("s_barrier" ::: "memory");   // of the last step, if the last batch begins in the one before
            } else {
                // The next 64 batches, from the lengths n of the steps from `from` on (lane i: step i), `skip` batches of the first
                // left out: lane j finds the step of batch j as the last one that begins no later.
                auto window = [&](uint32_t n, int from, int skip) __attribute__((always_inline)) {
                    const int batches = max(((int)n + BATCH - 1) / BATCH, 1) - (lane == 0 ? skip : 0);
                    const uint32_t begin = across((uint32_t)batches, sum) - (uint32_t)batches;
                    const auto either = [](uint32_t a, uint32_t b) { return a | b; };
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane(across(begin < 32 ? 1u << begin : 0u, either), 63);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane(across(begin >= 32 && begin < 64 ? 1u << (begin - 32) : 0u, either), 63);
                    const uint64_t begun = ((uint64_t)hi << 32 | lo) & (~0ull >> (63 - lane));   // (bit 0 is set)
                    const int i = __popcll(begun) - 1, batch = lane - (63 - __builtin_clzll(begun)) + (i == 0 ? skip : 0);
                    const int left = max(min((int)__shfl(n, i, 64) - batch * BATCH, BATCH), 0);
                    const uint32_t place = ((uint32_t)(chunk_begin + from + i) * PER_STEP + (uint32_t)batch) * BATCH_BYTES;
                    plan = place | (from + i >= all_steps ? PAST : batch == 0 ? FRESH : 0u);
                    ends = place + (uint32_t)(left + MMM_UNIT - 1) / MMM_UNIT * MMM_UNIT_BYTES;   // (behind the last step nothing is left)
                    asm volatile("" : "+v"(plan), "+v"(ends));   // waited for here
                    ahead_j = 0;
                };
                if (!active) {   // a wave past the last column only copies (through `turn` it would multiply too: 4096 x 4096 x 8, p = .3, bf16, 12.8 -> 12.2 us)
                    wait_vmem<0>();
                    asm volatile("s_barrier" ::: "memory");
                    if (more_to_copy()) copy_block();
                    for (int i = 1; i < all_steps; ++i) {
                        if (more_to_copy())
                            wait_vmem<(RING - 2) * DMA>();   // (the two blocks behind this one may be on their way)
                        else
                            wait_vmem<0>();
                        asm volatile("s_barrier" ::: "memory");
                        if (more_to_copy()) copy_block();
                    }
                } else {
                    window(first_lengths, 0, 0);
                    B0.what = (uint32_t)__builtin_amdgcn_readlane(plan, 0) & ~FRESH;   // (begun here)
                    request_planned(B1, 1);
                    request_planned(B2, 2);
                    ahead_j = 2;
                    wait_vmem<2 * OPS>();   // the blocks so far have landed
                    asm volatile("s_barrier" ::: "memory");
                    if (more_to_copy()) copy_block();
                    {   // (asked for as if all of its units held a slot; the entries of the others name the zero column)
                        const bool held = (uint32_t)lane * 16u < (uint32_t)__builtin_amdgcn_readlane(ends, 0) - (B0.what & PLACE);
#pragma unroll
                        for (int g = 0; g < (WIDE ? 0 : GW); ++g) B0.bh[g][0] = held ? B0.bh[g][0] : u32x4{0, 0, 0, 0};
                    }
                    while ((int)B2.what >= 0) {
                        turn(B0);
                        turn(B1);
                        turn(B2);
                        if (ahead_j > 60) {
                            const uint32_t place = (B2.what & PLACE) / BATCH_BYTES;
                            const int step = (int)(place / PER_STEP);
                            window(lengths(step), step - chunk_begin, (int)(place % PER_STEP));
                        }
                    }
                    if ((int)B0.what >= 0) {   // one batch or two are left
                        last_turn(B0);
                        if ((int)B1.what >= 0) last_turn(B1);
                    }
                }
            }
        }
        if constexpr (PARTED) {
            if (some_marked && active) {   // the marked steps, as floats put together again.  Seldom: no more than correct.
#pragma unroll 1
                for (int ch = chunk_begin; ch < chunk_end; ++ch) {
                    uint32_t m = cnt0[ch];
                    const uint32_t n = m & 0xffu;
                    if (GW > 1) m |= cnt0[p.KBA + ch];
                    if (a_marked) m |= step_marks[(ch - chunk_begin) >> 5] << (31 - ((ch - chunk_begin) & 31)) & 0x80000000u;
                    if ((int)m >= 0) continue;
                    const uint16_t *const list = p.bp_list + (seg0 + ch) * KC;
                    const char *const block = p.a_img + ((int64_t)tile_m * p.KBA + ch) * SLAB;   // (rows past M hold zeros)
#pragma unroll 1
                    for (uint32_t i = 0; i < n; i += 4) {
                        const uint32_t slot = min(i + (uint32_t)s, n - 1u);
                        const uint32_t col = mmm_list_entry_k(ESZ, list[mmm_list_pos(ESZ, slot)], (uint32_t)ch % (uint32_t)RING);
                        const bool there = i + (uint32_t)s < n;
                        float a[RT];
#pragma unroll
                        for (int r = 0; r < RT; ++r) {
                            const float v = mmm_whole_float(block + mmm_img_pos(2, col, (uint32_t)(r * 16 + c)), MMM_PART_BYTES);
                            a[r] = there ? v : 0.f;
                        }
#pragma unroll
                        for (int g = 0; g < GW; ++g) {   // (blocks that are off and columns past N hold zeros)
                            const char *const unit = p.bp_val + ((int64_t)(Gc + g) * p.KBA + ch) * SEGB + slot / MMM_UNIT * (PARTS * MMM_UNIT_BYTES);
                            const float v = mmm_whole_float(unit + mmm_value_pos(ESZ, slot, (uint32_t)c) * 2u, MMM_UNIT_BYTES);
                            const float b = there ? v : 0.f;
#pragma unroll
                            for (int r = 0; r < RT; ++r) acc[g][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b, acc[g][r], 0, 0, 0);
                        }
                    }
                }
            }
        }
        }
        if constexpr (PARTED) {
#pragma unroll
            for (int g = 0; g < GW; ++g)
#pragma unroll
                for (int r = 0; r < RT; ++r) acc[g][r] += rest[g][r];
        }
    } else if (KS > 1) {   // no step left for this range of K: only the barriers of the others
        for (int i = 0; i < all_steps; ++i) asm volatile("s_barrier" ::: "memory");
    }
    __syncthreads();   // the rings are free: what follows reuses them
    if constexpr (KS > 1) {   // sums of the later ranges of K, added in order
        tile_t *sums = reinterpret_cast<tile_t *>(rings + RING_BYTES);   // (the first ring is what the layout below uses)
        static_assert((KS - 1) * NW * 64 * GW * RT * (int)sizeof(tile_t) <= (KS - 1) * RING_BYTES, "room for them");
        if (ks > 0)
#pragma unroll
            for (int g = 0; g < GW; ++g)
#pragma unroll
                for (int r = 0; r < RT; ++r) sums[((((ks - 1) * NW + wave) * GW + g) * RT + r) * 64 + lane] = acc[g][r];
        __syncthreads();
        if (ks > 0) return;
#pragma unroll
        for (int q = 0; q < KS - 1; ++q)
#pragma unroll
            for (int g = 0; g < GW; ++g)
#pragma unroll
                for (int r = 0; r < RT; ++r) acc[g][r] += sums[(((q * NW + wave) * GW + g) * RT + r) * 64 + lane];
    }

    // ---- write C (or this split's partial sums): every element exactly once.
    // Accumulator layout of the 16x16 MFMA: lane holds rows 4*s + v (v = 0..3) of column c; doubles: rows s + 4*v.
    // Each wave lays 16 columns of its tile out row-major in its own piece of the (now free) ring, a few row tiles at a
    // time, then stores 64-byte row pieces with 16-byte lanes.
    // (A row of doubles is 128 bytes in 16 lanes as it is.)
    elem_t *out = p.split_k > 1 ? static_cast<elem_t *>(p.P) + (int64_t)split * p.M * p.N : static_cast<elem_t *>(p.C);
    const int64_t ldo = p.split_k > 1 ? p.N : p.ldc, row0 = (int64_t)tile_m * TM;
    const bool add = p.split_k == 1 && p.accumulate;
    constexpr int PIECE = RING * SLAB / NW;   // bytes of the (first) ring per wave
    constexpr int RP = PIECE / 1024 < RT ? PIECE / 1024 : RT;   // row tiles (1 KiB each) laid out at a time
    static_assert(RP >= 1 && RT % RP == 0, "whole passes");
    const bool vec_ok = !F64 && reinterpret_cast<uintptr_t>(out) % 16 == 0 && ldo % 4 == 0;
#pragma unroll
    for (int g = 0; g < GW; ++g) {
        const int64_t col0 = (int64_t)(G0 + g) * 16;
        if (vec_ok && col0 + 16 <= p.N) {
            float *mine = reinterpret_cast<float *>(ring + wave * PIECE);
#pragma unroll
            for (int r0 = 0; r0 < RT; r0 += RP) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();   // the pass before has been read
#pragma unroll
                for (int r = 0; r < RP; ++r)
#pragma unroll
                    for (int v = 0; v < 4; ++v) mine[(r * 16 + s * 4 + v) * 16 + c] = (float)acc[g][r0 + r][v];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int r = 0; r < RP; ++r) {
                    const int64_t row = row0 + (r0 + r) * 16 + (lane >> 2);
                    if (row < p.M) {
                        floatx4 val = *reinterpret_cast<const floatx4 *>(&mine[(r * 16 + (lane >> 2)) * 16 + 4 * (lane & 3)]);
                        floatx4 *dst = reinterpret_cast<floatx4 *>(reinterpret_cast<float *>(out) + row * ldo + col0 + 4 * (lane & 3));
                        if (add) val += *dst;
                        *dst = val;
                    }
                }
            }
        } else {
            const int64_t col = col0 + c;
            if (col >= p.N) continue;
#pragma unroll
            for (int r = 0; r < RT; ++r) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int64_t row = row0 + r * 16 + (F64 ? s + 4 * v : s * 4 + v);
                    if (row >= p.M) continue;
                    elem_t *dst = out + row * ldo + col;
                    *dst = add ? *dst + acc[g][r][v] : acc[g][r][v];
                }
            }
        }
    }
}

// Sum of the split-K partials in a fixed order (split 0, 1, ...), so the result
// does not depend on the order in which workgroups finish.  Bound by latency: a thread takes VEC neighbours of a row, and
// the loads of eight splits are in flight together.
template <typename E, int VEC>
__global__ __launch_bounds__(256) void mmm_splitk_reduce_kernel(const E *P, E *C, int64_t ldc, uint32_t M, uint32_t NV,
                                                                int32_t splits, int32_t accumulate)
{
    typedef E vec __attribute__((ext_vector_type(VEC)));
    typedef vec vec_u __attribute__((aligned(sizeof(E) * VEC)));
    const vec_u *parts = reinterpret_cast<const vec_u *>(P);
    const uint32_t col = blockIdx.x * 256u + threadIdx.x;
    if (col >= NV) return;
    const int64_t total = (int64_t)M * NV;
    for (uint32_t row = blockIdx.y; row < M; row += gridDim.y) {
        const int64_t e = (int64_t)row * NV + col;
        vec sum = parts[e];
        for (int32_t sp = 1; sp < splits; sp += 8) {
            vec v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = sp + i < splits ? parts[(int64_t)(sp + i) * total + e] : vec(0);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (sp + i < splits) sum += v[i];
        }
        vec_u *dst = reinterpret_cast<vec_u *>(C + (int64_t)row * ldc + (int64_t)col * VEC);
        *dst = accumulate ? *dst + sum : sum;
    }
}

template <typename E>
void launch_splitk_reduce(const void *P, void *C, int64_t ldc, int64_t M, int64_t N, int32_t splits, int32_t accumulate, hipStream_t s)
{
    constexpr int VEC = 16 / (int)sizeof(E);   // N is a multiple of 8
    const bool vec = reinterpret_cast<uintptr_t>(C) % 16 == 0 && ldc % VEC == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0;
    const uint32_t NV = (uint32_t)(vec ? N / VEC : N);
    const dim3 grid((NV + 255) / 256, (uint32_t)std::min<int64_t>(M, 65535));
    if (vec)
        hipLaunchKernelGGL((mmm_splitk_reduce_kernel<E, VEC>), grid, dim3(256), 0, s, static_cast<const E *>(P), static_cast<E *>(C), ldc, (uint32_t)M,
                           NV, splits, accumulate);
    else
        hipLaunchKernelGGL((mmm_splitk_reduce_kernel<E, 1>), grid, dim3(256), 0, s, static_cast<const E *>(P), static_cast<E *>(C), ldc, (uint32_t)M,
                           NV, splits, accumulate);
}

typedef void (*matmul_kernel_fn)(const MatmulParams);

struct VariantEntry {
    mmm_variant_info info;
    int32_t waves;              // of 16 columns each; 32-wide blocks: half as many waves of 32 columns
    matmul_kernel_fn fn[2][4];  // [bw == 32][element type]; null: not built
    matmul_kernel_fn filter[2]; // [bw == 32]: floats, without the columns of A that are zero in the tile
    matmul_kernel_fn parts[2];  // [bw == 32]: floats in parts
};

#define MMM_KERNELS(RT, GW, NW, KS)                                                                                       \
    mmm_matmul_kernel<RT, GW, NW, KS, float, false>, mmm_matmul_kernel<RT, GW, NW, KS, uint16_t, false>,                  \
        mmm_matmul_kernel<RT, GW, NW, KS, _Float16, false>
#define MMM_FILTERS(RT, NW, KS) {mmm_matmul_kernel<RT, 1, NW, KS, float, true>, mmm_matmul_kernel<RT, 2, NW / 2, KS, float, true>}
#define MMM_PARTED(RT, NW) {mmm_matmul_kernel<RT, 1, NW, 1, FloatParts, false>, mmm_matmul_kernel<RT, 2, NW / 2, 1, FloatParts, false>}
#define MMM_WHOLE(RT, NW) {nullptr, nullptr}
#define MMM_VARIANT(RT, NW, PARTS, PARTS_KERNELS)                                                                         \
    {                                                                                                                     \
        {"R" #RT "x16_TN" #NW "x16", TM, 16 * NW, KC, 16 * RT, 1, true, PARTS}, NW,                                             \
            {{MMM_KERNELS(RT, 1, NW, 1), mmm_matmul_kernel<RT, 1, NW, 1, double, false>},                                 \
             {MMM_KERNELS(RT, 2, NW / 2, 1), mmm_matmul_kernel<RT, 2, NW / 2, 1, double, false>}},                        \
            MMM_FILTERS(RT, NW, 1), PARTS_KERNELS(RT, NW)                                                                 \
    }
#define MMM_VARIANT_K2(RT, NW) /* two rings: not for doubles and floats in parts */                                                           \
    {                                                                                                                     \
        {"R" #RT "x16_TN" #NW "x16_K2", TM, 16 * NW, KC, 16 * RT, 2, false, PARTS_NO}, NW,                                                 \
            {{MMM_KERNELS(RT, 1, NW, 2), nullptr}, {MMM_KERNELS(RT, 2, NW / 2, 2), nullptr}}, MMM_FILTERS(RT, NW, 2), MMM_WHOLE(RT, NW) \
    }

// Floats in parts have 64 x 256 by themselves; the narrower tiles, which leave a compute unit 8 or 4 waves beside the same ring, where they
// are fixed while the operands are in parts (4096^3, p = .4: 323, 375 and 612 us; 1500 x 2100 x 1024, p_B = .5: 33.5, 29.8 and 49.3).
const VariantEntry g_variants[] = {
    MMM_VARIANT(4, 8, PARTS_FIXED, MMM_PARTED),   // 0: 64 x 128
    MMM_VARIANT(4, 16, PARTS_OWN, MMM_PARTED),     // 1: 64 x 256
    MMM_VARIANT(4, 4, PARTS_FIXED, MMM_PARTED),   // 2: 64 x 64
    MMM_VARIANT(2, 8, PARTS_NO, MMM_WHOLE),       // 3: 32 x 128   (matrices of at most 32 rows)
    MMM_VARIANT_K2(2, 8),   // 4: 32 x 128, K in two ranges
    MMM_VARIANT(2, 4, PARTS_NO, MMM_WHOLE),       // 5: 32 x 64
    MMM_VARIANT_K2(4, 8),   // 6: 64 x 128, K in two ranges
    MMM_VARIANT_K2(4, 4),   // 7: 64 x 64, K in two ranges
};
constexpr int32_t kVariants = (int32_t)(sizeof(g_variants) / sizeof(g_variants[0]));

}   // namespace

// Partial sums of the split-K multiplication for callers that cannot bring (or let the library
// carve out of a workspace) a buffer of their own: one array per GPU, held until the process
// ends.  Host code never uses the array's name as an address: the device address is looked up
// once per device and that pointer is what kernels and copies get.
static __device__ __align__(256) unsigned char scratch[MMM_STATIC_SCRATCH_BYTES];

hipError_t mmm_static_scratch(float **ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices];   // zero-initialised: not looked up yet
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (addr[dev] == nullptr) {   // the current device's own copy of the array
        void *q = nullptr;
        e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (q == nullptr) return hipErrorInvalidSymbol;
        addr[dev] = q;
    }
    *ptr = static_cast<float *>(addr[dev]);
    return hipSuccess;
}

int32_t mmm_variant_count() { return kVariants; }
const mmm_variant_info &mmm_variant(int32_t i) { return g_variants[i].info; }

hipError_t mmm_launch_matmul(const mmm_maps *m, const mmm_plan &pl, int32_t dtype, void *C, int64_t ldc, int32_t accumulate, void *partials,
                             size_t partial_bytes, hipStream_t s)
{
    if (pl.variant < 0 || pl.variant >= kVariants) return hipErrorInvalidValue;
    const VariantEntry &v = g_variants[pl.variant];
    if ((m->M > v.info.rows && v.info.rows < TM) || !mmm_packs(m->M, dtype)) return hipErrorInvalidValue;
    if (pl.workgroups <= 0 || pl.workgroups > 0x7fffffffLL) return hipErrorInvalidValue;   // (ahead of the divisors: products of fewer tiles are 32 bits wide)
    const bool f64 = dtype == MMM_F64;
    MatmulParams p{};
    p.C = C;
    p.ldc = ldc;
    p.P = partials;
    p.a_img = f64 ? m->a_img64 : m->a_img;
    p.bp_val = m->bp_val;
    p.bp_list = m->bp_list;
    p.bp_cnt = m->bp_cnt;
    p.kinfo = m->b_compact ? m->kinfo : nullptr;
    p.bt_bits = m->b_compact ? m->btc_bits : m->bt_bits;
    p.a_colany = m->a_colany;
    p.kmap = m->kmap;
    p.bw = m->bw;
    p.NB = m->NB;
    p.WA = m->WA;
    p.MT = m->MT;
    p.M = m->M;
    p.N = m->N;
    p.KBA = (int32_t)m->KBA;
    p.NG = (int32_t)m->NG;
    p.tiles_m = pl.tiles_m;
    p.tiles_n = pl.tiles_n;
    p.panel = pl.panel;
    p.split_k = pl.split_k;
    p.chunks_total = pl.chunks_total;
    p.chunks_per_split = pl.chunks_per_split;
    p.accumulate = accumulate;
    const uint32_t tiles = (uint32_t)pl.tiles_m * (uint32_t)pl.tiles_n;
    p.by_tiles = mmm_make_divisor(tiles);
    p.by_in_panel = mmm_make_divisor((uint32_t)pl.tiles_m * (uint32_t)pl.panel);
    p.by_panel = mmm_make_divisor((uint32_t)pl.panel);
    p.by_last_panel = mmm_make_divisor((uint32_t)((pl.tiles_n - 1) % pl.panel + 1));
    p.by_split = mmm_make_divisor((uint32_t)pl.split_k);
    if (pl.split_k > 1 && (size_t)pl.split_k * (size_t)m->M * (size_t)m->N * (f64 ? sizeof(double) : sizeof(float)) > partial_bytes)
        return hipErrorInvalidValue;
    const int wide = m->bw == 32 ? 1 : 0;
    const bool parts = m->b_form == MMM_FORM_PARTS;
    if (parts) p.a_wild = m->a_wild;
    matmul_kernel_fn fn = parts ? v.parts[wide] : pl.filter ? v.filter[wide] : v.fn[wide][f64 ? 3 : dtype == MMM_BF16 ? 1 : dtype == MMM_F16 ? 2 : 0];
    if (fn == nullptr) return hipErrorInvalidValue;
    (void)hipGetLastError();   // drop any stale error another library left on this thread
    hipLaunchKernelGGL(fn, dim3((uint32_t)pl.workgroups), dim3((uint32_t)(v.waves >> wide) * (uint32_t)v.info.k_ranges * 64), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (pl.split_k > 1) {
        if (f64)
            launch_splitk_reduce<double>(partials, C, ldc, m->M, m->N, pl.split_k, accumulate, s);
        else
            launch_splitk_reduce<float>(partials, C, ldc, m->M, m->N, pl.split_k, accumulate, s);
        e = hipGetLastError();
    }
    return e;
}
