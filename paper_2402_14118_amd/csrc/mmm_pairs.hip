// Masked GEMM on the vector ALUs, over exactly the surviving products:
//   C[i,j] = sum over k with a_bits[i,k] & b_bits[k, j div bw] of X[i,k] * Y[k,j]
// (paper, section 3 "Random sparsity in A": a zero element of A skips a whole row of B;
// section 3 "Block-Random Sparsity in B": an empty block of B is skipped; Fig. "MMM
// Pseudocode" does both).  No product with a zero element of A or an empty block of B is
// ever formed here, so the work is p_A * p_B of the dense work, and skipped operands cannot
// reach the arithmetic at all.
//
// Mapping onto a 64-lane wavefront.  A wave owns one row i of C and 64 consecutive columns
// = G = 64 / bw blocks of B, lane group g <-> block jb0 + g.  For a range of k the wave
// intersects the bitmap row of A with the transposed B map of each of its blocks (one 64-bit
// AND per 64 values of k, the words spread over the lanes of a group), ranks the survivors with
// a prefix sum inside the group and writes the surviving k of every block into a short list in
// LDS.  Then the G lists are walked side by side.  A lane takes 16 bytes of a row of Y, that is
// C16 = 2, 4 or 8 columns of one entry, so a group covers C16 entries of its list per load, and
// sums for its columns over the entries it has seen; at the end the lanes of a group exchange
// halves of their sums until each holds one column.  The bitmap intersection plays the role of the paper's
// pattern lookup: the branch per element is taken once, on 64 elements at a time.
//
// What bounds it.  Many waves: vector-memory issue, which a compute unit's waves share and which costs 8 cycles per
// instruction up to 4 bytes per lane and 16 above, so one element of one column per lane and load was eight
// times as many instructions as there had to be (maps built, 64 x 4096 x 2048 half precision: 11.8 -> 6.6 us); then the vector ALUs,
// which write the lists and widen 16-bit elements (32 x 16384 x 4096 bf16: 384 instructions per wave, more than half of 10.7 us).
// Few waves: the chain of memory round trips.  There is no staging and no workgroup barrier on the path that takes the map of A as built; the map
// words of the next range are requested before the lists of this one are walked, and the operands of up to four loads
// per lane are in flight together.  Waves of a workgroup that share a column span split K
// between them and add their partial sums in a fixed order at the end.
//
// The matrix-instruction kernel multiplies every listed row of B with all 64 rows of a tile of
// A, zeros included; this kernel pays two gathers per product instead.  It needs only the two
// bitmaps, not the blocked lists of A.  With FUSED the mask M is evaluated right here (eight elements per lane and
// trip: their bits are a byte of the row's bitmap in LDS), so no A-side map
// pass is needed.
#include <type_traits>

#include "mmm_internal.h"

namespace {

constexpr int MAX_WAVE_WORDS = 64;  // map words (64 k each) one wave intersects at a time, at most: 4096 values of k
constexpr int LIST_SLOTS = 1024;    // list entries per wave, shared by its G lists
constexpr int SUPER_WORDS = 1024;   // FUSED: bitmap words of the row kept in LDS at a time (65536 values of k)

struct PairsParams {
    const void *X;
    int64_t ldx;
    const void *Y;
    int64_t ldy;
    void *C;                  // float, or double for double inputs
    int64_t ldc;
    const uint64_t *a_bits;   // M x WA words (not FUSED)
    const uint64_t *keep_a;   // FUSED: optional keep bitmap of M, M x WA words
    const uint64_t *bt_bits;  // NB x WA words
    int64_t M, K, N, NB, WA;
    ElementTest test;         // FUSED: the predicate
    int32_t accumulate;
    mmm_divisor by_m;
    uint32_t workgroups;
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));

// 16 bytes of a row, which starts at any element
template <int ESZ> struct Row16;
template <> struct Row16<2> { typedef u32x4 type __attribute__((aligned(2), may_alias)); };
template <> struct Row16<4> { typedef u32x4 type __attribute__((aligned(4), may_alias)); };
template <> struct Row16<8> { typedef u32x4 type __attribute__((aligned(8), may_alias)); };

__device__ __forceinline__ float fma_acc(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_acc(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Per element type: the type products are accumulated in (float; double for double inputs), the exact widening of an
// element to it, and of the elements of 16 bytes; the bit pattern the predicate is decided on (as in the map builder).
template <typename T> struct Elem;
template <> struct Elem<float> {
    typedef float acc;
    typedef uint32_t pattern;
    static __device__ __forceinline__ acc value(float v) { return v; }
    static __device__ __forceinline__ void unpack(u32x4 v, acc *out)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = __uint_as_float(v[i]);
    }
};
template <> struct Elem<uint16_t> {   // bf16
    typedef float acc;
    typedef uint32_t pattern;
    static __device__ __forceinline__ acc value(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
    static __device__ __forceinline__ void unpack(u32x4 v, acc *out)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(v[i] << 16);
            out[2 * i + 1] = __uint_as_float(v[i] & 0xffff0000u);
        }
    }
};
template <> struct Elem<_Float16> {
    typedef float acc;
    typedef uint32_t pattern;
    static __device__ __forceinline__ acc value(_Float16 v) { return (float)v; }
    static __device__ __forceinline__ void unpack(u32x4 v, acc *out)
    {
        typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
        const halfx8 x = __builtin_bit_cast(halfx8, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = (float)x[i];
    }
};
template <> struct Elem<double> {
    typedef double acc;
    typedef uint64_t pattern;
    static __device__ __forceinline__ acc value(double v) { return v; }
    static __device__ __forceinline__ void unpack(u32x4 v, acc *out)
    {
        const doublex2 x = __builtin_bit_cast(doublex2, v);
        out[0] = x.x;
        out[1] = x.y;
    }
};

__device__ __forceinline__ uint32_t pairs_xcd_id(uint32_t b, uint32_t n)
{
    const uint32_t x = b & 7u, i = b >> 3, q = n >> 3, rem = n & 7u;
    return x * q + (x < rem ? x : rem) + i;
}

// CW: waves side by side (64 columns each); KS: waves that share a column span and take the
// 4096-wide ranges of k in turn (their partial sums are added in a fixed order at the end).
// WAVE_WORDS: map words one wave intersects at a time (a range of 64 * WAVE_WORDS values of k).
template <typename T, int BW, int CW, int KS, int WAVE_WORDS, bool FUSED>
__global__ __launch_bounds__(CW *KS * 64) __attribute__((amdgpu_waves_per_eu(FUSED ? 4 : 8, 8))) void mmm_pairs_kernel(const PairsParams p)
{
    static_assert(WAVE_WORDS <= MAX_WAVE_WORDS && WAVE_WORDS % BW == 0, "whole words per lane, offsets fit the lists");
    constexpr int NW = CW * KS;
    constexpr int G = 64 / BW;                 // blocks (lists) per wave
    constexpr int CAP = LIST_SLOTS / G;        // entries per list and pass
    constexpr int WPL = WAVE_WORDS / BW;       // words per lane and range
    constexpr uint32_t ESZ = (uint32_t)sizeof(T);
    constexpr int C16 = 16 / (int)ESZ;         // columns per lane = entries of a list per load
    constexpr int LPR = BW / C16;              // lanes per entry
    typedef typename Elem<T>::acc acc_t;
    typedef typename Elem<T>::pattern pattern;
    typedef typename Row16<(int)ESZ>::type row16;

    __shared__ __align__(8) uint8_t aw[FUSED ? SUPER_WORDS * 8 : 8];   // FUSED: bitmap of the row
    __shared__ __align__(16) uint16_t lists[NW][LIST_SLOTS];
    __shared__ acc_t red[KS > 1 ? (KS - 1) * CW * 64 : 1];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cw = wave % CW, ks = wave / CW;
    const int g = lane / BW, c = lane % BW;
    const int entry = c / LPR, part = c % LPR;   // of a load: which entry of the list, which 16 bytes of its block

    // Consecutive workgroups of one XCD work on consecutive rows of the same column span, so the
    // blocks of Y and the map words of that span stay in that XCD's L2.
    // (All waves of a compute unit share its scalar unit, and what they work out up to the first load stands in front of everything else: 32-bit
    // arithmetic where the sizes allow it - leading dimensions are below 2^22, so K and N are too -, the divisor from the host, and the
    // arguments asked for at once.)
    asm volatile("" ::"s"(p.X), "s"(p.ldx), "s"(p.ldy), "s"(p.a_bits), "s"(p.keep_a), "s"(p.bt_bits), "s"(p.K), "s"(p.N), "s"(p.NB), "s"(p.WA), "s"(p.by_m.mul), "s"(p.by_m.shift),
                 "s"(p.workgroups));
    if constexpr (FUSED) asm volatile("" ::"s"(p.test.mode), "s"(p.test.lo1), "s"(p.test.len1), "s"(p.test.lo2), "s"(p.test.len2));
    const uint32_t L = pairs_xcd_id(blockIdx.x, p.workgroups);
    const uint32_t ct = mmm_divided(L, p.by_m);
    const uint32_t row_i = L - ct * (uint32_t)p.M;
    const uint32_t col0 = (ct * CW + (uint32_t)cw) * 64u, NB = (uint32_t)p.NB, WA = (uint32_t)p.WA;
    const bool blk_ok = col0 / BW + (uint32_t)g < NB;   // this lane group's block column

    const T *Xrow = static_cast<const T *>(p.X) + (uint64_t)row_i * (uint32_t)p.ldx;
    // the map row of A; the map rows of the wave's blocks (K is below 2^22: a row is at most 2^19 bytes)
    const __amdgpu_buffer_rsrc_t ab = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(p.a_bits + (uint64_t)row_i * WA), 0, (int)(WA * 8u), 0x00020000);
    const uint32_t jb0 = min(col0 / BW, NB - 1u);
    const __amdgpu_buffer_rsrc_t bt = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint64_t *>(p.bt_bits + (uint64_t)jb0 * WA), 0,
                                                                        (int)(min(NB - jb0, (uint32_t)G) * WA * 8u), 0x00020000);
    const uint32_t bt_row = blk_ok ? (uint32_t)g * WA * 8u : 0x40000000u;   // past the end: reads as zero
    const uint32_t ldyb = (uint32_t)p.ldy * ESZ;
    const uint32_t ldy = (uint32_t)p.ldy;   // below 2^22: a 24-bit multiplier
    // first column of the wave (wave-uniform); a lane adds a 32-bit offset to it
    const char *Ycol = static_cast<const char *>(p.Y) + min(col0, (uint32_t)p.N - (uint32_t)BW) * ESZ;
    const uint32_t lane_off = blk_ok ? (uint32_t)(g * BW + part * C16) * ESZ : 0u;
    uint16_t *lst = &lists[wave][g * CAP];
    acc_t acc[C16];
#pragma unroll
    for (int q = 0; q < C16; ++q) acc[q] = 0;

    for (int sw0 = 0; sw0 < (int)WA; sw0 += SUPER_WORDS) {   // one trip unless FUSED and K > 65536
        const int sw = min(SUPER_WORDS, (int)WA - sw0);
        // This lane's map words of the range that starts at word rw0 of the trip: rw0 + c, rw0 + c + BW, ...  Past the end
        // of the row of A words read as zero, so what is read of the B map there does not matter.
        uint64_t wa[WPL], wb[WPL];
        auto fetch = [&](int rw0) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < WPL; ++j) {
                const uint32_t at = (uint32_t)(sw0 + rw0 + c + j * BW) * 8u;
                const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(bt, (int)(at + bt_row), 0, 0);
                wb[j] = (uint64_t)b.y << 32 | b.x;
                if (!FUSED) {
                    const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(ab, (int)at, 0, 0);
                    wa[j] = (uint64_t)a.y << 32 | a.x;
                }
            }
        };
        if constexpr (FUSED) {
            // Eight elements per lane: a byte of the bitmap.  The last, short one is read from K - 8 on and shifted.
            const T *xs = Xrow + (uint32_t)sw0 * 64u;
            const int left = min(SUPER_WORDS * 64, (int)p.K - sw0 * 64);   // elements of the trip
            // the row's keep bits, or without any (a row of the map of B, and) bits that keep all: a load on one side of a branch would be waited for there
            const uint8_t *const keep = reinterpret_cast<const uint8_t *>((p.keep_a != nullptr ? p.keep_a + (uint64_t)row_i * WA : p.bt_bits) + sw0);
            const uint32_t keep_all = p.keep_a != nullptr ? 0u : 0xffu;
            const pattern mask = p.test.mode == TEST_MAGNITUDE ? (pattern)(~(pattern)0 >> 1 >> (ESZ == 2 ? 16 : 0)) : ~(pattern)0;
            auto bits_of = [&](const u32x4 *v) -> uint32_t {
                uint32_t bits = 0;
#pragma unroll
                for (int q = 7; q >= 0; --q) {
                    pattern u;
                    if constexpr (ESZ == 2)
                        u = q & 1 ? v[0][q / 2] >> 16 : v[0][q / 2] & 0xffffu;
                    else if constexpr (ESZ == 4)
                        u = v[q / 4][q % 4];
                    else
                        u = (uint64_t)v[q / 2][(q & 1) * 2 + 1] << 32 | v[q / 2][(q & 1) * 2];
                    u &= mask;
                    bool in = u - (pattern)p.test.lo1 < (pattern)p.test.len1;
                    in |= u - (pattern)p.test.lo2 < (pattern)p.test.len2;
                    bits = bits * 2 + (in ? 1u : 0u);
                }
                return bits;
            };
            constexpr int V = 8 / C16;   // 16-byte pieces of eight elements
            constexpr int PU = ESZ == 8 ? 1 : 2;   // trips in flight together
            u32x4 v[PU][V];
            uint32_t kp[PU];
            auto load = [&](int w) __attribute__((always_inline)) {
#pragma unroll
                for (int q = 0; q < PU; ++q) {
                    const int k = (w + q * NW * 8) * 64 + lane * 8;
                    // (the trip of a short K behind a long one reaches back into that)
                    const row16 *at = reinterpret_cast<const row16 *>(xs + min(k, left - 8));
#pragma unroll
                    for (int z = 0; z < V; ++z) v[q][z] = at[z];
                    kp[q] = keep[min(k / 8, sw * 8 - 1)];
                }
            };
            // The elements are asked for first, the map words of B behind them: the other way round, and with the fewer than eight
            // elements below in the same loop, the elements waited for the map words to arrive (4 x 16384 x 4096 bf16: 6.38 -> 5.96 us).
            int w = wave * 8;
            const bool whole = p.K >= 8;
            if (whole && w < sw) load(w);
            fetch(ks * WAVE_WORDS);
            if (sw0 > 0) __syncthreads();   // the words of the previous trip are no longer needed
            if (whole) {
                while (w < sw) {
#pragma unroll
                    for (int q = 0; q < PU; ++q) {
                        const int k = (w + q * NW * 8) * 64 + lane * 8;
                        const int back = k - min(k, left - 8);   // elements before k that were read
                        const uint32_t bits = back < 8 ? bits_of(v[q]) >> back & (kp[q] | keep_all) : 0u;
                        if (k < sw * 64) aw[k / 8] = (uint8_t)bits;
                    }
                    w += PU * NW * 8;
                    if (w < sw) load(w);
                }
            } else if (w == 0) {   // fewer than eight elements in all
                int k = lane * 8;
                asm volatile("" : "+v"(k));   // (its addresses are not worked out in front of the loop)
                uint32_t bits = 0;
                for (int q = 0; q < 8; ++q) {
                    pattern u = 0;
                    __builtin_memcpy(&u, Xrow + min(k + q, (int)p.K - 1), ESZ);
                    u &= mask;
                    const bool in = u - (pattern)p.test.lo1 < (pattern)p.test.len1 || u - (pattern)p.test.lo2 < (pattern)p.test.len2;
                    bits |= k + q < p.K && in ? 1u << q : 0u;
                }
                if (lane < 8) aw[lane] = (uint8_t)(bits & (keep[lane] | keep_all));
            }
            __syncthreads();
        }
        // this wave's ranges of the trip: ranges ks, ks + KS, ... of WAVE_WORDS words each
        for (int rw0 = ks * WAVE_WORDS; rw0 < sw; rw0 += KS * WAVE_WORDS) {
            const int rw1 = min(sw, rw0 + WAVE_WORDS);
            if (!FUSED) fetch(rw0);
            uint64_t m[WPL];
            uint32_t cnt = 0;
#pragma unroll
            for (int j = 0; j < WPL; ++j) {
                const int wi = rw0 + c + j * BW;
                uint64_t a = wa[j];
                if (FUSED) a = wi < rw1 ? reinterpret_cast<const uint64_t *>(aw)[min(wi, rw1 - 1)] : 0ull;
                m[j] = a & wb[j];
                cnt += (uint32_t)__popcll(m[j]);
            }
            if (FUSED && rw0 + KS * WAVE_WORDS < sw) fetch(rw0 + KS * WAVE_WORDS);   // while the lists of this range are walked
            // ranks: exclusive prefix of the counts inside the lane group, and the group's total
            uint32_t incl = cnt;
            auto from_below = [&](auto ctrl, bool take) {   // (a row of the cross-lane moves is 16 lanes; past its end 0 comes in)
                const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)incl, decltype(ctrl)::value, 0xf, 0xf, true);
                incl += take ? o : 0u;
            };
            from_below(std::integral_constant<int, 0x111>{}, BW >= 16 || c >= 1);   // row_shr 1, 2, 4, 8
            from_below(std::integral_constant<int, 0x112>{}, BW >= 16 || c >= 2);
            from_below(std::integral_constant<int, 0x114>{}, BW >= 16 || c >= 4);
            if (BW >= 16) from_below(std::integral_constant<int, 0x118>{}, true);
            if (BW == 32) {   // the second row of a group adds the total of the first
                const uint32_t o = (uint32_t)__shfl((int)incl, (lane & 32) + 15, 64);
                incl += c >= 16 ? o : 0u;
            }
            const uint32_t first = incl - cnt;
            const uint32_t n_g = (uint32_t)__shfl((int)incl, BW - 1, BW);
            uint32_t nmax = 0;
#pragma unroll
            for (int q = 0; q < G; ++q) nmax = max(nmax, (uint32_t)__builtin_amdgcn_readlane((int)n_g, q * BW));
            if (nmax == 0) continue;

            const uint32_t k0 = (uint32_t)(sw0 + rw0) * 64u;     // first k of the range
            const char *Yr = Ycol + (uint64_t)k0 * ldyb;         // row k0 of Y at the wave's first column
            const char *Xr = reinterpret_cast<const char *>(Xrow + k0);

            // Lists longer than CAP are walked in several passes of CAP entries.
            for (uint32_t base = 0; base < nmax; base += CAP) {
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();   // the previous pass has read its entries
                uint32_t pos = first - base;       // rank of this lane's next survivor within the pass (wraps below 0)
                auto write = [&](auto whole) __attribute__((always_inline)) {   // whole: the lists fit one pass
#pragma unroll
                    for (int j = 0; j < 2 * WPL; ++j) {
                        uint32_t mm = (uint32_t)(m[j / 2] >> (32 * (j & 1)));
                        const uint32_t kw = (uint32_t)((c + j / 2 * BW) * 64 + (j & 1) * 32) * ESZ;   // entries are byte offsets into the row of X
                        while (mm != 0) {
                            const uint32_t bit = (uint32_t)__builtin_ctz(mm);
                            mm &= mm - 1;
                            if (decltype(whole)::value || pos < (uint32_t)CAP) lst[pos] = (uint16_t)(kw + bit * ESZ);
                            ++pos;
                        }
                    }
                };
                if (nmax <= (uint32_t)CAP)
                    write(std::true_type{});
                else
                    write(std::false_type{});
                const uint32_t n_here = n_g > base ? min(n_g - base, (uint32_t)CAP) : 0u;   // entries of this lane group
                const uint32_t rmax = min(nmax - base, (uint32_t)CAP);                      // of the longest list
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                // UN loads of C16 entries of every list.  Lanes past the end of their list read the first row of the
                // range, which exists, and count it for nothing.
                auto batch = [&](uint32_t t0, auto un) __attribute__((always_inline)) {
                    constexpr int UN = decltype(un)::value;
                    T x[UN];
                    u32x4 y[UN];
                    bool valid[UN];
#pragma unroll
                    for (int u = 0; u < UN; ++u) {
                        const uint32_t t = t0 + (uint32_t)(u * C16 + entry);
                        valid[u] = t < n_here;
                        const uint32_t kb = valid[u] ? lst[min(t, (uint32_t)CAP - 1)] : 0u;   // k * ESZ
                        x[u] = *reinterpret_cast<const T *>(Xr + kb);
                        y[u] = *reinterpret_cast<const row16 *>(Yr + (__umul24(kb, ldy) + lane_off));
                    }
#pragma unroll
                    for (int u = 0; u < UN; ++u) {
                        const acc_t xv = valid[u] ? Elem<T>::value(x[u]) : acc_t(0);
                        acc_t yv[C16];
                        Elem<T>::unpack(valid[u] ? y[u] : u32x4{0, 0, 0, 0}, yv);
#pragma unroll
                        for (int q = 0; q < C16; ++q) acc[q] = fma_acc(xv, yv[q], acc[q]);
                    }
                };
                uint32_t t = 0;
                if (FUSED)
                    for (; t + 2 * C16 < rmax; t += 4 * C16) batch(t, std::integral_constant<int, 4>{});
                for (; t + C16 < rmax; t += 2 * C16) batch(t, std::integral_constant<int, 2>{});
                if (t < rmax) batch(t, std::integral_constant<int, 1>{});
            }
        }
        if constexpr (FUSED) __builtin_amdgcn_s_waitcnt(0);   // nothing is under way at the start of a trip (else the first one waits for what might be)
    }

    // The lanes of a group that hold the same columns exchange halves of them: one column per lane is left.
#pragma unroll
    for (int half = C16 / 2, stride = BW / 2; half >= 1; half /= 2, stride /= 2) {
        const bool upper = (lane & stride) != 0;
#pragma unroll
        for (int q = 0; q < half; ++q) {
            const acc_t send = upper ? acc[q] : acc[q + half];
            acc[q] = (upper ? acc[q + half] : acc[q]) + __shfl_xor(send, stride, 64);
        }
    }
    const uint32_t col = col0 + (uint32_t)(g * BW + part * C16 + entry);
    if (KS > 1) {   // add the partial sums of the waves that shared this column span, in wave order
        if (ks > 0) red[((ks - 1) * CW + cw) * 64 + lane] = acc[0];
        __syncthreads();
        if (ks == 0)
#pragma unroll
            for (int q = 1; q < KS; ++q) acc[0] += red[((q - 1) * CW + cw) * 64 + lane];
    }
    if (ks == 0 && col < p.N) {
        acc_t *dst = static_cast<acc_t *>(p.C) + (int64_t)row_i * p.ldc + col;
        *dst = p.accumulate ? *dst + acc[0] : acc[0];
    }
}

typedef void (*pairs_kernel_fn)(const PairsParams);

struct PairsShape { int cw, ks, words; };

// Workgroup shapes: CW waves side by side (64 columns each), KS that share K, and the map words a wave intersects at a time.
//   8 x 1  512 columns: many rows, or a K so short that there is nothing to share out
//   2 x 4  few rows: 128 columns, K in four shares
//   8 x 2, 4 x 4, 2 x 8  few rows, mask evaluated here: the predicate work is shared by 512, 256, 128 columns
// Words: the fewest that still give every share a part of K (64 k each), so that no wave stands idle: a K of 4096 in ranges
// of 64 words was one range, for one wave in four.
template <typename T, int BW, bool FUSED> pairs_kernel_fn pick_shape(const PairsShape &sh)
{
    constexpr int W16 = BW == 32 ? 32 : 16;   // a lane takes at least one word
    const int w = sh.words;
    if (sh.ks == 1)
        return w == 16 ? mmm_pairs_kernel<T, BW, 8, 1, W16, FUSED> : w == 32 ? mmm_pairs_kernel<T, BW, 8, 1, 32, FUSED> : mmm_pairs_kernel<T, BW, 8, 1, 64, FUSED>;
    if constexpr (!FUSED) {
        return w == 16 ? mmm_pairs_kernel<T, BW, 2, 4, W16, FUSED> : w == 32 ? mmm_pairs_kernel<T, BW, 2, 4, 32, FUSED> : mmm_pairs_kernel<T, BW, 2, 4, 64, FUSED>;
    } else {
        if (sh.ks == 8) return w == 16 ? mmm_pairs_kernel<T, BW, 2, 8, W16, FUSED> : mmm_pairs_kernel<T, BW, 2, 8, 32, FUSED>;
        if (sh.ks == 4) return w <= 32 ? mmm_pairs_kernel<T, BW, 4, 4, 32, FUSED> : mmm_pairs_kernel<T, BW, 4, 4, 64, FUSED>;
        return w <= 32 ? mmm_pairs_kernel<T, BW, 8, 2, 32, FUSED> : mmm_pairs_kernel<T, BW, 8, 2, 64, FUSED>;
    }
}

template <typename T, bool FUSED> pairs_kernel_fn pick(int32_t bw, const PairsShape &sh)
{
    if (bw == 8) return pick_shape<T, 8, FUSED>(sh);
    if (bw == 16) return pick_shape<T, 16, FUSED>(sh);
    return pick_shape<T, 32, FUSED>(sh);
}

}   // namespace

bool mmm_pairs_supports(int32_t dtype, int64_t ldy)
{
    const int64_t esz = dtype == MMM_F64 ? 8 : dtype == MMM_F32 ? 4 : 2;
    return ldy * esz * (MAX_WAVE_WORDS * 64) + 256 <= 0xffffffffLL;
}

// fused: evaluate M (pred, threshold, keep_a) on X in the kernel; otherwise take a_bits from the maps.
hipError_t mmm_launch_pairs(const mmm_maps *m, int32_t dtype, const void *X, int64_t ldx, const void *Y, int64_t ldy,
                            void *C, int64_t ldc, int32_t accumulate, bool fused, int32_t pred, float threshold,
                            const uint64_t *keep_a, hipStream_t s)
{
    PairsParams p{};
    p.X = X;
    p.ldx = ldx;
    p.Y = Y;
    p.ldy = ldy;
    p.C = C;
    p.ldc = ldc;
    p.a_bits = m->a_bits;
    p.keep_a = keep_a;
    p.bt_bits = m->bt_bits;
    p.M = m->M;
    p.K = m->K;
    p.N = m->N;
    p.NB = m->NB;
    p.WA = m->WA;
    if (fused) p.test = mmm_element_test(dtype, pred, threshold);
    p.accumulate = accumulate;
    p.by_m = mmm_make_divisor((uint32_t)m->M);
    // Workgroups of 8 waves x 64 columns; when that gives the machine too little to do (few rows:
    // the decode shape), fewer columns per workgroup and K shared out over several waves, unless there is next to nothing of it.
    // With the mask evaluated here every column span repeats the predicate, so the spans are as wide as leaves every compute unit a
    // workgroup (4 x 16384 x 4096 bf16: 128, 256 columns: 5.7, 6.6 us; 16 x 8192 x 4096, where 128 make two rounds: 8.7, 5.6).
    const int64_t wide = (m->N + 511) / 512 * m->M;
    PairsShape sh{8, 1, 64};
    if (wide < 1024 && (fused || m->WA > 32)) {
        if (!fused)
            sh = {2, 4, 64};
        else if ((m->N + 127) / 128 * m->M <= 256)
            sh = {2, 8, 32};
        else if (m->M <= 16)
            sh = {4, 4, 64};
        else
            sh = {8, 2, 64};
    }
    if (m->WA <= 16 * sh.ks)
        sh.words = 16;
    else if (m->WA <= 32 * sh.ks)
        sh.words = 32;
    const int64_t span = sh.cw * 64;
    const int64_t ctiles = (m->N + span - 1) / span;
    const int64_t wgs = ctiles * m->M;
    if (wgs <= 0 || wgs > 0x7fffffffLL) return hipErrorInvalidValue;
    pairs_kernel_fn fn;
    if (fused)
        fn = dtype == MMM_F64 ? pick<double, true>(m->bw, sh) : dtype == MMM_BF16 ? pick<uint16_t, true>(m->bw, sh) : dtype == MMM_F16 ? pick<_Float16, true>(m->bw, sh)
                                                                                         : pick<float, true>(m->bw, sh);
    else
        fn = dtype == MMM_F64 ? pick<double, false>(m->bw, sh) : dtype == MMM_BF16 ? pick<uint16_t, false>(m->bw, sh) : dtype == MMM_F16 ? pick<_Float16, false>(m->bw, sh)
                                                                                          : pick<float, false>(m->bw, sh);
    p.workgroups = (uint32_t)wgs;
    (void)hipGetLastError();
    hipLaunchKernelGGL(fn, dim3((uint32_t)wgs), dim3((uint32_t)(sh.cw * sh.ks * 64)), 0, s, p);
    return hipGetLastError();
}
