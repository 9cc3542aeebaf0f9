// Host side of the C ABI declared in include/mmm.h: argument checks, workspace
// layout, launch planning.  All checks run before any device call, so they can
// be exercised on a machine without a GPU.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>

#include "mmm_internal.h"

namespace {

constexpr size_t kAlign = 256;
constexpr int64_t kMaxLd = (1LL << 22) - 1;   // largest leading dimension of X and Y the masked GEMM addresses
constexpr size_t kPartialCap = (size_t)64 << 20;   // split-K partial sums: at most 64 MiB

thread_local char g_detail[160] = "";

void note_device_error(const char *where, hipError_t e)
{
    std::snprintf(g_detail, sizeof(g_detail), "%s: %s (%d)", where, hipGetErrorName(e), (int)e);
}

std::atomic<int64_t> g_opt_variant{-1};
std::atomic<int64_t> g_opt_split{0};
std::atomic<int64_t> g_opt_path{-1};
std::atomic<int64_t> g_opt_form{-1};

inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct Layout {
    size_t a_bits, a_colany, a_cnt, a_ent, a_img, a_wild, b_bits, bt_bits, stats, kinfo, kmap, rows_copy, a_colany_c, btc_bits, bp_val, bp_list, bp_cnt, partials, partial_bytes, total;
};

bool shape_ok(int64_t M, int64_t K, int64_t N, int32_t bw)
{
    if (M < 1 || K < 1 || N < 1) return false;
    if (bw != 8 && bw != 16 && bw != 32) return false;
    if (N % bw != 0) return false;
    // 31-bit grids and 32-bit tile-relative offsets are used throughout
    if (M > (1LL << 30) || K > (1LL << 30) || N > (1LL << 30)) return false;
    return true;
}

// parts: with room for floats in parts
Layout make_layout(int64_t M, int64_t K, int64_t N, int32_t bw, bool parts)
{
    parts = parts && M > 64;
    const int64_t NB = N / bw, WA = (K + 63) / 64, WB = (NB + 63) / 64, MT = (M + MMM_COLANY_ROWS - 1) / MMM_COLANY_ROWS;
    Layout l{};
    size_t off = 0;
    l.a_bits = off;
    off += align_up((size_t)M * WA * 8);
    l.a_colany = off;
    off += align_up((size_t)MT * WA * 8);
    const size_t blocks = (size_t)((M + MMM_AB_ROWS - 1) / MMM_AB_ROWS) * (size_t)((K + MMM_AB_COLS - 1) / MMM_AB_COLS);
    l.a_cnt = off;
    off += align_up(blocks * 4);
    l.a_ent = off;
    off += align_up(blocks * MMM_AB_CAP * 8);
    l.a_img = off;   // (doubles have theirs in a_ent)
    off += align_up(blocks * MMM_AB_CAP * (parts ? MMM_PARTS_ESZ : 4));
    l.a_wild = off;
    off += align_up(blocks);
    l.b_bits = off;
    off += align_up((size_t)K * WB * 8);
    l.bt_bits = off;
    off += align_up((size_t)NB * WA * 8);
    l.stats = off;
    off += align_up(MMM_STATS_WORDS * 8);
    // row-compacted mode: numbering of the live rows and maps over it
    l.kinfo = off;
    off += align_up(64);
    l.kmap = off;
    off += align_up((size_t)K * 4);
    l.rows_copy = off;
    off += align_up((size_t)WA * 8);
    l.a_colany_c = off;
    off += align_up((size_t)MT * WA * 8);
    l.btc_bits = off;
    off += align_up((size_t)NB * WA * 8);
    // packed B: every row of every 16-column group, in the widest element type that is packed
    const size_t segs = (size_t)((N + MMM_GROUP_COLS - 1) / MMM_GROUP_COLS) * (size_t)((K + MMM_AB_COLS - 1) / MMM_AB_COLS);
    l.bp_val = off;
    off += align_up(segs * MMM_AB_COLS * MMM_GROUP_COLS * (mmm_packs(M, MMM_F64) ? 8 : 4));
    l.bp_list = off;
    off += align_up(segs * MMM_AB_COLS * 2);
    l.bp_cnt = off;
    off += align_up(segs * 4);
    l.partials = off;
    // room for up to 32 splits of C, capped
    size_t want = (size_t)M * (size_t)N * sizeof(float) * 32;
    if (want > kPartialCap) want = kPartialCap;
    l.partial_bytes = align_up(want);
    off += l.partial_bytes;
    l.total = off;
    return l;
}

bool dtype_ok(int32_t dt) { return dt == MMM_F32 || dt == MMM_BF16 || dt == MMM_F16 || dt == MMM_F64; }
size_t elem_size(int32_t dt) { return dt == MMM_F64 ? 8 : dt == MMM_F32 ? 4 : 2; }
size_t c_elem_size(int32_t dt) { return dt == MMM_F64 ? 8 : 4; }

// ---- Which kernel, which tile, how many splits of K -------------------------------------------
//
// A table of thresholds cannot follow this choice: it depends on the shape, both densities and how evenly the
// workgroups fall on 256 compute units.  So both kernels' times are estimated and the least is taken.  The
// estimates are sums of terms with a meaning each; their coefficients are a least-squares fit to random problems (200 to 4096
// in each dimension, few rows with K up to 16384, densities .05 to 1, all types), built and multiplied with every variant and
// a dozen splits.  What is chosen from them, against other random problems (profiles/kernel_choice.txt): the kernel takes 1 % longer
// than the faster one in the mean, 1 to 3 % where A keeps .2 to 5 % of its elements, outside the fit (a rule of thresholds fitted to
// 4096^3 floats decided there before: 5 % floats, 7 % doubles, 22 % 16-bit); the tile and split 1 % (16-bit) to 3 % longer than the best.
// The 2-byte row is from 700 problems (65 to 4096 rows, K to 16384, N to 8192) after the kernel took its batches from one queue, and
// scaled to lie above timings as the others do: tile and split 1.4 % longer than the best on 700 others, 19 % at worst; with the
// row from before, whose waiting per step is twice as long, 3.3 and 51 % (512 x 8192 x 4096, p = .1: 24.0 -> 21.9 us).
// The row of floats in parts is from 800 problems (65 to 4096 rows, K to 16384, densities .05 to .6, up to three splits each) after their batches were joined:
// 90 to 113 % of the timings of 800 others in nine of ten (with the row from before, whose batches were whole lists', 70 to 94 %).
// The other estimates lie 10 to 25 % from back-to-back timings, those of 2-byte types mostly above, which hide the launch.
struct MatrixCost {   // microseconds
    double launch;        // per call
    double latency;       // per step and batch of its longest lists: nobody hides the first wave's waiting
    double step;          // per step of each workgroup on the fullest compute unit: barrier, copy of a block of A
    double multiply;      // per 16 columns, row tile of 16 and list unit (quad of k; 16-bit: batch of 32) there
    double wave;          // per 16 columns of each workgroup there: prologue, writing C
    double workgroup;     // per workgroup there
    double reduce;        // second launch that adds the splits
    double reduce_mega;   // per 2^20 partial sums of C
    double image_giga;    // per 10^9 bytes of A copied to LDS
};
constexpr MatrixCost kMatrixCost[4] = {   // 2-, 4-, 8-byte elements, floats in parts
    {2.936, 0.0995, 0.0371, 0.0032, 0.0971, 0.866, 2.67, 1.241, 34.4},
    {3.524, 0.1805, 0.1198, 0.0031, 0.0747, 0.561, 2.0, 1.159, 24.9},
    {3.210, 0.3107, 0.4623, 0.0059, 0.1092, 1.362, 3.3, 2.257, 30.9},
    {5.009, 0.0222, 0.2541, 0.0133, 0.0, 1.607, 2.07, 1.861, 20.3},
};
struct PairsCost {   // microseconds
    double launch;     // per call
    double range;      // per range of 4096 k a wave goes through, one after another
    double word;       // per 10^5 ranges of all rows and 64-column spans: intersecting the maps
    double product[3]; // per 10^9 surviving products, blocks of 8, 16, 32
    double list;       // per 100 entries of one wave's lists, one after another
};
constexpr PairsCost kPairsCost[3] = {
    {3.39, 2.24, 26.3, {521, 275, 140}, 1.1},
    {1.75, 3.50, 24.7, {632, 312, 191}, 4.8},
    {3.90, 0.00, 30.2, {863, 549, 463}, 15.9},
};

int cost_class(int32_t dt, int32_t form) { return form == MMM_FORM_PARTS ? 3 : dt == MMM_F64 ? 2 : dt == MMM_F32 ? 1 : 0; }
bool stats_known(const mmm_maps *m) { return m->stats_a_valid && m->stats_b_valid; }

// Densities are known only after a mmm_maps_stats call (the counts of the most recent one are kept as the estimate, also
// across rebuilds: emergent sparsity levels are stable from step to step); without one a fifth of B is assumed.
struct MatrixProblem {
    int64_t steps;   // of 128 k that the kernel walks
    double units;    // per step and group: quads of listed k (16-bit: batches of 32)
    double batches;  // batches of 16 (32) slots
    double marked;   // floats in parts: share of the steps of a wave with an element that they do not hold
    double redone;   // and how long such a step takes, us
    bool look;       // workgroups look for columns of A that are zero in their tile (floats)
    bool filtered;   // and most will leave them out of their lists
};
MatrixProblem matrix_problem(const mmm_maps *m, int32_t dt, int32_t form)
{
    const size_t esz = form == MMM_FORM_PARTS ? 2 : elem_size(dt);   // as the lists are laid out
    const bool known = stats_known(m);
    const int64_t rows = known && m->b_compact ? std::max<int64_t>((int64_t)m->stats_rows_b, 1) : m->K;
    double p = known ? std::min(1.0, (double)m->stats_occ_b / ((double)rows * (double)m->NB)) : 0.2;
    if (m->bw == 8) p = 1.0 - (1.0 - p) * (1.0 - p);   // a group lists k if either of its blocks does
    const double batch = esz == 2 ? 32.0 : 16.0;
    double listed = p * MMM_AB_COLS;
    MatrixProblem q;
    // The form that looks takes longer where it finds nothing: its registers, arguments and the looking cost 0.5 to 8 us (4096^3,
    // p = .05 121.3 and 128.0 us, 256^3 10.8 and 11.6, 60 problems 4.8 %).  So only where the counts say that there is something.
    q.look = dt == MMM_F32 && form == MMM_FORM_PLAIN && known && m->stats_active < 0.9;
    q.filtered = q.look && mmm_filter_pays((float)listed, (float)(listed * m->stats_active), m->bw);
    if (q.filtered) listed *= m->stats_active;
    q.steps = (rows + MMM_AB_COLS - 1) / MMM_AB_COLS;
    q.batches = listed > 0.5 * batch ? listed / batch + 0.5 : 1.0;
    if (form == MMM_FORM_PARTS) q.batches = std::max(listed / MMM_UNIT + 0.5, 3.0) * MMM_UNIT / batch;   // (put together from units, three a step at least)
    q.units = esz == 2 ? q.batches : listed / 4.0 + 0.5;
    const double b_marked = m->bw == 32 ? 1.0 - (1.0 - m->stats_marked_b) * (1.0 - m->stats_marked_b) : m->stats_marked_b;   // (a wave has two groups)
    q.marked = form == MMM_FORM_PARTS && known ? 1.0 - (1.0 - m->stats_marked_a) * (1.0 - b_marked) : 0.0;
    q.redone = 1.65 * (listed / 4.0 + 0.5);
    return q;
}

double matrix_cost(const mmm_maps *m, int32_t dt, int32_t form, const MatrixProblem &q, const mmm_variant_info &vi, int64_t tiles, int64_t split)
{
    MatrixCost c = kMatrixCost[cost_class(dt, form)];
    const size_t esz = form == MMM_FORM_PARTS ? MMM_PARTS_ESZ : elem_size(dt);
    if (q.filtered) {   // lists made in the kernel (estimated from the timings at mmm_filter_pays, within 20 %)
        c.multiply *= 1.35;
        if (m->bw != 32) c.latency += 0.25, c.step += 0.2 * vi.TN / 256.0;
    }
    const int64_t per_split = (q.steps + split - 1) / split, steps = (per_split + vi.k_ranges - 1) / vi.k_ranges;
    const int64_t wgs = tiles * split, per_cu = (wgs + 255) / 256;
    const double groups = vi.TN / MMM_GROUP_COLS, work = (double)steps * vi.k_ranges;
    double t = c.launch + (double)steps * q.batches * c.latency +
               (double)per_cu * (work * (c.step + groups * (vi.rows / 16) * q.units * c.multiply) + groups * vi.k_ranges * c.wave + c.workgroup) +
               1e-9 * c.image_giga * (double)wgs * work * (double)(MMM_AB_ROWS * MMM_AB_COLS * esz);
    if (q.marked > 0.0) {
        // Marked steps are done again behind the loop, by a wave on its own and four k at a time.  The fullest compute unit has more of them
        // than the mean: by about three times its root.  4096^3, p = .4, multiplication, with 0, 1, 10, 100 % of the blocks of A marked
        // 314, 390, 762, 2908 us, of the segments of B 311, 454, 879, 2911; 2048^3, blocks of 32, p_B = .5, 56, 123, 214, 360 and 52, 97, 211, 358.
        const double all = (double)steps * (double)per_cu, mean = q.marked * all;
        t += q.redone * std::min(all, mean + 3.0 * std::sqrt(mean));
    }
    if (split > 1) t += c.reduce + 1e-6 * c.reduce_mega * (double)split * (double)m->M * (double)m->N;
    return t;
}

// Tile columns per panel.  Each of the 8 XCDs works on an eighth of the tiles, one after another in the order of the
// numbering, and what its L2 has to fetch is the block rows of A and the column tiles of B that eighth touches.  An
// eighth of T tiles in panels of w columns is about T / w rows by w columns: least for w = sqrt(T * a / b), with a and b
// the bytes of one row and one column tile.  (512 x 8192 x 4096 bf16, p = .1: one row and all of B per XCD, 143 MB in all
// against 67, and 27.8 -> 22.7 us; columns bf16 2048 x 1638 of 16384 x 4096 46.2 -> 42.5.)
// Of a long eighth it is the 32 tiles or so under way at a time that have to find their rows and columns in the L2: what
// earlier ones fetched does not stay (4096^3, a column tile of packed B is 4 MB).  Width 6 instead of all 16: bf16, p = .05,
// 64.9 -> 56.9 us, .4 99.5 -> 98.1; floats p = .05 89.1 -> 87.5, .2 239 -> 236.7, in parts .4 311 -> 307.  With 64 tiles
// 57.6, 89.2 and 237.0, with 16 57.0, 88.4 and 237.4 and the columns above 37.2 instead of 36.
int32_t panel_width(const mmm_maps *m, int32_t dt, int32_t form, const MatrixProblem &q, const mmm_plan &p)
{
    const double batch = elem_size(dt) == 2 || form == MMM_FORM_PARTS ? 32.0 : 16.0;
    const double a = (double)(MMM_AB_ROWS * MMM_AB_COLS), b = (double)mmm_variant(p.variant).TN * q.batches * batch;   // elements per step
    const double t = std::max(1.0, std::min((double)p.tiles_m * p.tiles_n / 8.0, 32.0));
    const int64_t panels = std::max<int64_t>(1, (int64_t)((double)p.tiles_n / std::sqrt(t * a / b) + 0.5));   // of about equal width
    return (int32_t)std::max<int64_t>(1, (p.tiles_n + panels - 1) / panels);
}

double pairs_cost(const mmm_maps *m, int32_t dt)
{
    const PairsCost &c = kPairsCost[cost_class(dt, MMM_FORM_PLAIN)];
    const double spans = (double)m->M * (double)((m->N + 63) / 64), products = (double)m->stats_macs;
    const int64_t ranges = (m->WA + 63) / 64, shares = (m->N + 511) / 512 * m->M >= 1024 ? 1 : 4;
    // (4 shares for few workgroups whatever K is, as the coefficients were fitted; mmm_launch_pairs takes 1 for K <= 2048.  With its
    // number here the choice was no better: 984 float problems 1.5 instead of 1.2 % longer than the faster kernel, refitted 1.6.)
    return c.launch + (double)((ranges + shares - 1) / shares) * c.range + 1e-5 * spans * (double)ranges * c.word +
           1e-9 * products * c.product[m->bw == 8 ? 0 : m->bw == 16 ? 1 : 2] + 0.01 * products / (spans * (double)shares * 64.0) * c.list;
}

mmm_plan tile_plan(const mmm_maps *m, int32_t variant)   // without the split
{
    const mmm_variant_info &vi = mmm_variant(variant);
    mmm_plan p{};
    p.variant = variant;
    p.tiles_m = (int32_t)((m->M + vi.TM - 1) / vi.TM);
    p.tiles_n = (int32_t)((m->N + vi.TN - 1) / vi.TN);
    p.chunks_total = (int32_t)((m->K + vi.KC - 1) / vi.KC);
    return p;
}

bool variant_usable(const mmm_maps *m, int32_t dt, int32_t form, int64_t v)
{
    if (v < 0 || v >= mmm_variant_count()) return false;
    const mmm_variant_info &vi = mmm_variant((int32_t)v);
    return !(vi.rows < MMM_AB_ROWS && m->M > vi.rows)        // computes too few rows for this matrix
           && !(dt == MMM_F64 && !vi.doubles) && !(form == MMM_FORM_PARTS && vi.parts == PARTS_NO);
}

void compute_plan(const mmm_maps *m, int32_t dt, int32_t form, int64_t variant, int64_t fixed_split, mmm_plan *plan, double *cost)
{
    const MatrixProblem q = matrix_problem(m, dt, form);
    const size_t c_bytes = (size_t)m->M * (size_t)m->N * c_elem_size(dt);
    double best = -1.0;
    for (int32_t v = 0; v < mmm_variant_count(); ++v) {
        if (!variant_usable(m, dt, form, v) || (variant_usable(m, dt, form, variant) && v != variant)) continue;
        if (form == MMM_FORM_PARTS && mmm_variant(v).parts != PARTS_OWN && v != variant) continue;
        mmm_plan p = tile_plan(m, v);
        const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
        static constexpr int64_t kSplits[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 28, 32};
        for (int64_t s : kSplits) {
            // an automatic split also fits the library's own scratch array, whichever entry point runs it
            int64_t split = fixed_split > 0 ? fixed_split : s;
            const size_t room = fixed_split > 0 ? m->partial_bytes : std::min(m->partial_bytes, (size_t)MMM_STATIC_SCRATCH_BYTES);
            split = std::min<int64_t>(split, (int64_t)(room / c_bytes));
            split = std::max<int64_t>(1, std::min<int64_t>(split, p.chunks_total));
            p.chunks_per_split = (int32_t)((p.chunks_total + split - 1) / split);
            split = (p.chunks_total + p.chunks_per_split - 1) / p.chunks_per_split;   // drop empty splits
            const double t = matrix_cost(m, dt, form, q, mmm_variant(v), tiles, split);
            if (best < 0.0 || t < best) {
                best = t;
                p.split_k = (int32_t)split;
                p.workgroups = tiles * split;
                *plan = p;
            }
            if (fixed_split > 0 || split < s) break;
        }
    }
    plan->panel = panel_width(m, dt, form, q, *plan);
    plan->filter = q.look ? 1 : 0;
    *cost = best;
}

mmm_plan make_plan(const mmm_maps *m, int32_t dt, int32_t form, double *cost = nullptr)
{
    const int64_t v = m->plan_variant >= 0 ? m->plan_variant : g_opt_variant.load();
    const int64_t split = m->plan_split > 0 ? m->plan_split : g_opt_split.load();
    std::lock_guard<std::mutex> lock(m->plan_mutex);
    const mmm_plan_key key{dt, v, split, m->stats_version, m->b_compact, form};
    if (!(m->plan_valid && key == m->plan_key)) {
        compute_plan(m, dt, form, v, split, &m->plan, &m->plan_cost);
        m->plan_key = key;
        m->plan_valid = true;
    }
    if (cost) *cost = m->plan_cost;
    return m->plan;
}

int32_t choose_path(const mmm_maps *m, int32_t dt, int32_t form)
{
    if (!mmm_packs(m->M, dt)) return MMM_PATH_PAIRS;
    const int64_t path = m->plan_path >= 0 ? m->plan_path : g_opt_path.load();
    if (path == MMM_PATH_MATRIX || path == MMM_PATH_PAIRS) return (int32_t)path;
    if (m->plan_variant >= 0 || g_opt_variant.load() >= 0) return MMM_PATH_MATRIX;   // a tile variant was asked for
    if (!stats_known(m)) {   // the shape alone: few rows make short lists
        if (dt == MMM_F64) return (double)m->M * (double)m->K * (double)m->N >= 134217728.0 ? MMM_PATH_MATRIX : MMM_PATH_PAIRS;
        return m->M <= 64 ? MMM_PATH_PAIRS : MMM_PATH_MATRIX;
    }
    // doubles of a few tiles: the matrix kernel leaves nearly all of the chip idle, and the estimates are poor there
    // (215 x 722 x 320: 7.1 against 8.7 us; from 28 tiles on it is the estimates that decide better)
    if (dt == MMM_F64 && ((m->M + 63) / 64) * ((m->N + 63) / 64) <= 24) return MMM_PATH_PAIRS;
    double matrix = 0.0;
    make_plan(m, dt, form, &matrix);
    return pairs_cost(m, dt) < matrix ? MMM_PATH_PAIRS : MMM_PATH_MATRIX;
}

// The form the operands are in, or would be if there are none yet.
int32_t form_of(const mmm_maps *m, int32_t dt)
{
    if (dt != MMM_F32) return MMM_FORM_PLAIN;
    return m->b_built && m->b_dtype == dt ? m->b_form : m->a_built && m->a_dtype == dt ? m->a_form : MMM_FORM_PLAIN;
}

struct RelaxedCapture {   // calls that another thread's stream capture would forbid, and that do not disturb it
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool exchanged = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~RelaxedCapture()
    {
        if (exchanged) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
};

// What only inspection reads is made when it is asked for.  These calls take no stream: the build may have run on one that is
// busy with something else by now or does not exist any more, and the caller may read on any.  So nothing is assumed about
// streams: the device's work is waited for, and then what was made.
mmm_status make_for_inspection(const char *what, const mmm_maps *maps, hipError_t (*launch)(const mmm_maps *, hipStream_t))
{
    RelaxedCapture relaxed;
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = launch(maps, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e == hipSuccess) return MMM_OK;
    note_device_error(what, e);
    return MMM_ERR_DEVICE;
}

bool capturing(hipStream_t s)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(s, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
}

// Whether this call is captured with a form.  (The null stream is never captured; asking takes 0.15 us.)
bool form_is_captured(const mmm_maps *m, int32_t dt, hipStream_t s)
{
    return mmm_may_part(m, dt) && s != nullptr && capturing(s);
}

void release_captures(mmm_captures *c)
{
    if (c->owners.fetch_sub(1) == 1) delete c;
}
void graph_is_gone(void *captures)   // (called by the runtime: no calls of it in here)
{
    mmm_captures *c = static_cast<mmm_captures *>(captures);
    c->graphs.fetch_sub(1);
    release_captures(c);
}

// The graph under capture holds a call with this form.  Where the runtime cannot tell when the graph goes, it is taken to stay.
void capture_form(const mmm_maps *m, int32_t form, hipStream_t s)
{
    m->form_captured = form;
    mmm_captures *c = m->captures;
    c->graphs.fetch_add(1);
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    hipGraph_t graph = nullptr;
    hipUserObject_t object = nullptr;
    if (hipStreamGetCaptureInfo_v2(s, &status, nullptr, &graph, nullptr, nullptr) == hipSuccess && graph != nullptr) {
        c->owners.fetch_add(1);
        if (hipUserObjectCreate(&object, c, graph_is_gone, 1, hipUserObjectNoDestructorSync) != hipSuccess)
            release_captures(c);
        else if (hipGraphRetainUserObject(graph, object, 1, hipGraphUserObjectMove) != hipSuccess) {
            c->graphs.fetch_add(1);   // (what the release takes back)
            (void)hipUserObjectRelease(object, 1);
        }
    }
    (void)hipGetLastError();
}

// The form a build gives floats: that of the side it does not build (the kernel takes both from one form), that of captured
// calls, or the one with which build and multiplication are estimated to take less; without counts the plain one.  Parts pay
// for long lists: 4096^3, blocks of 16, multiplication and build, plain and in parts: p = .4 475 + 41 and 319 + 57 us, .2 248 + 36 and
// 185 + 44, .1 138 + 33 and 155 + 39 (a list of 13 fills two of the three units it counts for).  They do not where more than a few steps hold an element that
// parts do not (see matrix_cost): mmm_maps_stats counts those too, in either form.
int32_t choose_form(mmm_maps *m, const mmm_build_args &a)
{
    if (!mmm_may_part(m, a.dtype)) return MMM_FORM_PLAIN;
    const int64_t opt = g_opt_form.load();
    const bool keeps_a = a.X == nullptr && m->a_built && m->a_dtype == MMM_F32 && !(m->b_compact || a.b_compact);
    const bool keeps_b = a.Y == nullptr && m->b_built && m->b_dtype == MMM_F32;
    int32_t form = MMM_FORM_PLAIN;
    if (keeps_a || keeps_b) {
        form = keeps_a ? m->a_form : m->b_form;
    } else if (m->captures->graphs.load() > 0) {
        form = m->form_captured;
    } else if (opt >= 0) {
        form = (int32_t)opt;
    } else if (stats_known(m)) {
        const int64_t v = m->plan_variant >= 0 ? m->plan_variant : g_opt_variant.load();
        const int64_t split = m->plan_split > 0 ? m->plan_split : g_opt_split.load();
        const int32_t path = m->plan_path >= 0 ? m->plan_path : (int32_t)g_opt_path.load();
        const mmm_plan_key key{a.dtype, v, split, m->stats_version, m->b_compact, MMM_FORM_PLAIN};
        if (!(m->form_valid && key == m->form_key && path == m->form_path)) {
            mmm_plan plan;
            double plain = 0.0, parts = 0.0;
            compute_plan(m, a.dtype, MMM_FORM_PLAIN, v, split, &plan, &plain);
            const bool filter = plan.filter != 0;
            compute_plan(m, a.dtype, MMM_FORM_PARTS, v, split, &plan, &parts);
            // What the build takes longer, fitted to 400 random problems of 65 to 4096 rows and columns, K up to 16384, densities .05 to 1 (on 800
            // others within 2.3 us in nine of ten): the image and packed B are half as large again, and the rows of B are read twice.
            // With 15 % and 2 us between the two, 253 of 3700 float problems (p_B .05 to .6) are built in parts; their passes are .784 of plain ones in the
            // mean, three take more than 2 % longer, 14 % at worst; 107 or more are plain where parts would be 5 % faster.  Less between them gives
            // some of those to parts, and slower ones with them (10 %: of 1200 problems 102 in parts instead of 82, four of them slower, 29 % at worst; the row of
            // the former kernel with lists joined: 145 and 19, 34 %), and more callers another order of rounding.
            const MatrixProblem q = matrix_problem(m, a.dtype, MMM_FORM_PARTS);
            const double b_rounds = std::ceil((double)q.steps * (double)((m->N + 255) / 256) / 512.0);
            const double longer = 2.68e-7 * (double)m->M * (double)m->K + 7.7e-7 * (double)m->stats_occ_b * m->bw + 0.6 * q.batches * b_rounds;
            const bool asked = v >= 0 && mmm_variant((int32_t)v).parts != PARTS_OWN;   // another tile: floats as they are
            const bool pairs = path == MMM_PATH_PAIRS || (path < 0 && v < 0 && pairs_cost(m, a.dtype) < std::min(plain, parts));
            m->form_chosen = !filter && !asked && !pairs && 1.15 * parts + longer + 2.0 < plain ? MMM_FORM_PARTS : MMM_FORM_PLAIN;
            m->form_key = key;
            m->form_path = path;
            m->form_valid = true;
        }
        form = m->form_chosen;
    }
    return form;
}

// The transposed B map over k is read by the pair kernel and by inspection only.  In row-compacted mode it is made with
// the B side where the pair kernel is what will run (always for at most 64 rows); where the matrix kernel is, by the first
// call that wants it all the same, once per build, on that call's stream (5 us; with every build it would cost the matrix
// path 1 to 2).  Calls on other streams wait for it, by an event, until it is seen to have run.  A call that is being
// captured makes its own: it runs when the graph does, and after builds that come in between.  And once a build has been
// captured every call makes its own: what is done when that graph runs again is not seen here.
hipError_t ensure_bt(const mmm_maps *m, hipStream_t s)
{
    if (!m->b_compact || m->M <= 64) return hipSuccess;
    if (m->build_captured || capturing(s)) return mmm_launch_expand_rows(m, s);
    if (m->bt_state.load(std::memory_order_acquire) == BT_MADE) return hipSuccess;
    std::lock_guard<std::mutex> lock(m->bt_mutex);
    RelaxedCapture relaxed;
    hipError_t result = hipSuccess;
    bool launch = true;
    if (m->bt_state == BT_LAUNCHED) {
        const hipError_t e = hipEventQuery(m->bt_event);
        if (e == hipSuccess) m->bt_state.store(BT_MADE, std::memory_order_release);
        launch = e != hipSuccess && !(e == hipErrorNotReady && hipStreamWaitEvent(s, m->bt_event, 0) == hipSuccess);
    } else if (m->bt_state == BT_MADE) {
        launch = false;
    }
    if (launch) {   // (where the event fails, each call makes it anew, to the same values)
        result = mmm_launch_expand_rows(m, s);
        if (result == hipSuccess && (m->bt_event != nullptr || hipEventCreateWithFlags(&m->bt_event, hipEventDisableTiming) == hipSuccess) &&
            hipEventRecord(m->bt_event, s) == hipSuccess)
            m->bt_state = BT_LAUNCHED;
    }
    (void)hipGetLastError();   // "not ready" is no error of the caller's
    return result;
}

}   // namespace

extern "C" {

const char *mmm_status_string(mmm_status st)
{
    switch (st) {
    case MMM_OK: return "ok";
    case MMM_ERR_INVALID_ARG: return "invalid argument";
    case MMM_ERR_SHAPE: return "invalid shape";
    case MMM_ERR_DTYPE: return "invalid element type or alignment";
    case MMM_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case MMM_ERR_MAPS_MISMATCH: return "maps not built or built for different inputs";
    case MMM_ERR_DEVICE: return "device error";
    }
    return "unknown status";
}

mmm_status mmm_maps_workspace_bytes(int64_t M, int64_t K, int64_t N, int32_t block_width, size_t *bytes)
{
    if (bytes == nullptr) return MMM_ERR_INVALID_ARG;
    if (!shape_ok(M, K, N, block_width)) return MMM_ERR_SHAPE;
    *bytes = make_layout(M, K, N, block_width, true).total;
    return MMM_OK;
}

mmm_status mmm_maps_workspace_bytes_for(int64_t M, int64_t K, int64_t N, int32_t block_width, mmm_dtype dt, size_t *bytes)
{
    if (bytes == nullptr) return MMM_ERR_INVALID_ARG;
    if (!shape_ok(M, K, N, block_width)) return MMM_ERR_SHAPE;
    if (!dtype_ok(dt)) return MMM_ERR_DTYPE;
    *bytes = make_layout(M, K, N, block_width, dt == MMM_F32).total;
    return MMM_OK;
}

mmm_status mmm_maps_init(void *dev_workspace, size_t workspace_bytes, int64_t M, int64_t K, int64_t N,
                         int32_t block_width, mmm_maps **out)
{
    if (out == nullptr) return MMM_ERR_INVALID_ARG;
    if (!shape_ok(M, K, N, block_width)) return MMM_ERR_SHAPE;
    Layout l = make_layout(M, K, N, block_width, true);
    const bool parts_room = workspace_bytes >= l.total;
    if (!parts_room) l = make_layout(M, K, N, block_width, false);
    if (dev_workspace == nullptr || reinterpret_cast<uintptr_t>(dev_workspace) % kAlign != 0 ||
        workspace_bytes < l.total)
        return MMM_ERR_WORKSPACE;
    mmm_captures *captures = new (std::nothrow) mmm_captures();
    mmm_maps *m = captures != nullptr ? new (std::nothrow) mmm_maps() : nullptr;
    if (m == nullptr) {
        delete captures;
        return MMM_ERR_INVALID_ARG;
    }
    m->captures = captures;
    m->M = M;
    m->K = K;
    m->N = N;
    m->bw = block_width;
    m->NB = N / block_width;
    m->WA = (K + 63) / 64;
    m->WB = (m->NB + 63) / 64;
    m->MT = (M + MMM_COLANY_ROWS - 1) / MMM_COLANY_ROWS;
    char *base = static_cast<char *>(dev_workspace);
    m->a_bits = reinterpret_cast<uint64_t *>(base + l.a_bits);
    m->a_colany = reinterpret_cast<uint64_t *>(base + l.a_colany);
    m->MBA = (M + MMM_AB_ROWS - 1) / MMM_AB_ROWS;
    m->KBA = (K + MMM_AB_COLS - 1) / MMM_AB_COLS;
    m->a_cnt = reinterpret_cast<uint32_t *>(base + l.a_cnt);
    m->NG = (N + MMM_GROUP_COLS - 1) / MMM_GROUP_COLS;
    m->a_img = base + l.a_img;
    m->a_wild = reinterpret_cast<uint8_t *>(base + l.a_wild);
    m->a_img64 = base + l.a_ent;
    m->a_ent = reinterpret_cast<uint64_t *>(base + l.a_ent);
    m->b_bits = reinterpret_cast<uint64_t *>(base + l.b_bits);
    m->bt_bits = reinterpret_cast<uint64_t *>(base + l.bt_bits);
    m->stats = reinterpret_cast<uint64_t *>(base + l.stats);
    m->kinfo = reinterpret_cast<uint32_t *>(base + l.kinfo);
    m->kmap = reinterpret_cast<uint32_t *>(base + l.kmap);
    m->a_colany_c = reinterpret_cast<uint64_t *>(base + l.a_colany_c);
    m->btc_bits = reinterpret_cast<uint64_t *>(base + l.btc_bits);
    m->rows_copy = reinterpret_cast<uint64_t *>(base + l.rows_copy);
    m->bp_val = base + l.bp_val;
    m->bp_list = reinterpret_cast<uint16_t *>(base + l.bp_list);
    m->bp_cnt = reinterpret_cast<uint32_t *>(base + l.bp_cnt);
    m->partials = reinterpret_cast<float *>(base + l.partials);
    m->partial_bytes = l.partial_bytes;
    m->parts_room = parts_room;
    m->ws = dev_workspace;
    m->ws_bytes = workspace_bytes;
    m->a_built = m->b_built = false;
    m->a_compact = m->b_compact = false;
    m->bt_state = BT_MADE;
    m->bt_event = nullptr;
    m->build_captured = false;
    m->a_dtype = m->b_dtype = -1;
    m->a_form = m->b_form = MMM_FORM_PLAIN;
    m->form_captured = MMM_FORM_PLAIN;
    m->form_valid = false;
    m->a_src = nullptr;
    m->a_src_ld = 0;
    m->b_src = nullptr;
    m->b_src_ld = 0;
    m->plan_variant = -1;
    m->plan_split = 0;
    m->plan_path = -1;
    m->stats_a_valid = m->stats_b_valid = false;
    m->stats_active = 1.0;
    m->stats_marked_a = m->stats_marked_b = 0.0;
    m->stats_nnz_a = m->stats_occ_b = m->stats_macs = m->stats_rows_b = m->stats_version = 0;
    m->plan_valid = false;
    *out = m;
    return MMM_OK;
}

void mmm_maps_release(mmm_maps *maps)
{
    if (maps == nullptr) return;
    if (maps->bt_event != nullptr) (void)hipEventDestroy(maps->bt_event);
    release_captures(maps->captures);
    delete maps;
}

mmm_status mmm_build_maps(mmm_maps *maps, mmm_dtype dt, const void *X, int64_t ldx, const mmm_mask_a *ma,
                          const void *Y, int64_t ldy, const mmm_mask_b *mb, void *hip_stream)
{
    if (maps == nullptr || (X == nullptr && Y == nullptr)) return MMM_ERR_INVALID_ARG;
    if (!dtype_ok(dt)) return MMM_ERR_DTYPE;
    const size_t esz = elem_size(dt);
    mmm_build_args a{};
    a.dtype = dt;
    if (X != nullptr) {
        if (ma == nullptr) return MMM_ERR_INVALID_ARG;
        if (ma->pred < MMM_PRED_NONZERO || ma->pred > MMM_PRED_ABS_GT) return MMM_ERR_INVALID_ARG;
        if (ldx < maps->K || ldx > kMaxLd) return MMM_ERR_SHAPE;
        if (reinterpret_cast<uintptr_t>(X) % esz != 0) return MMM_ERR_DTYPE;
        if (ma->keep_bits != nullptr && reinterpret_cast<uintptr_t>(ma->keep_bits) % 8 != 0) return MMM_ERR_INVALID_ARG;
        a.X = X;
        a.ldx = ldx;
        a.pred = ma->pred;
        a.threshold = ma->threshold;
        a.keep_a = ma->keep_bits;
    }
    if (Y != nullptr) {
        if (mb == nullptr) return MMM_ERR_INVALID_ARG;
        if (mb->block_width != maps->bw) return MMM_ERR_SHAPE;
        if (ldy < maps->N || ldy > kMaxLd) return MMM_ERR_SHAPE;
        if (reinterpret_cast<uintptr_t>(Y) % esz != 0) return MMM_ERR_DTYPE;
        if ((mb->keep_rows != nullptr && reinterpret_cast<uintptr_t>(mb->keep_rows) % 8 != 0) ||
            (mb->keep_blocks != nullptr && reinterpret_cast<uintptr_t>(mb->keep_blocks) % 8 != 0))
            return MMM_ERR_INVALID_ARG;
        a.Y = Y;
        a.ldy = ldy;
        a.keep_rows = mb->keep_rows;
        a.keep_blocks = mb->keep_blocks;
    }
    // Row-compacted mode: when keep_rows switches whole rows of B off, the live rows are numbered k' and the
    // matrix kernel walks k' (steps of 128 live rows instead of 128 rows of which few are live).  A is then laid
    // out over k', so its image is only good for the numbering it was made for.
    a.b_compact = Y != nullptr && mb->keep_rows != nullptr && dt != MMM_F64;
    const bool compact_after = Y != nullptr ? a.b_compact : maps->b_compact;
    a.a_compact = X != nullptr && compact_after;
    a.form = choose_form(maps, a);
    if (form_is_captured(maps, dt, static_cast<hipStream_t>(hip_stream))) capture_form(maps, a.form, static_cast<hipStream_t>(hip_stream));
    if (hipError_t e = mmm_launch_build(maps, a, static_cast<hipStream_t>(hip_stream)); e != hipSuccess) {
        note_device_error("map builder launch", e);
        return MMM_ERR_DEVICE;
    }
    if (Y != nullptr) {
        // an image of A made for another numbering of k (or for none) do not fit the new B side
        if (X == nullptr && (maps->b_compact || a.b_compact)) maps->a_built = false;
        maps->b_compact = a.b_compact;
        maps->b_form = a.form;
        maps->bt_state = a.b_compact ? BT_MISSING : BT_MADE;
        if (a.b_compact && !maps->build_captured) maps->build_captured = capturing(static_cast<hipStream_t>(hip_stream));
        if (a.b_compact && (maps->M <= 64 || choose_path(maps, dt, a.form) == MMM_PATH_PAIRS)) {
            if (hipError_t e = mmm_launch_expand_rows(maps, static_cast<hipStream_t>(hip_stream)); e != hipSuccess) {
                note_device_error("transposed map launch", e);
                return MMM_ERR_DEVICE;
            }
            maps->bt_state = BT_MADE;
        }
    }
    if (X != nullptr) {
        maps->a_compact = a.a_compact;
        maps->a_form = a.form;
        maps->a_built = true;
        maps->a_dtype = dt;
        maps->a_src = X;   // compared, never dereferenced
        maps->a_src_ld = ldx;
    }
    if (Y != nullptr) {
        maps->b_built = true;
        maps->b_dtype = dt;
        maps->b_src = Y;   // compared, never dereferenced
        maps->b_src_ld = ldy;
    }
    return MMM_OK;
}

mmm_status mmm_maps_view(const mmm_maps *maps, const uint64_t **a_bits, int64_t *a_row_words,
                         const uint64_t **b_bits, int64_t *b_row_words)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (a_bits) *a_bits = maps->a_bits;
    if (a_row_words) *a_row_words = maps->WA;
    if (b_bits) *b_bits = maps->b_bits;
    if (b_row_words) *b_row_words = maps->WB;
    return MMM_OK;
}

mmm_status mmm_maps_view_derived(const mmm_maps *maps, const uint64_t **a_colany, const uint64_t **bt_bits,
                                 int64_t *k_words)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (a_colany) *a_colany = maps->a_colany;
    if (bt_bits) *bt_bits = maps->bt_bits;
    if (k_words) *k_words = maps->WA;
    if (bt_bits != nullptr && maps->b_built && maps->b_compact && (maps->bt_state != BT_MADE || maps->build_captured)) {
        if (mmm_status st = make_for_inspection("transposed map", maps, mmm_launch_expand_rows); st != MMM_OK) return st;
        std::lock_guard<std::mutex> lock(maps->bt_mutex);
        maps->bt_state = BT_MADE;
    }
    return MMM_OK;
}

mmm_status mmm_maps_view_compacted(const mmm_maps *maps, int32_t *on, const uint32_t **live_count, const uint32_t **kmap,
                                   const uint64_t **a_colany_c, const uint64_t **btc_bits)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (on) *on = maps->b_compact ? 1 : 0;
    if (live_count) *live_count = maps->kinfo;
    if (kmap) *kmap = maps->kmap;
    if (a_colany_c) *a_colany_c = maps->a_colany_c;
    if (btc_bits) *btc_bits = maps->btc_bits;
    if (a_colany_c != nullptr && maps->a_built && maps->a_compact)
        return make_for_inspection("column-any words over the live rows", maps, mmm_launch_colany_compact);
    return MMM_OK;
}

mmm_status mmm_debug_k_lists(const mmm_maps *maps, void *out, size_t out_bytes, size_t *bytes_needed, void *hip_stream)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (!maps->a_built || !maps->b_built) return MMM_ERR_MAPS_MISMATCH;
    if (maps->a_dtype == MMM_F64 || !mmm_packs(maps->M, maps->b_dtype)) return MMM_ERR_DTYPE;
    size_t need = 0;
    const hipError_t e = mmm_launch_dump_lists(maps, static_cast<uint8_t *>(out), out_bytes, &need,
                                               static_cast<hipStream_t>(hip_stream));
    if (bytes_needed) *bytes_needed = need;
    if (e == hipErrorInvalidValue) return out == nullptr && bytes_needed != nullptr ? MMM_OK : MMM_ERR_WORKSPACE;
    if (e != hipSuccess) {
        note_device_error("k list dump launch", e);
        return MMM_ERR_DEVICE;
    }
    return MMM_OK;
}

mmm_status mmm_maps_view_lists(const mmm_maps *maps, const uint32_t **counts, const uint64_t **entries,
                               int64_t *blocks_m, int64_t *blocks_k, int64_t *capacity)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (counts) *counts = maps->a_cnt;
    if (entries) *entries = maps->a_ent;
    if (blocks_m) *blocks_m = maps->MBA;
    if (blocks_k) *blocks_k = maps->KBA;
    if (capacity) *capacity = MMM_AB_CAP;
    // the multiplication reads the image of A, not lists: they are made from the image
    if ((counts != nullptr || entries != nullptr) && maps->a_built && maps->a_dtype != MMM_F64)
        return make_for_inspection("lists of A", maps, mmm_launch_lists);
    return MMM_OK;
}

mmm_status mmm_maps_stats(const mmm_maps *maps, uint64_t *nnz_a, uint64_t *occupied_blocks_b,
                          uint64_t *useful_macs, void *hip_stream)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (!maps->a_built || !maps->b_built) return MMM_ERR_MAPS_MISMATCH;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    hipError_t e = mmm_launch_stats(maps, s);
    uint64_t host[MMM_STATS_WORDS] = {};
    if (e == hipSuccess) e = hipMemcpyAsync(host, maps->stats, sizeof(host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        note_device_error("statistics", e);
        return MMM_ERR_DEVICE;
    }
    maps->stats_nnz_a = host[0];
    maps->stats_occ_b = host[1];
    maps->stats_macs = host[2];
    maps->stats_rows_b = host[3];
    maps->stats_active = host[5] != 0 ? (double)host[4] / ((double)host[5] * (double)maps->MBA) : 1.0;
    const double steps = (double)((host[5] + MMM_AB_COLS - 1) / MMM_AB_COLS);
    maps->stats_marked_a = host[6] != 0 ? (double)host[6] / (steps * (double)maps->MBA) : 0.0;
    maps->stats_marked_b = host[7] != 0 ? (double)host[7] / (steps * (double)maps->NG) : 0.0;
    ++maps->stats_version;
    maps->stats_a_valid = maps->stats_b_valid = true;
    if (nnz_a) *nnz_a = host[0];
    if (occupied_blocks_b) *occupied_blocks_b = host[1];
    if (useful_macs) *useful_macs = host[2];
    return MMM_OK;
}

mmm_status mmm_matmul_plan(const mmm_maps *maps, mmm_dtype dt, int32_t *variant, int32_t *split_k, int64_t *workgroups)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (!dtype_ok(dt)) return MMM_ERR_DTYPE;
    const mmm_plan p = make_plan(maps, dt, form_of(maps, dt));
    if (variant) *variant = p.variant;
    if (split_k) *split_k = p.split_k;
    if (workgroups) *workgroups = p.workgroups;
    return MMM_OK;
}

}   // extern "C"

static mmm_status matmul_common(const mmm_maps *maps, mmm_dtype dt, const void *X, int64_t ldx, const void *Y, int64_t ldy,
                                void *C, int64_t ldc, int32_t accumulate, void *hip_stream, bool static_scratch)
{
    if (maps == nullptr || X == nullptr || Y == nullptr || C == nullptr) return MMM_ERR_INVALID_ARG;
    if (!dtype_ok(dt)) return MMM_ERR_DTYPE;
    if (ldx < maps->K || ldy < maps->N || ldc < maps->N) return MMM_ERR_SHAPE;
    if (ldx > kMaxLd || ldy > kMaxLd) return MMM_ERR_SHAPE;   // tile-relative offsets are 32-bit
    const size_t esz = elem_size(dt);
    if (reinterpret_cast<uintptr_t>(X) % esz != 0 || reinterpret_cast<uintptr_t>(Y) % esz != 0 ||
        reinterpret_cast<uintptr_t>(C) % c_elem_size(dt) != 0)
        return MMM_ERR_DTYPE;
    if (dt == MMM_F64 && !mmm_pairs_supports(dt, ldy)) return MMM_ERR_SHAPE;   // for every double Y, whichever kernel it is
    if (!maps->a_built || !maps->b_built) return MMM_ERR_MAPS_MISMATCH;
    if (maps->a_dtype != dt || maps->b_dtype != dt) return MMM_ERR_MAPS_MISMATCH;
    // the values of A travel in the image that was made from X at build time: another X is another A
    if (maps->a_src != X || maps->a_src_ld != ldx) return MMM_ERR_MAPS_MISMATCH;
    // The matrix kernel has the values of B in the packed form that was made from Y at build time; the pair kernel reads the
    // Y it is given, so that is what another Y (or the same at another leading dimension) is multiplied by.
    const bool packed_y = maps->b_src == Y && maps->b_src_ld == ldy, pairs_can = mmm_pairs_supports(dt, ldy);
    if (!packed_y && !pairs_can) return MMM_ERR_MAPS_MISMATCH;
    if (pairs_can && (!packed_y || choose_path(maps, dt, maps->b_form) == MMM_PATH_PAIRS)) {   // no scratch at all on this path
        hipError_t e = ensure_bt(maps, static_cast<hipStream_t>(hip_stream));
        if (e == hipSuccess)
            e = mmm_launch_pairs(maps, dt, X, ldx, Y, ldy, C, ldc, accumulate ? 1 : 0, false, 0, 0.f, nullptr,
                                 static_cast<hipStream_t>(hip_stream));
        if (e != hipSuccess) {
            note_device_error("masked GEMM (pairs) launch", e);
            return MMM_ERR_DEVICE;
        }
        return MMM_OK;
    }
    const mmm_plan p = make_plan(maps, dt, maps->b_form);
    if (form_is_captured(maps, dt, static_cast<hipStream_t>(hip_stream))) capture_form(maps, maps->b_form, static_cast<hipStream_t>(hip_stream));
    void *partials = maps->partials;
    size_t partial_bytes = maps->partial_bytes;
    if (static_scratch) {
        const size_t need = p.split_k > 1 ? (size_t)p.split_k * (size_t)maps->M * (size_t)maps->N * c_elem_size(dt) : 0;
        if (need > (size_t)MMM_STATIC_SCRATCH_BYTES) {
            std::snprintf(g_detail, sizeof(g_detail),
                          "mmm_matmul_static_scratch: %d partial sums of C need %zu bytes, the static scratch holds %zu",
                          (int)p.split_k, need, (size_t)MMM_STATIC_SCRATCH_BYTES);
            return MMM_ERR_WORKSPACE;
        }
        if (hipError_t e = mmm_static_scratch(reinterpret_cast<float **>(&partials)); e != hipSuccess) {
            note_device_error("address of the static scratch", e);
            return MMM_ERR_DEVICE;
        }
        partial_bytes = (size_t)MMM_STATIC_SCRATCH_BYTES;
    }
    if (hipError_t e = mmm_launch_matmul(maps, p, dt, C, ldc, accumulate ? 1 : 0, partials, partial_bytes,
                                         static_cast<hipStream_t>(hip_stream));
        e != hipSuccess) {
        note_device_error("masked GEMM launch", e);
        return MMM_ERR_DEVICE;
    }
    return MMM_OK;
}

extern "C" {

mmm_status mmm_matmul(const mmm_maps *maps, mmm_dtype dt, const void *X, int64_t ldx, const void *Y, int64_t ldy,
                      void *C, int64_t ldc, int32_t accumulate, void *hip_stream)
{
    return matmul_common(maps, dt, X, ldx, Y, ldy, C, ldc, accumulate, hip_stream, false);
}

mmm_status mmm_matmul_fused(const mmm_maps *maps, mmm_dtype dt, const void *X, int64_t ldx, const mmm_mask_a *ma,
                            const void *Y, int64_t ldy, void *C, int64_t ldc, int32_t accumulate, void *hip_stream)
{
    if (maps == nullptr || X == nullptr || Y == nullptr || C == nullptr || ma == nullptr) return MMM_ERR_INVALID_ARG;
    if (ma->pred < MMM_PRED_NONZERO || ma->pred > MMM_PRED_ABS_GT) return MMM_ERR_INVALID_ARG;
    if (ma->keep_bits != nullptr && reinterpret_cast<uintptr_t>(ma->keep_bits) % 8 != 0) return MMM_ERR_INVALID_ARG;
    if (!dtype_ok(dt)) return MMM_ERR_DTYPE;
    if (ldx < maps->K || ldy < maps->N || ldc < maps->N) return MMM_ERR_SHAPE;
    if (ldx > kMaxLd || ldy > kMaxLd) return MMM_ERR_SHAPE;
    const size_t esz = elem_size(dt);
    if (reinterpret_cast<uintptr_t>(X) % esz != 0 || reinterpret_cast<uintptr_t>(Y) % esz != 0 ||
        reinterpret_cast<uintptr_t>(C) % c_elem_size(dt) != 0)
        return MMM_ERR_DTYPE;
    if (!mmm_pairs_supports(dt, ldy)) return MMM_ERR_SHAPE;
    if (!maps->b_built || maps->b_dtype != dt) return MMM_ERR_MAPS_MISMATCH;
    hipError_t e = ensure_bt(maps, static_cast<hipStream_t>(hip_stream));
    if (e == hipSuccess)
        e = mmm_launch_pairs(maps, dt, X, ldx, Y, ldy, C, ldc, accumulate ? 1 : 0, true, ma->pred, ma->threshold, ma->keep_bits,
                             static_cast<hipStream_t>(hip_stream));
    if (e != hipSuccess) {
        note_device_error("fused masked GEMM launch", e);
        return MMM_ERR_DEVICE;
    }
    return MMM_OK;
}

mmm_status mmm_matmul_static_scratch(const mmm_maps *maps, mmm_dtype dt, const void *X, int64_t ldx, const void *Y,
                                     int64_t ldy, void *C, int64_t ldc, int32_t accumulate, void *hip_stream)
{
    return matmul_common(maps, dt, X, ldx, Y, ldy, C, ldc, accumulate, hip_stream, true);
}

mmm_status mmm_maps_set_plan(mmm_maps *maps, int32_t variant, int32_t split_k)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (variant < -1 || variant >= mmm_variant_count()) return MMM_ERR_INVALID_ARG;
    if (split_k < 0 || split_k > 4096) return MMM_ERR_INVALID_ARG;
    maps->plan_variant = variant;
    maps->plan_split = split_k;
    return MMM_OK;
}

mmm_status mmm_maps_set_path(mmm_maps *maps, int32_t path)
{
    if (maps == nullptr) return MMM_ERR_INVALID_ARG;
    if (path < -1 || path > MMM_PATH_PAIRS) return MMM_ERR_INVALID_ARG;
    maps->plan_path = path;
    return MMM_OK;
}

mmm_status mmm_matmul_path(const mmm_maps *maps, int32_t *path)
{
    if (maps == nullptr || path == nullptr) return MMM_ERR_INVALID_ARG;
    const int32_t dt = maps->a_built ? maps->a_dtype : maps->b_built ? maps->b_dtype : MMM_F32;
    *path = choose_path(maps, dt, form_of(maps, dt));
    return MMM_OK;
}

mmm_status mmm_matmul_form(const mmm_maps *maps, int32_t *form)
{
    if (maps == nullptr || form == nullptr) return MMM_ERR_INVALID_ARG;
    *form = maps->b_built ? maps->b_form : maps->a_built ? maps->a_form : MMM_FORM_PLAIN;
    return MMM_OK;
}

mmm_status mmm_set_option(const char *name, int64_t value)
{
    if (name == nullptr) return MMM_ERR_INVALID_ARG;
    if (std::strcmp(name, "matmul_path") == 0) {
        if (value < -1 || value > MMM_PATH_PAIRS) return MMM_ERR_INVALID_ARG;
        g_opt_path.store(value);
        return MMM_OK;
    }
    if (std::strcmp(name, "matmul_variant") == 0) {
        if (value < -1 || value >= mmm_variant_count()) return MMM_ERR_INVALID_ARG;
        g_opt_variant.store(value);
        return MMM_OK;
    }
    if (std::strcmp(name, "float_form") == 0) {
        if (value < -1 || value > MMM_FORM_PARTS) return MMM_ERR_INVALID_ARG;
        g_opt_form.store(value);
        return MMM_OK;
    }
    if (std::strcmp(name, "split_k") == 0) {
        if (value < 0 || value > 4096) return MMM_ERR_INVALID_ARG;
        g_opt_split.store(value);
        return MMM_OK;
    }
    return MMM_ERR_INVALID_ARG;
}

const char *mmm_last_device_error(void) { return g_detail; }

int32_t mmm_matmul_variant_count(void) { return mmm_variant_count(); }

const char *mmm_matmul_variant_name(int32_t i)
{
    if (i < 0 || i >= mmm_variant_count()) return nullptr;
    return mmm_variant(i).name;
}

}   // extern "C"
