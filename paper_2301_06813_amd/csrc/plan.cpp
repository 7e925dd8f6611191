// plan.cpp -- choice of output tile and reduction splits for the bf16 and fp32
// GEMMs.
//
// A launch fills MI355X's 256 compute units only if it has enough
// workgroups; many local shares of an SBP linear have small outputs and long
// reductions (e.g. a weight gradient of 1024 x 384 over 8192 tokens), so the
// planner trades tile size (MFMA efficiency per workgroup) against the
// number of workgroups and splits of the reduction. It evaluates a small
// analytic time model for every (tile, splits) candidate and keeps the
// fastest. Pure host code.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <new>
#include <unordered_map>

#include "gemm.h"
#include "model_instances.h"

namespace sbpi {

namespace {

// Generic kernel (register-staged): time of one 64-wide reduction step of a
// work item on a compute unit, measured on products with odd leading
// dimensions (see plan_generic).
struct GenericTile {
    int bm, bn;
    double step;
};
const GenericTile kGeneric[] = {
    {256, 128, 1.40e-6}, {128, 256, 1.40e-6}, {128, 128, 0.70e-6},
    {128, 64, 0.50e-6},  {64, 128, 0.50e-6},  {64, 64, 0.33e-6},
};
// Pipelined instances the model chooses among, with their times on MI355X in us:
// a 64-wide reduction step of a work item alone on its compute unit (`step[0]`),
// its share of the unit when two workgroups take turns there (`step[1]`) and when
// three or more do (`step[2]`; `res` at most), and the end of an item, `end`:
// what it takes however few items there are, then what the stores of an fp32 or
// a bf16 tile add when the whole chip stores (in proportion below one item per
// unit), what each adds where rows are not whole 64-byte blocks, what loading the
// old values adds where the product is added to its output, and what an item takes
// more in the shifted form, and there where rows are cut (0: has no such form).
//
// Fitted on 1483 random products and 1269 random backward pairs, each on some 40
// plans (measured from graphs of calls over three sets of operands in turn):
// extents log-uniform in 64 .. 8192, 60 % multiples of 64 and the others of 8, up
// to 2e11 operations; three orientations, fp32 and bf16 outputs, a third
// accumulating, a fifth batched as in attention (2 to 128 items of 64 .. 2048 rows).
// Fitted to the plans' times and to the time of the plan chosen: 9 % rms over
// plans within 1.5 times of the best. On 688 products and 591 pairs not fitted, the
// plan chosen takes 2.0 % (pairs 3.2 %) longer than the fastest measured on
// average, 6 % (10 %) at the ninth decile, 15 % (29 %) at the 99th percentile and
// 44 % (60 %) at worst. With the constants before, which knew neither rows cut by
// 64-byte blocks, nor chips part filled, nor the accumulating forms, it took 6.0 %
// (7.7 %) longer on average. The last two columns were fitted on 600 products in
// the shifted form (odd extents of 64 .. 4096); on 600 others the plan chosen takes
// 3.1 % longer than the fastest on average, without them 8.9 %.
struct PipeClass {
    int bm, bn, code, res;
    double step[3];
    struct {
        double least, f32, bf16, cut_f32, cut_bf16, add, shifted, cut_shifted;
    } end;
};
constexpr PipeClass kPipe[] = {
    {64, 64, 1, 2, {0.394, 0.241, 0.241}, {0.65, 0.14, 0.16, 0.22, 0.22, 0.07, 1.0, -0.3}},
    {64, 64, 4, 5, {0.418, 0.312, 0.233}, {0.13, 0.29, 0.24, 0.17, 0.15, 0.18, 0.0, 0.0}},
    {64, 64, 12, 1, {0.207, 0.207, 0.207}, {1.34, 0.75, 0.54, 0.32, 0.54, 0.07, 1.9, 1.8}},
    {64, 128, 4, 3, {0.760, 0.356, 0.339}, {0.79, 0.30, 0.24, 1.01, 0.58, 0.05, 0.0, 0.0}},
    {64, 128, 12, 1, {0.409, 0.409, 0.409}, {1.78, 1.26, 0.51, 0.25, 0.64, 0.36, 1.4, 2.8}},
    {128, 64, 4, 3, {0.755, 0.334, 0.309}, {0.60, 0.33, 0.21, 0.73, 0.22, 0.19, 0.0, 0.0}},
    {128, 64, 12, 1, {0.367, 0.367, 0.367}, {1.87, 1.24, 0.59, 0.29, 0.70, 0.30, 2.0, 3.6}},
    {128, 128, 4, 2, {0.792, 0.388, 0.388}, {2.07, 0.13, 0.28, 2.38, 1.07, 0.98, 1.0, 0.4}},
    {128, 128, 12, 1, {0.502, 0.502, 0.502}, {2.45, 1.70, 0.98, 0.56, 0.60, 1.75, 2.7, 7.7}},
    {256, 192, 1, 1, {1.061, 1.061, 1.061}, {3.75, 2.37, 3.33, 9.27, 5.25, 2.26, 0.0, 0.0}},
    {256, 256, 1, 1, {1.405, 1.405, 1.405}, {4.37, 2.58, 3.90, 10.89, 7.28, 3.67, 0.0, 0.0}},
};

constexpr double kCUs = 256.0;
constexpr double kFixed = 1.7;         // a launch (us)
constexpr double kHbm = 8.1e6;         // bytes per us, of which the compute units' time
constexpr double kOverlap = 0.17;      // hides all but this share of the smaller
constexpr double kReduce = 2.15;       // the split reduction's launch (us), ...
constexpr double kReduceLoads = 0.30;  // each four slices it reads one after another
constexpr double kReduceRate = 4.45e6; // and its bytes per us, partials written and read

thread_local int ov_bm = 0, ov_bn = 0, ov_splits = 1, ov_kernel = 0, ov_occ = 0;
thread_local int ov_orients = 7;   // orientations the override applies to (bit per Orient)
thread_local int ov_bwd_mode = 0, ov_bwd_splits_w = 1;   // see set_bwd_override

// Pipelined instances reachable through the plan override, by kernel code
// (see sbp_set_plan_override): code, tile, stages (0 = the tile's default),
// reduction groups, epilogue.
struct Instance {
    int code, bm, bn, ns, kg, epi, bk = 64;
};
using sbpk::EPI_DIRECT;
using sbpk::EPI_ROWQ;
using sbpk::EPI_STAGED;

constexpr Instance kInstances[] = {
    {1, 256, 256, 0, 1, EPI_DIRECT}, {1, 256, 192, 0, 1, EPI_DIRECT},
    {1, 256, 128, 0, 1, EPI_DIRECT}, {1, 128, 256, 0, 1, EPI_DIRECT},
    {1, 128, 128, 0, 1, EPI_DIRECT}, {1, 128, 64, 0, 1, EPI_DIRECT},
    {1, 64, 128, 0, 1, EPI_DIRECT},  {1, 64, 64, 0, 1, EPI_DIRECT},
    {4, 128, 128, 2, 1, EPI_DIRECT}, {5, 256, 128, 0, 2, EPI_STAGED},
    {5, 128, 256, 0, 2, EPI_STAGED}, {5, 128, 128, 0, 2, EPI_STAGED}, {6, 256, 256, 0, 1, EPI_ROWQ},
    {6, 128, 128, 2, 1, EPI_ROWQ},   {7, 256, 128, 0, 2, EPI_ROWQ},   {7, 128, 256, 0, 2, EPI_ROWQ},
    {7, 128, 128, 0, 2, EPI_ROWQ},   {8, 256, 256, 5, 1, EPI_DIRECT, 32},
    {9, 256, 128, 6, 2, EPI_STAGED, 32}, {9, 128, 256, 6, 2, EPI_STAGED, 32},
    {9, 128, 128, 8, 2, EPI_STAGED, 32}, {10, 128, 128, 2, 2, EPI_STAGED},
    {4, 128, 64, 2, 1, EPI_DIRECT},      {4, 64, 128, 2, 1, EPI_DIRECT},
    {4, 64, 64, 2, 1, EPI_DIRECT},       {11, 128, 64, 6, 1, EPI_DIRECT},
    {11, 64, 128, 6, 1, EPI_DIRECT},     {11, 64, 64, 8, 1, EPI_DIRECT},
    {5, 128, 64, 0, 2, EPI_STAGED},      {5, 64, 128, 0, 2, EPI_STAGED},
    {5, 64, 64, 0, 2, EPI_STAGED},       {7, 128, 64, 0, 2, EPI_ROWQ},
    {7, 64, 128, 0, 2, EPI_ROWQ},        {7, 64, 64, 0, 2, EPI_ROWQ},
    {12, 128, 128, 2, 2, EPI_STAGED, 128}, {12, 128, 64, 3, 2, EPI_STAGED, 128},
    {12, 64, 128, 3, 2, EPI_STAGED, 128},  {12, 64, 64, 4, 2, EPI_STAGED, 128},
    {13, 128, 128, 2, 2, EPI_ROWQ, 128},   {13, 128, 64, 3, 2, EPI_ROWQ, 128},
    {13, 64, 128, 3, 2, EPI_ROWQ, 128},    {13, 64, 64, 4, 2, EPI_ROWQ, 128},
};

// kPipe names each instance of SBP_MODEL_INSTANCES (those with the grouped
// attention launch and the accumulating form) once, and no other.
constexpr bool model_lists_agree() {
    struct Row {
        int bm, bn, bk, ns, kg, epi;
    };
#define SBP_ROW(BM_, BN_, BKD_, NS_, WGM_, WGN_, KG_, EPI_) {BM_, BN_, BKD_, NS_, KG_, EPI_},
    const Row rows[] = {SBP_MODEL_INSTANCES(SBP_ROW)};
#undef SBP_ROW
    constexpr int N = sizeof(rows) / sizeof(rows[0]);
    bool used[N] = {};
    int n = 0;
    for (const PipeClass &c : kPipe)
        for (const Instance &i : kInstances) {
            if (i.code != c.code || i.bm != c.bm || i.bn != c.bn) continue;
            for (int r = 0; r < N; ++r)
                if (rows[r].bm == i.bm && rows[r].bn == i.bn && rows[r].bk == i.bk &&
                    (i.ns == 0 || rows[r].ns == i.ns) && rows[r].kg == i.kg &&
                    rows[r].epi == i.epi) {
                    n += !used[r];
                    used[r] = true;
                    break;   // the first match is the one launched
                }
        }
    return n == N && n == (int)(sizeof(kPipe) / sizeof(kPipe[0]));
}
static_assert(model_lists_agree(), "kPipe and SBP_MODEL_INSTANCES list different instances");

// Plans measured fastest on MI355X for the local products of the paper's
// workloads (generated by paper_2301_06813_amd/tune.py): orientation, fp32
// output, m, n, k, pipelined-kernel eligibility -> tile, kernel code, splits,
// persistent workgroups per CU. Other products use the model below.
struct Tuned {
    int orient, out_f32;
    int64_t m, n, k;
    int dma, bm, bn, code, splits, occ;
    int64_t nbatch = 1;   // batched products (attention core): batches x heads
};
const Tuned kTuned[] = {
#include "tuned_plans.inc"
    {-1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}   // end marker
};

// Backward pairs measured fastest as one grouped launch: backward-data
// product (m, n, k, fp32 output), backward-weight product (same) -> shared
// tile and kernel code, splits of each product. Pairs not listed run as two
// launches where both products have tuned plans, else as the model expects to be
// faster (plan_bwd_uncached).
struct TunedBwd {
    int64_t md, nd, kd;
    int fd;
    int64_t mw, nw, kw;
    int fw, bm, bn, code, sd, sw;
};
const TunedBwd kTunedBwd[] = {
#include "tuned_bwd_plans.inc"
    {-1, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}   // end marker
};

// Instances with a shifted-index-space form (gemm_bf16_launch.h
// SBP_DMA_SHIFT_INSTANCES): tile, reduction step, stages (0: the tile's
// default), reduction groups, epilogue.
struct ShiftInstance {
    int bm, bn, bk, ns, kg, epi;
};
const ShiftInstance kShiftInstances[] = {
    {64, 64, 64, 0, 1, EPI_DIRECT},     {128, 128, 64, 2, 1, EPI_DIRECT},
    {64, 64, 128, 4, 2, EPI_STAGED},    {128, 64, 128, 3, 2, EPI_STAGED},
    {64, 128, 128, 3, 2, EPI_STAGED},   {128, 128, 128, 2, 2, EPI_STAGED},
};

bool shift_capable(int bm, int bn, int bk, int ns, int kg, int epi) {
    for (const ShiftInstance &i : kShiftInstances)
        if (i.bm == bm && i.bn == bn && i.bk == bk && i.ns == ns && i.kg == kg && i.epi == epi)
            return true;
    return false;
}
bool shift_capable(const Plan &p) { return shift_capable(p.bm, p.bn, p.bk, p.ns, p.kg, p.epi); }

const Instance *find_instance(int code, int bm, int bn) {
    for (const Instance &i : kInstances)
        if (i.code == code && i.bm == bm && i.bn == bn) return &i;
    return nullptr;
}

int kblocks(int64_t k) { return (int)((k + 63) / 64); }

// Splits actually launched when asking for s, and blocks per split.
void split_of(int kb_total, int s, int *splits, int *per) {
    if (kb_total <= 0) {
        *splits = 1;
        *per = 1;
        return;
    }
    s = std::max(1, std::min(s, kb_total));
    int p = (kb_total + s - 1) / s;
    *per = p;
    *splits = (kb_total + p - 1) / p;
}

// Workspace floats available to a product: the caller's, capped at the
// preferred size so that plans do not depend on workspaces beyond it.
double ws_budget(const Gemm &g) {
    return (double)std::min(g.ws_floats, WS_FLOATS_PREFERRED);
}

bool fits_ws(const Gemm &g, int splits) {
    if (splits == 1) return true;
    if (g.nbatch() > 1) return false;   // batched launches never split
    return (double)splits * (double)g.m * (double)partial_ld(g.n) <= ws_budget(g);
}

double out_elem(const Gemm &g) { return g.out_dtype == DT_F32 ? 4.0 : 2.0; }

// Bytes read and written per element of the output.
double out_traffic(const Gemm &g) { return out_elem(g) * (g.accumulate ? 2.0 : 1.0); }

double algo_bytes(const Gemm &g) {
    return (2.0 * ((double)g.m * g.k + (double)g.k * g.n) + out_traffic(g) * g.m * g.n) *
           (double)g.nbatch();
}

double step_of(const PipeClass &c, double r) { return c.step[r > 2.0 ? 2 : r > 1.0 ? 1 : 0]; }

// Work items of a product under class c: their number, one's reduction steps and
// the time of its end (see PipeClass) where `q` items of the launch come on a unit.
double items_of(const Gemm &g, const PipeClass &c, int splits) {
    const double tiles = (double)((g.m + c.bm - 1) / c.bm) * (double)((g.n + c.bn - 1) / c.bn);
    return tiles * splits * (double)g.nbatch();
}
double end_of(const Gemm &g, const PipeClass &c, int splits, double q, bool shift) {
    const bool split = splits > 1, f32 = split || g.out_dtype == DT_F32;
    // a row is taken to be as long as the output is wide; partials have padded rows
    const bool cut = !split && std::fmod((double)g.n * out_elem(g), 64.0) != 0.0;
    double t = f32 ? c.end.f32 : c.end.bf16;
    if (cut) t += (f32 ? c.end.cut_f32 : c.end.cut_bf16) + (shift ? c.end.cut_shifted : 0.0);
    return c.end.least + std::min(1.0, q) * t + (g.accumulate && !split ? c.end.add : 0.0) +
           (shift ? c.end.shifted : 0.0);
}
double reduce_time(const Gemm &g, int splits) {
    return splits > 1 ? (4.0 * splits + out_traffic(g)) * g.m * g.n / kReduceRate : 0.0;
}

double reduce_loads(int splits) { return kReduceLoads * ((splits + 3) / 4); }

// Time t of the compute units beside `bytes` of memory traffic.
double overlapped(double t, double bytes) {
    const double h = bytes / kHbm;
    return std::max(t, h) + kOverlap * std::min(t, h);
}

// One product: the busiest unit's items in turn (beyond four the units even
// out), not faster than its bytes, then the split reduction.
double model_time(const Gemm &g, const PipeClass &c, int splits, int per, bool shift) {
    const double q = items_of(g, c, splits) / kCUs, busy = q > 4.0 ? q + 0.5 : std::ceil(q);
    const double r = std::min((double)c.res, std::ceil(q));
    const double t = busy * (per * step_of(c, r) + end_of(g, c, splits, q, shift));
    return kFixed + overlapped(t, algo_bytes(g)) +
           (splits > 1 ? kReduce + reduce_loads(splits) + reduce_time(g, splits) : 0.0);
}

// Two products sharing one grid: the longer items are dispatched first and
// the shorter fill in behind them. The whole lasts at least as long as the
// even share of a unit plus half a short item, and as one long item, whose
// steps wait for the other workgroups of its unit (0.78 of taking turns with all
// of them to the end: they finish sooner).
double model_pair(const Gemm &gd, const Gemm &gw, const PipeClass &c, int sd, int pd, int sw,
                  int pw, bool shift) {
    const double nd = items_of(gd, c, sd), nw = items_of(gw, c, sw);
    const double q = (nd + nw) / kCUs, r = std::min((double)c.res, std::ceil(q));
    const double step = step_of(c, r);
    const double ed = end_of(gd, c, sd, q, shift), ew = end_of(gw, c, sw, q, shift);
    const double cd = pd * step + ed, cw = pw * step + ew;
    const bool data_first = pd >= pw;
    const double n1 = data_first ? nd : nw, c1 = data_first ? cd : cw;
    const double c2 = data_first ? cw : cd;
    double t = std::max(c1, c2);
    if (q > 1.0)
        t = std::max(std::max(t, std::ceil(n1 / kCUs) * c1),
                     (nd * cd + nw * cw) / kCUs + 0.58 * c2);
    const double wait = std::max(c.step[0], r > 1.0 ? 0.78 * r * step : 0.0);
    t = std::max(t, std::max(pd * wait + ed, pw * wait + ew));
    return kFixed + overlapped(t, algo_bytes(gd) + algo_bytes(gw)) +
           (sd > 1 || sw > 1 ? kReduce + reduce_loads(std::max(sd, sw)) : 0.0) +
           reduce_time(gd, sd) + reduce_time(gw, sw);
}

}  // namespace

static bool pipe_class(int bm, int bn, int code) {
    for (const PipeClass &c : kPipe)
        if (c.bm == bm && c.bn == bn && c.code == code) return true;
    return false;
}

// Whether plan p adds to its output in the GEMM itself, which only the model's
// instances (and the generic kernel) have a form for; a split plan's reduction
// does it.
static bool adds(const Gemm &g, const Plan &p) { return g.accumulate && p.splits == 1; }

bool tile_supported(int bm, int bn, bool dma) {
    if (dma) {
        return find_instance(1, bm, bn) != nullptr;
    } else {
        for (const GenericTile &t : kGeneric)
            if (t.bm == bm && t.bn == bn) return true;
    }
    return false;
}

bool override_supported(int bm, int bn, int kernel) {
    if (kernel == 0 || kernel == 2) return tile_supported(bm, bn, true);
    return find_instance(kernel, bm, bn) != nullptr;
}

int kernel_code(const Plan &p) {
    if (!p.dma) return 2;
    for (const Instance &i : kInstances)
        if (i.bm == p.bm && i.bn == p.bn && i.kg == p.kg && i.epi == p.epi && i.bk == p.bk &&
            (i.ns == p.ns || (i.ns == 0 && p.ns == 0)))
            return i.code;
    return 1;
}

void set_override_occ(int occ) { ov_occ = occ < 0 ? 0 : occ; }

void set_override_orients(int mask) { ov_orients = mask & 7; }

void set_bwd_override(int mode, int splits_w) {
    ov_bwd_mode = mode;
    ov_bwd_splits_w = splits_w < 1 ? 1 : splits_w;
}

void set_override(int bm, int bn, int splits, int kernel) {
    ov_bm = bm;
    ov_bn = bn;
    ov_splits = std::max(1, splits);
    ov_kernel = kernel;
}

static bool kmajor_a(int orient) { return orient != OR_BWD_WEIGHT; }
static bool kmajor_b(int orient) { return orient == OR_BWD_DATA; }

int block_offset(const void *p) {
    return (int)((reinterpret_cast<uintptr_t>(p) >> 1) & 7);
}

bool dma_eligible(const Gemm &g) {
    if (g.in_dtype != DT_BF16) return false;
    // every row of an operand starts at the same offset within a 16-byte block
    if (g.lda % 8 || g.ldb % 8) return false;
    if ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B)) & 1) return false;
    const int oa = block_offset(g.A), ob = block_offset(g.B);
    if (g.nbatch() > 1) {
        // batched: every item's operand bases 16-byte aligned, ends on chunks
        if (oa || ob) return false;
        if (g.sa_b % 8 || g.sa_h % 8 || g.sb_b % 8 || g.sb_h % 8) return false;
        if ((kmajor_a(g.orient) ? g.k : g.m) % 8 || (kmajor_b(g.orient) ? g.k : g.n) % 8)
            return false;
    }
    // An offset along m or n shifts the output index; along the reduction
    // both operands must be k-major with the same offset (a k-major A with
    // an n-major B needs an aligned A).
    if (g.orient == OR_FWD && oa) return false;
    if (g.orient == OR_BWD_DATA && oa != ob) return false;
    // per-tile buffer offsets stay below 2^31 bytes
    return g.lda <= (int64_t(1) << 21) && g.ldb <= (int64_t(1) << 21);
}

int dma_mode(const Gemm &g) {
    if (!dma_eligible(g)) return 0;
    const int64_t a_contig = kmajor_a(g.orient) ? g.k : g.m;
    const int64_t b_contig = kmajor_b(g.orient) ? g.k : g.n;
    const bool aligned = block_offset(g.A) == 0 && block_offset(g.B) == 0 && a_contig % 8 == 0 &&
                         b_contig % 8 == 0;
    return aligned ? 1 : 2;
}

static Plan plan_uncached(const Gemm &g);
static Plan plan_model(const Gemm &g, double *time);

// Tuned entry of product g under pipelined-kernel mode `mode` (nullptr if none).
// The rows were measured storing their outputs: an unsplit one does not hold for
// a product that is added to its output (a split one's reduction does that).
static const Tuned *tuned_for(const Gemm &g, int mode) {
    if (g.in_dtype != DT_BF16) return nullptr;
    const int f32 = g.out_dtype == DT_F32 ? 1 : 0;
    for (const Tuned &t : kTuned) {
        if (t.orient < 0) break;
        if (t.orient == g.orient && t.out_f32 == f32 && t.m == g.m && t.n == g.n && t.k == g.k &&
            t.dma == mode && t.nbatch == g.nbatch() && !(g.accumulate && t.splits == 1))
            return &t;
    }
    return nullptr;
}

int device_cus() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            n <= 0)
            n = 256;
        cached[dev] = n;
    }
    return cached[dev];
}

namespace {
struct Key {
    int64_t v[11];
    bool operator==(const Key &o) const {
        for (int i = 0; i < 11; ++i)
            if (v[i] != o.v[i]) return false;
        return true;
    }
};
struct KeyHash {
    size_t operator()(const Key &k) const {
        size_t h = 1469598103934665603ull;
        for (int i = 0; i < 11; ++i) h = (h ^ (size_t)k.v[i]) * 1099511628211ull;
        return h;
    }
};
Key key_of(const Gemm &g, int mode) {
    return Key{{g.orient, g.in_dtype, g.out_dtype + 2 * (g.accumulate ? 1 : 0), g.m, g.n, g.k, mode,
                ov_bm * 1000 + ov_bn, ((ov_splits * 100 + ov_kernel) * 100 + ov_occ) * 8 + ov_orients,
                g.nbatch(), (int64_t)std::min(g.ws_floats, WS_FLOATS_PREFERRED)}};
}
thread_local std::unordered_map<Key, Plan, KeyHash> plan_cache;

struct PairKey {
    Key d, w;
    int64_t bwd;   // the backward override
    bool operator==(const PairKey &o) const { return d == o.d && w == o.w && bwd == o.bwd; }
};
struct PairHash {
    size_t operator()(const PairKey &k) const {
        return (KeyHash()(k.d) * 31 + KeyHash()(k.w)) * 31 + (size_t)k.bwd;
    }
};
struct PairPlan {
    bool grouped;
    Plan d{}, w{};
};
thread_local std::unordered_map<PairKey, PairPlan, PairHash> pair_cache;
}  // namespace

static Plan plan_f32_uncached(const Gemm &g, int mode);
static bool plan_f32_bwd_uncached(const Gemm &gd, const Gemm &gw, int mode_d, int mode_w, Plan *pd,
                                  Plan *pw);

// Keeps a plan for later calls; where there is no memory to keep it in, it is
// found again next time (nothing may be thrown through the C entry points).
template <class Cache, class K, class P>
static void keep(Cache &cache, const K &key, const P &plan) {
    try {
        if (cache.size() > 4096) cache.clear();
        cache.emplace(key, plan);
    } catch (const std::bad_alloc &) {
    }
}

static Plan cached_plan(const Gemm &g, int mode) {
    const Key k = key_of(g, mode);
    auto it = plan_cache.find(k);
    if (it != plan_cache.end()) return it->second;
    const Plan p = g.in_dtype == DT_F32 ? plan_f32_uncached(g, mode) : plan_uncached(g);
    keep(plan_cache, k, p);
    return p;
}

Plan plan_bf16(const Gemm &g) { return cached_plan(g, dma_mode(g)); }

// Leading dimensions whose tile offsets reach 2^31 bytes.
static bool f32_big_ld(const Gemm &g) {
    constexpr int64_t kMaxLd = int64_t(1) << 21;
    return g.lda > kMaxLd || g.ldb > kMaxLd;
}

bool f32_vec4(const Gemm &g) {
    const int64_t ca = g.orient == OR_BWD_WEIGHT ? g.m : g.k;
    const int64_t cb = g.orient == OR_BWD_DATA ? g.k : g.n;
    return ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.B)) & 15) == 0 &&
           g.lda % 4 == 0 && g.ldb % 4 == 0 && ca % 4 == 0 && cb % 4 == 0;
}

// What an fp32 plan depends on beside the sizes.
enum { F32_BIG_LD = 1, F32_VEC4 = 2 };
static int f32_mode(const Gemm &g) {
    return (f32_big_ld(g) ? F32_BIG_LD : 0) | (f32_vec4(g) ? F32_VEC4 : 0);
}

Plan plan_f32(const Gemm &g) { return cached_plan(g, f32_mode(g)); }

static double work_items(const Gemm &g, const Plan &p) {
    return (double)((g.m + p.bm - 1) / p.bm + 1) * (double)((g.n + p.bn - 1) / p.bn + 1) *
           p.splits * (double)g.nbatch();
}

// Grouped plan of both products on instance `in` (tile bm x bn) with the
// given splits; false if it does not fit the workspace.
static bool grouped_plan(const Gemm &gd, const Gemm &gw, const Instance *in, int bm, int bn,
                         int sd, int sw, Plan *pd, Plan *pw) {
    const bool sh = dma_mode(gd) == 2 || dma_mode(gw) == 2;
    if (sh && !shift_capable(bm, bn, in->bk, in->ns, in->kg, in->epi)) return false;
    for (int w = 0; w < 2; ++w) {
        const Gemm &g = w ? gw : gd;
        Plan &p = w ? *pw : *pd;
        p = Plan{bm, bn, 1, 1, true, in->ns, in->kg, in->epi, 0, in->bk};
        p.shift = sh;
        split_of(kblocks(g.k), w ? sw : sd, &p.splits, &p.kblk_per_split);
        if (adds(g, p) && !pipe_class(bm, bn, in->code)) return false;
    }
    // a batched product is never split, and all work items fit a 31-bit index
    if ((gd.nbatch() > 1 && pd->splits > 1) || (gw.nbatch() > 1 && pw->splits > 1)) return false;
    if (work_items(gd, *pd) + work_items(gw, *pw) > 2147483647.0) return false;
    return (double)plan_ws_floats(gd, *pd) + (double)plan_ws_floats(gw, *pw) <= ws_budget(gd);
}

size_t plan_ws_floats(const Gemm &g, const Plan &p) {
    return p.splits > 1 ? (size_t)p.splits * (size_t)g.m * (size_t)partial_ld(g.n) : 0;
}

static bool plan_bwd_uncached(const Gemm &gd, const Gemm &gw, Plan *pd, Plan *pw) {
    *pd = plan_bf16(gd);
    *pw = plan_bf16(gw);
    const bool attn = gd.orient == OR_FWD;   // dQ beside dK
    if (ov_bwd_mode == 1) return false;
    if (ov_bm != 0 && (ov_kernel == 2 || ((attn || gd.nbatch() > 1) && ov_bwd_mode != 2)))
        return false;
    if (!dma_eligible(gd) || !dma_eligible(gw)) return false;
    if (attn && (gd.out_dtype != gw.out_dtype || dma_mode(gd) == 2 || dma_mode(gw) == 2))
        return false;
    if (ov_bm != 0 && ov_bwd_mode == 2) {
        // tuning: grouped on the override's instance, backward-data splits from
        // the plan override, backward-weight splits from the backward override
        const Instance *in = find_instance(ov_kernel == 0 ? 1 : ov_kernel, ov_bm, ov_bn);
        if (attn && !pipe_class(ov_bm, ov_bn, in ? in->code : 0)) return false;
        return in && grouped_plan(gd, gw, in, ov_bm, ov_bn, ov_splits, ov_bwd_splits_w, pd, pw);
    }
    if (ov_bm == 0) {
        const int fd = gd.out_dtype == DT_F32, fw = gw.out_dtype == DT_F32;
        for (const TunedBwd &t : kTunedBwd) {
            if (t.md < 0 || gd.nbatch() > 1 || attn) break;
            if ((gd.accumulate && t.sd == 1) || (gw.accumulate && t.sw == 1)) continue;
            if (t.md == gd.m && t.nd == gd.n && t.kd == gd.k && t.fd == fd && t.mw == gw.m &&
                t.nw == gw.n && t.kw == gw.k && t.fw == fw) {
                const Instance *in = find_instance(t.code, t.bm, t.bn);
                if (in && grouped_plan(gd, gw, in, t.bm, t.bn, t.sd, t.sw, pd, pw)) return true;
                *pd = plan_bf16(gd);
                *pw = plan_bf16(gw);
                break;
            }
        }
        // measured plans of both products: they run as measured, one after the
        // other (batched pairs were measured without a grouped form)
        if (gd.nbatch() == 1 && tuned_for(gd, dma_mode(gd)) && tuned_for(gw, dma_mode(gw)))
            return false;
    }
    const bool sh = dma_mode(gd) == 2 || dma_mode(gw) == 2;
    if (ov_bm != 0) {
        // an override fixes the tile (and the splits of both products)
        if (!pd->dma || !pw->dma) return false;
        pw->bm = pd->bm;
        pw->bn = pd->bn;
        pw->ns = pd->ns;
        pw->kg = pd->kg;
        pw->epi = pd->epi;
        pw->bk = pd->bk;
        if (sh && !shift_capable(*pd)) return false;
        pd->shift = pw->shift = sh;
        pd->occ = pw->occ = 0;   // the grouped launch runs one workgroup per item
        if ((adds(gd, *pd) || adds(gw, *pw)) && !pipe_class(pd->bm, pd->bn, kernel_code(*pd)))
            return false;
        return (double)plan_ws_floats(gd, *pd) + (double)plan_ws_floats(gw, *pw) <=
               ws_budget(gd);
    }
    // grouped where the model expects it to beat the two products in turn
    double best_d, best_w;
    plan_model(gd, &best_d);
    plan_model(gw, &best_w);
    double best = best_d + best_w;
    bool grouped = false;
    const int kd = kblocks(gd.k), kw = kblocks(gw.k);
    for (const PipeClass &c : kPipe) {
        const Instance &in = *find_instance(c.code, c.bm, c.bn);
        int last_d = 0;
        for (int a = 1; a <= (gd.nbatch() > 1 ? 1 : 16); ++a) {
            int sd, perd;
            split_of(kd, a, &sd, &perd);
            if (sd == last_d) continue;
            last_d = sd;
            if (sd > 1 && perd < 2) continue;
            int last_w = 0;
            for (int b = 1; b <= (gw.nbatch() > 1 ? 1 : 16); ++b) {
                int sw, perw;
                split_of(kw, b, &sw, &perw);
                if (sw == last_w) continue;
                last_w = sw;
                if (sw > 1 && perw < 2) continue;
                const double tm = model_pair(gd, gw, c, sd, perd, sw, perw, sh);
                if (tm >= best * 0.999) continue;
                Plan qd, qw;
                if (!grouped_plan(gd, gw, &in, c.bm, c.bn, sd, sw, &qd, &qw)) continue;
                best = tm;
                grouped = true;
                *pd = qd;
                *pw = qw;
            }
        }
    }
    return grouped;
}

// Plans are pure functions of the key, kept per thread so that a repeated
// call does not search again (a pair weighs some 2,000 candidates).
static bool cached_pair(const Gemm &gd, const Gemm &gw, int mode_d, int mode_w, Plan *pd,
                        Plan *pw) {
    const PairKey k{key_of(gd, mode_d), key_of(gw, mode_w),
                    ov_bwd_mode * 65536 + ov_bwd_splits_w};
    auto it = pair_cache.find(k);
    PairPlan p;
    if (it != pair_cache.end()) {
        p = it->second;
    } else {
        p.grouped = gd.in_dtype == DT_F32
                        ? plan_f32_bwd_uncached(gd, gw, mode_d, mode_w, &p.d, &p.w)
                        : plan_bwd_uncached(gd, gw, &p.d, &p.w);
        keep(pair_cache, k, p);
    }
    *pd = p.d;
    *pw = p.w;
    return p.grouped;
}

bool plan_bf16_bwd(const Gemm &gd, const Gemm &gw, Plan *pd, Plan *pw) {
    return cached_pair(gd, gw, dma_mode(gd), dma_mode(gw), pd, pw);
}

bool plan_f32_bwd(const Gemm &gd, const Gemm &gw, Plan *pd, Plan *pw) {
    return cached_pair(gd, gw, f32_mode(gd), f32_mode(gw), pd, pw);
}

// Generic kernel: the busiest compute unit's share of the work items, each
// `per` steps (the workgroups of a unit share its load path, so their steps
// add up: 0.70 us per 128 x 128 step alone and with two workgroups), plus a
// fixed cost and the split reduction. Measured: 2051 x 2502 x 1024 forward 27.7
// us on 128 x 128 tiles, 35.6 on 64 x 64 ones, 32.0 on 256 x 128; 250 x 511 x
// 6001 12.7 us on 64 x 64 split 8 ways.
static Plan plan_generic(const Gemm &g) {
    const int kb_total = kblocks(g.k);
    Plan best{64, 64, 1, std::max(1, kb_total), false};
    double best_t = 1e30;
    for (const GenericTile &t : kGeneric) {
        const double nt = (double)((g.m + t.bm - 1) / t.bm) * (double)((g.n + t.bn - 1) / t.bn) *
                          (double)g.nbatch();
        int last = 0;
        for (int s = 1; s <= 32; ++s) {
            int splits, per;
            split_of(kb_total, s, &splits, &per);
            if (splits == last) continue;
            last = splits;
            if (splits > 1 && (per < 2 || !fits_ws(g, splits))) continue;
            const double q = nt * splits / kCUs, busy = q > 4.0 ? q + 0.5 : std::ceil(q);
            double tm = busy * per * t.step + 5e-6;
            if (splits > 1) tm += (splits * 2.0 + 0.5) * 4.0 * g.m * g.n / 6e12 + 3e-6;
            if (tm < best_t * 0.999) {
                best_t = tm;
                best = Plan{t.bm, t.bn, splits, per, false};
            }
        }
    }
    return best;
}

static Plan plan_uncached(const Gemm &g) {
    const int kb_total = kblocks(g.k);
    const int mode = dma_mode(g);
    const bool dma = mode > 0;
    if (ov_bm != 0 && ((ov_orients >> g.orient) & 1)) {
        // kernel: 0 or 1 the tile's default pipelined instance (if eligible),
        // 2 generic, other codes the instance of kInstances (if eligible);
        // a product the pipelined kernel cannot read runs the generic kernel,
        // and so does one that needs the shifted form of an instance without
        // one
        bool use_dma = dma && ov_kernel != 2;
        const Instance *in = nullptr;
        if (use_dma) {
            in = find_instance(ov_kernel == 0 ? 1 : ov_kernel, ov_bm, ov_bn);
            if (!in) in = find_instance(1, ov_bm, ov_bn);
            if (mode == 2 && !shift_capable(ov_bm, ov_bn, in->bk, in->ns, in->kg, in->epi))
                use_dma = false;
        }
        Plan p{ov_bm, ov_bn, 1, 1, use_dma};
        if (use_dma) {
            p.ns = in->ns;
            p.kg = in->kg;
            p.epi = in->epi;
            p.bk = in->bk;
            p.occ = ov_occ;
            p.shift = mode == 2;
        } else if (!tile_supported(p.bm, p.bn, false)) {
            p.bn = 128;   // 256x256 only pipelined
        }
        split_of(kb_total, ov_splits, &p.splits, &p.kblk_per_split);
        while (p.splits > 1 && !fits_ws(g, p.splits))
            split_of(kb_total, p.splits - 1, &p.splits, &p.kblk_per_split);
        if (use_dma && adds(g, p) && !pipe_class(p.bm, p.bn, in->code)) {
            // no accumulating form: the tile's model instance, or the generic kernel
            const int code = pipe_class(p.bm, p.bn, 4) ? 4 : 1;
            const Instance *a = find_instance(code, p.bm, p.bn);
            if (pipe_class(p.bm, p.bn, code) &&
                (mode == 1 || shift_capable(p.bm, p.bn, a->bk, a->ns, a->kg, a->epi))) {
                p.ns = a->ns;
                p.kg = a->kg;
                p.epi = a->epi;
                p.bk = a->bk;
            } else {
                Plan q{p.bm, tile_supported(p.bm, p.bn, false) ? p.bn : 128, 1, p.kblk_per_split,
                       false};
                return q;
            }
        }
        return p;
    }
    if (const Tuned *t = tuned_for(g, mode)) {
        Plan p{t->bm, t->bn, 1, 1, dma && t->code != 2};
        const Instance *in = p.dma ? find_instance(t->code, t->bm, t->bn) : nullptr;
        if (in && mode == 2 && !shift_capable(t->bm, t->bn, in->bk, in->ns, in->kg, in->epi))
            in = nullptr;
        if ((!p.dma && tile_supported(t->bm, t->bn, false)) || in) {
            if (in) {
                p.ns = in->ns;
                p.kg = in->kg;
                p.epi = in->epi;
                p.bk = in->bk;
                p.occ = t->occ;
                p.shift = mode == 2;
            }
            split_of(kb_total, t->splits, &p.splits, &p.kblk_per_split);
            if (fits_ws(g, p.splits)) return p;
        }
    }
    double time;
    return dma ? plan_model(g, &time) : plan_generic(g);
}

// The pipelined plan the model expects to be fastest, and its time in us.
static Plan plan_model(const Gemm &g, double *time) {
    const int kb_total = kblocks(g.k);
    const bool shift = dma_mode(g) == 2;
    Plan best{64, 64, 1, std::max(1, kb_total), true};
    best.shift = shift;
    *time = 1e30;
    for (const PipeClass &c : kPipe) {
        const Instance &in = *find_instance(c.code, c.bm, c.bn);
        if (shift && !shift_capable(c.bm, c.bn, in.bk, in.ns, in.kg, in.epi)) continue;
        int last_splits = 0;
        for (int s = 1; s <= 32; ++s) {
            int splits, per;
            split_of(kb_total, s, &splits, &per);
            if (splits == last_splits) continue;
            last_splits = splits;
            if (splits > 1 && per < 2) continue;            // keep >= 128 reduction per split
            if (!fits_ws(g, splits)) continue;
            const double tm = model_time(g, c, splits, per, shift);
            if (tm < *time * 0.999) {
                *time = tm;
                best = Plan{c.bm, c.bn, splits, per, true, in.ns, in.kg, in.epi, 0, in.bk};
                best.shift = shift;
            }
        }
    }
    return best;
}

// fp32 products (gemm_f32.hip). Measured on MI355X, a 32-wide reduction step of
// a 128 x 128 tile takes a compute unit 2.1 us however many workgroups share
// it (fp32 MFMA bound); one of a 64 x 64 tile 0.55 us when two or more
// workgroups share the unit and 0.76 us alone, where nothing hides its load
// latency. So small outputs split their reduction until every unit has
// several 64 x 64 workgroups (1024 x 1024 x 4096: 98 us unsplit, 79 us split
// four ways), and outputs of a whole wave of 128 x 128 tiles take those
// (4096^3: 1028 us against 1068 us; 1024 x 4096 x 1024: 75 us for both).
namespace {
// Time in us of a 32-wide step of a t x t tile with `q` work items per unit.
double f32_step(int t, double q) { return t == 128 ? 2.1 : q <= 1.0 ? 0.76 : 0.55; }
double f32_reduce(const Gemm &g, int splits) {
    return splits > 1 ? (splits * 2.0 + 1.0) * 4.0 * g.m * g.n / 8e6 : 0.0;
}
double f32_tiles(const Gemm &g, int t) {
    return (double)((g.m + t - 1) / t) * (double)((g.n + t - 1) / t);
}
constexpr double kF32Fixed = 6.0, kF32Reduce = 2.5;   // us
// Steps below which a 128 x 128 tile's stores bound it, which more, smaller tiles
// hide behind one another's loads (2048 x 2048 over 64 13.2 us, on 64 x 64 tiles 10.6;
// over 160 18.7 and 16.8; 4096 x 4096 over 64 32.3 and 28.9, over 160 54.8 and 54.1).
constexpr int kF32Steps128 = 6;

// Reductions so short that the stores bound the launch, where the plain FMA
// kernel's are faster than the matrix-core kernel's on 64 x 64 tiles: large outputs
// (4096 x 4096 over 5 19.9 against 26.2 us, over 16 22.4 against 22.0; 960 x 1084
// over 4 by 16-byte loads 5.8 against 5.0) and weight gradients by 4-byte loads (1123
// x 82 over 1 4.1 against 4.6). Where the product is added to the output the
// matrix-core kernel is faster at all sizes (2176 x 2036 over 8 10.2 against 15.6).
bool f32_fma(const Gemm &g, int mode) {
    if (mode & F32_BIG_LD) return true;
    if (g.accumulate || g.k == 0) return false;
    const double out = (double)g.m * (double)g.n;
    if (mode & F32_VEC4) return g.k <= 8 && out >= 1 << 22;
    return g.k <= 12 && (g.orient == OR_BWD_WEIGHT || out >= 1 << 20);
}
}  // namespace

// The matrix-core plan the model expects to be fastest, and its time in us.
static Plan plan_f32_model(const Gemm &g, double *time);

static Plan plan_f32_uncached(const Gemm &g, int mode) {
    if (f32_fma(g, mode)) {
        Plan p{64, 64, 1, std::max(1, (int)((g.k + 31) / 32)), false};
        p.bk = 32;
        return p;
    }
    double t;
    return plan_f32_model(g, &t);
}

// The two backward products in one launch: as model_pair, with the fp32 steps.
static bool plan_f32_bwd_uncached(const Gemm &gd, const Gemm &gw, int mode_d, int mode_w, Plan *pd,
                                  Plan *pw) {
    if ((mode_d | mode_w) & F32_BIG_LD || ov_bwd_mode == 1) return false;
    double best, tw;
    *pd = plan_f32_model(gd, &best);
    *pw = plan_f32_model(gw, &tw);
    best += tw;
    bool grouped = false;
    const int kd = (int)((gd.k + 31) / 32), kw = (int)((gw.k + 31) / 32);
    for (const int t : {64, 128}) {
        int last_d = 0;
        for (int a = 1; a <= 16; ++a) {
            int sd, perd;
            split_of(kd, a, &sd, &perd);
            if (sd == last_d) continue;
            last_d = sd;
            if (sd > 1 && perd < 4) continue;
            int last_w = 0;
            for (int b = 1; b <= 16; ++b) {
                int sw, perw;
                split_of(kw, b, &sw, &perw);
                if (sw == last_w) continue;
                last_w = sw;
                if (sw > 1 && perw < 4) continue;
                const double nd = f32_tiles(gd, t) * sd, nw = f32_tiles(gw, t) * sw;
                if (nd + nw > 2147483647.0) continue;
                const double q = (nd + nw) / kCUs, step = f32_step(t, q);
                const double lo = std::max(perd, perw), sh = std::min(perd, perw);
                const double nlo = perd >= perw ? nd : nw;
                // a long item waits for the other workgroups of its unit
                const double r = std::min(t == 128 ? 2.0 : 4.0, std::ceil(q));
                double busy = q <= 1.0 ? lo
                                       : std::max(std::ceil(nlo / kCUs) * lo,
                                                  (nd * perd + nw * perw) / kCUs + 0.5 * sh);
                // whole rounds of both leave no tail
                if (q > 1.0)
                    busy = std::min(busy, std::ceil(nd / kCUs) * perd + std::ceil(nw / kCUs) * perw);
                busy = std::max(busy, lo * std::max(1.0, 0.7 * r));
                const double tm = busy * step + kF32Fixed +
                                  (sd > 1 || sw > 1 ? kF32Reduce : 0.0) + f32_reduce(gd, sd) +
                                  f32_reduce(gw, sw);
                if (tm >= best * 0.999) continue;
                Plan qd{t, t, sd, perd, true}, qw{t, t, sw, perw, true};
                qd.bk = qw.bk = 32;
                if ((double)plan_ws_floats(gd, qd) + (double)plan_ws_floats(gw, qw) >
                    ws_budget(gd))
                    continue;
                best = tm;
                grouped = true;
                *pd = qd;
                *pw = qw;
            }
        }
    }
    return grouped;
}

static Plan plan_f32_model(const Gemm &g, double *time) {
    const int kb = (int)((g.k + 31) / 32);
    Plan best{64, 64, 1, std::max(1, kb), true};
    best.bk = 32;
    *time = 1e30;
    for (const int t : {64, 128}) {
        const double nt = f32_tiles(g, t);
        int last = 0;
        for (int s = 1; s <= 32; ++s) {
            int splits, per;
            split_of(kb, s, &splits, &per);
            if (splits == last) continue;
            last = splits;
            if (splits > 1 && (per < 4 || !fits_ws(g, splits))) continue;
            if (t == 128 && per < kF32Steps128) continue;
            // work items of the busiest unit; beyond four the units even out
            const double q = nt * splits / kCUs, busy = q > 4.0 ? q + 0.5 : std::ceil(q);
            const double tm = busy * per * f32_step(t, q) + kF32Fixed +
                              (splits > 1 ? kF32Reduce : 0.0) + f32_reduce(g, splits);
            if (tm < *time * 0.999) {
                *time = tm;
                best.bm = best.bn = t;
                best.splits = splits;
                best.kblk_per_split = per;
            }
        }
    }
    return best;
}

}  // namespace sbpi
