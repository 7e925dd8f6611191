// gemm_f32.hip -- fp32-input path of the local matmul and the bf16 dispatch
// by orientation.
//
// The fp32 path serves fp32 training (the paper's P100 runs are fp32). Two
// kernels: the matrix-core kernel below for every product whose tiles fit
// 31-bit buffer offsets, and a plain FMA kernel for leading dimensions beyond
// that (2^21 elements) and for reductions so short that the stores bound the launch
// (plan.cpp f32_fma).
//
// Matrix-core kernel (gemm_f32_mfma_kernel), bound by the fp32 MFMA rate:
//   * v_mfma_f32_32x32x2_f32: fp32 products and sums, 256 flop/clk/CU -- the
//     same fp32 arithmetic as FMAs, in another order of k.
//   * Four waves (2 x 2), 128 x 128 or 64 x 64 output tile, 32-wide reduction
//     steps; two stages of both operand tiles in LDS, loaded by buffer loads
//     that write LDS directly. A 128 x 128 step is 4096 cycles of MFMA per
//     32 KB of operands, so one stage ahead and a second workgroup per CU
//     (four or five of the 64 x 64 ones) cover the memory latency, barriers
//     and epilogues. More stages (three to eight) with fewer workgroups per
//     CU, or two reduction groups of waves, were no faster; 128 x 64 tiles
//     lay between the two.
//   * The two backward products of a linear share one launch where the model
//     expects it to pay: two 256-tile products of 128 x 128 tiles 148 -> 136 us.
//   * Measured, against the FMA kernel below: 1024 x 4096 x 1024 forward
//     240 -> 75 us, 256 x 4096 x 3136 forward 660 -> 63 us, 4096^3 134
//     TFLOP/s (the library product reaches 141); the largest error against
//     64 bits over fp32 layers of those sizes 1.1e-6 -> 8.1e-7.
//   * V = 4: 16 bytes per lane, where both operands' base, ld and contiguous
//     extent are multiples of 4 floats. V = 1: 4 bytes per lane with per-element
//     bounds, for any other operand: four times the load instructions, which
//     still fit under the MFMA time of a step.
//   * k-major tiles: 128-byte rows (32 reduction values) of eight 16-byte
//     chunks, chunk c of row r at c ^ ((r / 2) % 8), so a 16-row
//     ds_read_b128 phase covers all 64 banks; lane l takes chunk 2 j + l / 32,
//     i.e. MFMA e of group j multiplies k = 8 j + e (lower half-wave) and
//     8 j + 4 + e (upper half).
//   * m/n-major tiles: rows of BM (BN) values per reduction index, read with
//     ds_read_b32 at the same k; chunks of rows with odd k / 4 are shifted by
//     8 so that the two half-waves use different banks.
//   * Split reduction as in the bf16 kernels (split_reduce.hip adds the fp32
//     partials in split order).
#include "gemm.h"
#include "gemm_bf16_dma.h"
#include "profile.h"

namespace sbpk {

struct F32Args {
    const float *A;
    const float *B;
    float *C;
    int64_t lda, ldb, ldc;
    int32_t m, n, k;
    int32_t tiles_m, tiles_n;
    int32_t splits, kchunk;   // reduction elements per split (a multiple of 32)
    float *ws;                // split partials, row stride partial_ld(n)
    int32_t accumulate;       // add the product to C's contents
};

// One 4-byte-per-lane buffer load that writes LDS directly (see dma16).
__device__ __forceinline__ void dma4(i32x4 r, char *lds, int voff) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(SBP_LDS void *)lds);
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(m0), "v"(voff), "s"(r)
                 : "memory", "m0");
}

constexpr int FK = 32;   // reduction elements per step

// Operand tile of BMN output indices x FK reduction indices (layouts above).
template <int BMN, bool KMAJ, int V>
struct F32Tile {
    static constexpr int LOADS = BMN * FK / (64 * V * 4);   // per wave (4 waves)

    __device__ __forceinline__ static int swz(int row) {
        return KMAJ ? (row >> 1) & 7 : ((row >> 2) & 1) << 3;
    }

    __device__ __forceinline__ static void issue(const float *base, int64_t ld, int mn0,
                                                 int mn_lim, int k0, int k_lim, char *lds,
                                                 int wave, int lane) {
        constexpr int ROW = KMAJ ? FK : BMN;   // floats per LDS row
        const i32x4 r = make_rsrc(KMAJ ? base + (int64_t)mn0 * ld + k0
                                       : base + (int64_t)k0 * ld + mn0);
        // rows left along the row index, elements left along the contiguous one
        const int rows = KMAJ ? mn_lim - mn0 : k_lim - k0;
        const int cols = KMAJ ? k_lim - k0 : mn_lim - mn0;
        const int ldi = (int)ld;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int seg = (i * 4 + wave) * 64 * V;
            const int pos = seg + lane * V;
            const int row = pos / ROW, in = pos % ROW;
            const int col = (((in >> 2) ^ swz(row)) << 2) + (in & 3);
            const bool ok = row < rows && col + V <= cols;
            const int voff = ok ? (row * ldi + col) * 4 : OOB;
            if constexpr (V == 4) dma16(r, lds + seg * 4, voff);
            else dma4(r, lds + seg * 4, voff);
        }
    }

    // Values k = 8 j + 4 (lane / 32) + 0..3 of output index c0 + lane % 32.
    __device__ __forceinline__ static f32x4 frag(const char *lds, int c0, int j, int lane) {
        const int mn = c0 + (lane & 31);
        if constexpr (KMAJ) {
            const int c = 2 * j + (lane >> 5);
            return *reinterpret_cast<const f32x4 *>(lds + mn * FK * 4 + ((c ^ swz(mn)) << 4));
        } else {
            const int k = 8 * j + 4 * (lane >> 5);   // rows k .. k+3 share one swizzle
            const float *p = reinterpret_cast<const float *>(lds) + k * BMN +
                             ((((mn >> 2) ^ swz(k)) << 2) | (mn & 3));
            f32x4 v = {p[0], p[BMN], p[2 * BMN], p[3 * BMN]};
            return v;
        }
    }
};

// Adds a lane's 16 elements of a 32 x 32 MFMA block (rows rbase + 8 (r / 4) + r % 4
// of the block that starts at row r0, column col) to the output `out`, row stride
// ldo, rows below m, as the bf16 kernels' direct epilogue does: all old values
// loaded before any is stored, no bounds checks kept between the two. (2000 x 1003
// over 16, 7.8 -> 5.8 us against bounds-checked loads; the FMA kernel takes 11.4.)
__device__ __forceinline__ void add_block(void *out, int64_t ldo, int rbase, int col, int r0, int m,
                                          const f32x16 v) {
    typedef __attribute__((address_space(1))) float GlobalFloat;
    float old[16];
    r0 = __builtin_amdgcn_readfirstlane(r0);
    if (r0 + 32 <= m) {
        GlobalFloat *d = (GlobalFloat *)out + ((int64_t)rbase * ldo + col);
        asm volatile("" : "+v"(d) : : "memory");
#pragma unroll
        for (int r = 0; r < 16; ++r) old[r] = d[(8 * (r >> 2) + (r & 3)) * ldo];
        asm volatile("" : "+v"(d) : : "memory");
#pragma unroll
        for (int r = 0; r < 16; ++r) d[(8 * (r >> 2) + (r & 3)) * ldo] = old[r] + v[r];
        return;
    }
    GlobalFloat *const c = (GlobalFloat *)out + col;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = rbase + 8 * (r >> 2) + (r & 3);
        old[r] = c[(int64_t)min(row, m - 1) * ldo];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = rbase + 8 * (r >> 2) + (r & 3);
        if (row < m) c[(int64_t)row * ldo] = old[r] + v[r];
    }
}

// One work item (an output tile and a reduction split; L its logical index).
// ACCUM: as in the bf16 tile body.
template <int BM, int BN, bool A_KMAJ, bool B_KMAJ, int V, int ACCUM>
__device__ __forceinline__ void f32_tile_body(const F32Args &g, const int L, char *smem) {
    using TA = F32Tile<BM, A_KMAJ, V>;
    using TB = F32Tile<BN, B_KMAJ, V>;
    constexpr int A_BYTES = BM * FK * 4, STAGE = (BM + BN) * FK * 4;
    constexpr int WM = BM / 2, WN = BN / 2, MI = WM / 32, NI = WN / 32;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    const int tiles = g.tiles_m * g.tiles_n;
    const int split = L / tiles;
    const int t = L % tiles;
    constexpr int GROUP = SBP_TILE_GROUP;
    const int grp = t / (GROUP * g.tiles_n);
    const int first_m = grp * GROUP;
    const int gsize = min(g.tiles_m - first_m, GROUP);
    const int tg = t - grp * GROUP * g.tiles_n;
    const int m0 = (first_m + tg % gsize) * BM, n0 = (tg / gsize) * BN;
    const int k_begin = split * g.kchunk;
    const int k_lim = min(g.k, k_begin + g.kchunk);
    const int nkb = max(0, (k_lim - k_begin + FK - 1) / FK);

    auto issue = [&](int kb, int stage) {
        char *base = smem + stage * STAGE;
        const int k0 = k_begin + kb * FK;
        TA::issue(g.A, g.lda, m0, g.m, k0, k_lim, base, wave, lane);
        TB::issue(g.B, g.ldb, n0, g.n, k0, k_lim, base + A_BYTES, wave, lane);
    };
    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    if (nkb > 0) issue(0, 0);
    for (int it = 0; it < nkb; ++it) {
        // this thread's loads of step `it` are done, then everyone's; the
        // stage read last step is free to refill
        wait_vm<0>();
        __syncthreads();
        if (it + 1 < nkb) issue(it + 1, (it + 1) & 1);
        const char *cur = smem + (it & 1) * STAGE;
#pragma unroll
        for (int j = 0; j < FK / 8; ++j) {
            f32x4 a[MI], b[NI];
#pragma unroll
            for (int i = 0; i < MI; ++i) a[i] = TA::frag(cur, wm * WM + i * 32, j, lane);
#pragma unroll
            for (int i = 0; i < NI; ++i) b[i] = TB::frag(cur + A_BYTES, wn * WN + i * 32, j, lane);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int jj = 0; jj < NI; ++jj)
                        acc[i][jj] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[jj][e],
                                                                          acc[i][jj], 0, 0, 0);
        }
    }

    // lane holds column lane % 32 of a 32 x 32 block, register r row
    // 8 (r / 4) + 4 (lane / 32) + r % 4
    const bool partial = ACCUM != ACC_ALL && g.splits > 1;
    const bool add = ACCUM == ACC_ALL || (ACCUM == ACC_SOME && g.accumulate && !partial);
    const int64_t ldo = partial ? sbpi::partial_ld(g.n) : g.ldc;
    float *const out = partial ? g.ws + (size_t)split * (size_t)g.m * (size_t)ldo : g.C;
    const __amdgpu_buffer_rsrc_t pr = part_rsrc(out);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int col = n0 + wn * WN + j * 32 + (lane & 31);
            const int rbase = m0 + wm * WM + i * 32 + 4 * (lane >> 5);
            if (col >= g.n) continue;
            if constexpr (ACCUM != ACC_NONE) {
                if (add) {
                    // opaque: shared with the plain stores, 47 more registers hold
                    // row addresses in the pair's 64 x 64 form, four workgroups a
                    // unit for five
                    int rb = rbase;
                    asm volatile("" : "+v"(rb));
                    add_block(out, ldo, rb, col, m0 + wm * WM + i * 32, g.m, acc[i][j]);
                    continue;
                }
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = rbase + 8 * (r >> 2) + (r & 3);
                if (row >= g.m) continue;
                if (partial) st_part(pr, (int64_t)row * ldo + col, acc[i][j][r]);
                else st_nt(out + (int64_t)row * ldo + col, acc[i][j][r]);
            }
        }
}

// Two workgroups of 128 x 128 tiles per CU (64 KB of LDS each), four or five of 64 x 64 ones.
template <int BM, bool A_KMAJ, bool B_KMAJ, int V, int ACCUM>
__global__ __launch_bounds__(256, BM == 64 ? 4 : 2) void gemm_f32_mfma_kernel(F32Args g) {
    __shared__ __attribute__((aligned(1024))) char smem[4 * BM * FK * 4];
    const int total = g.tiles_m * g.tiles_n * g.splits;
    f32_tile_body<BM, BM, A_KMAJ, B_KMAJ, V, ACCUM>(g, remap_xcd(blockIdx.x, total), smem);
}

// Both backward products of one linear in one launch, the product with the
// longer work items first (as gemm_bf16_dma_bwd_kernel): a product of 256 tiles
// alone puts one workgroup on each CU, which then waits for every load.
template <int BM, int V, int ACCUM>
__global__ __launch_bounds__(256, BM == 64 ? 4 : 2) void gemm_f32_mfma_bwd_kernel(
    F32Args gd, F32Args gw, int data_first) {
    __shared__ __attribute__((aligned(1024))) char smem[4 * BM * FK * 4];
    const int wd = gd.tiles_m * gd.tiles_n * gd.splits;
    const int ww = gw.tiles_m * gw.tiles_n * gw.splits;
    const int b = blockIdx.x;
    if (data_first ? b < wd : b >= ww)
        f32_tile_body<BM, BM, true, true, V, ACCUM>(gd, remap_xcd(data_first ? b : b - ww, wd),
                                                    smem);
    else
        f32_tile_body<BM, BM, false, false, V, ACCUM>(gw, remap_xcd(data_first ? b - wd : b, ww),
                                                      smem);
}

// Plain LDS-tiled FMA kernel (leading dimensions beyond 2^21, shortest reductions): 64 x 64
// output tile, reduction step 16, 256 threads each owning a 4 x 4 strided
// sub-block.
constexpr int F_BM = 64, F_BN = 64, F_BK = 16;

template <bool A_KMAJ, bool B_KMAJ>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Args g) {
    __shared__ float As[F_BK][F_BM + 1];
    __shared__ float Bs[F_BK][F_BN + 1];
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int tm = blockIdx.x / g.tiles_n, tn = blockIdx.x % g.tiles_n;
    const int m0 = tm * F_BM, n0 = tn * F_BN;
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

    for (int k0 = 0; k0 < g.k; k0 += F_BK) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = tid + 256 * q;
            int i, kk;
            if (A_KMAJ) { i = e / F_BK; kk = e % F_BK; } else { kk = e / F_BM; i = e % F_BM; }
            const int gi = m0 + i, gk = k0 + kk;
            float v = 0.f;
            if (gi < g.m && gk < g.k)
                v = A_KMAJ ? g.A[(int64_t)gi * g.lda + gk] : g.A[(int64_t)gk * g.lda + gi];
            As[kk][i] = v;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = tid + 256 * q;
            int j, kk;
            if (B_KMAJ) { j = e / F_BK; kk = e % F_BK; } else { kk = e / F_BN; j = e % F_BN; }
            const int gj = n0 + j, gk = k0 + kk;
            float v = 0.f;
            if (gj < g.n && gk < g.k)
                v = B_KMAJ ? g.B[(int64_t)gj * g.ldb + gk] : g.B[(int64_t)gk * g.ldb + gj];
            Bs[kk][j] = v;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < F_BK; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = As[kk][ty + 16 * i];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx + 16 * j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = m0 + ty + 16 * i;
        if (row >= g.m) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = n0 + tx + 16 * j;
            if (col >= g.n) continue;
            float *c = g.C + (int64_t)row * g.ldc + col;
            *c = g.accumulate ? *c + acc[i][j] : acc[i][j];
        }
    }
}

}  // namespace sbpk

namespace sbpi {

hipError_t launch_bf16_fwd(const Gemm &, const Plan &, float *, hipStream_t);
hipError_t launch_bf16_bwd_data(const Gemm &, const Plan &, float *, hipStream_t);
hipError_t launch_bf16_bwd_weight(const Gemm &, const Plan &, float *, hipStream_t);

hipError_t launch_bf16(const Gemm &g, const Plan &p, float *ws, hipStream_t s) {
    switch (g.orient) {
        case OR_FWD: return launch_bf16_fwd(g, p, ws, s);
        case OR_BWD_DATA: return launch_bf16_bwd_data(g, p, ws, s);
        case OR_BWD_WEIGHT: return launch_bf16_bwd_weight(g, p, ws, s);
    }
    return hipErrorInvalidValue;
}

static sbpk::F32Args f32_args(const Gemm &g, const Plan &p, float *ws) {
    sbpk::F32Args a;
    a.A = static_cast<const float *>(g.A);
    a.B = static_cast<const float *>(g.B);
    a.C = static_cast<float *>(g.C);
    a.lda = g.lda;
    a.ldb = g.ldb;
    a.ldc = g.ldc;
    a.m = (int32_t)g.m;
    a.n = (int32_t)g.n;
    a.k = (int32_t)g.k;
    a.tiles_m = (int32_t)((g.m + p.bm - 1) / p.bm);
    a.tiles_n = (int32_t)((g.n + p.bn - 1) / p.bn);
    a.splits = p.splits;
    a.kchunk = p.kblk_per_split * p.bk;
    a.ws = ws;
    a.accumulate = g.accumulate;
    return a;
}

template <bool AK, bool BK_>
static hipError_t launch_f32_orient(const Gemm &g, const Plan &p, float *ws, hipStream_t s) {
    const char *tf[2] = {"false", "true"};
    char name[96];
    const sbpk::F32Args a = f32_args(g, p, ws);
    const dim3 grid((unsigned)(a.tiles_m * a.tiles_n * a.splits));
    if (!p.dma) {
        if (profiling()) snprintf(name, sizeof(name), "gemm_f32_kernel<%s, %s>", tf[AK], tf[BK_]);
        return launch_kernel(sbpk::gemm_f32_kernel<AK, BK_>, name, grid, dim3(256), s, a);
    }
    const bool v4 = f32_vec4(g), add = g.accumulate && p.splits == 1;
    hipError_t e = hipErrorInvalidValue;
#define SBP_F32_TILE(BM_, V_, ACC_)                                                           \
    if (p.bm == BM_ && v4 == (V_ == 4) && add == (ACC_ == sbpk::ACC_ALL)) {                   \
        if (profiling())                                                                     \
            snprintf(name, sizeof(name), "gemm_f32_mfma_kernel<%d, %s, %s, %d, %d>", BM_,    \
                     tf[AK], tf[BK_], V_, ACC_);                                             \
        e = launch_kernel(sbpk::gemm_f32_mfma_kernel<BM_, AK, BK_, V_, ACC_>, name, grid,    \
                          dim3(256), s, a);                                                  \
    }
    SBP_F32_TILE(128, 4, sbpk::ACC_NONE)
    SBP_F32_TILE(128, 1, sbpk::ACC_NONE)
    SBP_F32_TILE(64, 4, sbpk::ACC_NONE)
    SBP_F32_TILE(64, 1, sbpk::ACC_NONE)
    SBP_F32_TILE(128, 4, sbpk::ACC_ALL)
    SBP_F32_TILE(128, 1, sbpk::ACC_ALL)
    SBP_F32_TILE(64, 4, sbpk::ACC_ALL)
    SBP_F32_TILE(64, 1, sbpk::ACC_ALL)
#undef SBP_F32_TILE
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_split_reduce(g, p.splits, ws, s);
}

hipError_t launch_f32(const Gemm &g, const Plan &p, float *ws, hipStream_t s) {
    switch (g.orient) {
        case OR_FWD: return launch_f32_orient<true, false>(g, p, ws, s);
        case OR_BWD_DATA: return launch_f32_orient<true, true>(g, p, ws, s);
        case OR_BWD_WEIGHT: return launch_f32_orient<false, false>(g, p, ws, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_f32_bwd_group(const Gemm &gd, const Plan &pd, const Gemm &gw, const Plan &pw,
                                float *ws, hipStream_t s) {
    if (!pd.dma || !pw.dma || pd.bm != pw.bm) return hipErrorInvalidValue;
    char name[96];
    float *const ws_w = ws + plan_ws_floats(gd, pd);
    const sbpk::F32Args d = f32_args(gd, pd, ws), w = f32_args(gw, pw, ws_w);
    const dim3 grid((unsigned)(d.tiles_m * d.tiles_n * d.splits + w.tiles_m * w.tiles_n * w.splits));
    const int data_first = pd.kblk_per_split >= pw.kblk_per_split;
    const bool v4 = f32_vec4(gd) && f32_vec4(gw);
    const bool add = (gd.accumulate && pd.splits == 1) || (gw.accumulate && pw.splits == 1);
    hipError_t e = hipErrorInvalidValue;
#define SBP_F32_PAIR(BM_, V_, ACC_)                                                          \
    if (pd.bm == BM_ && v4 == (V_ == 4) && add == (ACC_ == sbpk::ACC_SOME)) {                \
        if (profiling())                                                                     \
            snprintf(name, sizeof(name), "gemm_f32_mfma_bwd_kernel<%d, %d, %d>", BM_, V_,    \
                     ACC_);                                                                  \
        e = launch_kernel(sbpk::gemm_f32_mfma_bwd_kernel<BM_, V_, ACC_>, name, grid,         \
                          dim3(256), s, d, w, data_first);                                   \
    }
    SBP_F32_PAIR(128, 4, sbpk::ACC_NONE)
    SBP_F32_PAIR(128, 1, sbpk::ACC_NONE)
    SBP_F32_PAIR(64, 4, sbpk::ACC_NONE)
    SBP_F32_PAIR(64, 1, sbpk::ACC_NONE)
    SBP_F32_PAIR(128, 4, sbpk::ACC_SOME)
    SBP_F32_PAIR(128, 1, sbpk::ACC_SOME)
    SBP_F32_PAIR(64, 4, sbpk::ACC_SOME)
    SBP_F32_PAIR(64, 1, sbpk::ACC_SOME)
#undef SBP_F32_PAIR
    if (e != hipSuccess) return e;
    if (pd.splits > 1 && pw.splits > 1)
        return launch_split_reduce_pair(gd, pd.splits, ws, gw, pw.splits, ws_w, s);
    if (pd.splits > 1) return launch_split_reduce(gd, pd.splits, ws, s);
    if (pw.splits > 1) return launch_split_reduce(gw, pw.splits, ws_w, s);
    return hipSuccess;
}

}  // namespace sbpi
