// Layer contractions of the forward pass (QKV, O, SwiGLU gate/up, down) on the MFMA kernel
// template of gemm_mfma.h: activations are the row operand, weights [out, in] the column
// operand.  The workgroup tile is picked per shape so that the grid fills the 256 CUs: big
// tiles (least LDS traffic per FLOP) when whole rounds of them come out, smaller ones for
// the short-M stage-1 pass and the narrow O / down projections.
#include "gemm_mfma.h"

namespace {

using namespace mfma;

struct TileCfg {
    int bm, bn;
    const char *name;
};
// index = value returned by gemm_bf16_tile
constexpr TileCfg kTiles[] = {
    {128, 128, "128x128, LDS rings 2/3"},   // two workgroups per CU
    {256, 256, "256x256, LDS rings 2/3"},   // least LDS traffic per FLOP; fills the 160 KB
    {256, 192, "256x192, LDS rings 2/4"},
    {128, 192, "128x192, LDS rings 2/2"},   // two workgroups per CU
    {128, 64, "128x64, LDS rings 4/4"},     // lone workgroup per CU: fetches several stages ahead
    {128, 128, "128x128, LDS rings 4/4"},
    {64, 64, "64x64, LDS rings 4/4"},
    {256, 128, "256x128, LDS rings 3/4"},   // one full round of 256 workgroups for 2048 x 4096 outputs
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// launches `tile`; launch_cfg's arguments
template <int EPI, typename... Args>
void launch_tile(int tile, Args... args) {
    switch (tile) {
        case 1: return launch_cfg<256, 256, 2, 2, EPI, 2, 3>(args...);
        case 2: return launch_cfg<256, 192, 2, 2, EPI, 2, 4>(args...);
        case 3: return launch_cfg<128, 192, 2, 2, EPI, 2, 2, 2>(args...);
        case 4: return launch_cfg<128, 64, 2, 2, EPI, 4, 4>(args...);
        case 5: return launch_cfg<128, 128, 2, 2, EPI, 4, 4>(args...);
        case 6: return launch_cfg<64, 64, 2, 2, EPI, 4, 4>(args...);
        case 7: return launch_cfg<256, 128, 2, 2, EPI, 3, 4>(args...);
        default: return launch_cfg<128, 128, 2, 2, EPI, 2, 3, 2>(args...);
    }
}

template <int EPI>
void dispatch(const bf16_t *A, const bf16_t *W, const bf16_t *W2, int M, int Nout, int Kin, int lda, int ldw,
              const float *bias, bf16_t *out, float *resid, int ldo, hipStream_t st) {
    launch_tile<EPI>(gemm_bf16_tile(M, Nout, EPI, Kin), A, W, W2, M, Nout, Kin, lda, ldw, bias, out, resid, ldo, Top1Args(), st);
}

}   // namespace

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
static int g_force_tile = -1, g_force_splits = 0, g_group_m = 4;
// tile < 0: automatic.  Otherwise bits 0-7 the tile, bits 8-15 the K-split of the residual hook, bits 16-23 the band
// height of the tile order (0 = leave it)
void gemm_bf16_force_tile(int tile) {
    g_force_tile = tile < 0 ? -1 : (tile & 0xff) == 0xff ? -1 : (tile & 0xff);
    g_force_splits = tile < 0 ? 0 : ((tile >> 8) & 0xff);
    if (tile < 0) g_group_m = 4;
    else if ((tile >> 16) & 0xff) g_group_m = (tile >> 16) & 0xff;
}
int gemm_tile_group_m() { return g_group_m; }
int gemm_bf16_tile_count() { return kNumTiles; }
const char *gemm_bf16_tile_name(int tile) {
    return tile >= 0 && tile < kNumTiles ? kTiles[tile].name : tile == kNumTiles ? "all of up to 128 rows, streams the weights" : "?";
}

int gemm_bf16_tile(int64_t M, int Nout, int epi, int Kin) {
    if (g_force_tile >= 0 && g_force_tile < kNumTiles) return g_force_tile;
    const bool dual = epi == EPI_SWIGLU;
    const int64_t cols = dual ? 2 * (int64_t)Nout : Nout;
    auto tiles = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((cols + bn - 1) / bn); };
    // SwiGLU reads two weight operands against one activation tile: the big tile as soon as it
    // reaches half of the CUs
    // (a single row tile is a pure weight stream: the deep equal rings keep more of it in flight)
    // A partial round costs a whole one, and a round of 256x192 tiles (96 gate and 96 up columns) 0.84 of a round of 256x256: it
    // wins where it needs no more rounds (2 x 12288 outputs, K = 4096: 512 rows 103 -> 96 us, 300 rows 94.5 -> 88, 700 rows
    // 175 -> 153; 1671 rows 280 against 316 and 2048 rows 303 against 338 stay on 256x256).
    if (dual) {
        const int64_t big = tiles(256, 256);
        if (big < 128) return M <= 128 ? 5 : 0;
        return (tiles(256, 192) + 255) / 256 <= (big + 255) / 256 ? 2 : 1;
    }
    // At most one 128x128 workgroup per CU: the contraction is bound by fetch latency, not by the
    // matrix cores; small tiles reach every CU and the deep rings keep several stages in flight.
    if (tiles(128, 128) <= 256) {
        const int64_t t = tiles(128, 64);
        return t <= 128 ? 6 : t <= 256 ? 4 : 5;
    }
    // Otherwise: rounds of workgroups over the 256 CUs times the work of one round, weighted by the
    // rate each tile sustains on a full machine (PFLOP/s with weights streamed cold from HBM, from a
    // sweep over the layer shapes of the benchmark configurations).  A tile that runs two workgroups per
    // CU does a round of 512 in the time of two.
    struct Cand {
        int tile, per_round;
        double rate;
    };
    // Residual contractions (fp32 read-modify-write epilogue), measured at 2048 x 4096 and 6144 x 3584 outputs: 256x192 beats
    // 128x192 by 2 - 8 % and three rounds of 256x128 (K = 18944: 790 against 820 us, K = 3584: 155 against 163); one full round of
    // 256x128 beats two 128x128 workgroups per CU (K = 4096: 66 against 75 us, in the 16x16x32 MFMA form; K = 12288, where the
    // 32x32x16 form is level with it, 236 against 238).  Kin = 0: unknown, taken as long.  Store epilogues: the 256x128 tile is
    // ahead of 128x128 per round of workgroups (512 x 12288 outputs: 53 against 68 us) and behind 256x192.
    // (With the activation ring one stage deeper, 3/4 against 2/4, the 256x128 tile takes 236 us instead of 264 on 2048 x 4096
    // outputs at K = 12288, 66 instead of 73 at K = 4096, and 53 instead of 56 on 512 x 12288.)
    const bool resid = epi == EPI_RESIDUAL;
    const Cand cand[] = {{1, 256, 1.25}, {2, 256, 1.16}, {3, 512, resid ? 1.12 : 1.15}, {0, 512, 1.00},
                         {7, 256, !resid ? 1.06 : (Kin == 0 || Kin > 4096) ? 1.12 : 1.05}};
    int best = 0;
    double best_cost = 0;
    for (const Cand &c : cand) {
        const int64_t n = tiles(kTiles[c.tile].bm, kTiles[c.tile].bn);
        const int64_t rounds = (n + c.per_round - 1) / c.per_round;
        const double cost = (double)rounds * (c.per_round / 256) * kTiles[c.tile].bm * kTiles[c.tile].bn / c.rate;
        if (best_cost == 0 || cost < best_cost) {
            best_cost = cost;
            best = c.tile;
        }
    }
    return best;
}

// A residual contraction over at most 128 rows is cut along K: part 0 adds into resid, the others store partial sums that the next
// reader of resid adds in order.  The parts are those the streaming kernel plans for 128 rows, whatever the number of rows: a
// sequence's sums must not depend on how many rows share its call.  At most four: eight cost the norm more than they save here
// (8B cached iteration 9.42 ms, with four 9.04, with the plan of each row count 9.06).
int gemm_bf16_splits(int64_t M, int Nout, int Kin) {
    int splits = 1;
    if (g_force_splits > 0) splits = g_force_splits;
    else if (g_force_tile < 0 && M <= 128) splits = stream_plan(128, Nout, Kin, EPI_RESIDUAL, 1, 4).splits;
    if (splits > 8 || splits < 1 || Kin % (splits * BK) != 0) splits = 1;
    return splits;
}

void launch_gemm_bf16_split(const bf16_t *A, const bf16_t *W, int64_t M, int Nout, int Kin, int lda, int ldw, float *resid, int ldo,
                            float *partial, int splits, hipStream_t st) {
    if (g_force_splits == 0 && g_force_tile < 0) {
        const StreamPlan plan = stream_plan(M, Nout, Kin, EPI_RESIDUAL, splits, splits);
        if (plan.tiles && ldo % 4 == 0 && aligned16(resid) && aligned16(partial))
            return launch_gemm_stream(plan, A, W, nullptr, M, Nout, Kin, lda, ldw, EPI_RESIDUAL, nullptr, nullptr, resid, ldo, partial, st);
    }
    launch_cfg<128, 128, 2, 2, EPI_RESIDUAL, 4, 4>(A, W, nullptr, (int)M, Nout, Kin, lda, ldw, nullptr, nullptr, resid, ldo, Top1Args(), st,
                                                   splits, partial);
}

// QKV projection with rotary and the V transpose in its epilogue (EPI_QKV).  The tile is the one the plain store
// would get, provided every tile then holds whole heads of one kind: the tile width a multiple of d_head and the first
// V column a multiple of the tile width.  -1: no such tile, run the store epilogue and the separate kernel instead.
int gemm_bf16_qkv_tile(int64_t M, int Nout, int d_head, int v_start, int rows_per_seq) {
    if ((d_head != 64 && d_head != 128) || rows_per_seq % 16 != 0 || Nout % 8 != 0) return -1;
    int tile = gemm_bf16_tile(M, Nout, EPI_STORE);
    // the 192-column tiles cut heads in two: the 256x256 tile takes over where the plain store would have picked one of
    // them (2048 x 6144 outputs: 87 us + 24 us for the separate rotary / transpose kernel against 95 us in one)
    if (tile == 2 || tile == 3) tile = 1;
    const int bn = kTiles[tile].bn;
    if (bn % d_head != 0 || v_start % bn != 0) return -1;
    return tile;
}

// A partial last round of 256x256 tiles costs almost a whole one.  Where the column tiles of the whole rounds come out even
// enough, the columns behind them run as a launch of their own in smaller tiles, one round of which is shorter (2048 x 12288
// outputs, K = 4096: 384 tiles in 179 us; 256 of them in 99, the other 4096 columns in 57 on 256x128 tiles).  Costs as in
// gemm_bf16_tile; the second launch takes some 3 us, 2000 units at that K.  Returns the second launch's first column, 0: one launch.
int gemm_bf16_qkv_cut(int64_t M, int Nout, int Kin, int tile) {
    if (tile != 1 || g_force_tile >= 0) return 0;
    const int64_t tm = (M + 255) / 256, n = tm * ((Nout + 255) / 256), whole = n / 256 * 256 / tm;
    const int c0 = (int)whole * 256;
    if (n % 256 == 0 || n >= 8 * 256 || whole == 0 || c0 >= Nout) return 0;
    auto cost = [&](int64_t tiles, double area, double rate) { return (double)((tiles + 255) / 256) * area / rate; };
    const double rest = cost(tm * ((Nout - c0 + 127) / 128), 32768, 1.06);
    return cost(whole * tm, 65536, 1.25) + rest + 2000.0 * 4096 / Kin < cost(n, 65536, 1.25) ? c0 : 0;
}

void launch_gemm_bf16_qkv(const bf16_t *A, const bf16_t *W, int64_t M, int Nout, int Kin, int lda, int ldw, const float *bias, bf16_t *qkv,
                          int ld_qkv, int d_head, int v_start, int rows_per_seq, int pos0, const float *cos_t, const float *sin_t,
                          const KvDest &kv, int tile, hipStream_t st) {
    QkvArgs qa;
    qa.d_head = d_head;
    qa.v_start = v_start;
    qa.N = rows_per_seq;
    qa.pos0 = pos0;
    qa.cos_t = cos_t;
    qa.sin_t = sin_t;
    qa.vT = kv.vT;
    qa.ld_vt = kv.ld_vt;
    qa.vt_seq = kv.vt_seq;
    qa.k_dst = kv.k;
    qa.ld_k = kv.ld_k;
    qa.k_start = kv.k_start;
    qa.k_seq = kv.k_seq;
    const int m = (int)M;
    // columns [c0, c0 + cols) on tile t
    auto part = [&](int t, int c0, int cols) {
        QkvArgs q = qa;
        q.v_start -= c0;
        q.k_start -= c0;
        launch_tile<EPI_QKV>(t, A, W + (int64_t)c0 * ldw, (const bf16_t *)nullptr, m, cols, Kin, lda, ldw, bias ? bias + c0 : nullptr, qkv + c0,
                             (float *)nullptr, ld_qkv, Top1Args(), st, 1, (float *)nullptr, q);
    };
    const int c0 = gemm_bf16_qkv_cut(M, Nout, Kin, tile);
    if (c0 == 0) return part(tile, 0, Nout);
    part(1, 0, c0);
    part(7, c0, Nout - c0);
}

// the streaming kernel's plan for a contraction that it takes, tiles = 0 otherwise (16-byte accesses to out, resid and bias)
static StreamPlan stream_choice(int64_t M, int Nout, int Kin, int epi, const float *bias, const bf16_t *out, const float *resid, int ldo) {
    if (M > 128 || g_force_tile >= 0 || ldo % 4 || !aligned16(epi == EPI_RESIDUAL ? (const void *)resid : (const void *)out) ||
        (epi == EPI_BIAS && !aligned16(bias)))
        return StreamPlan();
    return stream_plan(M, Nout, Kin, epi, 1, 1);
}

int gemm_bf16_kernel(int64_t M, int Nout, int Kin, int epi, const float *bias, const bf16_t *out, const float *resid, int ldo) {
    return stream_choice(M, Nout, Kin, epi, bias, out, resid, ldo).tiles ? kNumTiles : gemm_bf16_tile(M, Nout, epi, Kin);
}

void launch_gemm_bf16(const bf16_t *A, const bf16_t *W, const bf16_t *W2, int64_t M, int Nout, int Kin, int lda, int ldw, int epi,
                      const float *bias, bf16_t *out, float *resid, int ldo, hipStream_t st) {
    const int m = (int)M;
    const StreamPlan plan = stream_choice(M, Nout, Kin, epi, bias, out, resid, ldo);
    if (plan.tiles) return launch_gemm_stream(plan, A, W, W2, M, Nout, Kin, lda, ldw, epi, bias, out, resid, ldo, nullptr, st);
    switch (epi) {
        case EPI_STORE: dispatch<EPI_STORE>(A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, st); break;
        case EPI_BIAS: dispatch<EPI_BIAS>(A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, st); break;
        case EPI_RESIDUAL: dispatch<EPI_RESIDUAL>(A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, st); break;
        default: dispatch<EPI_SWIGLU>(A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, st); break;
    }
}

// ---------------------------------------------------------------------------------------------
// Calibration: what a loop of nothing but v_mfma_f32_32x32x16_bf16 sustains on this device when
// the operands are real data (16 independent accumulators per wavefront, 4 wavefronts per CU,
// operand registers rotated every iteration).  The MFMA clock is power-managed, so this is well
// below the rate the same loop reaches on all-zero operands; it is the ceiling a contraction
// kernel can be judged against besides the published peak.
namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void mfma_rate_kernel(const u32x4_t *__restrict__ src, int n_src, int iters,
                                                        floatx16 *__restrict__ sink) {
    bf16x8 a[4], b[4];
    for (int i = 0; i < 4; ++i) {
        a[i] = __builtin_bit_cast(bf16x8, src[(threadIdx.x * 8 + i) % n_src]);
        b[i] = __builtin_bit_cast(bf16x8, src[(threadIdx.x * 8 + 4 + i) % n_src]);
    }
    floatx16 acc[4][4];
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j)
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        bf16x8 t = a[0];
        a[0] = a[1]; a[1] = a[2]; a[2] = a[3]; a[3] = t;
        t = b[0];
        b[0] = b[1]; b[1] = b[2]; b[2] = b[3]; b[3] = t;
    }
    floatx16 s = acc[0][0];
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j)
            if (i || j) s += acc[i][j];
    sink[blockIdx.x * 256 + threadIdx.x] = s;
}

}   // namespace

void launch_mfma_rate(const void *operands, int n_vec16, int iters, void *sink, hipStream_t st) {
    hipLaunchKernelGGL(mfma_rate_kernel, dim3(256), dim3(256), 0, st, (const u32x4_t *)operands, n_vec16, iters,
                       (floatx16 *)sink);
}
