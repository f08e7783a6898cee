// Layer contractions of the forward pass (QKV, O, SwiGLU gate/up, down) on the MFMA kernel
// template of gemm_mfma.h: activations are the row operand, weights [out, in] the column
// operand.  The workgroup tile is picked per shape so that the grid fills the 256 CUs: big
// tiles (least LDS traffic per FLOP) when whole rounds of them come out, smaller ones for
// the short-M stage-1 pass and the narrow O / down projections.
#include <stdio.h>

#include "gemm_mfma.h"

namespace {

using namespace mfma;

struct TileCfg {
    int bm, bn;
    double stage;       // us for 64 of K with every CU at work (the model of gemm_bf16_tile)
    const char *name;
};
// index = value returned by gemm_bf16_tile.  One workgroup per CU: two of 128x128 or 128x192 with shallower rings were never ahead
// by more than 2 % of the best of these.
constexpr TileCfg kTiles[] = {
    {192, 256, 1.054, "192x256, LDS rings 2/3"},
    {256, 256, 1.349, "256x256, LDS rings 2/3"},   // least LDS and fetch traffic per FLOP; fills the 160 KB
    {256, 192, 1.067, "256x192, LDS rings 2/4"},
    {128, 192, 0.683, "128x192, LDS rings 4/4"},
    {128, 64, 0.341, "128x64, LDS rings 4/4"},
    {128, 128, 0.527, "128x128, LDS rings 4/4"},
    {64, 64, 0.208, "64x64, LDS rings 4/4"},
    {256, 128, 0.786, "256x128, LDS rings 3/4"},
    {96, 128, 0.435, "96x128, LDS rings 4/4"},
    {192, 128, 0.643, "192x128, LDS rings 3/4"},
    {192, 192, 0.841, "192x192, LDS rings 2/4"},
    {192, 64, 0.465, "192x64, LDS rings 4/4"},
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// launches `tile`; launch_cfg's arguments
template <int EPI, typename... Args>
void launch_tile(int tile, Args... args) {
    switch (tile) {
        case 0: return launch_cfg<192, 256, 2, 2, EPI, 2, 3>(args...);
        case 1: return launch_cfg<256, 256, 2, 2, EPI, 2, 3>(args...);
        case 2: return launch_cfg<256, 192, 2, 2, EPI, 2, 4>(args...);
        case 3: return launch_cfg<128, 192, 2, 2, EPI, 4, 4>(args...);
        case 4: return launch_cfg<128, 64, 2, 2, EPI, 4, 4>(args...);
        case 6: return launch_cfg<64, 64, 2, 2, EPI, 4, 4>(args...);
        case 7: return launch_cfg<256, 128, 2, 2, EPI, 3, 4>(args...);
        case 8: return launch_cfg<96, 128, 2, 2, EPI, 4, 4>(args...);
        case 9: return launch_cfg<192, 128, 2, 2, EPI, 3, 4>(args...);
        case 10: return launch_cfg<192, 192, 2, 2, EPI, 2, 4>(args...);
        case 11: return launch_cfg<192, 64, 2, 2, EPI, 4, 4>(args...);
        default: return launch_cfg<128, 128, 2, 2, EPI, 4, 4>(args...);
    }
}

// What the CUs that the last round of tiles leaves idle read ahead of `next`: items are cut to the bytes that they fetch in half of the
// round (45 GB/s a CU, 2 TB/s together), so that the tiles end last and keep most of the HBM rate (3 TB/s over 60 % of it gave
// the 7B cached batch 17.6 - 17.9 ms, 4 TB/s over 90 % 17.8, this 17.5, nothing 18.1; 8B prefill 8.47, nothing 8.59).  A launch over
// more than 2048 rows is bound by the matrix cores, and its tiles need the HBM rate for themselves.  The rows of a launch decide, not
// those of the contraction: what a cut leaves to its second launch (540 of 6684 rows of the 8B SwiGLU, half of the CUs) reads ahead as any other of
// its size.
// Nothing is read ahead where that and the weights that the round fetches itself exceed 200 MB: the last-level cache holds 256, so one pushes the other
// out again and the round has lost its HBM rate for nothing.  Three or four layers, nothing ahead / everything / this rule (us): d 6144, d_ffn 24 576, 136 rows 1612 / 1707
// / 1612; d 7168, d_ffn 18 432, 192 rows 1426 / 1479 / 1423; d 5120, d_ffn 25 600, 512 rows 1875 / 1939 / 1864; d 4096, d_ffn 14 336, 384 rows 976 / 954 / 940; d 2560, d_ffn 9728,
// 192 rows 573 / 541 / 541.  Over 12 layer shapes of d 2048 - 8192 at 136 - 2048 rows it is within 0.2 % of the best of these on average, and at most 1 % (noise
// is 1 - 2 % there) behind nothing ahead at any; with 240 or 270 MB, or with reads cut to what is left of 200 or 256, up to 1.6 % more than with it.
Warm spare_reads(Warm next, int tile, int64_t M, int64_t cols, int Kin) {
    const TileCfg &t = kTiles[tile];
    const int64_t n = ((M + t.bm - 1) / t.bm) * ((cols + t.bn - 1) / t.bn);
    const int idle = (int)((256 - n % 256) % 256);
    const double rate = idle * 45e3 < 2e6 ? idle * 45e3 : 2e6;     // bytes per us
    int64_t left = idle < 16 || M > 2048 ? 0 : (int64_t)(rate * (Kin / mfma::BK) * t.stage * 0.5) / 1024;    // KB
    int64_t want = 0;
    for (int i = 0; i < next.n; ++i) want += (int64_t)next.rows[i] * next.kb[i];
    const double own = (double)cols * Kin * 2 / 1024 * (n % 256) / n;    // KB of weights that the last round fetches
    if (own + (want < left ? want : left) > 200e6 / 1024) left = 0;
    for (int i = 0; i < next.n; ++i) {
        const int64_t fit = left / next.rows[i];
        if (next.kb[i] > fit) next.kb[i] = (int)fit;
        left -= (int64_t)next.rows[i] * next.kb[i];
        if (next.kb[i]) next.wgs = idle;
        else next.rows[i] = 0;
    }
    return next;
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
// Numbers of what runs: a tile, kNumTiles the streaming kernel, behind it the pairs of tiles of a contraction in two launches
static int pair_number(int first, int rest) { return kNumTiles + 1 + first * kNumTiles + rest; }
int gemm_bf16_kernel_count() { return pair_number(kNumTiles - 1, kNumTiles - 1) + 1; }
const char *gemm_bf16_tile_name(int tile) {
    static const struct Pairs {
        char name[kNumTiles * kNumTiles][80];
        Pairs() {
            for (int i = 0; i < kNumTiles * kNumTiles; ++i)
                snprintf(name[i], sizeof(name[i]), "two launches, %s and %s", kTiles[i / kNumTiles].name, kTiles[i % kNumTiles].name);
        }
    } pairs;
    if (tile < 0 || tile >= gemm_bf16_kernel_count()) return "?";
    if (tile == kNumTiles) return "all of up to 128 rows, streams the weights";
    return tile < kNumTiles ? kTiles[tile].name : pairs.name[tile - pair_number(0, 0)];
}

// Time of a launch (us).  Every workgroup has a CU to itself, so a launch takes whole rounds of 256 of them: K / 64 stages of the tile's
// time, plus prologue and epilogue, which are bound by memory and so by the outputs of the tile (256x256: 20 us for the read and
// write of the fp32 stream, 6.5 us for bf16 outputs).  A partial last round is shorter than a whole one, but not by much: the CUs
// run faster with others idle (clock, caches), down to 3/4 of the time (4/5 for small tiles).  Stage times fitted to a sweep of
// all tiles over the layer shapes of the benchmark configurations, 160 - 12 288 rows, cold weights: the tile chosen is within 1 %
// of the fastest on average, within 10 % everywhere but for 640 rows of the residual contractions (25 %).
static double tile_time(const TileCfg &t, int64_t M, int64_t cols, int Kin, int epi) {
    const unsigned n = (((unsigned)M + t.bm - 1) / t.bm) * (((unsigned)cols + t.bn - 1) / t.bn), whole = n / 256;   // (32 bits, as the grid)
    const double part = (double)(n % 256) / 256, area = t.bm * t.bn / 65536.0, least = area >= 0.375 ? 0.75 : 0.8;
    const double stages = (Kin / mfma::BK) * t.stage, ends = area * (epi == EPI_RESIDUAL ? 20 : 6.5) + 0.7;
    return 1.5 + stages * (whole + (part > 0 ? least + (1 - least) * part : 0)) + ends * (whole + (part > 0));
}

// the fastest tile among those that `fits` takes, -1: none
template <typename F>
static int fastest_tile(int64_t M, int64_t cols, int Kin, int epi, F fits) {
    int best = -1;
    double best_time = 0;
    for (int t = 0; t < kNumTiles; ++t) {
        if (!fits(kTiles[t])) continue;
        const double time = tile_time(kTiles[t], M, cols, Kin, epi);
        if (best < 0 || time < best_time) {
            best = t;
            best_time = time;
        }
    }
    return best;
}

// K of the model where the outputs are bf16: the depth does not move the choice there (the same regret with every shape's own K), and
// callers that ask for a tile by rows and outputs alone get the one that runs
constexpr int kStoreK = 4096;

int gemm_bf16_tile(int64_t M, int Nout, int epi, int Kin) {
    if (g_force_tile >= 0 && g_force_tile < kNumTiles) return g_force_tile;
    // SwiGLU reads two weight operands against one activation tile, half of the tile's columns each
    return fastest_tile(M, epi == EPI_SWIGLU ? 2 * (int64_t)Nout : Nout, epi == EPI_RESIDUAL && Kin ? Kin : kStoreK, epi, [](const TileCfg &) { return true; });
}

// A partial last round costs most of a whole one.  A contraction of some rounds may run as two launches instead: rows (or columns) that
// come out as whole rounds of one of the two largest tiles, and the others in the tiles that suit them.  Looked for from 1000 rows on
// (below, idle CUs read weights ahead: the 7B cached batch, 768 rows, is level), where a launch takes 50 us or more (the search
// takes some 5 us of the host's time) and up to 16 rounds; taken where the model, which adds 1.5 us for the gap, says 2.5 %.  8B
// ragged steps (6684 and 1671 rows) 125.7 -> 122.1 ms, 7B iteration (6144 and 1024) 78.3 -> 77.4.
SplitPlan gemm_bf16_plan(int64_t M, int Nout, int epi, int Kin) {
    SplitPlan best;
    best.tile = gemm_bf16_tile(M, Nout, epi, Kin);
    if (g_force_tile >= 0 || M < 1000 || (double)M * Nout * Kin < 3e10) return best;
    const int dual = epi == EPI_SWIGLU ? 2 : 1, K = epi == EPI_RESIDUAL && Kin ? Kin : kStoreK;
    const int64_t cols = (int64_t)Nout * dual;
    const auto any = [](const TileCfg &) { return true; };
    double least = tile_time(kTiles[best.tile], M, cols, K, epi) * 0.975 - 1.5;
    for (int t : {0, 1}) {
        const TileCfg &c = kTiles[t];
        const int64_t tm = (M + c.bm - 1) / c.bm, tn = (cols + c.bn - 1) / c.bn;
        if (tm * tn > 16 * 256) continue;
        for (int64_t r = 1; r * 256 < tm * tn; ++r) {
            const int64_t m0 = r * 256 / tn * c.bm, c0 = r * 256 / tm * c.bn;
            if (m0 > 0 && m0 < M) {
                const int rest = fastest_tile(M - m0, cols, K, epi, any);
                const double time = tile_time(c, m0, cols, K, epi) + tile_time(kTiles[rest], M - m0, cols, K, epi);
                if (time < least) {
                    least = time;
                    best.tile = t;
                    best.rows = m0;
                    best.cols = 0;
                    best.rest = rest;
                }
            }
            if (c0 > 0 && c0 < cols) {
                const int rest = fastest_tile(M, cols - c0, K, epi, any);
                const double time = tile_time(c, M, c0, K, epi) + tile_time(kTiles[rest], M, cols - c0, K, epi);
                if (time < least) {
                    least = time;
                    best.tile = t;
                    best.rows = 0;
                    best.cols = c0 / dual;
                    best.rest = rest;
                }
            }
        }
    }
    return best;
}

Warm gemm_bf16_ahead(const SplitPlan &p, int64_t M, int Nout, int epi, int Kin, const Warm &next) {
    const int64_t cols = Nout - p.cols;
    return spare_reads(next, p.rows || p.cols ? p.rest : p.tile, M - p.rows, epi == EPI_SWIGLU ? 2 * cols : cols, Kin);
}

namespace {

template <int EPI>
void dispatch(const bf16_t *A, const bf16_t *W, const bf16_t *W2, int M, int Nout, int Kin, int lda, int ldw,
              const float *bias, bf16_t *out, float *resid, int ldo, hipStream_t st, const Warm &next) {
    const SplitPlan p = gemm_bf16_plan(M, Nout, EPI, Kin);
    // rows [m0, m0 + rows) and output columns [c0, c0 + cols) on `tile`
    auto part = [&](int tile, int64_t m0, int rows, int c0, int cols, const Warm &ahead) {
        const int64_t o = m0 * ldo + c0, w = (int64_t)c0 * ldw;
        launch_tile<EPI>(tile, A + m0 * lda, W + w, W2 ? W2 + w : W2, rows, cols, Kin, lda, ldw, bias ? bias + c0 : bias, out ? out + o : out,
                         resid ? resid + o : resid, ldo, Top1Args(), st, 1, (float *)nullptr, QkvArgs(), ahead);
    };
    const Warm ahead = gemm_bf16_ahead(p, M, Nout, EPI, Kin, next);
    if (p.rows) {
        part(p.tile, 0, (int)p.rows, 0, Nout, Warm());
        part(p.rest, p.rows, M - (int)p.rows, 0, Nout, ahead);
    } else if (p.cols) {
        part(p.tile, 0, M, 0, (int)p.cols, Warm());
        part(p.rest, 0, M, (int)p.cols, Nout - (int)p.cols, ahead);
    } else {
        part(p.tile, 0, M, 0, Nout, ahead);
    }
}

}   // namespace

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

// QKV projection with rotary and the V transpose in its epilogue (EPI_QKV): every tile has to hold whole heads of one kind, so the
// tile width is a multiple of d_head and the first V column a multiple of the tile width.  -1: no such tile, run the store epilogue
// and the separate kernel instead.
static int qkv_tile(int64_t M, int Nout, int d_head, int v_start) {
    return fastest_tile(M, Nout, kStoreK, EPI_STORE, [&](const TileCfg &t) { return t.bn % d_head == 0 && v_start % t.bn == 0; });
}

int gemm_bf16_qkv_tile(int64_t M, int Nout, int d_head, int v_start, int rows_per_seq) {
    if ((d_head != 64 && d_head != 128) || rows_per_seq % 16 != 0 || Nout % 8 != 0) return -1;
    if (g_force_tile >= 0 && g_force_tile < kNumTiles) {
        const int bn = kTiles[g_force_tile].bn;
        return bn % d_head == 0 && v_start % bn == 0 ? g_force_tile : -1;
    }
    return qkv_tile(M, Nout, d_head, v_start);
}

// Few rows in one round of tiles of 128 columns or more (heads of 128), or in two of 64 columns (more than 256 heads of 64): tiles that walk all of K alone, against a stream over the weights and a launch that
// rotates, transposes and, for a KV cache, stores.  Fitted to both forms over 18 layer shapes of d 512 - 8192, 16 - 96 rows (us; 6.2 ns per K; 0.13 per
// MB of weights up to 64 rows, 0.24 above; 7 for the launches behind the stream where they store into caches, 3 where not): the choice is within
// 0.2 us of the faster form on average, within 6.4 everywhere.  7B shape (3584 -> 4608), 32 rows: fused 10.5 - 11 us a layer behind, MHA of 4096 at 96 rows
// 6 ahead; 96 heads of 64, d 6144, 48 and 49 rows 16 and 18 behind.  From 97 rows on and in one round of 64 columns the fused form is level or ahead.
bool gemm_bf16_qkv_in_two(int64_t M, int Nout, int Kin, int tile, bool into_cache) {
    const TileCfg &t = kTiles[tile];
    if (g_force_tile >= 0 || M > 96 || (t.bn < 128 && (M + t.bm - 1) / t.bm * ((Nout + t.bn - 1) / t.bn) <= 256)) return false;
    const double mb = (double)Nout * Kin * 2e-6;
    return 0.0062 * Kin > mb * (M <= 64 ? 0.13 : 0.24) + (into_cache ? 7 : 3);
}

// A partial last round of 256x256 tiles costs almost a whole one.  Where the column tiles of the whole rounds come out even
// enough, the columns behind them run as a launch of their own in the tiles that suit them (2048 x 12288 outputs, K = 4096: 384
// tiles in 172 us; 256 of them in 93, the other 4096 columns in 55 on 256x128 tiles), if that is faster than `tile` alone.
// Returns the second launch's first column, 0: one launch.
int gemm_bf16_qkv_cut(int64_t M, int Nout, int d_head, int v_start, int tile) {
    if (g_force_tile >= 0) return 0;
    const TileCfg &big = kTiles[1];
    if (big.bn % d_head != 0 || v_start % big.bn != 0) return 0;
    const int64_t tm = (M + 255) / 256, n = tm * ((Nout + 255) / 256), whole = n / 256 * 256 / tm;
    const int c0 = (int)whole * 256;
    if (n % 256 == 0 || n >= 8 * 256 || whole == 0 || c0 >= Nout) return 0;
    const int rest = qkv_tile(M, Nout - c0, d_head, v_start > c0 ? v_start - c0 : 0);
    if (rest < 0) return 0;
    const double two = tile_time(big, M, c0, kStoreK, EPI_STORE) + tile_time(kTiles[rest], M, Nout - c0, kStoreK, EPI_STORE);
    return two < tile_time(kTiles[tile], M, Nout, kStoreK, EPI_STORE) ? c0 : 0;
}

void launch_gemm_bf16_qkv(const bf16_t *A, const bf16_t *W, int64_t M, int Nout, int Kin, int lda, int ldw, const float *bias, bf16_t *qkv,
                          int ld_qkv, int d_head, int v_start, int rows_per_seq, int pos0, const float *cos_t, const float *sin_t,
                          const KvDest &kv, int tile, hipStream_t st, const Warm &next) {
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
                             (float *)nullptr, ld_qkv, Top1Args(), st, 1, (float *)nullptr, q, c0 + cols == Nout ? spare_reads(next, t, M, cols, Kin) : Warm());
    };
    const int c0 = gemm_bf16_qkv_cut(M, Nout, d_head, v_start, tile);
    if (c0 == 0) return part(tile, 0, Nout);
    part(1, 0, c0);
    part(qkv_tile(M, Nout - c0, d_head, v_start > c0 ? v_start - c0 : 0), c0, Nout - c0);
}

// the streaming kernel's plan for a contraction that it takes, tiles = 0 otherwise (16-byte accesses to out, resid and bias)
static StreamPlan stream_choice(int64_t M, int Nout, int Kin, int epi, const float *bias, const bf16_t *out, const float *resid, int ldo) {
    if (M > 128 || g_force_tile >= 0 || ldo % 4 || !aligned16(epi == EPI_RESIDUAL ? (const void *)resid : (const void *)out) ||
        (epi == EPI_BIAS && !aligned16(bias)))
        return StreamPlan();
    return stream_plan(M, Nout, Kin, epi, 1, 1);
}

int gemm_bf16_kernel(int64_t M, int Nout, int Kin, int epi, const float *bias, const bf16_t *out, const float *resid, int ldo) {
    if (stream_choice(M, Nout, Kin, epi, bias, out, resid, ldo).tiles) return kNumTiles;
    const SplitPlan p = gemm_bf16_plan(M, Nout, epi, Kin);
    return p.rows || p.cols ? pair_number(p.tile, p.rest) : p.tile;
}

void launch_gemm_bf16(const bf16_t *A, const bf16_t *W, const bf16_t *W2, int64_t M, int Nout, int Kin, int lda, int ldw, int epi,
                      const float *bias, bf16_t *out, float *resid, int ldo, hipStream_t st, const Warm &next) {
    const int m = (int)M;
    const StreamPlan plan = stream_choice(M, Nout, Kin, epi, bias, out, resid, ldo);
    if (plan.tiles) return launch_gemm_stream(plan, A, W, W2, M, Nout, Kin, lda, ldw, epi, bias, out, resid, ldo, nullptr, st);
    switch (epi) {
        case EPI_STORE: dispatch<EPI_STORE>(A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, st, next); break;
        case EPI_BIAS: dispatch<EPI_BIAS>(A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, st, next); break;
        case EPI_RESIDUAL: dispatch<EPI_RESIDUAL>(A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, st, next); break;
        default: dispatch<EPI_SWIGLU>(A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, st, next); break;
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
