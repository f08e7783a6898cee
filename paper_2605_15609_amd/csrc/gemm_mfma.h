// bf16 contraction D[i, j] = sum_k X[i, k] * Y[j, k] on the gfx950 matrix cores
// (v_mfma_f32_16x16x32_bf16, fp32 accumulation).  Both operands are K-contiguous ("NT"
// form, row strides ldx / ldy elements), the natural MFMA feed: every lane fetches 8 consecutive k
// (16 bytes) of one row.
//
// What bounds it: large shapes the power limit (256x256 tiles: the matrix cores are busy 70 - 80 % of the cycles and the clock has
// come down to 1.8 GHz), so what counts is energy per MFMA as much as issue slots; short ones the fetches of a CU (about 65 GB/s
// from behind its L2, whatever is in flight).  Hence four wavefronts a workgroup, each with the largest share of the tile that the
// 512 registers of a SIMD's lane hold: 128x128 of a 256x256 tile, 256 accumulators, two thirds of the LDS reads of eight
// wavefronts.  One wavefront a SIMD has nobody to hide behind, so the main loop is laid out by hand: MFMAs as inline asm in a
// fixed order, LDS reads and fetches between them one at a time, each read at least a quarter of a stage before its use.
// Against eight wavefronts scheduled by the compiler, cold weights: 20480 rows, SwiGLU of 12288 2877 -> 2755 us (1.50 PFLOP/s),
// store of 12288 1485 -> 1383, residual 4096 x 12288 1629 -> 1413 (1.46 PFLOP/s), 4096 x 4096 618 -> 544; 512 rows SwiGLU
// 91 -> 80, residual 86 -> 77.5 and 33 -> 28; 2048 rows, residual 4096 x 12288 236 -> 161.
//
// Tiling: a workgroup of 4 wavefronts owns a BM x BN tile; K advances 64 at a time.  Each
// operand tile has its own ring of LDS stages (NSA for X, NSB for Y) filled by direct global -> LDS
// loads, one barrier per stage.  The rings differ in depth because the operands differ in where
// they come from: activations were just written and sit in cache, weights arrive cold from HBM and
// need their fetches several stages ahead.
// LDS rows are 128 bytes; the 16-byte chunk c of row r sits at chunk slot c ^ ((r >> 1) & 7),
// so the 16 rows a wavefront touches per fragment fetch spread over all 64 banks.  Workgroup ids are remapped so
// that each of the 8 XCDs (which receive consecutive ids round-robin) works on a compact
// range of tiles and its private L2 sees the operand reuse.
//
// The weights are the row operand of the MFMA, so after the K loop a lane holds, for every 16x16 subtile, row lane % 16 of X and the
// 4 consecutive columns 4 * (lane / 16) ..: 8- and 16-byte accesses in the epilogues (EPI_TOP1 has the operands the other way
// round: a lane holds one column and 4 consecutive rows).  K runs in order in every accumulator: the same bits for every tile.
// The epilogue is a template policy:
//   EPI_STORE / EPI_BIAS   out = bf16(acc (+ bias[j]))                     QKV projection
//   EPI_RESIDUAL           resid[i, j] += acc           (fp32 stream)       O and down projections
//                          With k_splits > 1 the K range is cut into equal parts, one workgroup per (tile,
//                          part): part 0 adds into resid, part s > 0 stores its sum to partial[s - 1] (same
//                          shape, dense rows), and whoever reads the stream next adds the partials in order.
//   EPI_SWIGLU             out = bf16(silu(X Yg^T) * (X Yu^T))              gate and up in one pass
//   EPI_TOP1               per column j: running (max, argmax, sum-exp) over the rows i
//                          (LM-head with X = W_lm, Y = hidden rows; logits never stored)
//   EPI_QKV                QKV projection with what used to be a second pass over its output folded in: the tile
//                          (+ bias) is rounded to bf16 into LDS (the operand rings are free by then); a tile of q / k
//                          heads is read back row-wise, rotated (rotary position of row m: pos0 + m % N) and stored
//                          with 16-byte accesses; a tile of V heads is read back column-wise and stored transposed,
//                          key-contiguous, in the slot order the attention kernel's second MFMA wants.  Same values
//                          as EPI_STORE / EPI_BIAS followed by the separate rotary / transpose kernel, bit for bit.
#pragma once
#include <utility>

#include "psd_internal.h"
#include "device_types.h"
#include "rope_device.h"
#include "warm_device.h"

// row tiles per band of the tile order (see the kernel); 4 unless a tuning run changes it (measured over the layer
// contractions of the 8B shapes at 2048 - 163 840 rows: bands of 4 and 8 within 1 %, 1 and 16 about 5 % slower)
int gemm_tile_group_m();

namespace mfma {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int EPI_TOP1 = 4;
constexpr int EPI_QKV = 5;
constexpr int BK = 64;                  // k extent per stage (bf16) = 128 bytes per LDS row

struct Top1Args {
    float scale;        // logits = scale * acc
    int mask_id;        // row (vocab id) that is never predicted
    float *pmax;        // [slabs, cols] partial maxima
    float *psum;        // [slabs, cols] partial sum exp(z - pmax)
    int32_t *parg;      // [slabs, cols] partial argmax (lowest id on ties)
    int cols_total;
};

struct QkvArgs {
    int d_head;           // 64 or 128; every tile holds whole heads (BN % d_head == 0)
    int v_start;          // columns [0, v_start) are q and k heads, [v_start, Nout) V heads; a multiple of BN
    int N, pos0;          // rows per sequence (a multiple of 16 if vT) and the rotary position of a sequence's first row
    const float *cos_t, *sin_t;   // [positions, d_head / 2]
    bf16_t *vT;           // value column c, key i of sequence s at vT[s * vt_seq + c * ld_vt + slot(i)]; NULL: values row-major in `out`
    int ld_vt;
    int64_t vt_seq;
    // k heads (columns [k_start, v_start)): k_dst = NULL: into `out` next to q; otherwise into a KV cache, row i of sequence s
    // at k_dst[s * k_seq + i * ld_k + column - k_start]
    bf16_t *k_dst;
    int ld_k, k_start;
    int64_t k_seq;
};

// Swizzle key of an LDS row: 64 banks x 4 bytes = 256 bytes per bank line, rows are 128 bytes, so rows r and r+1 cover
// the two halves of a bank line and the chunk slot is rotated by (r >> 1) over the 8 slots of a row: 16 consecutive rows
// fetching the same logical 16-byte chunk hit 16 distinct bank groups.
__device__ __forceinline__ int row_key(int row) { return (row >> 1) & 7; }

// merge two (max, argmax, sum-exp) triples; ties go to the lower index
__device__ __forceinline__ void top1_merge(float &b, int &a, float &s, float b2, int a2, float s2) {
    const float bn = fmaxf(b, b2);
    const float s_new = (bn == -INFINITY) ? 0.f : s * __expf(b - bn) + s2 * __expf(b2 - bn);
    if (b2 > b || (b2 == b && a2 < a)) a = a2;
    b = bn;
    s = s_new;
}

// f(0), f(1) .. f(N - 1) with constant arguments (the loops of the main loop are longer than what the compiler unrolls by itself)
template <typename F, int... I>
__device__ __forceinline__ void static_for(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for(f, std::make_integer_sequence<int, N>());
}
// The bf16 epilogues go through LDS.  A lone wavefront a SIMD waits out the latency of every read, so a thread takes up to `most` of its `per` units
// at a time, all reads before the first store (one unit at a time the QKV projection was up to 10 % behind eight wavefronts a workgroup:
// 8192 rows, K = 1024, 3072 outputs 57 -> 63 us, with batches 60; 1536 outputs 34 -> 37, 35; 4096 rows, K = 2048, 6144 outputs 91 -> 97, 92; 2048 rows, K = 4096,
// 12288 outputs 160 -> 163, 158).
constexpr int batch_of(int per, int most) {
    int b = 1;
    for (int i = 2; i <= most; ++i)
        if (per % i == 0) b = i;
    return b;
}
// of n events spread over `span` steps, the first one at step t or later
constexpr int event_at(int t, int n, int span) { return (t * n + span - 1) / span < n ? (t * n + span - 1) / span : n; }

// One MFMA, accumulated in place.  Written as inline asm because the register allocator otherwise gives the result a register of its
// own and moves it back (v_accvgpr_read / write: more instructions than MFMAs, half the rate); the operands are ordinary values, so the
// compiler still places the waits for the LDS reads that produce them.  Consecutive MFMAs never touch the same accumulator, and the
// one wait state count that matters (result -> ordinary read) is spent after the main loop.
__device__ __forceinline__ void mfma_acc(floatx4 &acc, bf16x8 a, bf16x8 b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// WPS: wavefronts per SIMD that the registers must allow (workgroups per CU)
template <int BM, int BN, int WGM, int WGN, int EPI, int NSA, int NSB, int WPS>
__global__ __launch_bounds__(WGM * WGN * 64, WPS) void gemm_bf16_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ Y,
                                                        const bf16_t *__restrict__ Y2, int M, int Nout, int Kin, int ldx, int ldy,
                                                        const float *__restrict__ bias, bf16_t *__restrict__ out,
                                                        float *__restrict__ resid, int ldo, int tiles_n, int n_tiles,
                                                        Top1Args t1, int k_splits, float *__restrict__ partial, int group_m,
                                                        QkvArgs qa, Warm next) {
    if constexpr (EPI != EPI_TOP1) {
        if ((int)blockIdx.x >= (int)gridDim.x - next.wgs) return warm_part(next, blockIdx.x - (gridDim.x - next.wgs));   // spare workgroups
    }
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int ROW_BYTES = BK * 2;                     // an LDS row: one tile row of one stage
    constexpr int LPR = ROW_BYTES / 16, RPI = 64 / LPR;   // lanes per LDS row (8) and rows per DMA instruction (8: 1 KB)
    constexpr bool DUAL = EPI == EPI_SWIGLU;
    constexpr bool SWAP = EPI != EPI_TOP1;                // weights as the row operand: a lane holds 4 consecutive outputs of one row
    constexpr int BN_OUT = DUAL ? BN / 2 : BN;            // output columns per tile
    constexpr int A_BYTES = BM * ROW_BYTES, B_BYTES = BN * ROW_BYTES, B_RING = NSA * A_BYTES;   // X ring first, then the Y ring
    constexpr int MI = 16;
    constexpr int WTM = BM / WGM, WTN = BN / WGN, TM = WTM / MI, TN = WTN / MI, NV = 4;
    constexpr int NW = WGM * WGN, T = TM * TN, R = TM + TN;
    static_assert(NW == 4 && TM >= 1 && TN >= 1 && (!DUAL || TN % 2 == 0), "tile shape");
    static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "every wavefront moves whole row groups of both tiles");

    // XCD-aware tile id: ids i, i+8, i+16 ... land on the same XCD; give that XCD a contiguous tile range (XCD x has one id more than
    // n_tiles / 8 while x < n_tiles % 8)
    int pid = blockIdx.x, split = 0;
    if (EPI == EPI_RESIDUAL && k_splits > 1) {
        split = pid / n_tiles;
        pid -= split * n_tiles;
    }
    const int k_len = Kin / k_splits, k_beg = split * k_len;   // this workgroup's K range
    pid = (pid % 8) * (n_tiles / 8) + min(pid % 8, n_tiles % 8) + pid / 8;
    // Each XCD has its own L2 and runs about 32 consecutive tile ids of its range at a time, all walking K roughly in
    // step, so those 32 tiles should share operand tiles both ways: ids are laid out in bands of `group_m` row tiles,
    // column-major inside a band, which makes 32 consecutive ids a patch of group_m x (32 / group_m) tiles (every
    // activation K-slice is fetched once for 32 / group_m workgroups, every weight K-slice once for group_m).  With
    // at most group_m row tiles this is the plain "rows fastest" order.
    const int tiles_m = n_tiles / tiles_n;
    const int band = group_m * tiles_n;
    const int first_m = (pid / band) * group_m;
    const int rows_in_band = min(tiles_m - first_m, group_m);
    const int tile_m = first_m + (pid % band) % rows_in_band;
    const int tile_n = (pid % band) / rows_in_band;
    const int m0 = tile_m * BM, n0 = tile_n * BN_OUT;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    floatx4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // Operand tiles go from global memory straight into LDS (buffer_load ... lds): no staging
    // registers and no ds_write traffic on the wavefronts' issue ports.  One such instruction moves
    // 64 lanes x 16 bytes = 8 tile rows x 128 bytes into 1 KB of consecutive LDS, lane l landing at
    // offset 16*l, i.e. row l/8, chunk slot l%8.  The XOR swizzle therefore lives on the global
    // side: the lane fetches logical chunk (l%8) ^ key(row), key(row) = (row >> 1) & 7.  Row groups
    // are dealt to the NW wavefronts round-robin (group g = NW*j + wave), which makes the key a
    // per-lane constant: ((wave & 1) * 4 + l/16) & 7.  The per-lane byte offset is one VGPR; the
    // group and K position are wave-uniform and ride in a scalar offset.  Rows past the matrix edge
    // are rejected by the descriptor's range check (they only feed outputs that are never stored), and so are stages past the
    // end of K, whose offset no descriptor takes: no traffic, and the counts of fetches in flight stay what the waits assume.
    const int rows_x = min(BM, M - m0), rows_y = min(BN_OUT, Nout - n0);
    const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(X) + (int64_t)m0 * ldx + k_beg, 0, ((rows_x - 1) * ldx + Kin - k_beg) * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(Y) + (int64_t)n0 * ldy + k_beg, 0, ((rows_y - 1) * ldy + Kin - k_beg) * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_y2 = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(DUAL ? Y2 : Y) + (int64_t)n0 * ldy + k_beg, 0, ((rows_y - 1) * ldy + Kin - k_beg) * 2, 0x00020000);
    const int dma_key = (((wave & 1) << 2) + (lane >> 4)) & 7;
    const int voff_x = (lane / LPR) * ldx * 2 + (((lane % LPR) ^ dma_key) << 4);
    const int voff_y = (lane / LPR) * ldy * 2 + (((lane % LPR) ^ dma_key) << 4);
    constexpr int VOFF_NONE = 0x7ffffff0;
    constexpr int GA = BM / RPI / NW, GB = BN / RPI / NW, NLD = GA + GB;
    static_assert(!DUAL || (BN / 2) % (RPI * NW) == 0, "a fetch of the wavefronts holds gate or up rows");
    typedef __attribute__((address_space(3))) void lds_void;
    const int nk = k_len / BK;
    auto dma_a = [&](int j, int slot, int kt) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_x, (lds_void *)(lds + slot * A_BYTES + (j * NW + wave) * 1024), 16, kt < nk ? voff_x : VOFF_NONE,
                                                 ((j * NW + wave) * RPI * ldx + kt * BK) * 2, 0, 0);
    };
    auto dma_b = [&](int j, int slot, int kt) {
        unsigned char *d = lds + B_RING + slot * B_BYTES + (j * NW + wave) * 1024;
        const int v = kt < nk ? voff_y : VOFF_NONE;
        if (DUAL && j * (RPI * NW) >= BN / 2)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_y2, (lds_void *)d, 16, v, (((j * NW + wave) * RPI - BN / 2) * ldy + kt * BK) * 2, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_y, (lds_void *)d, 16, v, ((j * NW + wave) * RPI * ldy + kt * BK) * 2, 0, 0);
    };
    // Every iteration issues the fetch of the shallower ring first.  Memory returns in issue order, so
    // once the counter says that at most WAIT younger DMA instructions are in flight, both tiles of the
    // next stage have landed: with the X ring shallower, its stage kt+1 was issued NSA-2 iterations ago
    // and only that iteration's Y fetch plus NSA-2 whole iterations are younger (and mirrored).
    constexpr int WAIT = NSA < NSB ? (NSA - 2) * NLD + GB : NSA > NSB ? (NSB - 2) * NLD + GA : (NSA - 2) * NLD;
    constexpr int WAIT0 = WAIT + NLD;
    static_assert(NSA >= 2 && NSB >= 2 && WAIT0 <= 63, "fetches in flight must fit the vmcnt counter");

    const int lrow = lane & 15, lq = lane >> 4;
    const int rsw = row_key(lrow);
    // fragment addresses: the 16-row subtiles of a wavefront lie 2048 bytes apart, immediates of the reads
    const int a0 = (wm * WTM + lrow) * ROW_BYTES, b0 = B_RING + ((DUAL ? wn * (WTN / 2) : wn * WTN) + lrow) * ROW_BYTES;
    const int c0 = (lq ^ rsw) << 4, c1 = ((4 + lq) ^ rsw) << 4;
    constexpr int UP = DUAL ? (BN / 2 - (TN / 2) * MI) * ROW_BYTES : 0;   // second half of the subtiles: up rows of the same columns
    // Small tiles (DEEP) hold all fragments of a stage and all of the next one: with a few MFMAs per k-step the LDS latency would show
    // otherwise (128x64 over 512 rows, K = 12288: 86 -> 77.5 us).  Larger ones hold two k-steps of 32.
    constexpr bool DEEP = T <= 8;
    // Where the Y ring is one stage deeper, its fetches go out in the first half of a stage and those of X in the second (20480 rows,
    // 256x256, K = 12288: 1475 -> 1413 us against all of them in the second).
    constexpr bool EARLYB = !DEEP && NSB == NSA + 1;
    constexpr int NSET = DEEP ? 4 : 2;
    bf16x8 fa[NSET][TM], fb[NSET][TN];
    auto read = [&](int set, int r, int sa, int sb, int c) {   // fragment r of a k-step: the Y ones first
        if (r < TN) fb[set][r] = *reinterpret_cast<const bf16x8 *>(lds + sb * B_BYTES + b0 + c + r * (MI * ROW_BYTES) + (DUAL && r >= TN / 2 ? UP : 0));
        else fa[set][r - TN] = *reinterpret_cast<const bf16x8 *>(lds + sa * A_BYTES + a0 + c + (r - TN) * (MI * ROW_BYTES));
    };
    auto mfma = [&](int set, int t) {   // rows of subtiles in turn, every other one backwards: one operand stays from one MFMA to the next
        const int i = t / TN, j = (i & 1) ? TN - 1 - t % TN : t % TN;
        if constexpr (SWAP) mfma_acc(acc[i][j], fb[set][j], fa[set][i]);
        else mfma_acc(acc[i][j], fa[set][i], fb[set][j]);
    };
// this wavefront's fragment reads are done and its share of the stage wanted has landed (at most n younger fetches are in flight); then
// all wavefronts agree, and the compiler must not move LDS accesses across the point
#define PSD_GEMM_SYNC(n)                                                                                       \
    {                                                                                                          \
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(n) : "memory");                                    \
        __builtin_amdgcn_s_barrier();                                                                          \
        asm volatile("" ::: "memory");                                                                         \
    }
    // prologue: the stages that iterations before the first would have fetched, in their order
    constexpr int NS = NSA > NSB ? NSA : NSB;
#pragma unroll
    for (int q = -NS; q < 0; ++q) {
        auto a = [&]() {
            if (q + NSA >= 0)
#pragma unroll
                for (int j = 0; j < GA; ++j) dma_a(j, q + NSA, q + NSA);
        };
        auto b = [&]() {
            if (q + NSB >= 0 && (!EARLYB || q < -1))
#pragma unroll
                for (int j = 0; j < GB; ++j) dma_b(j, q + NSB, q + NSB);
        };
        if (NSA <= NSB) { a(); b(); } else { b(); a(); }
    }
    constexpr int LGKM0 = 0xc07f;   // s_waitcnt lgkmcnt(0)
    int sa = 0, sb = 0;             // ring slots of the stage
    if constexpr (DEEP) {
        PSD_GEMM_SYNC(WAIT0)
#pragma unroll
        for (int r = 0; r < 2 * R; ++r) read(r / R, r % R, 0, 0, r / R ? c1 : c0);
        // Stage kt computes from registers.  Meanwhile stage kt + 1 has landed and is read, and later stages go into the slots of
        // stage kt, which every wavefront has read before the barrier.
        auto stage = [&](int kt, int set) {
            PSD_GEMM_SYNC(WAIT)
            const int na = sa + 1 == NSA ? 0 : sa + 1, nb = sb + 1 == NSB ? 0 : sb + 1;
            static_for<2 * T>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
#pragma unroll
                for (int r = event_at(t, 2 * R, 2 * T); r < event_at(t + 1, 2 * R, 2 * T); ++r) read((set ^ 2) + r / R, r % R, na, nb, r / R ? c1 : c0);
#pragma unroll
                for (int d = event_at(t, NLD, 2 * T); d < event_at(t + 1, NLD, 2 * T); ++d) {
                    const int e = NSA <= NSB ? d : (d < GB ? d + GA : d - GB);
                    if (e < GA) dma_a(e, sa, kt + NSA);
                    else dma_b(e - GA, sb, kt + NSB);
                }
                mfma(set + t / T, t % T);
            });
            sa = na;
            sb = nb;
        };
        int kt = 0;
        for (; kt + 2 <= nk; kt += 2) {
            stage(kt, 0);
            stage(kt + 1, 2);
        }
        if (kt < nk) stage(kt, 0);
    } else {
        PSD_GEMM_SYNC(EARLYB ? WAIT0 - GB : WAIT0)
#pragma unroll
        for (int r = 0; r < R; ++r) read(0, r, 0, 0, c0);
        __builtin_amdgcn_s_waitcnt(LGKM0);
        // Two k-steps a stage.  The first one computes while the second one's fragments are read; after the barrier the second one
        // computes while the first fragments of the next stage are read and fetches go into the slots that are free now.
        constexpr int SPAN = T * 3 / 4;   // MFMAs over which the reads of a k-step are spread
        for (int kt = 0; kt < nk; ++kt) {
            const int na = sa + 1 == NSA ? 0 : sa + 1, nb = sb + 1 == NSB ? 0 : sb + 1;
            const int fill_b = sb == 0 ? NSB - 1 : sb - 1;
            static_for<T>([&](auto tc) {
                constexpr int t = decltype(tc)::value;
                mfma(0, t);
#pragma unroll
                for (int r = event_at(t, R, SPAN); r < event_at(t + 1, R, SPAN); ++r) read(1, r, sa, sb, c1);
                if constexpr (EARLYB)
#pragma unroll
                    for (int d = event_at(t, GB, T); d < event_at(t + 1, GB, T); ++d) dma_b(d, fill_b, kt + NSB - 1);
            });
            PSD_GEMM_SYNC(WAIT)
            static_for<T>([&](auto tc) {
                constexpr int t = decltype(tc)::value, ND = EARLYB ? GA : NLD;
                mfma(1, t);
#pragma unroll
                for (int r = event_at(t, R, SPAN); r < event_at(t + 1, R, SPAN); ++r) read(0, r, na, nb, c0);
#pragma unroll
                for (int d = event_at(t, ND, T); d < event_at(t + 1, ND, T); ++d) {
                    const int e = (EARLYB || NSA <= NSB) ? d : (d < GB ? d + GA : d - GB);
                    if (e < GA) dma_a(e, sa, kt + NSA);
                    else dma_b(e - GA, sb, kt + NSB);
                }
            });
            __builtin_amdgcn_s_waitcnt(LGKM0);
            sa = na;
            sb = nb;
        }
    }
    // No DMA may outlive the loop, and an MFMA's result may be read 8 wait states after its issue only, which the compiler does not know of
    // the asm lines.  (Copies that it places in front of this wait are checked in a listing by a test.)
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) asm volatile("" : "+a"(acc[i][j]));
#undef PSD_GEMM_SYNC

    constexpr int NT = NW * 64, LDC = BN_OUT * 2 + 16;   // LDC: bytes per row of the tile staged row-major (bf16 outputs)
    // the staged tile to `out`, 16 bytes per lane
    auto store_rows = [&]() {
        constexpr int W8 = BN_OUT / 8, PER = BM * W8 / NT, BATCH = batch_of(PER, 8);
        static_assert(BM * W8 % NT == 0, "whole units per thread");
        for (int u0 = tid; u0 < PER * NT; u0 += BATCH * NT) {
            u32x4 x[BATCH];
#pragma unroll
            for (int e = 0; e < BATCH; ++e) {
                const int u = u0 + e * NT;
                x[e] = *reinterpret_cast<const u32x4 *>(lds + u / W8 * LDC + u % W8 * 16);
            }
#pragma unroll
            for (int e = 0; e < BATCH; ++e) {
                const int u = u0 + e * NT, m = m0 + u / W8, n = n0 + u % W8 * 8;
                if (m < M && n < Nout) *reinterpret_cast<u32x4 *>(out + (int64_t)m * ldo + n) = x[e];
            }
        }
    };
    if constexpr (EPI == EPI_TOP1) {
        // per column j: (max, lowest argmax, sum exp) over this tile's rows; rows ascend with (i, v)
        // inside a lane, so a strict comparison keeps the lowest index on ties
        __syncthreads();   // every wavefront is done with the operand rings
        float(*s_b)[BN] = reinterpret_cast<float(*)[BN]>(lds), (*s_s)[BN] = s_b + WGM;
        int(*s_a)[BN] = reinterpret_cast<int(*)[BN]>(s_s + WGM);
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            float best = -INFINITY;
            int arg = 0x7fffffff;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int m = m0 + wm * WTM + i * MI + 4 * lq + v;
                    float z = acc[i][j][v] * t1.scale;
                    if (m >= M || m == t1.mask_id) z = -INFINITY;
                    acc[i][j][v] = z;
                    if (z > best) {
                        best = z;
                        arg = m;
                    }
                }
            float sum = 0.f;
            if (best > -INFINITY) {
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int v = 0; v < NV; ++v) sum += __expf(acc[i][j][v] - best);
            }
            // the 64 / MI lanes that hold this column own disjoint row sets
#pragma unroll
            for (int off = 32; off >= MI; off >>= 1) {
                const float b2 = __shfl_xor(best, off, 64);
                const int a2 = __shfl_xor(arg, off, 64);
                const float s2 = __shfl_xor(sum, off, 64);
                top1_merge(best, arg, sum, b2, a2, s2);
            }
            if (lq == 0) {
                const int col = wn * WTN + j * MI + lrow;
                s_b[wm][col] = best;
                s_a[wm][col] = arg;
                s_s[wm][col] = sum;
            }
        }
        __syncthreads();
        if (tid < BN && n0 + tid < Nout) {
            float best = s_b[0][tid], sum = s_s[0][tid];
            int arg = s_a[0][tid];
#pragma unroll
            for (int w = 1; w < WGM; ++w) top1_merge(best, arg, sum, s_b[w][tid], s_a[w][tid], s_s[w][tid]);
            const int64_t o = (int64_t)tile_m * t1.cols_total + n0 + tid;
            t1.pmax[o] = best;
            t1.psum[o] = sum;
            t1.parg[o] = arg;
        }
    } else if constexpr (EPI == EPI_QKV) {
        constexpr int LDT = BM * 2 + 8;    // bytes per column of the column-major one
        static_assert(BM * LDC <= (NSA * BM + NSB * BN) * ROW_BYTES && BN * LDT <= (NSA * BM + NSB * BN) * ROW_BYTES, "staging tile fits the rings");
        __syncthreads();                   // every wavefront is done with the operand rings
        if (n0 < qa.v_start || !qa.vT) {
            // ---- q / k heads: stage row-major, rotate pairs (j, j + d_head / 2), store 16 bytes per access
            // (V heads whose reader wants them row-major: the same without the rotation)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = wn * WTN + j * MI + 4 * lq;
                float bn[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) bn[v] = bias ? bias[min(n0 + col + v, Nout - 1)] : 0.f;
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const floatx4 x = acc[i][j];
                    *reinterpret_cast<uint2 *>(lds + (wm * WTM + i * MI + lrow) * LDC + col * 2) =
                        make_uint2(pack_bf16x2(x[0] + bn[0], x[1] + bn[1]), pack_bf16x2(x[2] + bn[2], x[3] + bn[3]));
                }
            }
            __syncthreads();
            if (n0 >= qa.v_start) return store_rows();
            // A unit is 8 pair indices of one head of one row, BN / 16 units to a row.
            constexpr int ROW_UNITS = BN / 16, PER = BM * ROW_UNITS / NT, BATCH = batch_of(PER, 4);
            static_assert(BM * ROW_UNITS % NT == 0, "whole units per thread");
            const int half = qa.d_head >> 1, pick = half == 64 ? 3 : 2;   // 8 or 4 units to a head
            for (int u0 = tid; u0 < PER * NT; u0 += BATCH * NT) {
                uint4 a[BATCH], b[BATCH];
                float4 c0[BATCH], c1[BATCH], s0[BATCH], s1[BATCH];
#pragma unroll
                for (int e = 0; e < BATCH; ++e) {
                    const int u = u0 + e * NT, row = u / ROW_UNITS, c = u % ROW_UNITS, g = c & ((1 << pick) - 1);
                    const unsigned char *src = lds + row * LDC + ((c >> pick) * qa.d_head + g * 8) * 2;
                    a[e] = *reinterpret_cast<const uint4 *>(src);
                    b[e] = *reinterpret_cast<const uint4 *>(src + half * 2);
                    const int64_t t = (int64_t)(qa.pos0 + (m0 + row) % qa.N) * half + g * 8;   // (rows past M: a position of the sequence, not stored)
                    c0[e] = *reinterpret_cast<const float4 *>(qa.cos_t + t);
                    c1[e] = *reinterpret_cast<const float4 *>(qa.cos_t + t + 4);
                    s0[e] = *reinterpret_cast<const float4 *>(qa.sin_t + t);
                    s1[e] = *reinterpret_cast<const float4 *>(qa.sin_t + t + 4);
                }
#pragma unroll
                for (int e = 0; e < BATCH; ++e) {
                    const int u = u0 + e * NT, row = u / ROW_UNITS, c = u % ROW_UNITS, g = c & ((1 << pick) - 1);
                    const int m = m0 + row, n = n0 + (c >> pick) * qa.d_head + g * 8;
                    if (m >= M || n >= Nout) continue;
                    uint4 ra, rb;
                    rope_rotate8(a[e], b[e], c0[e], c1[e], s0[e], s1[e], ra, rb);
                    bf16_t *dst = out + (int64_t)m * ldo + n;
                    if (qa.k_dst && n >= qa.k_start) dst = qa.k_dst + (m / qa.N) * qa.k_seq + (int64_t)(m % qa.N) * qa.ld_k + (n - qa.k_start);
                    *reinterpret_cast<uint4 *>(dst) = ra;
                    *reinterpret_cast<uint4 *>(dst + half) = rb;
                }
            }
        } else {
            // ---- V heads: stage column-major, store transposed.  Inside every group of 16 keys the slots hold keys 0-3, 8-11, 4-7, 12-15.
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int col = wn * WTN + j * MI + 4 * lq + v;
                    const float bn = bias ? bias[min(n0 + col, Nout - 1)] : 0.f;
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        *reinterpret_cast<uint16_t *>(lds + col * LDT + (wm * WTM + i * MI + lrow) * 2) = from_float<bf16_t>(acc[i][j][v] + bn).bits;
                }
            __syncthreads();
            constexpr int G16 = BM / 16, PER = BN * G16 * 2 / NT, BATCH = batch_of(PER, 8);
            static_assert(BN * G16 * 2 % NT == 0, "whole units per thread");
            for (int u0 = tid; u0 < PER * NT; u0 += BATCH * NT) {
                uint2 lo[BATCH], hi[BATCH];
#pragma unroll
                for (int e = 0; e < BATCH; ++e) {
                    const int u = u0 + e * NT, h = u & 1, g = (u >> 1) % G16, col = u / (2 * G16);
                    const unsigned char *src = lds + col * LDT + (g * 16 + 4 * h) * 2;
                    lo[e] = *reinterpret_cast<const uint2 *>(src);
                    hi[e] = *reinterpret_cast<const uint2 *>(src + 16);
                }
#pragma unroll
                for (int e = 0; e < BATCH; ++e) {
                    const int u = u0 + e * NT, h = u & 1, g = (u >> 1) % G16, col = u / (2 * G16);
                    const int m = m0 + g * 16, n = n0 + col;
                    if (m >= M || n >= Nout) continue;
                    const int sq = m / qa.N, i0 = m % qa.N;   // N % 16 == 0: the 16 keys belong to one sequence
                    bf16_t *dst = qa.vT + sq * qa.vt_seq + (int64_t)(n - qa.v_start) * qa.ld_vt + i0 + 8 * h;
                    *reinterpret_cast<uint4 *>(dst) = make_uint4(lo[e].x, lo[e].y, hi[e].x, hi[e].y);
                }
            }
        }
    } else if constexpr (EPI == EPI_RESIDUAL) {
        // fp32 read-modify-write of the stream, 16 bytes per lane.  A row of subtiles is fetched ahead of the one being written: written
        // as one load-add-store per value every load would wait for the store before it (the compiler cannot tell rows apart).
        float *dst = split == 0 ? resid : partial + (int64_t)(split - 1) * M * Nout;
        const int ldd = split == 0 ? ldo : Nout;
        const int nb = n0 + wn * WTN + 4 * lq, mb = m0 + wm * WTM + lrow;
        if ((ldd & 3) == 0 && (Nout & 3) == 0 && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {   // uniform
            float4 old[2][TN];
            auto fetch = [&](int i) {
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    old[i & 1][j] = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (split == 0 && nb + j * MI < Nout && mb + i * MI < M)
                        old[i & 1][j] = *reinterpret_cast<const float4 *>(dst + (int64_t)(mb + i * MI) * ldd + nb + j * MI);
                }
            };
            fetch(0);
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (i + 1 < TM) fetch(i + 1);
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const float4 o = old[i & 1][j];
                    const floatx4 x = acc[i][j];
                    if (nb + j * MI < Nout && mb + i * MI < M)
                        *reinterpret_cast<float4 *>(dst + (int64_t)(mb + i * MI) * ldd + nb + j * MI) = make_float4(o.x + x[0], o.y + x[1], o.z + x[2], o.w + x[3]);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int n = nb + j * MI + v, m = mb + i * MI;
                        if (n < Nout && m < M) {
                            float *p = dst + (int64_t)m * ldd + n;
                            *p = split == 0 ? *p + acc[i][j][v] : 0.f + acc[i][j][v];
                        }
                    }
        }
    } else {
        constexpr int TN_OUT = DUAL ? TN / 2 : TN;
        constexpr int WTN_OUT = DUAL ? WTN / 2 : WTN;
        auto value = [&](int i, int j, int v, float bn) {
            float x = acc[i][j][v];
            if (EPI == EPI_BIAS) x += bn;
            if (DUAL) x = x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)) * acc[i][j + TN / 2 * (DUAL ? 1 : 0)][v];   // silu(x) * u; v_rcp_f32 (1 ulp) instead of a full division
            return x;
        };
        // bf16 outputs.  Where rows allow 16-byte accesses the tile is staged in LDS (the operand rings are free; rows padded by 16 bytes)
        // and stored with 16 bytes per lane.
        static_assert(BM * LDC <= (NSA * BM + NSB * BN) * ROW_BYTES, "staging tile fits the rings");
        const bool wide = (ldo & 7) == 0 && (Nout & 7) == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;   // uniform
        if (wide) {
            __syncthreads();   // every wavefront is done with the operand rings
#pragma unroll
            for (int j = 0; j < TN_OUT; ++j) {
                const int col = wn * WTN_OUT + j * MI + 4 * lq;
                float bn[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) bn[v] = (EPI == EPI_BIAS) ? bias[min(n0 + col + v, Nout - 1)] : 0.f;
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    *reinterpret_cast<uint2 *>(lds + (wm * WTM + i * MI + lrow) * LDC + col * 2) =
                        make_uint2(pack_bf16x2(value(i, j, 0, bn[0]), value(i, j, 1, bn[1])), pack_bf16x2(value(i, j, 2, bn[2]), value(i, j, 3, bn[3])));
            }
            __syncthreads();
            store_rows();
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN_OUT; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int n = n0 + wn * WTN_OUT + j * MI + 4 * lq + v, m = m0 + wm * WTM + i * MI + lrow;
                        if (n >= Nout || m >= M) continue;
                        out[(int64_t)m * ldo + n] = from_float<bf16_t>(value(i, j, v, (EPI == EPI_BIAS) ? bias[n] : 0.f));
                    }
        }
    }
}

template <int BM, int BN, int WGM, int WGN, int EPI, int NSA, int NSB, int WPS = 1>
void launch_cfg(const bf16_t *X, const bf16_t *Y, const bf16_t *Y2, int M, int Nout, int Kin, int ldx, int ldy, const float *bias,
                bf16_t *out, float *resid, int ldo, Top1Args t1, hipStream_t st, int k_splits = 1, float *partial = nullptr,
                QkvArgs qa = QkvArgs(), const Warm &next = Warm()) {
    constexpr int BN_OUT = (EPI == EPI_SWIGLU) ? BN / 2 : BN;
    const int tiles_m = (M + BM - 1) / BM, tiles_n = (Nout + BN_OUT - 1) / BN_OUT;
    const int n_tiles = tiles_m * tiles_n;
    constexpr int smem = (NSA * BM + NSB * BN) * BK * 2;
    static_assert(smem <= 160 * 1024, "LDS ring exceeds the 160 KB of a CU");
    auto kern = gemm_bf16_kernel<BM, BN, WGM, WGN, EPI, NSA, NSB, WPS>;
    static std::atomic<uint64_t> lds_raised{0};   // one per instantiation
    ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem, lds_raised);
    if (EPI != EPI_RESIDUAL) k_splits = 1;
    hipLaunchKernelGGL(kern, dim3(n_tiles * k_splits + next.wgs), dim3(WGM * WGN * 64), smem, st, X, Y, Y2, M, Nout, Kin, ldx, ldy, bias, out, resid,
                       ldo, tiles_n, n_tiles, t1, k_splits, partial, gemm_tile_group_m(), qa, next);
}

}   // namespace mfma
