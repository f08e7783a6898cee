// Contractions over at most 128 rows (block rows of the KV-cached calls, the block rows behind the last attention): the weights
// are read once and everything else is small, so the kernel is built as a stream over them.
//
// What bounds it: a CU gets about 64 KB of fetches in flight back from HBM every 1.2 us, whatever waits for them, and returns come
// in order.  So the time is the bytes a CU fetches -- its share of the weights AND the activations it multiplies them with -- at
// about 55 GB/s per CU, or the whole weight matrix at the HBM rate, whichever is longer.  A workgroup therefore takes all rows and a
// narrow slice of the weight rows, as wide as spreads the slices evenly over the 256 CUs; a residual contraction is also cut along
// K, which shortens the activations a workgroup reads (its partial sums are added by the next norm).  stream_plan weighs the two.
// Against the 128x64 / 128x128 tiles and the eight-fold K cut before it, inside a model call of the 8B shape: 12288 x 4096 (QKV)
// 32 -> 22 us at 32 rows, 34.6 -> 34 at 128; the SwiGLU pair of that size 49 -> 42 and 53 -> 48; the output and down
// projections of a layer together 52 on average over both row counts, now 29 and 46.
//
// Four wavefronts share one ring of NS stages of 64 k in LDS, filled by direct global -> LDS loads, 128-byte rows with the 16-byte
// chunks swizzled as in gemm_mfma.h; one barrier per stage, the fragments of the next stage in registers while one computes.  With
// weights as the row operand of v_mfma_f32_16x16x32_bf16 a lane holds 4 consecutive outputs of one row.  K runs in order in every
// accumulator, as in the tiled kernel: the same bits.
#include "gemm_mfma.h"

namespace {

using namespace mfma;

constexpr double CU_RATE = 55e9;   // bytes a CU fetches per second (42 - 55 GB/s measured)

// (deeper rings than these, up to the whole LDS, changed nothing)
constexpr int ring_stages(int rows) {
    const int n = 78 * 1024 / (rows * 128);   // two workgroups per CU where that leaves a ring worth the name
    return n < 3 ? 3 : n > 10 ? 10 : n;
}

// MR: rows of X, rounded up (32, 64 or 128); NT: 16-row tiles of Y (and of Y2) per workgroup
template <int MR, int NT, int EPI>
__global__ __launch_bounds__(256, 2) void gemm_stream_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ Y,
                                                          const bf16_t *__restrict__ Y2, int M, int Nout, int Kin, int ldx, int ldy,
                                                          const float *__restrict__ bias, bf16_t *__restrict__ out,
                                                          float *__restrict__ resid, int ldo, int k_splits, float *__restrict__ partial) {
    constexpr bool DUAL = EPI == EPI_SWIGLU;
    constexpr int NC = NT * 16, ROWS = MR + NC * (DUAL ? 2 : 1), STAGE = ROWS * 128, NS = ring_stages(ROWS);
    constexpr int MG = MR / 32 < 2 ? 2 : 4, NG = 4 / MG;      // wavefronts along the rows and along the tiles
    constexpr int TM = MR / (16 * MG), TNO = (NT + NG - 1) / NG, TN = TNO * (DUAL ? 2 : 1);
    constexpr int GX = MR / 32, GYT = NC / 8 * (DUAL ? 2 : 1), GY = (GYT + 3) / 4, NL = GX + GY;   // fetches per wavefront and stage
    static_assert((NS - 1) * NL <= 63, "fetches in flight must fit the vmcnt counter");
    extern __shared__ __align__(16) unsigned char lds[];
    typedef __attribute__((address_space(3))) void lds_void;

    // (parts of K vary fastest: an XCD gets every eighth workgroup, so with 2, 4 or 8 parts it reads one part of the activations)
    const int split = blockIdx.x % k_splits, n0 = blockIdx.x / k_splits * NC;
    const int k_len = Kin / k_splits, k_beg = split * k_len, nk = k_len / BK;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mg = wave % MG, ng = wave / MG, lrow = lane & 15, lq = lane >> 4;

    const int rows_y = min(NC, Nout - n0);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(X) + k_beg, 0,
                                                                        (int)((((int64_t)M - 1) * ldx + Kin - k_beg) * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(Y) + (int64_t)n0 * ldy + k_beg, 0,
                                                                        ((rows_y - 1) * ldy + Kin - k_beg) * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t ry2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(DUAL ? Y2 : Y) + (int64_t)n0 * ldy + k_beg, 0,
                                                                         ((rows_y - 1) * ldy + Kin - k_beg) * 2, 0x00020000);
    // groups of 8 rows, one fetch each, dealt to the wavefronts in turn: the swizzle key of a group is a constant of the wavefront
    const int key = (((wave & 1) << 2) + (lane >> 4)) & 7;
    const int voff_x = (lane >> 3) * ldx * 2 + (((lane & 7) ^ key) << 4), voff_y = (lane >> 3) * ldy * 2 + (((lane & 7) ^ key) << 4);
    // A stage past the end of K is fetched from offsets that every descriptor rejects: no traffic, and the counts of fetches in
    // flight stay what the waits assume.  (At its own offsets it would read the next part of K or the next row: with a ring of 9
    // stages 41 stages for the 32 of a half of K = 4096.)
    const int voff_none = 0x7ffffff0;
    auto fetch = [&](int slot, int kt) {
        unsigned char *s = lds + slot * STAGE + wave * 1024;
        const int k0 = kt * BK;
        const int vx = kt < nk ? voff_x : voff_none, vy = kt < nk ? voff_y : voff_none;
#pragma unroll
        for (int j = 0; j < GX; ++j)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (lds_void *)(s + j * 4096), 16, vx, ((j * 4 + wave) * 8 * ldx + k0) * 2, 0, 0);
#pragma unroll
        for (int j = 0; j < GY; ++j) {
            const int g = j * 4 + wave;
            if (GYT % 4 == 0 || g < GYT) {
                if (DUAL && g >= NC / 8)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(ry2, (lds_void *)(s + (GX + j) * 4096), 16, vy, ((g * 8 - NC) * ldy + k0) * 2, 0, 0);
                else
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(ry, (lds_void *)(s + (GX + j) * 4096), 16, vy, (g * 8 * ldy + k0) * 2, 0, 0);
            }
        }
    };
    const bool full = GYT % 4 == 0 || wave < GYT % 4;   // this wavefront issues NL fetches a stage, otherwise one less
// at most n stages younger than the one wanted are in flight, and this wavefront's fragment reads are done; then all agree
#define PSD_STREAM_SYNC(n)                                                                                     \
    {                                                                                                          \
        if (full) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((n) * NL) : "memory");                   \
        else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((n) * (NL - 1)) : "memory");                  \
        __builtin_amdgcn_s_barrier();                                                                          \
        asm volatile("" ::: "memory");                                                                         \
    }

    floatx4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;
    // LDS offset of fragment row lrow of the wavefront's tiles; a stage holds X, Y and Y2 rows one after the other
    int offx[TM], offy[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) offx[i] = (mg * (MR / MG) + i * 16 + lrow) * 128;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int t = min((j % TNO) * NG + ng, NT - 1);   // (a wavefront without a last tile repeats one and drops it)
        offy[j] = (MR + (j >= TNO ? NC : 0) + t * 16 + lrow) * 128;
    }
    bf16x8 fx[2][2][TM], fy[2][2][TN];   // [set][k-step]
    auto frags = [&](int slot, int set) {
        const unsigned char *s = lds + slot * STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int c = ((ks * 4 + lq) ^ row_key(lrow)) << 4;
#pragma unroll
            for (int i = 0; i < TM; ++i) fx[set][ks][i] = *reinterpret_cast<const bf16x8 *>(s + offx[i] + c);
#pragma unroll
            for (int j = 0; j < TN; ++j) fy[set][ks][j] = *reinterpret_cast<const bf16x8 *>(s + offy[j] + c);
        }
    };
    auto compute = [&](int set) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fy[set][ks][j], fx[set][ks][i], acc[i][j], 0, 0, 0);
    };

#pragma unroll
    for (int p = 0; p < NS; ++p) fetch(p, p);
    PSD_STREAM_SYNC(NS - 1)
    frags(0, 0);
    // Stage kt computes from registers.  Meanwhile stage kt + 1 has landed and is read, and stage kt + NS goes into the slot of
    // stage kt, which every wavefront has read before the barrier.
    int slot = 0;
    auto step = [&](int kt, int set) {
        PSD_STREAM_SYNC(NS - 2)
        fetch(slot, kt + NS);
        slot = slot + 1 == NS ? 0 : slot + 1;
        frags(slot, set ^ 1);
        compute(set);
    };
    int kt = 0;
    for (; kt + 2 <= nk; kt += 2) {
        step(kt, 0);
        step(kt + 1, 1);
    }
    if (kt < nk) step(kt, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no fetch may outlive the loop
#undef PSD_STREAM_SYNC

    float *dst = split == 0 ? resid : partial + (int64_t)(split - 1) * M * Nout;
    const int ldd = split == 0 ? ldo : Nout;
#pragma unroll
    for (int j = 0; j < TNO; ++j) {
        if (NT % NG != 0 && j * NG + ng >= NT) continue;
        const int n = n0 + (j * NG + ng) * 16 + lq * 4;
        if (n >= Nout) continue;
        float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
        if (EPI == EPI_BIAS) b = *reinterpret_cast<const float4 *>(bias + n);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = mg * (MR / MG) + i * 16 + lrow;
            if (m >= M) continue;
            floatx4 x = acc[i][j];
            if constexpr (EPI == EPI_RESIDUAL) {
                float4 r = make_float4(x[0], x[1], x[2], x[3]);
                float4 *p = reinterpret_cast<float4 *>(dst + (int64_t)m * ldd + n);
                if (split == 0) {
                    const float4 old = *p;
                    r = make_float4(old.x + x[0], old.y + x[1], old.z + x[2], old.w + x[3]);
                }
                *p = r;
            } else {
                if constexpr (EPI == EPI_BIAS) {
                    x[0] += b.x; x[1] += b.y; x[2] += b.z; x[3] += b.w;
                }
                if constexpr (DUAL) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) x[v] = x[v] * __builtin_amdgcn_rcpf(1.0f + __expf(-x[v])) * acc[i][j + TNO][v];
                }
                *reinterpret_cast<uint2 *>(out + (int64_t)m * ldo + n) = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
            }
        }
    }
}

template <int MR, int NT, int EPI>
void launch_stream_cfg(const bf16_t *X, const bf16_t *Y, const bf16_t *Y2, int M, int Nout, int Kin, int ldx, int ldy, const float *bias,
                       bf16_t *out, float *resid, int ldo, int splits, float *partial, hipStream_t st) {
    constexpr int rows = MR + NT * 16 * (EPI == EPI_SWIGLU ? 2 : 1), smem = ring_stages(rows) * rows * 128;
    static_assert(smem <= 160 * 1024, "LDS ring exceeds the 160 KB of a CU");
    auto kern = gemm_stream_kernel<MR, NT, EPI>;
    static std::atomic<uint64_t> lds_raised{0};   // one per instantiation
    ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem, lds_raised);
    hipLaunchKernelGGL(kern, dim3((Nout + NT * 16 - 1) / (NT * 16) * splits), dim3(256), smem, st, X, Y, Y2, M, Nout, Kin, ldx, ldy, bias,
                       out, resid, ldo, splits, partial);
}

template <int EPI>
void launch_stream_epi(const StreamPlan &p, const bf16_t *X, const bf16_t *Y, const bf16_t *Y2, int M, int Nout, int Kin, int ldx, int ldy,
                       const float *bias, bf16_t *out, float *resid, int ldo, float *partial, hipStream_t st) {
    auto go = [&](auto mr, auto nt) {
        launch_stream_cfg<decltype(mr)::value, decltype(nt)::value, EPI>(X, Y, Y2, M, Nout, Kin, ldx, ldy, bias, out, resid, ldo, p.splits, partial, st);
    };
    auto rows = [&](auto nt) {
        using std::integral_constant;
        if (M <= 32) go(integral_constant<int, 32>(), nt);
        else if (M <= 64) go(integral_constant<int, 64>(), nt);
        else go(integral_constant<int, 128>(), nt);
    };
    using std::integral_constant;
    switch (p.tiles) {
        case 1: return rows(integral_constant<int, 1>());
        case 2: return rows(integral_constant<int, 2>());
        case 3: return rows(integral_constant<int, 3>());
        case 4: return rows(integral_constant<int, 4>());
        case 5: return rows(integral_constant<int, 5>());
        default: return rows(integral_constant<int, 6>());
    }
}

}   // namespace

// Slice width and K parts: the shortest of the widths 16 .. 96 and (residual contractions whose reader adds partial sums) of
// min_splits, twice that, .. max_splits parts, by the rates in the head of this file.  max_splits = 1: no partial sums.  tiles = 0: not
// for this kernel.
StreamPlan stream_plan(int64_t M, int Nout, int Kin, int epi, int min_splits, int max_splits) {
    StreamPlan best;
    if (M > 128 || M < 1 || Nout % 4) return best;
    const int dual = epi == EPI_SWIGLU ? 2 : 1, rows = M <= 32 ? 32 : M <= 64 ? 64 : 128;
    const double stream = (double)dual * Nout * Kin * 2 / 5.5e12;
    double best_t = 0;
    for (int s = min_splits; s <= max_splits; s *= 2) {
        if (Kin % (s * mfma::BK)) break;
        for (int t = 1; t <= 6; ++t) {
            const int64_t groups = (int64_t)((Nout + t * 16 - 1) / (t * 16)) * s;
            const double fetch = (double)((groups + 255) / 256) * (rows + t * 16 * dual) * (Kin / s) * 2 / CU_RATE;
            const double sums = (s - 1) * (double)M * Nout * 8 / 4e12;
            const double time = (fetch > stream ? fetch : stream) + 0.1 * fetch + sums;   // (of equally fast streams the one that fetches less)
            if (best.tiles == 0 || time < best_t) {
                best.tiles = t;
                best.splits = s;
                best_t = time;
            }
        }
    }
    // few and narrow outputs under many rows: workgroups of half the rows fetch less than those of all of them (4608 outputs,
    // K = 3584, 128 rows: 20 us in 64x64 tiles, 23 here; 12288 outputs, K = 4096: 35 us in 128x64 tiles, 31 here)
    if (dual == 1 && max_splits == 1 && M > 64) {
        const int64_t tiles = (M + 63) / 64 * ((Nout + 63) / 64);
        if ((double)((tiles + 255) / 256) * 128 * Kin * 2 / CU_RATE < best_t) best.tiles = 0;
    }
    return best;
}

void launch_gemm_stream(const StreamPlan &p, const bf16_t *A, const bf16_t *W, const bf16_t *W2, int64_t M, int Nout, int Kin, int lda,
                        int ldw, int epi, const float *bias, bf16_t *out, float *resid, int ldo, float *partial, hipStream_t st) {
    const int m = (int)M;
    switch (epi) {
        case EPI_STORE: return launch_stream_epi<EPI_STORE>(p, A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, partial, st);
        case EPI_BIAS: return launch_stream_epi<EPI_BIAS>(p, A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, partial, st);
        case EPI_RESIDUAL: return launch_stream_epi<EPI_RESIDUAL>(p, A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, partial, st);
        default: return launch_stream_epi<EPI_SWIGLU>(p, A, W, W2, m, Nout, Kin, lda, ldw, bias, out, resid, ldo, partial, st);
    }
}
