// Attention of whole bf16 sequences whose length is no multiple of 8: fp32 scores, fp32 probabilities and every sum in the order of
// plain_attention_kernel, so that the two give the same bits.  These lengths have always been computed that way, and bf16
// probabilities (attention_mfma.hip) or sums in another order move the confidences of a deep model by a percent, which swaps
// positions whose confidences nearly tie.
//
// v_mfma_f32_32x32x2_f32 and v_mfma_f32_16x16x4_f32 round like a chain of fmaf over their k in ascending order (also with
// denormals, infinities and NaN), so a dot product over consecutive instructions is the plain kernel's loop.  What it takes
// over from that kernel besides: one product with the scale per score, expf of the difference to the maximum, the sum as
// 64 strided partial sums added in a butterfly, the values accumulated key after key and divided at the end.
//
// Bound by the fp32 matrix instructions (a sixteenth of the bf16 rate, twice what fmaf reaches without packed instructions) and by the
// latency of what feeds them.  A workgroup takes QT queries of one head; the scores of all keys stay in LDS, because the sums need
// the final maximum and their order, so two workgroups fit a CU at 557 keys: each has eight wavefronts, four to a SIMD, to cover
// the fetches of one with the MFMAs of another.  Keys and values go from global memory straight into the registers that the
// instructions read, by buffer loads with the position in a scalar offset; a value fetch is two channels wide where that leaves
// every wavefront an output tile.  12 x 557 tokens, 32 heads of 128: 688 us a layer (89 TFLOP/s; scores 320, softmax 120, values
// 250, each of the products 200 at the rate of the instructions), with four wavefronts and a pass of its own for the maximum 883, the
// plain kernel 8546, bf16 matrix instructions 126.  Half of a key's row per lane and an exchange between the lanes instead of
// the whole row in both: no change.
#include <type_traits>

#include "psd_internal.h"
#include "device_types.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int NW = 8;                // wavefronts per workgroup
constexpr int RED = NW * 32;         // floats of LDS in front of the scores

template <int QT>
using acc_t = std::conditional_t<QT == 32, f32x16, f32x4>;

// QT x QT outputs; a lane holds row (a) / column (b) lane % QT at k = lane / QT, and of the result column lane % QT, rows
// 8 * (v / 4) + 4 * (lane / QT) + v % 4
__device__ __forceinline__ f32x16 mma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// of 8 consecutive channels the ones with k = h of the instructions that contract them, ascending
template <int QT>
__device__ __forceinline__ void pick(const u32x4 u, int h, float *f) {
    auto half = [](uint32_t w, int high) { return __uint_as_float(high ? w & 0xffff0000u : w << 16); };
    if constexpr (QT == 32) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[i] = half(u[i], h);
    } else {
        f[0] = half(h & 2 ? u[1] : u[0], h & 1);
        f[1] = half(h & 2 ? u[3] : u[2], h & 1);
    }
}

template <int DH, int QT>
__global__ __launch_bounds__(NW * 64, 4) void attention_ordered_kernel(const bf16_t *__restrict__ qkv, int ld, int N, int n_heads,
                                                                       int n_kv_heads, bf16_t *__restrict__ out) {
    constexpr int KPI = 64 / QT, NV = QT * QT / 64;     // k per instruction, outputs per lane
    constexpr int GROUPS = NW * 64 / QT;                // threads per query in the softmax
    constexpr int STRIDED = 64 / GROUPS;                // of the 64 partial sums, those of one thread
    static_assert(STRIDED >= 1 && GROUPS >= 2 * NW, "threads per query");
    extern __shared__ __align__(16) float smem[];
    float *red = smem, *sc = smem + RED;                // sc[key][query]

    // (KV head, sequence) units dealt to the XCDs, as in attention_kernel
    int qblk = blockIdx.x, head = blockIdx.y, s = blockIdx.z;
    const int group = n_heads / n_kv_heads;
    {
        const int units = n_kv_heads * (int)gridDim.z, per_unit = (int)gridDim.x * group;
        if (units % 8 == 0) {
            const int pid = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
            const int slot = pid >> 3, unit = (slot / per_unit) * 8 + (pid & 7), within = slot % per_unit;
            qblk = within % (int)gridDim.x;
            head = (unit % n_kv_heads) * group + within / (int)gridDim.x;
            s = unit / n_kv_heads;
        }
    }
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane % QT, h = lane / QT;
    const bf16_t *seq = qkv + (int64_t)s * N * ld;
    // keys and values of the KV head, rows of the sequence; rows past its end read as zero
    const int64_t kv_off = (n_heads + head / group) * DH;
    const int kv_bytes = ((N - 1) * ld + DH) * 2;
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(seq) + kv_off, 0, kv_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(seq) + kv_off + n_kv_heads * DH, 0, kv_bytes, 0x00020000);

    // ---- scores: the wavefronts deal the tiles of QT keys
    float mx = -INFINITY;   // of the scores of query lrow that this lane has seen
    {
        float qf[DH / KPI];
        const bf16_t *q = seq + (int64_t)min(qblk * QT + lrow, N - 1) * ld + head * DH;   // (past the last query: it again, not stored)
#pragma unroll
        for (int j = 0; j < DH / 8; ++j) pick<QT>(*reinterpret_cast<const u32x4 *>(q + j * 8), h, qf + j * (8 / KPI));
        const float scale = 1.0f / sqrtf((float)DH);
        const int row_off = lrow * ld * 2;
        for (int k0 = wave * QT; k0 < N; k0 += NW * QT) {
            u32x4 kf[DH / 8];
            const int base = k0 * ld * 2;
#pragma unroll
            for (int j = 0; j < DH / 8; ++j) kf[j] = __builtin_amdgcn_raw_buffer_load_b128(kr, row_off + j * 16, base, 0);
            acc_t<QT> acc;
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[v] = 0.f;
#pragma unroll
            for (int j = 0; j < DH / 8; ++j) {
                float f[8 / KPI];
                pick<QT>(kf[j], h, f);
#pragma unroll
                for (int i = 0; i < 8 / KPI; ++i) acc = mma(f[i], qf[j * (8 / KPI) + i], acc);
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const int key = k0 + 8 * (v >> 2) + 4 * h + (v & 3);
                if (key < N) {
                    const float z = acc[v] * scale;
                    sc[key * QT + lrow] = z;
                    mx = fmaxf(mx, z);
                }
            }
        }
    }
    // the maximum does not depend on the order of its parts
#pragma unroll
    for (int off = 32; off >= QT; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    if (h == 0) red[wave * QT + lrow] = mx;
    __syncthreads();

    // ---- softmax: GROUPS threads per query
    const int tq = threadIdx.x % QT, tg = threadIdx.x / QT;
    mx = red[tq];
#pragma unroll
    for (int w = 1; w < NW; ++w) mx = fmaxf(mx, red[w * QT + tq]);
    float sum[STRIDED];   // [t]: keys = tg + GROUPS * t modulo 64
#pragma unroll
    for (int t = 0; t < STRIDED; ++t) sum[t] = 0.f;
    for (int j0 = tg; j0 < N; j0 += 64)
#pragma unroll
        for (int t = 0; t < STRIDED; ++t) {
            const int j = j0 + GROUPS * t;
            if (j < N) {
                const float e = expf(sc[j * QT + tq] - mx);
                sc[j * QT + tq] = e;
                sum[t] += e;
            }
        }
#pragma unroll
    for (int off = STRIDED / 2; off > 0; off >>= 1)
#pragma unroll
        for (int t = 0; t < off; ++t) sum[t] += sum[t + off];
    // the partial sums of the threads, upper half onto lower half, through `red` in rounds of NW until NW are left
#pragma unroll
    for (int n = GROUPS / 2; n >= NW; n >>= 1)
#pragma unroll
        for (int r = 0; r < n; r += NW) {
            __syncthreads();   // what `red` held is read
            if (tg >= n + r && tg < n + r + NW) red[(tg - n - r) * QT + tq] = sum[0];
            __syncthreads();
            if (tg >= r && tg < r + NW) sum[0] += red[(tg - r) * QT + tq];
        }
    __syncthreads();
    if (tg < NW) red[tg * QT + tq] = sum[0];
    __syncthreads();

    // ---- values: 16 x 16 outputs each, CPL tiles of channels and one of queries per wavefront; a lane holds channels
    // c0 + CPL * (lane % 16) + t of the keys lane / 16 (so the tiles interleave), and walks the keys, FLIGHT instructions per round of fetches
    constexpr int QTILES = QT / 16, TILES = QTILES * (DH / 16), CPL = TILES >= 2 * NW ? 2 : 1;
    constexpr int FLIGHT = 8, STEP = FLIGHT * 4;
    static_assert(TILES / CPL <= NW, "one round of output tiles");
    if (wave >= TILES / CPL) return;
    const int l16 = lane & 15, h4 = lane >> 4;
    const int q16 = wave % QTILES * 16, c0 = wave / QTILES * (16 * CPL);
    float part[NW];
#pragma unroll
    for (int g = 0; g < NW; ++g) part[g] = red[g * QT + q16 + l16];   // this lane's query as a column of the output
#pragma unroll
    for (int off = NW / 2; off > 0; off >>= 1)
#pragma unroll
        for (int g = 0; g < off; ++g) part[g] += part[g + off];
    const float inv = 1.0f / part[0];
    f32x4 acc[CPL];
#pragma unroll
    for (int t = 0; t < CPL; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int v_off = (h4 * ld + c0 + CPL * l16) * 2;
    const float *p = sc + h4 * QT + q16 + l16;
    uint32_t next[FLIGHT];
    auto fetch = [&](int j0) {   // (past the last key: anything, dropped below)
#pragma unroll
        for (int i = 0; i < FLIGHT; ++i) {
            const int at = min(j0 + 4 * i, N - 1) * ld * 2;
            if constexpr (CPL == 2) next[i] = __builtin_amdgcn_raw_buffer_load_b32(vr, v_off, at, 0);
            else next[i] = __builtin_amdgcn_raw_buffer_load_b16(vr, v_off, at, 0);
        }
    };
    fetch(0);
    int j0 = 0;
    for (; j0 + STEP <= N; j0 += STEP) {
        uint32_t u[FLIGHT];
        float pv[FLIGHT];
#pragma unroll
        for (int i = 0; i < FLIGHT; ++i) u[i] = next[i];
        fetch(j0 + STEP);
#pragma unroll
        for (int i = 0; i < FLIGHT; ++i) pv[i] = p[(j0 + 4 * i) * QT];
#pragma unroll
        for (int i = 0; i < FLIGHT; ++i) {
            acc[0] = mma(__uint_as_float(u[i] << 16), pv[i], acc[0]);
            if constexpr (CPL == 2) acc[1] = mma(__uint_as_float(u[i] & 0xffff0000u), pv[i], acc[1]);
        }
    }
#pragma unroll
    for (int i = 0; i < FLIGHT; ++i) {
        if (j0 + i * 4 < N) {   // (uniform) the last keys; 0 x 0 for those that do not exist
            const bool in = j0 + i * 4 + h4 < N;
            const float pr = in ? p[(j0 + 4 * i) * QT] : 0.f;
            if (!in) next[i] = 0;
            acc[0] = mma(__uint_as_float(next[i] << 16), pr, acc[0]);
            if constexpr (CPL == 2) acc[1] = mma(__uint_as_float(next[i] & 0xffff0000u), pr, acc[1]);
        }
    }
    const int q = qblk * QT + q16 + l16;
    if (q < N) {
        bf16_t *o = out + ((int64_t)s * N + q) * (n_heads * DH) + head * DH + c0 + CPL * 4 * h4;   // result rows 4 h4 + v: channels CPL * (4 h4 + v) + t
        if constexpr (CPL == 2)
            *reinterpret_cast<uint4 *>(o) = make_uint4(pack_bf16x2(acc[0][0] * inv, acc[1][0] * inv), pack_bf16x2(acc[0][1] * inv, acc[1][1] * inv),
                                                       pack_bf16x2(acc[0][2] * inv, acc[1][2] * inv), pack_bf16x2(acc[0][3] * inv, acc[1][3] * inv));
        else
            *reinterpret_cast<uint2 *>(o) = make_uint2(pack_bf16x2(acc[0][0] * inv, acc[0][1] * inv), pack_bf16x2(acc[0][2] * inv, acc[0][3] * inv));
    }
}

constexpr int MAX_LDS = 160 * 1024;
constexpr int lds_bytes(int qt, int N) { return (RED + N * qt) * 4; }

template <int DH, int QT>
void launch_ordered(const bf16_t *qkv, int ld_qkv, int S, int N, int n_heads, int n_kv_heads, bf16_t *out, hipStream_t st) {
    auto kern = attention_ordered_kernel<DH, QT>;
    static std::atomic<uint64_t> lds_raised{0};   // one per instantiation
    ensure_dynamic_lds(reinterpret_cast<const void *>(kern), MAX_LDS, lds_raised);
    hipLaunchKernelGGL(kern, dim3((N + QT - 1) / QT, n_heads, S), dim3(NW * 64), lds_bytes(QT, N), st, qkv, ld_qkv, N, n_heads, n_kv_heads, out);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}   // namespace

// 32 queries per workgroup read the keys and values half as often as 16 (with four wavefronts 1109 against 1327 us at 12 x 557 tokens,
// 32 heads of 128; 44 against 52 at 20 x 197, 8 heads of 64); 16 where the scores of 32 do not fit LDS (above 1272 keys), and the plain kernel where
// those of 16 do not (above 2544).
bool launch_attention_ordered(const bf16_t *qkv, int ld_qkv, int S, int N, int n_heads, int n_kv_heads, int d_head, bf16_t *out,
                              hipStream_t st) {
    if (N < 1 || lds_bytes(16, N) > MAX_LDS || (d_head != 64 && d_head != 128) || ld_qkv % 8 || !aligned16(qkv) || !aligned16(out)) return false;
    if ((int64_t)N * ld_qkv * 2 > 0x7fffffff) return false;   // (byte offsets inside a sequence are 32 bits)
    auto go = [&](auto dh, auto qt) {
        launch_ordered<decltype(dh)::value, decltype(qt)::value>(qkv, ld_qkv, S, N, n_heads, n_kv_heads, out, st);
        return true;
    };
    using std::integral_constant;
    const bool wide = lds_bytes(32, N) <= MAX_LDS;
    if (d_head == 128) return wide ? go(integral_constant<int, 128>(), integral_constant<int, 32>()) : go(integral_constant<int, 128>(), integral_constant<int, 16>());
    return wide ? go(integral_constant<int, 64>(), integral_constant<int, 32>()) : go(integral_constant<int, 64>(), integral_constant<int, 16>());
}
