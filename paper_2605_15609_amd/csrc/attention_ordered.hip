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
// Bound by the fp32 matrix instructions (a sixteenth of the bf16 rate, twice what fmaf reaches without packed instructions) and the
// 2-byte fetches of the values.  A workgroup takes QT queries of one head; the scores of all keys stay in LDS, because the sums need
// the final maximum and their order.  Keys and values go from global memory straight into the registers that the instructions
// read.  12 x 557 tokens, 32 heads of 128: 1109 us a layer (55 TFLOP/s), the plain kernel 8546, bf16 matrix instructions 126.
#include <type_traits>

#include "psd_internal.h"
#include "device_types.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NW = 4;   // wavefronts per workgroup

template <int QT>
using acc_t = std::conditional_t<QT == 32, f32x16, f32x4>;

// QT x QT outputs; a lane holds row (a) / column (b) lane % QT at k = lane / QT, and of the result column lane % QT, rows
// 8 * (v / 4) + 4 * (lane / QT) + v % 4
__device__ __forceinline__ f32x16 mma(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// of 8 consecutive channels the ones with k = h of the instructions that contract them, ascending
template <int QT>
__device__ __forceinline__ void pick(const uint4 u, int h, float *f) {
    auto half = [](uint32_t w, int high) { return __uint_as_float(high ? w & 0xffff0000u : w << 16); };
    if constexpr (QT == 32) {
        f[0] = half(u.x, h);
        f[1] = half(u.y, h);
        f[2] = half(u.z, h);
        f[3] = half(u.w, h);
    } else {
        f[0] = half(h & 2 ? u.y : u.x, h & 1);
        f[1] = half(h & 2 ? u.w : u.z, h & 1);
    }
}

template <int DH, int QT>
__global__ __launch_bounds__(NW * 64, 2) void attention_ordered_kernel(const bf16_t *__restrict__ qkv, int ld, int N, int n_heads,
                                                                       int n_kv_heads, bf16_t *__restrict__ out) {
    constexpr int KPI = 64 / QT, NV = QT * QT / 64;     // k per instruction, outputs per lane
    constexpr int GROUPS = NW * 64 / QT;                // threads per query in the softmax
    constexpr int STRIDED = 64 / GROUPS;                // of the 64 partial sums, those of one thread
    extern __shared__ __align__(16) float smem[];
    float *red = smem, *sc = smem + GROUPS * QT;        // sc[key][query]

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
    const bf16_t *kp = seq + (n_heads + head / group) * DH, *vp = kp + n_kv_heads * DH;

    // ---- scores: the wavefronts deal the tiles of QT keys
    {
        float qf[DH / KPI];
        const bf16_t *q = seq + (int64_t)min(qblk * QT + lrow, N - 1) * ld + head * DH;   // (past the last query: it again, not stored)
#pragma unroll
        for (int j = 0; j < DH / 8; ++j) pick<QT>(*reinterpret_cast<const uint4 *>(q + j * 8), h, qf + j * (8 / KPI));
        const float scale = 1.0f / sqrtf((float)DH);
        for (int k0 = wave * QT; k0 < N; k0 += NW * QT) {
            const bf16_t *k = kp + (int64_t)min(k0 + lrow, N - 1) * ld;
            uint4 kf[DH / 8];
#pragma unroll
            for (int j = 0; j < DH / 8; ++j) kf[j] = *reinterpret_cast<const uint4 *>(k + j * 8);
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
                if (key < N) sc[key * QT + lrow] = acc[v] * scale;
            }
        }
    }
    __syncthreads();

    // ---- softmax: GROUPS threads per query
    const int tq = threadIdx.x % QT, tg = threadIdx.x / QT;
    float mx = -INFINITY;
    for (int j = tg; j < N; j += GROUPS) mx = fmaxf(mx, sc[j * QT + tq]);
    red[tg * QT + tq] = mx;
    __syncthreads();
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) mx = fmaxf(mx, red[g * QT + tq]);
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
    __syncthreads();   // the maxima are read
    red[tg * QT + tq] = sum[0];
    __syncthreads();
    float part[GROUPS];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) part[g] = red[g * QT + lrow];   // this lane's query as a column of the output
#pragma unroll
    for (int off = GROUPS / 2; off > 0; off >>= 1)
#pragma unroll
        for (int g = 0; g < off; ++g) part[g] += part[g + off];
    const float inv = 1.0f / part[0];

    // ---- values: a wavefront takes tiles of QT channels and walks the keys, FLIGHT instructions per round of fetches
    constexpr int FLIGHT = 8, STEP = FLIGHT * KPI;
    for (int c0 = wave * QT; c0 < DH; c0 += NW * QT) {
        acc_t<QT> acc;
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v] = 0.f;
        const bf16_t *v = vp + c0 + lrow;
        uint16_t next[FLIGHT];
        auto fetch = [&](int j0) {   // (past the last key: it again, dropped below)
#pragma unroll
            for (int i = 0; i < FLIGHT; ++i) next[i] = v[(int64_t)min(j0 + i * KPI + h, N - 1) * ld].bits;
        };
        fetch(0);
        int j0 = 0;
        for (; j0 + STEP <= N; j0 += STEP) {
            float a[FLIGHT];
#pragma unroll
            for (int i = 0; i < FLIGHT; ++i) a[i] = bf16_bits_to_float(next[i]);
            fetch(j0 + STEP);
#pragma unroll
            for (int i = 0; i < FLIGHT; ++i) acc = mma(a[i], sc[(j0 + i * KPI + h) * QT + lrow], acc);
        }
#pragma unroll
        for (int i = 0; i < FLIGHT; ++i) {
            if (j0 + i * KPI < N) {   // (uniform) the last keys; 0 x 0 for those that do not exist
                const bool in = j0 + i * KPI + h < N;
                acc = mma(in ? bf16_bits_to_float(next[i]) : 0.f, in ? sc[(j0 + i * KPI + h) * QT + lrow] : 0.f, acc);
            }
        }
        const int q = qblk * QT + lrow;
        if (q < N) {
            bf16_t *o = out + ((int64_t)s * N + q) * (n_heads * DH) + head * DH + c0 + 4 * h;
#pragma unroll
            for (int g = 0; g < NV / 4; ++g)
                *reinterpret_cast<uint2 *>(o + 8 * g) = make_uint2(pack_bf16x2(acc[4 * g] * inv, acc[4 * g + 1] * inv),
                                                                   pack_bf16x2(acc[4 * g + 2] * inv, acc[4 * g + 3] * inv));
        }
    }
}

constexpr int MAX_LDS = 160 * 1024;
constexpr int lds_bytes(int qt, int N) { return (NW * 64 + N * qt) * 4; }

template <int DH, int QT>
void launch_ordered(const bf16_t *qkv, int ld_qkv, int S, int N, int n_heads, int n_kv_heads, bf16_t *out, hipStream_t st) {
    auto kern = attention_ordered_kernel<DH, QT>;
    static std::atomic<uint64_t> lds_raised{0};   // one per instantiation
    ensure_dynamic_lds(reinterpret_cast<const void *>(kern), MAX_LDS, lds_raised);
    hipLaunchKernelGGL(kern, dim3((N + QT - 1) / QT, n_heads, S), dim3(NW * 64), lds_bytes(QT, N), st, qkv, ld_qkv, N, n_heads, n_kv_heads, out);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}   // namespace

// 32 queries per workgroup read the keys and values half as often as 16 (1109 against 1327 us at 12 x 557 tokens, 32 heads of 128;
// 44 against 52 at 20 x 197, 8 heads of 64); 16 where the scores of 32 do not fit LDS (above 1272 keys), and the plain kernel where
// those of 16 do not (above 2544).
bool launch_attention_ordered(const bf16_t *qkv, int ld_qkv, int S, int N, int n_heads, int n_kv_heads, int d_head, bf16_t *out,
                              hipStream_t st) {
    if (N < 1 || lds_bytes(16, N) > MAX_LDS || (d_head != 64 && d_head != 128) || ld_qkv % 8 || !aligned16(qkv) || !aligned16(out)) return false;
    auto go = [&](auto dh, auto qt) {
        launch_ordered<decltype(dh)::value, decltype(qt)::value>(qkv, ld_qkv, S, N, n_heads, n_kv_heads, out, st);
        return true;
    };
    using std::integral_constant;
    const bool wide = lds_bytes(32, N) <= MAX_LDS;
    if (d_head == 128) return wide ? go(integral_constant<int, 128>(), integral_constant<int, 32>()) : go(integral_constant<int, 128>(), integral_constant<int, 16>());
    return wide ? go(integral_constant<int, 64>(), integral_constant<int, 32>()) : go(integral_constant<int, 64>(), integral_constant<int, 16>());
}
