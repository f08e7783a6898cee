// Attention of block rows against a KV cache (bf16): a sequence has at most 64 rows of its own, every one of them sees the pre.len
// cached positions and all own rows.  Same transposed problem, fragment layouts and probabilities as attention_mfma.hip; what
// differs is how the work is cut, because a launch is a chain of latencies and nothing else (128 rows of the 8B shape read 2 MB).
//
// What bounds it: the serial chain fetch -> scores -> softmax -> values of a wavefront, about 2.5 us per tile of 64 keys through
// LDS, and the launch that rotated the own rows and transposed their values before it.  So four wavefronts deal the tiles, operands
// of cached keys go from global memory straight into the registers the MFMAs read (a lane's 16 bytes of a K row or of a transposed
// value row are a fragment as they are: no ring, barrier or swizzle), and the partial results meet once in LDS.  The own rows pass
// through LDS, rotated on the way, while a wavefront's first keys are under way.
// One wavefront per SIMD: a tile's keys, values, scores and outputs are 224 registers a lane, and at 256 the compiler spills 53 of
// them (22 us instead of 14).  With it, against rotary + transpose launch and key-split kernel: 32 heads of 128, 32 rows, 448
// cached positions, 1 sequence 17.0 -> 14.3 us, 4 sequences 19.9 -> 14.2.  The next tile's operands fetched ahead into a second register set: 5 - 8 % slower; eight wavefronts spill.
#include "psd_internal.h"
#include "device_types.h"
#include "rope_device.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int BKV = 64;   // keys per tile
constexpr int KSP = 4;    // wavefronts per workgroup, which deal the tiles among themselves

template <int DH>
__global__ __launch_bounds__(KSP * 64, 1) void attention_block_kernel(const bf16_t *__restrict__ qkv, int ld_qkv, int N, int n_heads,
                                                                   int n_kv_heads, bf16_t *__restrict__ out, KvPrefix pre, int pos0,
                                                                   const float *__restrict__ cos_t, const float *__restrict__ sin_t) {
    constexpr int KS = DH / 16, CT = DH / 32, NF = CT * 16;   // k-steps of the scores, output subtiles, output values per lane
    static_assert(NF % KSP == 0 && NF / KSP % 4 == 0, "the merge deals groups of 4 values to the wavefronts");
    // LDS: first the own rows (32 queries and 64 keys rotated, 64 rows of values; padded by 16 bytes against bank conflicts), then
    // the partial results [wavefront][max, sum, NF values][64 lanes]
    constexpr int LD = DH + 8;
    extern __shared__ __align__(16) unsigned char lds[];
    bf16_t *sq = reinterpret_cast<bf16_t *>(lds), *sk = sq + 32 * LD, *sv = sk + 64 * LD;
    float *part = reinterpret_cast<float *>(lds);

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
    const int kvh = head / group;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5;
    const bf16_t *seq = qkv + (int64_t)s * N * ld_qkv;
    const int64_t cache = pre.len > 0 ? (pre.seq_rows ? pre.seq_rows[s] : s) / pre.seqs_per_cache : 0;
    const bf16_t *k_pre = (const bf16_t *)pre.k + cache * pre.stride_k + kvh * DH;
    const bf16_t *v_pre = (const bf16_t *)pre.vt + cache * pre.stride_vt + (int64_t)kvh * DH * pre.ld_vt;

    // lane (row, half) of a fragment holds channels 16 ks + 8 half .. + 7 of its row
    auto load_row = [&](uint4 *f, const bf16_t *row) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) f[ks] = *reinterpret_cast<const uint4 *>(row + ks * 16 + lhalf * 8);
    };
    // a tile: kf[kt] the K rows of keys k0 + 32 kt .., vf[kg][ct] the values of 16 keys in the slot order of vt_key_slot
    // (rows past the last key repeat it; a value row is as long as whole tiles)
    const int n_pre = (pre.len + BKV - 1) / BKV;
    uint4 kf[2][KS];
    auto load_keys = [&](int k0) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) load_row(kf[kt], k_pre + (int64_t)min(k0 + kt * 32 + lrow, pre.len - 1) * pre.ld_k);
    };
    if (wave < n_pre) load_keys(wave * BKV);

    // the own rows into LDS while that is under way, queries and keys rotated: a thread takes 8 rotary pairs of a row
    {
        constexpr int G = DH / 16, V8 = DH / 8;
        const bf16_t *v_own = seq + (n_heads + n_kv_heads + kvh) * DH;
        const int nv = N * V8;
        uint4 v0 = make_uint4(0, 0, 0, 0);
        if ((int)threadIdx.x < nv) v0 = *reinterpret_cast<const uint4 *>(v_own + (int64_t)(threadIdx.x / V8) * ld_qkv + threadIdx.x % V8 * 8);
        for (int u = threadIdx.x; u < (32 + N) * G; u += KSP * 64) {
            const int r = u / G, j = u % G * 8;
            const bool query = r < 32;
            const int i = query ? min(qblk * 32 + r, N - 1) : r - 32;   // (queries past the last one repeat it and store nothing)
            const bf16_t *row = seq + (int64_t)i * ld_qkv + (query ? head : n_heads + kvh) * DH + j;
            const int64_t at = (int64_t)(pos0 + i) * (DH / 2) + j;
            const float4 *c = reinterpret_cast<const float4 *>(cos_t + at), *n = reinterpret_cast<const float4 *>(sin_t + at);
            uint4 a, b;
            rope_rotate8(*reinterpret_cast<const uint4 *>(row), *reinterpret_cast<const uint4 *>(row + DH / 2), c[0], c[1], n[0], n[1], a, b);
            bf16_t *to = sq + r * LD + j;   // (the keys follow the queries)
            *reinterpret_cast<uint4 *>(to) = a;
            *reinterpret_cast<uint4 *>(to + DH / 2) = b;
        }
        if ((int)threadIdx.x < nv) *reinterpret_cast<uint4 *>(sv + threadIdx.x / V8 * LD + threadIdx.x % V8 * 8) = v0;
        for (int u = threadIdx.x + KSP * 64; u < nv; u += KSP * 64)
            *reinterpret_cast<uint4 *>(sv + u / V8 * LD + u % V8 * 8) = *reinterpret_cast<const uint4 *>(v_own + (int64_t)(u / V8) * ld_qkv + u % V8 * 8);
    }
    __syncthreads();
    const int q = qblk * 32 + lrow;
    floatx16 acc_o[CT];
#pragma unroll
    for (int i = 0; i < CT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_o[i][v] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;
    const float sl2 = 1.4426950408889634f / sqrtf((float)DH);   // softmax scale folded into exp2

    auto tile = [&](int left, auto values) {   // left: keys of the tile that exist
        uint4 vf[4][CT];
        values(vf);
        floatx16 acc_s[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_s[kt][v] = 0.f;
        asm volatile("" ::: "memory");   // the queries are read per tile: kept in registers they would push the tile's operands out
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 qf = *reinterpret_cast<const bf16x8 *>(sq + lrow * LD + ks * 16 + lhalf * 8);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
                acc_s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[kt][ks]), qf, acc_s[kt], 0, 0, 0);
        }
        if (left < BKV) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (kt * 32 + 8 * (v >> 2) + 4 * lhalf + (v & 3) >= left) acc_s[kt][v] = -INFINITY;
        }
        float mx = acc_s[0][0];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc_s[kt][v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run, mx), m_s = m_new * sl2;
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * sl2);
        float psum = 0.f;
        uint4 pf[4];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
            float p[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                p[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(acc_s[kt][v], sl2, -m_s));
                psum += p[v];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
                pf[kt * 2 + u] = make_uint4(pack_bf16x2(p[8 * u + 0], p[8 * u + 1]), pack_bf16x2(p[8 * u + 2], p[8 * u + 3]),
                                            pack_bf16x2(p[8 * u + 4], p[8 * u + 5]), pack_bf16x2(p[8 * u + 6], p[8 * u + 7]));
        }
        l_run = l_run * alpha + psum;
        m_run = m_new;
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_o[ct][v] *= alpha;
#pragma unroll
        for (int kg = 0; kg < 4; ++kg)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                uint4 w = vf[kg][ct];
                if (left < BKV) {   // slots past the end hold anything: their probabilities are zero, but 0 x NaN is NaN
                    const int n_lo = left - (kg * 16 + 4 * lhalf), n_hi = n_lo - 8;
                    w.x &= n_lo >= 2 ? 0xffffffffu : n_lo == 1 ? 0x0000ffffu : 0u;
                    w.y &= n_lo >= 4 ? 0xffffffffu : n_lo == 3 ? 0x0000ffffu : 0u;
                    w.z &= n_hi >= 2 ? 0xffffffffu : n_hi == 1 ? 0x0000ffffu : 0u;
                    w.w &= n_hi >= 4 ? 0xffffffffu : n_hi == 3 ? 0x0000ffffu : 0u;
                }
                acc_o[ct] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, pf[kg]),
                                                                   acc_o[ct], 0, 0, 0);
            }
    };

    for (int t = wave; t < n_pre; t += KSP) {
        if (t != wave) load_keys(t * BKV);
        tile(pre.len - t * BKV, [&](uint4 (&vf)[4][CT]) {
#pragma unroll
            for (int kg = 0; kg < 4; ++kg)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    vf[kg][ct] = *reinterpret_cast<const uint4 *>(v_pre + (int64_t)(ct * 32 + lrow) * pre.ld_vt + t * BKV + kg * 16 + lhalf * 8);
        });
    }
    if (wave == n_pre % KSP) {   // the own rows: one tile (what lies behind the last row in LDS is masked)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) load_row(kf[kt], sk + (kt * 32 + lrow) * LD);
        tile(N, [&](uint4 (&vf)[4][CT]) {
#pragma unroll
            for (int kg = 0; kg < 4; ++kg)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    uint32_t x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = sv[(kg * 16 + 8 * (e >> 2) + 4 * lhalf + (e & 3)) * LD + ct * 32 + lrow].bits;
                    vf[kg][ct] = make_uint4(x[0] | x[1] << 16, x[2] | x[3] << 16, x[4] | x[5] << 16, x[6] | x[7] << 16);
                }
        });
    }
    __syncthreads();   // the own rows are done with

    // The partial results meet in LDS, each wavefront merges and stores a share of the channels, in wavefront order.  A wavefront
    // without tiles contributes max = -inf, sum = 0.
    l_run += __shfl_xor(l_run, 32, 64);   // the half-waves of a query hold disjoint keys
    float *mine = part + wave * (2 + NF) * 64 + lane;
    mine[0] = m_run;
    mine[64] = l_run;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int v = 0; v < 16; ++v) mine[(2 + ct * 16 + v) * 64] = acc_o[ct][v];
    __syncthreads();
    float scale[KSP], m_all = -INFINITY, l_all = 0.f;
#pragma unroll
    for (int w = 0; w < KSP; ++w) {
        scale[w] = part[w * (2 + NF) * 64 + lane];
        m_all = fmaxf(m_all, scale[w]);
    }
#pragma unroll
    for (int w = 0; w < KSP; ++w) {
        scale[w] = __builtin_amdgcn_exp2f((scale[w] - m_all) * sl2);
        l_all += part[(w * (2 + NF) + 1) * 64 + lane] * scale[w];
    }
    const float inv = 1.0f / l_all;
    bf16_t *op = out + ((int64_t)s * N + q) * (n_heads * DH) + head * DH;
#pragma unroll
    for (int g = 0; g < NF / KSP / 4; ++g) {
        const int f = wave * (NF / KSP) + g * 4;   // values f .. f + 3: subtile f / 16, channels 8 (f % 16 / 4) + 4 half ..
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < KSP; ++w)
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] += part[(w * (2 + NF) + 2 + f + v) * 64 + lane] * scale[w];
        if (q < N)
            *reinterpret_cast<uint2 *>(op + (f >> 4) * 32 + 8 * ((f & 15) >> 2) + 4 * lhalf) =
                make_uint2(pack_bf16x2(o[0] * inv, o[1] * inv), pack_bf16x2(o[2] * inv, o[3] * inv));
    }
}

template <int DH>
void launch_block(const bf16_t *qkv, int ld_qkv, int S, int N, int n_heads, int n_kv_heads, bf16_t *out, const KvPrefix &pre, int pos0,
                  const float *cos_t, const float *sin_t, hipStream_t st) {
    constexpr int merge = KSP * (2 + DH / 2) * 64 * 4, own = 160 * (DH + 8) * 2, smem = merge > own ? merge : own;
    static_assert(smem <= 160 * 1024, "own rows or partial results exceed the LDS of a CU");
    auto kern = attention_block_kernel<DH>;
    static std::atomic<uint64_t> lds_raised{0};   // one per instantiation
    ensure_dynamic_lds(reinterpret_cast<const void *>(kern), smem, lds_raised);
    hipLaunchKernelGGL(kern, dim3((N + 31) / 32, n_heads, S), dim3(KSP * 64), smem, st, qkv, ld_qkv, N, n_heads, n_kv_heads, out, pre, pos0,
                       cos_t, sin_t);
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}   // namespace

// Long prefixes and many workgroups are throughput, where the tiles that attention_kernel shares in LDS win.  The lines must not
// depend on the number of sequences, or a sequence's bits would (beyond the 128 rows where the contractions change too).
// Up to 32 rows: three tiles a wavefront.  32 heads of 128, 1 to 128 sequences: 10.7 against 15.7 us (1 sequence, 128 positions), 23.9
// against 25.2 (1, 768), 434 against 447 (128, 768), behind at 37 against 31 (8, 1216).  28 heads on 4 KV heads: 21 against 24 (1, 768),
// but 4 to 11 % behind at 64 sequences and more against 256, 576 or 768 positions, where a wavefront has one tile more than the
// others.
// 33 to 64 rows, whose keys two workgroups fetch: while the call has at most 128 rows and such a call is one round of workgroups
// (d_head 128, 64 rows: 22.6 against 33.6 us at 768 positions; 16 sequences 92 against 60), and for heads of 64 up to 7 tiles (8 heads: 9.5
// against 17.7 us with 1 sequence, 23.8 against 26.9 with 64, 49 against 45 with 128).
bool attention_block_fits(const bf16_t *qkv, int ld_qkv, int S, int N, int n_heads, int d_head, const bf16_t *out, const KvPrefix &pre,
                          const float *cos_t, const float *sin_t) {
    if (N < 1 || N > 64) return false;
    const bool one_round = (int64_t)S * N <= 128 && 2 * n_heads * (128 / N) <= 256;
    if (N <= 32 ? pre.len > 3 * KSP * BKV : !one_round && (d_head != 64 || pre.len > 7 * BKV)) return false;
    return (d_head == 64 || d_head == 128) && ld_qkv % 8 == 0 && aligned16(qkv) && aligned16(out) && aligned16(cos_t) &&
           aligned16(sin_t) &&
           (pre.len == 0 || (aligned16(pre.k) && aligned16(pre.vt) && pre.ld_k % 8 == 0 && pre.ld_vt % 64 == 0 && pre.ld_vt >= pre.len &&
                             pre.stride_k % 8 == 0 && pre.stride_vt % 8 == 0));
}

void launch_attention_block(const bf16_t *qkv, int ld_qkv, int S, int N, int n_heads, int n_kv_heads, int d_head, bf16_t *out,
                            const KvPrefix &pre, int pos0, const float *cos_t, const float *sin_t, hipStream_t st) {
    if (d_head == 128) launch_block<128>(qkv, ld_qkv, S, N, n_heads, n_kv_heads, out, pre, pos0, cos_t, sin_t, st);
    else launch_block<64>(qkv, ld_qkv, S, N, n_heads, n_kv_heads, out, pre, pos0, cos_t, sin_t, st);
}
