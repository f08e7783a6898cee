// Decision kernels of the PSD step: transfer policy (Eq. 1), speculative ordering and
// draft assembly (Eq. 2), hierarchical acceptance and state advance (Alg. 1, stage 3);
// EOS early stopping and the truncated token count of the evaluation protocol (App. B.1).
//
// A 64-lane wavefront looks at one sequence's block (L <= 64): lane j is block position j.
// Rankings are rank-by-counting inside the wavefront -- position j's rank among the
// masked positions is the number of masked positions that come before it in the order
// (confidence descending, lower position first on ties) -- so no sort is needed and ties
// are resolved identically everywhere.  All comparisons are on the fp32 confidences as
// stored, the precision the decisions are defined in.
#include "psd_internal.h"

namespace {

constexpr int WAVE = 64;

// rank of lane j among the live lanes below L by (c desc, lane asc); meaningful for live lanes.  Every live lane's confidence is
// broadcast through a scalar register; lanes that are not live broadcast NaN, which comes before nothing.  (With
// two shuffles through LDS per lane select_unmask took 6.8 us, now 4.4.)
__device__ __forceinline__ int rank_by_confidence(bool live, float c, int L) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int key = __float_as_int(live ? c : __builtin_nanf(""));
    int r = 0;
#pragma unroll
    for (int base = 0; base < WAVE; base += 16) {
        if (base >= L) break;
#pragma unroll
        for (int i = base; i < base + 16; ++i) {
            const float ci = __int_as_float(__builtin_amdgcn_readlane(key, i));
            r += (i < lane ? ci >= c : ci > c) ? 1 : 0;
        }
    }
    return r;
}

// would the policy commit a live lane of this rank and confidence?
__device__ __forceinline__ bool policy_commits(bool live, int rank, float c, const psd_policy &p) {
    bool ok = live && (c > p.tau || rank < p.k_min);
    if (p.k_max > 0) ok = ok && rank < p.k_max;
    return ok;
}

// ------------------------------------------------------------------ stage 1 commit (Eq. 1)
__global__ __launch_bounds__(WAVE) void select_unmask_kernel(int32_t *__restrict__ tokens, int N, BlockStart bs, int L,
                                                             const int32_t *__restrict__ top1,
                                                             const float *__restrict__ conf, psd_policy policy,
                                                             int32_t mask_id, uint8_t *__restrict__ transfer_mask,
                                                             int32_t *__restrict__ n_selected,
                                                             int32_t *__restrict__ n_left,
                                                             int32_t *__restrict__ devstats,
                                                             const int32_t *__restrict__ only) {
    const int b = blockIdx.x;
    const int j = threadIdx.x;
    if (only && only[b] == 0) return;   // uniform per workgroup: this sequence had no stage-1 call
    const int block_start = bs.of_row(b);
    int32_t *row = tokens + (int64_t)b * N + block_start;
    const bool in = j < L;
    // a sequence that stopped on an EOS token keeps its masks: its predictions are stale, nothing is committed
    const bool stopped = devstats && devstats[(int64_t)b * PSD_DEVSTAT_WORDS + PSD_DEVSTAT_EOS] > 0;
    const bool live = in && !stopped && row[j] == mask_id;
    const float c = in ? conf[(int64_t)b * L + j] : -2.0f;
    const int rank = rank_by_confidence(live, c, L);
    const bool take = policy_commits(live, rank, c, policy);
    if (take) row[j] = top1[(int64_t)b * L + j];
    if (in && transfer_mask) transfer_mask[(int64_t)b * L + j] = take ? 1 : 0;
    const int n_take = __popcll(__ballot(take));
    const int n_live = __popcll(__ballot(live));
    if (j == 0) {
        if (n_selected) n_selected[b] = n_take;
        if (n_left) n_left[b] = n_live - n_take;
        if (devstats) devstats[(int64_t)b * PSD_DEVSTAT_WORDS + PSD_DEVSTAT_POLICY] += n_take;
    }
}

// ------------------------------------------------------------------ stage 2 drafts (Eq. 2)
// grid (K, B): every (sequence, node) pair recomputes the ranking and writes its own draft row with coalesced 4-byte
// stores.  Bound by the latency of its loads: four wavefronts copy the row (one took 20 rounds of loads over 1280 tokens),
// the first one ranks and speculates meanwhile (13.6 -> 5.6 us at 16 sequences of 1280 tokens, K = 8).
constexpr int DRAFT_WAVES = 4;
__global__ __launch_bounds__(WAVE *DRAFT_WAVES) void build_drafts_kernel(const int32_t *__restrict__ tokens, int N, BlockStart bs,
                                                            int L, const int32_t *__restrict__ top1,
                                                            const float *__restrict__ conf, GraphArg g, int32_t mask_id,
                                                            int32_t *__restrict__ sigma, int32_t *__restrict__ m_out,
                                                            int32_t *__restrict__ drafts, int32_t *__restrict__ m_host) {
    const int k = blockIdx.x;
    const int b = blockIdx.y;
    const int j = threadIdx.x;
    const int block_start = bs.of_row(b);
    const int32_t *row = tokens + (int64_t)b * N;
    int32_t *out = drafts + ((int64_t)b * g.K + k) * N;
    // copy the sequence outside the block; the block gets the speculated tokens
#pragma unroll 4
    for (int i = j; i < N; i += WAVE * DRAFT_WAVES)
        if (i < block_start || i >= block_start + L) out[i] = row[i];
    if (j >= WAVE) return;
    const bool in = j < L;
    const int32_t tok = in ? row[block_start + j] : 0;
    const float c = in ? conf[(int64_t)b * L + j] : -2.0f;
    const int32_t pred = in ? top1[(int64_t)b * L + j] : 0;
    const bool live = in && tok == mask_id;
    const int rank = rank_by_confidence(live, c, L);
    const int m = __popcll(__ballot(live));
    if (in) {
        const bool spec = live && rank < m && ((g.rank_set[k] >> rank) & 1ull);
        out[block_start + j] = spec ? pred : tok;
    }
    if (k == 0) {   // uniform per workgroup
        __shared__ int s_pos[WAVE];
        s_pos[j] = -1;
        __builtin_amdgcn_wave_barrier();   // LDS accesses of one wavefront stay in order
        if (live) s_pos[rank] = j;
        __builtin_amdgcn_wave_barrier();
        if (in) sigma[(int64_t)b * L + j] = (j < m) ? s_pos[j] : -1;
        if (j == 0) {
            m_out[b] = m;
            if (m_host) m_host[b] = m;
        }
    }
}

// ------------------------------------------------------------------ stage 3 acceptance + advance
// One workgroup per sequence, one wavefront per node (up to ACCEPT_WAVES at a time): all loads of the K drafts and verifier tables
// are in flight together and the rankings run side by side.  The kernel is a chain of memory latencies and nothing else; with one
// wavefront walking the nodes in turn it was K such chains (58 -> 8.3 us at 16 sequences, K = 8).
constexpr int ACCEPT_WAVES = 16;
__global__ __launch_bounds__(WAVE *ACCEPT_WAVES) void accept_kernel(
    int32_t *__restrict__ tokens, const int32_t *__restrict__ drafts, int N, BlockStart bs, int L, const int32_t *__restrict__ sigma,
    const int32_t *__restrict__ m_in, GraphArg g, psd_policy policy, int32_t mask_id, const int32_t *__restrict__ v_top1,
    const float *__restrict__ v_conf, int32_t *__restrict__ k_star_out, uint8_t *__restrict__ accepted_out, int32_t *__restrict__ n_left,
    int32_t *__restrict__ devstats, int32_t *__restrict__ adopt_top1, float *__restrict__ adopt_conf, int32_t *__restrict__ n_left_host) {
    __shared__ int s_rank[WAVE];                               // block position -> rank in sigma, or -1
    __shared__ int32_t s_tok[PSD_MAX_NODES][WAVE];             // the drafts' blocks
    __shared__ int32_t s_top[PSD_MAX_NODES][WAVE];             // the verifier's predictions on them
    __shared__ uint64_t s_S[PSD_MAX_NODES];                    // S_k as a bit set over block positions
    __shared__ uint64_t s_ok[PSD_MAX_NODES][PSD_MAX_NODES];    // [p][k]: positions where edge test passes
    __shared__ uint64_t s_commit[PSD_MAX_NODES];               // positions pi commits on p's output

    const int b = blockIdx.x;
    const int j = threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), n_waves = blockDim.x / WAVE;
    const int block_start = bs.of_row(b);
    const int K = g.K;
    const int m = m_in[b];
    const bool in = j < L;
    if (m <= 0) {   // nothing was speculated for this sequence: leave its state alone
        if (wave > 0) return;
        if (j == 0) {
            if (k_star_out) k_star_out[b] = 0;
            if (n_left_host) n_left_host[b] = n_left[b];
        }
        if (accepted_out && j < K) accepted_out[(int64_t)b * K + j] = (j == 0) ? 1 : 0;
        return;
    }
    const int32_t *dbase = drafts + (int64_t)b * K * N + block_start;
    if (wave == 0) {
        const int pos = in && j < m ? sigma[(int64_t)b * L + j] : -1;
        s_rank[j] = -1;
        __builtin_amdgcn_wave_barrier();   // LDS accesses of one wavefront stay in order
        if (pos >= 0 && pos < L) s_rank[pos] = j;
    }
    // policy outcome on every node's verifier output
    for (int p = wave; p < K; p += n_waves) {
        const int64_t row = ((int64_t)b * K + p) * L + j;
        const int32_t dtok = in ? dbase[(int64_t)p * N + j] : 0;
        const float c = in ? v_conf[row] : -2.0f;
        const int32_t vt = in ? v_top1[row] : -1;
        s_tok[p][j] = dtok;
        s_top[p][j] = vt;
        const bool live = in && dtok == mask_id;
        const int rank = rank_by_confidence(live, c, L);
        const uint64_t commit = __ballot(policy_commits(live, rank, c, policy));
        if (j == 0) s_commit[p] = commit;
    }
    __syncthreads();
    // node sets, per-edge token agreement
    const int my_rank = s_rank[j];
    for (int p = wave; p < K; p += n_waves) {
        const uint64_t Sp = __ballot(my_rank >= 0 && ((g.rank_set[p] >> my_rank) & 1ull));
        const uint64_t commit = s_commit[p];
        const int32_t vt = s_top[p][j];
        uint64_t mine = 0;   // lane k keeps the set of edge (p, k)
        for (int k = 0; k < K; ++k) {
            const uint64_t agree = __ballot(in && vt == s_tok[k][j]);
            if (j == k) mine = agree & commit;
        }
        if (j < K) s_ok[p][j] = mine;
        if (j == 0) s_S[p] = Sp;
    }
    __syncthreads();
    if (wave > 0) return;

    // lane k: the parents of node k whose edge holds.  A parent's set is a strict subset of k's, so spreading acceptance from
    // the root until nothing changes accepts what a sweep in order of |S_k| does.
    const uint64_t Sk = j < K ? s_S[j] : 0;
    uint64_t parents = 0;
    if (j > 0 && j < K)
        for (int p = 0; p < K; ++p) {
            const uint64_t Sp = s_S[p];
            const bool strict_subset = (Sp & ~Sk) == 0 && Sp != Sk;
            if (strict_subset && ((Sk & ~Sp) & ~s_ok[p][j]) == 0) parents |= 1ull << p;
        }
    uint64_t acc = 1;
    for (;;) {
        const uint64_t next = __ballot(j == 0 || (parents & acc) != 0);
        if (next == acc) break;
        acc = next;
    }
    // k*: the largest accepted set, ties to the lowest node
    int key = j < K && ((acc >> j) & 1ull) ? (__popcll(Sk) << 8) | (255 - j) : -1;
    for (int off = 32; off > 0; off >>= 1) key = max(key, __shfl_xor(key, off, WAVE));
    const int k_star = 255 - (__builtin_amdgcn_readfirstlane(key) & 255);
    if (accepted_out && j < K) accepted_out[(int64_t)b * K + j] = (uint8_t)((acc >> j) & 1ull);

    // advance: x <- draft k*, then pi once more on k*'s verifier output
    const int32_t dtok = s_tok[k_star][j], vt = s_top[k_star][j];
    const bool live = in && dtok == mask_id;
    const bool take = live && ((s_commit[k_star] >> j) & 1ull);
    if (in) tokens[(int64_t)b * N + block_start + j] = take ? vt : dtok;
    // single-forward loop: k*'s verifier output becomes the table the next drafts are drawn from
    if (adopt_top1 && in) {
        adopt_top1[(int64_t)b * L + j] = vt;
        adopt_conf[(int64_t)b * L + j] = v_conf[((int64_t)b * K + k_star) * L + j];
    }
    const int n_live = __popcll(__ballot(live));
    const int n_take = __popcll(__ballot(take));
    if (j == 0) {
        const int depth = __popcll(s_S[k_star]);
        if (k_star_out) k_star_out[b] = k_star;
        if (n_left) n_left[b] = n_live - n_take;
        if (n_left_host) n_left_host[b] = n_live - n_take;
        if (devstats) {
            int32_t *ds = devstats + (int64_t)b * PSD_DEVSTAT_WORDS;
            ds[PSD_DEVSTAT_DRAFT] += depth;
            ds[PSD_DEVSTAT_POST] += n_take;
            ds[PSD_DEVSTAT_HIST + depth] += 1;
        }
    }
}

// ------------------------------------------------------------------ EOS early stopping (App. B.1)
// After a state update: a sequence whose block holds the EOS token is finished, whatever is still masked.
// Its mask counts are zeroed, which is what takes it out of the following model calls, and the position is
// flagged in its counters, which is what keeps the stage-1 commit from touching it again.
__global__ __launch_bounds__(WAVE) void eos_stop_kernel(const int32_t *__restrict__ tokens, int N, BlockStart bs, int L,
                                                        int32_t eos_id, int32_t *__restrict__ n_left,
                                                        int32_t *__restrict__ m, int32_t *__restrict__ devstats) {
    const int b = blockIdx.x, j = threadIdx.x;
    const int block_start = bs.of_row(b);
    const bool hit = j < L && tokens[(int64_t)b * N + block_start + j] == eos_id;
    const uint64_t hits = __ballot(hit);
    if (hits != 0ull && j == 0) {
        if (n_left) n_left[b] = 0;
        if (m) m[b] = 0;
        devstats[(int64_t)b * PSD_DEVSTAT_WORDS + PSD_DEVSTAT_EOS] = __ffsll((unsigned long long)hits);
    }
}

// A sequence leaves its block (resolved, stopped on an EOS token, or the call ends): the first EOS position of the
// block (when stopping on EOS is on) and the number of positions resolved since the block was entered at or before
// it -- all resolved positions without an EOS -- are added to the sequence's counters.  The positions masked on
// entry are in the counters as a 64-bit set.  only != NULL: just the sequences b with only[b] != 0.
__device__ __forceinline__ void finish_counts(const int32_t *__restrict__ tokens, int N, const BlockStart &bs, int L, int32_t mask_id, int32_t eos_stop,
                                              int32_t eos_id, int32_t *__restrict__ devstats) {
    const int b = blockIdx.x, j = threadIdx.x;
    const int block_start = bs.of_row(b);
    const int32_t tok = j < L ? tokens[(int64_t)b * N + block_start + j] : mask_id;
    const uint64_t hits = __ballot(eos_stop && j < L && tok == eos_id);
    const uint64_t resolved = __ballot(j < L && tok != mask_id);
    if (j == 0) {
        int32_t *ds = devstats + (int64_t)b * PSD_DEVSTAT_WORDS;
        const int eos = hits ? __ffsll((unsigned long long)hits) - 1 : -1;
        const int limit = eos >= 0 ? eos : L - 1;
        const uint64_t upto = limit >= 63 ? ~0ull : ((1ull << (limit + 1)) - 1ull);
        const uint64_t entry = (uint64_t)(uint32_t)ds[PSD_DEVSTAT_ENTRY] | ((uint64_t)(uint32_t)ds[PSD_DEVSTAT_ENTRY + 1] << 32);
        ds[PSD_DEVSTAT_EOS] = eos + 1;
        ds[PSD_DEVSTAT_COUNTED] += __popcll(entry & resolved & upto);
    }
}

__global__ __launch_bounds__(WAVE) void finish_counts_kernel(const int32_t *__restrict__ tokens, int N, BlockStart bs, int L,
                                                             int32_t mask_id, int32_t eos_stop, int32_t eos_id,
                                                             int32_t *__restrict__ devstats, const int32_t *__restrict__ only) {
    if (only && only[blockIdx.x] == 0) return;
    finish_counts(tokens, N, bs, L, mask_id, eos_stop, eos_id, devstats);
}

__global__ __launch_bounds__(WAVE) void finish_export_kernel(const int32_t *__restrict__ tokens, int N, BlockStart bs, int L, int32_t mask_id,
                                                             int32_t *devstats, SeqSet who, int32_t *__restrict__ host_stats) {
    if (who.has(blockIdx.x)) finish_counts(tokens, N, bs, L, mask_id, 0, 0, devstats);
    __syncthreads();
    const int64_t at = (int64_t)blockIdx.x * PSD_DEVSTAT_WORDS;
    for (int i = threadIdx.x; i < PSD_DEVSTAT_WORDS; i += WAVE) host_stats[at + i] = devstats[at + i];
}

}   // namespace

void launch_eos_stop(const int32_t *tokens, int B, int N, BlockStart block_start, int L, int32_t eos_id, int32_t *n_left, int32_t *m,
                     int32_t *devstats, hipStream_t st) {
    hipLaunchKernelGGL(eos_stop_kernel, dim3(B), dim3(WAVE), 0, st, tokens, N, block_start, L, eos_id, n_left, m, devstats);
}

void launch_finish_counts(const int32_t *tokens, int B, int N, BlockStart block_start, int L, int32_t mask_id, int32_t eos_stop,
                          int32_t eos_id, int32_t *devstats, const int32_t *only, hipStream_t st) {
    hipLaunchKernelGGL(finish_counts_kernel, dim3(B), dim3(WAVE), 0, st, tokens, N, block_start, L, mask_id, eos_stop, eos_id,
                       devstats, only);
}

void launch_finish_export(const int32_t *tokens, int B, int N, BlockStart block_start, int L, int32_t mask_id, int32_t *devstats, const SeqSet &who,
                          int32_t *host_stats, hipStream_t st) {
    hipLaunchKernelGGL(finish_export_kernel, dim3(B), dim3(WAVE), 0, st, tokens, N, block_start, L, mask_id, devstats, who, host_stats);
}

void launch_select_unmask(int32_t *tokens, int B, int N, BlockStart block_start, int L, const int32_t *top1, const float *conf,
                          psd_policy policy, int32_t mask_id, uint8_t *transfer_mask, int32_t *n_selected,
                          int32_t *n_left, int32_t *devstats, const int32_t *only, hipStream_t st) {
    hipLaunchKernelGGL(select_unmask_kernel, dim3(B), dim3(WAVE), 0, st, tokens, N, block_start, L, top1, conf, policy,
                       mask_id, transfer_mask, n_selected, n_left, devstats, only);
}

void launch_build_drafts(const int32_t *tokens, int B, int N, BlockStart block_start, int L, const int32_t *top1,
                         const float *conf, const GraphArg &g, int32_t mask_id, int32_t *sigma, int32_t *m,
                         int32_t *drafts, hipStream_t st, int32_t *m_host) {
    hipLaunchKernelGGL(build_drafts_kernel, dim3(g.K, B), dim3(WAVE * DRAFT_WAVES), 0, st, tokens, N, block_start, L, top1, conf, g,
                       mask_id, sigma, m, drafts, m_host);
}

void launch_accept(int32_t *tokens, const int32_t *drafts, int B, int N, BlockStart block_start, int L, const int32_t *sigma,
                   const int32_t *m, const GraphArg &g, psd_policy policy, int32_t mask_id, const int32_t *v_top1,
                   const float *v_conf, int32_t *k_star, uint8_t *accepted, int32_t *n_left, int32_t *devstats,
                   int32_t *adopt_top1, float *adopt_conf, hipStream_t st, int32_t *n_left_host) {
    hipLaunchKernelGGL(accept_kernel, dim3(B), dim3(WAVE * (g.K < ACCEPT_WAVES ? g.K : ACCEPT_WAVES)), 0, st, tokens, drafts, N, block_start, L, sigma, m, g, policy,
                       mask_id, v_top1, v_conf, k_star, accepted, n_left, devstats, adopt_top1, adopt_conf, n_left_host);
}
