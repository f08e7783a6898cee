"""Kernel-level parity at the full shapes of the benchmark configurations, on sampled outputs
that the fp64 oracle computes one by one (the whole result at these sizes would take the CPU
minutes).  Through the C ABI's kernel hooks, in the launch configuration the forward uses."""
import numpy as np
import pytest
import torch

import psd_inputs as inp
from oracle import psd_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bf16_round_trip(a):
    return inp.round_to_bf16(np.asarray(a, dtype=np.float32))


def dev_bf16(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV).to(torch.bfloat16)


def host_f64(t):
    return t.float().cpu().numpy().astype(np.float64)


GEMM_CASES = [
    # label, M, N, K, epilogue           (config 3 verify / stage-1, config 4 verify, ragged M)
    ("c3v-qkv", 2048, 12288, 4096, 0), ("c3v-o", 2048, 4096, 4096, 2), ("c3v-swiglu", 2048, 12288, 4096, 3),
    ("c3v-down", 2048, 4096, 12288, 2), ("c3s-qkv", 512, 12288, 4096, 0), ("c3s-o", 512, 4096, 4096, 2),
    ("c3s-down", 512, 4096, 12288, 2), ("c4v-qkv-bias", 6144, 4608, 3584, 1), ("c4v-swiglu", 6144, 18944, 3584, 3),
    ("c4s-down", 1024, 3584, 18944, 2), ("ragged", 200, 1408, 512, 3), ("ragged-store", 333, 1536, 512, 0),
    ("ragged-resid", 77, 512, 1408, 2),
]


@pytest.mark.parametrize("label,M,N,K,epi", GEMM_CASES, ids=[c[0] for c in GEMM_CASES])
def test_gemm_sampled_rows(label, M, N, K, epi):
    from paper_2605_15609_amd import binding as B
    print(f"[kernels] gemm {label} M={M} N={N} K={K} epi={epi}", flush=True)
    rng = np.random.default_rng(hash(label) % 2 ** 31)
    A = bf16_round_trip(rng.standard_normal((M, K), dtype=np.float32))
    W = bf16_round_trip(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    W2 = bf16_round_trip(rng.standard_normal((N, K), dtype=np.float32) * 0.05) if epi == 3 else None
    bias = rng.standard_normal(N).astype(np.float32) if epi == 1 else None
    resid0 = rng.standard_normal((M, N)).astype(np.float32) if epi == 2 else None
    dA, dW = dev_bf16(A), dev_bf16(W)
    if epi == 2:
        d_res = torch.from_numpy(resid0).to(DEV)
        B.kernel_gemm_bf16(dA, dW, epi, resid=d_res)
        got = d_res.cpu().numpy().astype(np.float64)
    else:
        out = B.kernel_gemm_bf16(dA, dW, epi, W2=None if W2 is None else dev_bf16(W2),
                                 bias=None if bias is None else torch.from_numpy(bias).to(DEV))
        got = host_f64(out)
    torch.cuda.synchronize()
    rows = sorted(set([0, M - 1, M // 2] + [int(r) for r in rng.integers(0, M, size=13)]))
    a = A[rows].astype(np.float64)
    ref = a @ W.astype(np.float64).T
    if epi == 1:
        ref = ref + bias
    if epi == 3:
        ref = orc.silu(ref) * (a @ W2.astype(np.float64).T)
    if epi == 2:
        ref = ref + resid0[rows]
        tol = 1e-3 * np.sqrt(K / 4096) + 1e-6 * np.abs(ref)             # fp32 accumulation only
    else:
        tol = 2.0 ** -8 * np.abs(ref) + 2e-3 * np.sqrt(K / 4096)        # one bf16 rounding of the result
    err = np.abs(got[rows] - ref)
    assert (err <= tol).all(), f"{label}: max err {err.max():.3e} at {np.unravel_index(err.argmax(), err.shape)}"


@pytest.mark.parametrize("epi", [0, 2, 3], ids=["store", "residual", "swiglu"])
def test_gemm_every_tile_configuration(epi):
    """Each workgroup tile / LDS ring depth the dispatcher can pick, forced in turn on one ragged shape
    (several tiles in both directions, K = 18 stages so every ring wraps) and checked in full."""
    from paper_2605_15609_amd import binding as B
    lib = B.load_library()
    M, N, K = 333, 832, 1152
    rng = np.random.default_rng(40 + epi)
    A = bf16_round_trip(rng.standard_normal((M, K), dtype=np.float32))
    W = bf16_round_trip(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    W2 = bf16_round_trip(rng.standard_normal((N, K), dtype=np.float32) * 0.05) if epi == 3 else None
    resid0 = rng.standard_normal((M, N)).astype(np.float32) if epi == 2 else None
    a = A.astype(np.float64)
    ref = a @ W.astype(np.float64).T
    if epi == 3:
        ref = orc.silu(ref) * (a @ W2.astype(np.float64).T)
    if epi == 2:
        ref = ref + resid0
        tol = 1e-3 + 1e-6 * np.abs(ref)
    else:
        tol = 2.0 ** -8 * np.abs(ref) + 2e-3
    dA, dW = dev_bf16(A), dev_bf16(W)
    dW2 = None if W2 is None else dev_bf16(W2)
    try:
        for tile in range(lib.psd_kernel_gemm_tile_count()):
            print(f"[kernels] gemm tile {tile} epi={epi}", flush=True)
            lib.psd_debug_force_gemm_tile(tile)
            if epi == 2:
                d_res = torch.from_numpy(resid0).to(DEV)
                B.kernel_gemm_bf16(dA, dW, epi, resid=d_res)
                got = d_res.cpu().numpy().astype(np.float64)
            else:
                got = host_f64(B.kernel_gemm_bf16(dA, dW, epi, W2=dW2))
            err = np.abs(got - ref)
            assert (err <= tol).all(), f"tile {tile}: max err {err.max():.3e} at {np.unravel_index(err.argmax(), err.shape)}"
    finally:
        lib.psd_debug_force_gemm_tile(-1)


@pytest.mark.parametrize("epi,M,N,K", [(2, 5000, 4032, 3072), (2, 6143, 3584, 6144), (3, 1037, 18944, 2048), (3, 1021, 19008, 2048), (3, 6684, 12288, 1024), (1, 5001, 12288, 2048)])
def test_contraction_in_two_launches_changes_no_bit(epi, M, N, K):
    """Contractions whose last round of tiles is partial run as two launches, cut along the rows or the output columns.  Against one
    launch on one tile (forced), bit for bit, with rows and columns that no tile divides."""
    import ctypes as C
    from paper_2605_15609_amd import binding as B
    lib = B.load_library()
    rows, cols = C.c_int64(), C.c_int64()
    assert lib.psd_debug_gemm_cut(M, N, K, epi, C.byref(rows), C.byref(cols)) == 0
    assert 0 < rows.value < M or 0 < cols.value < N, "one launch"
    g = torch.Generator(device=DEV)
    g.manual_seed(M + N)
    def draw(*s, std=1.0):
        return torch.empty(s, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=g)
    A, W, W2 = draw(M, K), draw(N, K, std=0.05), draw(N, K, std=0.05) if epi == 3 else None
    bias = torch.empty(N, device=DEV).normal_(generator=g) if epi == 1 else None
    resid = torch.empty(M, N, device=DEV).normal_(generator=g) if epi == 2 else None
    got = []
    try:
        for tile in (-1, 5):
            lib.psd_debug_force_gemm_tile(tile)
            if epi == 2:
                got.append(resid.clone())
                B.kernel_gemm_bf16(A, W, epi, resid=got[-1])
            else:
                got.append(B.kernel_gemm_bf16(A, W, epi, W2=W2, bias=bias))
    finally:
        lib.psd_debug_force_gemm_tile(-1)
    assert torch.equal(got[0], got[1])


SPLITK_CASES = [("c3-block-down", 128, 4096, 12288, (0, 8)), ("c3-block-o", 128, 4096, 4096, (0, 8)),
                ("c3-stage1-block-down", 32, 4096, 12288, (0, 4)), ("c4-block-down", 192, 3584, 18944, (0, 2, 4)),
                ("c4-block-o", 96, 3584, 3584, (0,)), ("ragged", 77, 832, 1536, (1, 2, 3, 4, 6, 8))]


@pytest.mark.parametrize("label,M,N,K,splits", SPLITK_CASES, ids=[c[0] for c in SPLITK_CASES])
def test_gemm_residual_split_along_k(label, M, N, K, splits):
    """Residual contraction over few rows cut along K (one workgroup per column tile and K part, partial sums
    added in order afterwards): every row against the fp64 product, and bit-for-bit repeatable."""
    from paper_2605_15609_amd import binding as B
    rng = np.random.default_rng(len(label) * 1000 + M)
    A = bf16_round_trip(rng.standard_normal((M, K), dtype=np.float32))
    W = bf16_round_trip(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
    resid0 = rng.standard_normal((M, N)).astype(np.float32)
    dA, dW = dev_bf16(A), dev_bf16(W)
    ref = A.astype(np.float64) @ W.astype(np.float64).T + resid0
    tol = 1e-3 * np.sqrt(K / 4096) + 1e-6 * np.abs(ref)
    for s in splits:
        print(f"[kernels] split-K gemm {label} k_splits={s}", flush=True)
        outs = []
        for _ in range(2):
            d_res = torch.from_numpy(resid0).to(DEV)
            used = B.kernel_gemm_residual_splitk(dA, dW, d_res, s)
            outs.append(d_res.cpu().numpy())
        assert s == 0 or used == s
        assert not (s == 0 and M <= 128 and K >= 4096) or used > 1, "few rows and a long K must be split"
        err = np.abs(outs[0].astype(np.float64) - ref)
        assert (err <= tol).all(), f"{label} k_splits={s} (used {used}): max err {err.max():.3e}"
        assert np.array_equal(outs[0], outs[1]), f"{label} k_splits={s}: two runs differ"


@pytest.mark.parametrize("N,K", [(4096, 4096), (4096, 12288), (3584, 3584), (3584, 18944), (512, 512), (512, 1408), (512, 640)])
def test_sums_of_few_rows_do_not_depend_on_their_number(N, K):
    """The residual contractions of a cached call, cut along K as the forward cuts them: a row's sum has the same bits whether 1, 16, ..
    or 128 rows share the call (every row class of the streaming kernel, its edges and one over)."""
    from paper_2605_15609_amd import binding as B
    g = torch.Generator(device=DEV)
    g.manual_seed(N + K)
    A = torch.empty((128, K), dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    W = torch.empty((N, K), dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
    full = torch.zeros((128, N), dtype=torch.float32, device=DEV)
    parts = B.kernel_gemm_residual_splitk(A, W, full)
    for M in (1, 16, 17, 32, 33, 48, 64, 65, 127):
        got = torch.zeros((M, N), dtype=torch.float32, device=DEV)
        assert B.kernel_gemm_residual_splitk(A[:M], W, got) == parts, f"{M} rows: another number of parts"
        assert torch.equal(got, full[:M]), f"{M} rows: other bits"


@pytest.mark.parametrize("epi", [0, 1, 2, 3], ids=["store", "bias", "residual", "swiglu"])
def test_gemm_few_rows(epi):
    """The streaming kernel of contractions over at most 128 rows: every row class (32, 64, 128) full, one over and one short of the
    class below, slices of every width the plan gives (from a few to thousands of outputs, ragged last ones), K of one stage (the
    ring is longer than K), of an odd number of stages, and long enough that the ring wraps several times."""
    from paper_2605_15609_amd import binding as B
    lib = B.load_library()
    for M, N, K in [(1, 64, 64), (31, 832, 64), (32, 4160, 192), (33, 9024, 320), (64, 12352, 128), (65, 12352, 1152), (100, 16448, 448),
                    (127, 20544, 192), (128, 12288, 704)]:
        assert lib.psd_debug_gemm_plan(M, N, K, epi, None) == lib.psd_kernel_gemm_tile_count(), "not on the streaming kernel"
        print(f"[kernels] few rows M={M} N={N} K={K} epi={epi}", flush=True)
        rng = np.random.default_rng(M + N + K)
        A = bf16_round_trip(rng.standard_normal((M, K), dtype=np.float32))
        W = bf16_round_trip(rng.standard_normal((N, K), dtype=np.float32) * 0.05)
        W2 = bf16_round_trip(rng.standard_normal((N, K), dtype=np.float32) * 0.05) if epi == 3 else None
        bias = rng.standard_normal(N).astype(np.float32)
        resid0 = rng.standard_normal((M, N)).astype(np.float32)
        a = A.astype(np.float64)
        ref = a @ W.astype(np.float64).T
        if epi == 1:
            ref += bias
        if epi == 3:
            ref = orc.silu(ref) * (a @ W2.astype(np.float64).T)
        if epi == 2:
            ref += resid0
            d_res = torch.from_numpy(resid0).to(DEV)
            B.kernel_gemm_bf16(dev_bf16(A), dev_bf16(W), epi, resid=d_res)
            got, tol = d_res.cpu().numpy().astype(np.float64), 1e-3 * np.sqrt(K / 4096) + 1e-6 * np.abs(ref)
        else:
            got = host_f64(B.kernel_gemm_bf16(dev_bf16(A), dev_bf16(W), epi, W2=None if W2 is None else dev_bf16(W2),
                                              bias=torch.from_numpy(bias).to(DEV) if epi == 1 else None))
            tol = 2.0 ** -8 * np.abs(ref) + 2e-3 * np.sqrt(K / 4096)
        err = np.abs(got - ref)
        assert (err <= tol).all(), f"M={M} N={N} K={K}: max err {err.max():.3e} at {np.unravel_index(err.argmax(), err.shape)}"


ATTN_CASES = [("c3v", 4, 512, 32, 32, 128), ("c4v-gqa", 6, 1024, 28, 4, 128), ("c2v", 4, 384, 8, 8, 64),
              ("c5-len", 2, 1280, 32, 32, 128), ("ragged", 3, 200, 4, 2, 64)]


@pytest.mark.parametrize("label,S,N,H,Hkv,dh", ATTN_CASES, ids=[c[0] for c in ATTN_CASES])
def test_attention_sampled_queries(label, S, N, H, Hkv, dh):
    from paper_2605_15609_amd import binding as B
    print(f"[kernels] attention {label}", flush=True)
    rng = np.random.default_rng(len(label) + N)
    qkv = bf16_round_trip(rng.standard_normal((S * N, (H + 2 * Hkv) * dh), dtype=np.float32))
    d_qkv = dev_bf16(qkv)
    out = host_f64(B.kernel_attention_bf16(d_qkv, S, N, H, Hkv, dh))
    # the forward keeps qkv with padded rows: same result from a row-strided view
    padded = torch.zeros((S * N, qkv.shape[1] + 64), dtype=torch.bfloat16, device=DEV)
    padded[:, :qkv.shape[1]] = d_qkv
    out_padded = B.kernel_attention_bf16(padded[:, :qkv.shape[1]], S, N, H, Hkv, dh)
    assert torch.equal(out_padded.cpu(), torch.from_numpy(out).to(torch.bfloat16)), f"{label}: row-strided qkv changes the result"
    torch.cuda.synchronize()
    group = H // Hkv
    worst = 0.0
    for _ in range(24):
        s, hd, i = int(rng.integers(S)), int(rng.integers(H)), int(rng.integers(N))
        if _ == 0:
            s, hd, i = S - 1, H - 1, N - 1
        seq = qkv[s * N: (s + 1) * N].astype(np.float64)
        q = seq[i, hd * dh: (hd + 1) * dh]
        k = seq[:, (H + hd // group) * dh: (H + hd // group + 1) * dh]
        v = seq[:, (H + Hkv + hd // group) * dh: (H + Hkv + hd // group + 1) * dh]
        ref = orc.attention(q[None, None, :], k[:, None, :], v[:, None, :])[0, 0]
        got = out[s * N + i, hd * dh: (hd + 1) * dh]
        worst = max(worst, np.abs(got - ref).max())
    # probabilities and outputs are rounded to bf16 once each: relative 2^-8 on O(1) values
    assert worst < 2e-2, f"{label}: max err {worst:.3e}"


HEAD_CASES = [("c3-stage1", 32, 126464, 4096), ("c3-verify", 128, 126464, 4096), ("c4-verify", 192, 152064, 3584),
              ("c2-verify", 128, 32000, 512), ("ragged", 77, 5000, 512), ("many-rows", 300, 3001, 512),
              ("c5-block64", 64, 126464, 4096), ("rows-256", 250, 5000, 576), ("one-row", 1, 3001, 64)]


@pytest.mark.parametrize("path", ["stream", "tiled"])
@pytest.mark.parametrize("label,rows,V,d", HEAD_CASES, ids=[c[0] for c in HEAD_CASES])
def test_fused_head_sampled_rows(label, rows, V, d, path):
    from paper_2605_15609_amd import binding as B
    print(f"[kernels] head {label}", flush=True)
    rng = np.random.default_rng(rows + V)
    y = bf16_round_trip(rng.standard_normal((rows, d), dtype=np.float32))
    W = bf16_round_trip(rng.standard_normal((V, d), dtype=np.float32) * 0.02)
    mask_id = V - 1
    scale = 1.7
    dW, dy = dev_bf16(W), dev_bf16(y)
    if path == "tiled":
        row_sum, row_arg = B.kernel_head_confidence_bf16(dy, dW, scale, mask_id)
    else:
        if rows > 192:
            pytest.skip("the streaming head takes at most 192 rows")
        row_sum, row_arg = B.kernel_head_stream_bf16(dy, B.kernel_pack_rows(dW), V, scale, mask_id)
    torch.cuda.synchronize()
    row_sum, row_arg = row_sum.cpu().numpy().astype(np.float64), row_arg.cpu().numpy()
    sample = sorted(set([0, rows - 1] + [int(r) for r in rng.integers(0, rows, size=6)]))
    Wd = W.astype(np.float64)
    for r in sample:
        z = scale * (y[r].astype(np.float64) @ Wd.T)
        x_hat, c = orc.top1_confidence(z[None], mask_id)
        zz = z.copy()
        zz[mask_id] = -np.inf
        top2 = np.partition(zz, -2)[-2:]
        if top2[1] - top2[0] >= 1e-3:
            assert row_arg[r] == x_hat[0], f"{label}: row {r} argmax {row_arg[r]} vs {x_hat[0]}"
        assert row_arg[r] != mask_id
        assert abs((1.0 / row_sum[r]) / c[0] - 1.0) < 2e-3, f"{label}: row {r} confidence {1 / row_sum[r]} vs {c[0]}"


HEAD_TILES = [(V, d, rows) for V, d in [(129, 64), (16384, 576), (16385, 576), (65024, 128), (65025, 64), (70001, 448)] for rows in (129, 160, 192, 193)]
HEAD_TILES += [(65537, 192, 65), (98304, 64, 128), (98305, 64, 100)]                              # two columns of 64 rows, and past them
HEAD_TILES += [(3001, 2048, 257), (32768, 2048, 200), (32769, 2048, 200), (9001, 2112, 1025)]    # above 192 rows, tiles of 128 or 256


@pytest.mark.parametrize("V,d,rows", HEAD_TILES)
def test_head_tiles_against_fp64(V, d, rows):
    """129 - 192 hidden rows in one column of tiles or two, ids in tiles of 128 or 256 that no vocabulary here divides (and one that it does), one K stage
    to nine; above 192 rows, tiles of 128 rows and of 256, partial ones among them.  Every row against fp64 logits: fp32 sums of d products are off by at most d * 2^-24 * sum |y w| each, a logit
    error of e changes the confidence by a factor exp(2 e), and the exponentials add 1e-5."""
    from paper_2605_15609_amd import binding as B
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + V)
    y = torch.empty((rows, d), dtype=torch.bfloat16, device=DEV).normal_(generator=g)
    W = torch.empty((V, d), dtype=torch.bfloat16, device=DEV).normal_(0.0, 0.02, generator=g)
    scale, mask_id = 1.7, V // 2
    row_sum, row_arg = B.kernel_head_confidence_bf16(y, W, scale, mask_id)
    z = scale * (y.double() @ W.double().T.contiguous())
    e = scale * d * 2.0 ** -24 * float((y.double().abs() @ W.double().abs().T.contiguous()).max())
    z[:, mask_id] = -float("inf")
    best = z.max(-1).values
    conf = 1.0 / torch.exp(z - best[:, None]).sum(-1)
    assert float((1.0 / row_sum.double() / conf - 1.0).abs().max()) <= np.expm1(2 * e) + 1e-5
    assert bool((z.gather(1, row_arg.long()[:, None])[:, 0] >= best - 2 * e).all())


def test_head_ties_go_to_the_lowest_token_id_and_mask_is_excluded():
    from paper_2605_15609_amd import binding as B
    d, V = 64, 1000
    y = np.zeros((40, d), dtype=np.float32)
    y[:, 0] = 1.0
    W = np.zeros((V, d), dtype=np.float32)
    W[[17, 300, 700, 999], 0] = 2.0            # exact ties across different vocabulary slabs; 999 is [M]
    W[999, 0] = 8.0
    for path in ("tiled", "stream"):
        if path == "tiled":
            row_sum, row_arg = B.kernel_head_confidence_bf16(dev_bf16(y), dev_bf16(W), 1.0, 999)
        else:
            row_sum, row_arg = B.kernel_head_stream_bf16(dev_bf16(y), B.kernel_pack_rows(dev_bf16(W)), V, 1.0, 999)
        torch.cuda.synchronize()
        assert (row_arg.cpu().numpy() == 17).all(), path
        expect = 3 + (V - 4) * np.exp(-2.0)
        np.testing.assert_allclose(row_sum.cpu().numpy(), expect, rtol=1e-5)


def test_kernel_hooks_reject_bad_shapes():
    from paper_2605_15609_amd import binding as B
    a = torch.zeros((8, 100), dtype=torch.bfloat16, device=DEV)
    w = torch.zeros((64, 100), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(B.PsdError, match="multiples of 64"):
        B.kernel_gemm_bf16(a, w)
    with pytest.raises(B.PsdError):
        B.kernel_attention_bf16(torch.zeros((10, 3 * 64), dtype=torch.bfloat16, device=DEV), 1, 10, 1, 1, 64)
