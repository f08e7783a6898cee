"""Numeric parity of the HIP forward + top-1 confidence with the fp64 oracle, through the C ABI.

Tolerances (from the benchmark spec): logits within 1e-4 max-abs on the fp32 debug path and
2e-2 on the bf16 MFMA path; top-1 tokens equal except where the oracle's own top-1 margin
is below 1e-3 (logged and excluded).  Confidences are compared relatively: a logit error
of e changes a softmax probability by at most a factor exp(2e).
"""
import dataclasses

import numpy as np
import pytest
import torch

import psd_inputs as inp
from oracle import psd_oracle as orc

pytestmark = pytest.mark.gpu

SMALL = inp.WORKLOADS[2].shape
SHAPES = {
    # d_head 64, MHA, ragged sequence length (200 = 128 + 72), ragged vocab tail vs 128/256 slabs
    "small-2l": (inp.cut_down(SMALL, n_layers=2, vocab=5000, seed=21), 200, 96, 32),
    # d_head 128, grouped KV heads + QKV bias (Dream layout), 136 tokens
    "gqa-bias": (inp.cut_down(inp.WORKLOADS[4].shape, n_layers=2, d_model=512, n_heads=4, n_kv_heads=2, d_ffn=640,
                              vocab=3001, seed=22), 136, 40, 64),
    # full config-2 model (8 layers, vocab 32000)
    "cfg2-full": (SMALL, 384, 128, 32),
}


def _state(shape, N, block_start, L, seed, n_committed):
    rng = np.random.default_rng(seed)
    t = np.full(N, shape.mask_id, dtype=np.int32)
    t[:block_start] = inp.draw_prompt(shape.vocab, block_start, seed)
    idx = rng.choice(L, size=n_committed, replace=False)
    t[block_start + idx] = rng.integers(0, shape.vocab - 1, size=n_committed)
    return t


def _margins(z, mask_id):
    z = z.copy()
    z[:, mask_id] = -np.inf
    part = np.partition(z, -2, axis=-1)
    return part[:, -1] - part[:, -2]


def oracle_reference(host, t, block_start, L, calibrate=False):
    """What the oracle says about one sequence: (top1, conf, exact logits, bf16-operand logits or None)."""
    o_top1, o_conf, z = orc.forward_confidence(host, t, block_start, L, return_logits=True)
    z_b = orc.block_logits(host, t, block_start, L, operands="bf16") if calibrate else None
    return o_top1, o_conf, z, z_b


def check_sequence(ref, logits, top1, conf, t, mask_id, block_start, L, tol_logits, label):
    """One sequence's HIP outputs (logits [L, V], top1 [L], conf [L]) against oracle_reference's.  Returns
    (max-abs logit error, tolerance used, near-tie rows, mismatches outside near-ties but inside the logit band).

    With bf16-operand logits in `ref` the tolerance is calibrated by the oracle alone.  That is for the 4096-wide
    configurations, where bf16 arithmetic itself cannot hold 2e-2: the logits have a standard deviation of 1.3
    there, and the fp64 evaluation of the network with bf16-rounded contraction operands (the oracle's
    operands="bf16") already differs from exact arithmetic by 5e-2 (2 layers) to 1.3e-1 (32 layers) max-abs.  The
    HIP logits may then be at most 1.5x (max-abs) and 1.25x (rms) as far from the exact logits as that
    bf16-operand evaluation is."""
    from tests.gpu_common import say
    o_top1, o_conf, z, z_b = ref
    err = np.abs(logits - z).max()
    if z_b is not None:
        inherent, inherent_rms = np.abs(z_b - z).max(), np.sqrt(np.mean((z_b - z) ** 2))
        rms = np.sqrt(np.mean((logits - z) ** 2))
        say(f"[forward] {label}: HIP vs exact oracle max-abs {err:.3e} rms {rms:.3e}; bf16-operand oracle vs exact "
            f"max-abs {inherent:.3e} rms {inherent_rms:.3e}; HIP vs bf16-operand oracle max-abs {np.abs(logits - z_b).max():.3e}")
        assert rms <= 1.25 * inherent_rms, f"{label}: logits rms error {rms:.3e} > 1.25 x {inherent_rms:.3e}"
        tol_logits = 1.5 * inherent
    assert err <= tol_logits, f"{label}: logits max-abs error {err:.3e} > {tol_logits}"
    blk = t[block_start: block_start + L]
    masked = blk == mask_id
    # sentinels
    assert (top1[~masked] == blk[~masked]).all()
    assert (conf[~masked] == -1.0).all()
    margin = _margins(z, mask_id)
    near_ties = int((masked & (margin < 1e-3)).sum())
    # a mismatch must stay within the band that the logit tolerance implies (2 * tol below the top)
    differ = masked & (top1 != o_top1)
    wide = 0
    for j in np.nonzero(differ)[0]:
        gap = z[j, o_top1[j]] - z[j, top1[j]]
        assert gap <= 2 * tol_logits, f"{label}: top-1 mismatch with oracle logit gap {gap:.3e}"
        wide += int(margin[j] >= 1e-3)
    # such mismatches are the tail of the logit noise: a handful per block (measured 2 of 32 and 4 of 64 rows at full depth)
    assert wide <= max(2, int(masked.sum()) // 8), f"{label}: {wide} top-1 mismatches beyond near-ties among {int(masked.sum())} rows"
    safe = masked & ~differ
    assert (top1[masked] != mask_id).all()
    rel = np.abs(conf[safe] / o_conf[safe] - 1.0).max() if safe.any() else 0.0
    assert rel <= np.expm1(2 * tol_logits) + 1e-5, f"{label}: confidence off by {rel:.3e}"
    return err, tol_logits, near_ties, wide


def hip_forward(model, tokens_list, block_start, L):
    """(logits [S, L, V], top1 [S, L], conf [S, L]) of one batched HIP forward, on the host."""
    import paper_2605_15609_amd as psd
    from tests.gpu_common import to_dev
    d_tokens = to_dev(np.stack(tokens_list))
    logits = psd.psd_forward_logits(model, d_tokens, block_start, L).cpu().numpy().reshape(len(tokens_list), L, -1)
    top1, conf = psd.psd_forward_confidence(model, d_tokens, block_start, L)
    torch.cuda.synchronize()
    return logits, top1.cpu().numpy(), conf.cpu().numpy()


def _compare(model, host, tokens_list, block_start, L, tol_logits, label, check=None, calibrate=False):
    """GPU forward over all of tokens_list in one batch; the oracle runs (and is compared) on the sequences
    listed in `check` (default: all)."""
    from tests.gpu_common import say
    logits, top1, conf = hip_forward(model, tokens_list, block_start, L)
    worst, near_ties, wide, tol = 0.0, 0, 0, tol_logits
    for s, t in enumerate(tokens_list):
        if check is not None and s not in check:
            continue
        ref = oracle_reference(host, t, block_start, L, calibrate)
        err, tol, nt, wd = check_sequence(ref, logits[s], top1[s], conf[s], t, host.shape.mask_id, block_start, L, tol_logits,
                                          f"{label} seq {s}")
        worst, near_ties, wide = max(worst, err), near_ties + nt, wide + wd
    say(f"[forward] {label}: logits max-abs err {worst:.3e} (tol {tol:.3e}), near-tie rows (margin < 1e-3): {near_ties}, "
        f"mismatches beyond that but inside the logit band: {wide}")
    return worst


def test_fp32_debug_path_config1():
    from tests.gpu_common import make_models
    w = inp.WORKLOADS[1]
    host, model = make_models(w.shape, w.seq_len)
    states = [inp.initial_state(w)[0], _state(w.shape, w.seq_len, 16, 32, 5, 11)]
    _compare(model, host, states, 16, 32, 1e-4, "cfg1-fp32")


@pytest.mark.parametrize("d,heads,kv,dh,ffn,vocab,N,S", [(72, 3, 1, 16, 88, 101, 33, 3),      # partial tiles, 8-k chunks for some wavefronts only
                                                         (8, 1, 1, 8, 8, 33, 5, 1),            # one chunk: three wavefronts have nothing
                                                         (264, 4, 2, 64, 520, 300, 65, 2),     # more than eight chunks a wavefront
                                                         (36, 3, 1, 12, 48, 50, 20, 2)])       # K no multiple of 8: the general kernel
def test_fp32_contractions_at_the_edges_of_their_tiles(d, heads, kv, dh, ffn, vocab, N, S):
    from tests.gpu_common import make_models
    shape = inp.cut_down(inp.WORKLOADS[1].shape, d_model=d, n_heads=heads, n_kv_heads=kv, d_head=dh, d_ffn=ffn, vocab=vocab, seed=31)
    host, model = make_models(shape, N)
    L = min(12, N - 1)
    states = [_state(shape, N, N - L, L, 90 + s, s) for s in range(S)]
    _compare(model, host, states, N - L, L, 1e-4, f"fp32 d={d} N={N}")


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("plain", [7, 6, 5, 3, 0], ids=["all-plain", "mfma-gemm", "mfma-attn", "fused-head", "all-mfma"])
def test_bf16_paths(name, plain):
    from tests.gpu_common import make_models, say
    shape, N, bs, L = SHAPES[name]
    if name == "cfg2-full" and plain not in (7, 0):
        pytest.skip("full config 2 is checked on the all-plain and all-MFMA paths only")
    say(f"[forward] {name} plain_mask={plain}")
    host, model = make_models(shape, N)
    model.set_plain(plain)
    states = [_state(shape, N, bs, L, 1, 0), _state(shape, N, bs, L, 2, L // 3)]
    if name != "cfg2-full":
        states.append(_state(shape, N, bs, L, 3, L - 1))
    _compare(model, host, states, bs, L, 2e-2, f"{name}/mask{plain}")


@pytest.mark.parametrize("name,N", [("small-2l", 33), ("small-2l", 65), ("small-2l", 127), ("small-2l", 197), ("small-2l", 20),
                                    ("gqa-bias", 141), ("gqa-bias", 257), ("gqa-bias", 30)])
def test_sequences_of_no_round_length_run_on_the_matrix_core_attention(name, N):
    """Lengths that are no multiple of 8 or 16: partial query and key tiles at every edge (one past a tile, one short of it,
    less than one), several sequences so that a sequence's neighbours in memory must not leak into its last tile."""
    from tests.gpu_common import make_models
    shape, L = SHAPES[name][0], 12
    host, model = make_models(shape, N)
    states = [_state(shape, N, N - L, L, 70 + s, 4 * s) for s in range(3)]
    _compare(model, host, states, N - L, L, 2e-2, f"{name} N={N}")


@pytest.mark.parametrize("name", ["small-2l", "gqa-bias"])
@pytest.mark.parametrize("N,S", [(9, 3), (31, 2), (33, 1), (63, 4), (70, 3), (127, 1), (197, 5), (1271, 1), (1273, 1), (2543, 1), (2545, 1)])
def test_sequences_of_no_round_length_keep_the_plain_kernels_bits(name, N, S):
    """fp32 probabilities and every sum in the plain kernel's order: logits of the product path equal those with the plain
    attention kernel (bit 1 of the debug mask) bit for bit.  Lengths around tiles of 16 and 32 keys and queries, around the
    64 partial sums, and on both sides of the two lengths where the scores of 32 and of 16 queries stop fitting LDS."""
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev
    shape, L = SHAPES[name][0], 8
    _, model = make_models(shape, N)
    d = to_dev(np.stack([_state(shape, N, N - L, L, 60 + s, s) for s in range(S)]))
    out = {}
    for mask in (0, 2):
        model.set_plain(mask)
        out[mask] = psd.psd_forward_logits(model, d, N - L, L).cpu().numpy()
    model.set_plain(0)
    assert np.isfinite(out[0]).all() and (out[0] == out[2]).all(), f"{(out[0] != out[2]).mean():.3f} of the logits differ"


@pytest.mark.parametrize("name,N,S", [("small-2l", 192, 1), ("small-2l", 48, 11), ("small-2l", 384, 4), ("gqa-bias", 144, 1),
                                      ("gqa-bias", 272, 5), ("gqa-bias", 1280, 2)])
def test_rotary_and_value_transpose_in_the_qkv_epilogue_change_no_bit(name, N, S):
    """The QKV projection applies the rotary embedding and stores V transposed from its own epilogue; bit 3 of the debug mask
    asks for the older form (plain store, then a second kernel over the output).  Both must give the same logits bit for
    bit -- the rounding points are the same -- for head widths 64 and 128, with and without biases and grouped KV heads,
    for tiles that hold several sequences (N = 48), ragged last tiles, and rows past one tile."""
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev, say
    shape = SHAPES[name][0]
    L = 16
    bs = N - 2 * L
    host, model = make_models(shape, N)
    states = np.stack([_state(shape, N, bs, L, 40 + s, (3 * s) % L) for s in range(S)])
    d = to_dev(states)
    out = {}
    for mask in (0, 8):
        model.set_plain(mask)
        out[mask] = psd.psd_forward_logits(model, d, bs, L).cpu().numpy()
    model.set_plain(0)
    assert np.isfinite(out[0]).all()
    assert (out[0] == out[8]).all(), f"{name} N={N} S={S}: max difference {np.abs(out[0] - out[8]).max():.3e}"
    # and the result is the model's: one sequence against the oracle
    z = orc.block_logits(host, states[S - 1], bs, L)
    err = float(np.abs(out[0].reshape(S, L, -1)[S - 1] - z).max())
    say(f"[forward] fused QKV epilogue {name} N={N} S={S}: bit-identical to the two-pass form; max-abs logit error vs oracle {err:.3e}")
    assert err < 2e-2


@pytest.mark.parametrize("name,N,S", [("small-2l", 197, 5), ("small-2l", 77, 11), ("small-2l", 1285, 1), ("gqa-bias", 331, 3), ("gqa-bias", 133, 16)])
def test_rotary_in_the_qkv_epilogue_of_odd_lengths_changes_no_bit(name, N, S):
    """Lengths that are no multiple of 8: the projection rotates q and k in its epilogue and leaves V row-major, for the attention that
    reads it so; bit 3 asks for the plain store and the separate rotary launch.  Sequences begin anywhere inside a tile."""
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev
    shape = SHAPES[name][0]
    L = 16
    bs = N - 2 * L
    host, model = make_models(shape, N)
    d = to_dev(np.stack([_state(shape, N, bs, L, 140 + s, (3 * s) % L) for s in range(S)]))
    out = {}
    for mask in (0, 8):
        model.set_plain(mask)
        out[mask] = psd.psd_forward_logits(model, d, bs, L).cpu().numpy()
    model.set_plain(0)
    assert np.isfinite(out[0]).all() and (out[0] == out[8]).all()


@pytest.mark.parametrize("d_model", [128, 320, 512, 576])
@pytest.mark.parametrize("N,S", [(40, 1), (72, 3)])
def test_norms_of_narrow_models(d_model, N, S):
    """Rows of up to 512 values are normed by a wavefront each, four to a workgroup (40 and 216 rows, a batch of 3 and the last layer's
    48 block rows), wider ones by a workgroup: logits against the oracle, and a sequence does not depend on its neighbours."""
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev
    shape = inp.cut_down(inp.WORKLOADS[2].shape, n_layers=2, d_model=d_model, n_heads=d_model // 64, n_kv_heads=d_model // 64, d_ffn=192, vocab=997,
                         seed=91)
    L = 16
    bs = N - 2 * L
    host, model = make_models(shape, N)
    states = np.stack([_state(shape, N, bs, L, 160 + s, s) for s in range(S)])
    z = psd.psd_forward_logits(model, to_dev(states), bs, L).cpu().numpy().reshape(S, L, -1)
    for s in range(S):
        assert float(np.abs(z[s] - orc.block_logits(host, states[s], bs, L)).max()) < 2e-2
        assert (psd.psd_forward_logits(model, to_dev(states[s: s + 1]), bs, L).cpu().numpy().reshape(L, -1) == z[s]).all()


@pytest.mark.parametrize("vocab", [128, 997, 5000, 66001])
def test_head_in_tiles(vocab):
    """The head over 32 to 192 hidden rows (each width of a tile, whole and partial): few ids in tiles of 128, one tile and ragged last ones,
    many in tiles of 256.  Against the softmax of the call's own logits, which another kernel computes from the same hidden rows: two fp32 sums
    of 512 products differ by at most 2 * 512 * 2^-24 * sum |y w| < 1e-3 (the sum is about 15), and a logit error of e changes a
    probability by a factor exp(2 e) at most.  And a sequence's bits do not depend on how many stand in the call."""
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev
    shape = inp.cut_down(SMALL, n_layers=2, vocab=vocab, seed=93)
    N, bs, L = 64, 32, 32
    host, model = make_models(shape, N)
    states = np.stack([_state(shape, N, bs, L, 170 + s, (3 * s) % 8) for s in range(6)])
    first = None
    for S in (1, 2, 3, 4, 5, 6):
        d = to_dev(states[:S])
        top1, conf = (x.cpu().numpy().reshape(S, L) for x in psd.psd_forward_confidence(model, d, bs, L))
        z = psd.psd_forward_logits(model, d, bs, L).cpu().numpy().reshape(S, L, -1).astype(np.float64)
        z[..., shape.mask_id] = -np.inf
        p = np.exp(z - z.max(-1, keepdims=True))
        p = p.max(-1) / p.sum(-1)
        masked = states[:S, bs: bs + L] == shape.mask_id
        assert (np.abs(conf - p) <= np.expm1(2e-3) * p)[masked].all() and (conf == -1)[~masked].all()
        assert (np.take_along_axis(z, top1[..., None], -1)[..., 0] >= z.max(-1) - 2e-3)[masked].all()
        if first is None:
            first = top1[0], conf[0]
        assert (top1[0] == first[0]).all() and (conf[0] == first[1]).all()


@pytest.mark.parametrize("d_model", [2048, 4160])
def test_head_streamed_in_the_model(d_model):
    """Models whose head is streamed from the packed copy up to 128 rows (65 025 ids and more): copy, the final norm's second output and the merge, for
    8 to 128 rows, and the switch to tiles at 160 and 192 on the same handle; the whole-sequence call and the block rows against an approximate
    cache.  Against the head on the plain kernel (debug bit 2) over the same hidden rows, a row's logit being off by at most 2 * d * 2^-24 * sum |y w|
    between the two (the sum is about d * 0.64 * 0.02), and a logit error of e changing a probability by a factor exp(2 e)."""
    import ctypes as C
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev
    shape = inp.cut_down(SMALL, n_layers=1, d_model=d_model, n_heads=4, n_kv_heads=4, d_head=64, d_ffn=128, vocab=65100, seed=95)
    N, L = 64, 32
    host, model = make_models(shape, N)
    e = 2 * d_model * 2.0 ** -24 * d_model * 0.64 * 0.02 * 1.5
    states = np.stack([_state(shape, N, 32, L, 180 + s, (3 * s) % 8) for s in range(6)])
    ids, width = C.c_int32(), C.c_int32()
    for S, bs, n in ((1, 40, 8), (1, 32, L), (2, 32, L), (3, 32, L), (4, 32, L), (5, 32, L), (6, 32, L)):
        streamed = model.lib.psd_debug_head_plan(S * n, shape.vocab, d_model, C.byref(ids), C.byref(width))
        assert streamed == (S * n <= 128)
        d = to_dev(states[:S])
        cache = psd.KvCache(model, S, N - n) if n % 16 == 0 else None
        calls = [lambda: psd.psd_forward_confidence(model, d, bs, n)]
        if cache is not None:
            psd.psd_forward_confidence_approx(model, d, bs, n, cache, refresh=True)
            calls.append(lambda: psd.psd_forward_confidence_approx(model, d, bs, n, cache, refresh=False))
        for call in calls:
            top1, conf = (x.cpu().numpy() for x in call())
            model.set_plain(4)
            p_top1, p_conf = (x.cpu().numpy() for x in call())
            model.set_plain(0)
            masked = states[:S, bs: bs + n] == shape.mask_id
            assert masked.any() and (conf[~masked] == -1).all() and (top1[~masked] == p_top1[~masked]).all()
            assert (np.abs(conf - p_conf) <= (np.expm1(2 * e) + 1e-5) * p_conf)[masked].all()
            assert (top1 == p_top1)[masked].mean() > 0.95     # (a near tie may fall either way)


@pytest.mark.parametrize("name,N,S", [("small-2l", 96, 5), ("gqa-bias", 272, 3)])
def test_qkv_epilogue_on_every_tile_configuration(name, N, S):
    """The same comparison with every workgroup tile forced in turn (the forced tile serves all contractions of both runs):
    every instantiation of the rotary / transpose epilogue that a shape can reach is run, ragged last tiles included."""
    import paper_2605_15609_amd as psd
    from paper_2605_15609_amd import binding as B
    from tests.gpu_common import make_models, to_dev, say
    lib = B.load_library()
    shape = SHAPES[name][0]
    L = 16
    bs = N - 2 * L
    host, model = make_models(shape, N)
    states = np.stack([_state(shape, N, bs, L, 60 + s, (5 * s) % L) for s in range(S)])
    d = to_dev(states)
    reference = None
    try:
        for tile in range(lib.psd_kernel_gemm_tile_count()):
            lib.psd_debug_force_gemm_tile(tile)
            out = {}
            for mask in (0, 8):
                model.set_plain(mask)
                out[mask] = psd.psd_forward_logits(model, d, bs, L).cpu().numpy()
            assert (out[0] == out[8]).all(), f"{name} tile {tile}: max difference {np.abs(out[0] - out[8]).max():.3e}"
            # a sequence's sums do not depend on the tile either
            if reference is None:
                reference = out[0]
            assert (out[0] == reference).all(), f"{name}: tile {tile} changes the logits"
    finally:
        lib.psd_debug_force_gemm_tile(-1)
        model.set_plain(0)
    say(f"[forward] fused QKV epilogue {name}: bit-identical on all {lib.psd_kernel_gemm_tile_count()} tile configurations")


@pytest.mark.parametrize("heads,kv_heads", [(32, 32), (60, 12)], ids=["cut-at-v", "cut-inside-k"])
def test_qkv_projection_in_two_launches_changes_no_bit(heads, kv_heads):
    """2048 rows whose 256x256 tiles are one whole round and a part of one: the columns behind the whole round run as a launch
    of their own.  The cut falls on the first V column, or on a k head with both k and V columns behind it."""
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev
    N, S, L = 512, 4, 16
    shape = inp.cut_down(inp.WORKLOADS[4].shape, n_layers=1, d_model=512, n_heads=heads, n_kv_heads=kv_heads, d_ffn=640, vocab=3001,
                         seed=23)
    assert shape.d_head == 128 and 256 < S * N // 256 * ((heads + 2 * kv_heads) * 128 // 256) < 512
    host, model = make_models(shape, N)
    cut = model.lib.psd_debug_qkv_cut(S * N, (heads + 2 * kv_heads) * 128, 512, 128, (heads + kv_heads) * 128, N)
    assert cut == 8192 and (cut == (heads + kv_heads) * 128 if heads == 32 else heads * 128 < cut < (heads + kv_heads) * 128)
    d = to_dev(np.stack([_state(shape, N, N - 2 * L, L, 80 + s, 5 * s) for s in range(S)]))
    out = {}
    for mask in (0, 8):
        model.set_plain(mask)
        out[mask] = psd.psd_forward_logits(model, d, N - 2 * L, L).cpu().numpy()
    model.set_plain(0)
    assert np.isfinite(out[0]).all() and (out[0] == out[8]).all()


def test_batched_forward_equals_single(monkeypatch):
    """Batching S sequences must not change any sequence's (top1, conf) by more than rounding
    of the tile schedule; the decisions of the all-MFMA path must agree exactly here."""
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev
    shape, N, bs, L = SHAPES["small-2l"]
    host, model = make_models(shape, N)
    states = np.stack([_state(shape, N, bs, L, s, s * 3) for s in range(5)])
    t_all, c_all = psd.psd_forward_confidence(model, to_dev(states), bs, L)
    for s in range(5):
        t1, c1 = psd.psd_forward_confidence(model, to_dev(states[s: s + 1]), bs, L)
        assert (t1[0] == t_all[s]).all()
        assert torch.allclose(c1[0], c_all[s], rtol=1e-5, atol=0)


def test_logit_scale_is_applied_inside_the_fused_head():
    import paper_2605_15609_amd as psd
    from tests.gpu_common import make_models, to_dev
    shape, N, bs, L = SHAPES["small-2l"]
    shape = dataclasses.replace(shape, logit_scale=6.0)
    host, model = make_models(shape, N)
    t = _state(shape, N, bs, L, 4, 5)
    top1, conf = psd.psd_forward_confidence(model, to_dev(t[None]), bs, L)
    o_top1, o_conf, z = orc.forward_confidence(host, t, bs, L, return_logits=True)
    masked = t[bs: bs + L] == shape.mask_id
    safe = masked & (_margins(z, shape.mask_id) >= 6e-3)
    assert (top1[0].cpu().numpy()[safe] == o_top1[safe]).all()
    rel = np.abs(conf[0].cpu().numpy()[safe] / o_conf[safe] - 1).max()
    assert rel < np.expm1(2 * 6 * 2e-2)
