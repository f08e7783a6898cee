"""The C-ABI library loads and exports every symbol that include/psd.h declares (CPU only)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    import paper_2605_15609_amd as psd
    if not os.path.exists(psd.library_path()):
        from paper_2605_15609_amd import build
        build.build()
    return psd.load_library()


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "psd.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(psd_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = declared_symbols()
    assert {"psd_forward_confidence", "psd_select_unmask", "psd_build_drafts", "psd_verify_accept",
            "psd_decode_block"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


def test_structure_layouts_agree_with_the_binding(lib):
    from paper_2605_15609_amd import binding as B
    n = lib.psd_struct_sizes(None, 0)
    got = (ctypes.c_int32 * n)()
    assert lib.psd_struct_sizes(got, n) == n == 8
    assert list(got) == [ctypes.sizeof(t) for t in (B._Config, B._Weights, B._Policy, B._Graph, B._Stats, B._Work, B._GraphScore,
                                                    B._DebugLayout)]
    assert got[2] == 24 and got[6] == 40           # psd_policy: float + 5 x int32; psd_graph_score: 3 doubles + 2 x int64


def test_host_only_entry_points(lib):
    import paper_2605_15609_amd as psd
    assert lib.psd_status_string(0) == b"ok" and lib.psd_status_string(-3).startswith(b"workspace")
    g = psd.chain_graph(4)
    assert g.rank_sets == (0, 1, 3, 7)
    assert psd.chain_graph(3, 2).rank_sets == (0, 3, 15)
    with pytest.raises(psd.PsdError):
        psd.chain_graph(40)
    # subset lattice: every subset of the top ranks exactly once, root first, by size
    import itertools
    for depth in range(0, 6):
        sets = psd.lattice_graph(depth).rank_sets
        want = [sum(1 << r for r in c) for n in range(depth + 1) for c in itertools.combinations(range(depth), n)]
        assert sorted(sets) == sorted(want) and len(sets) == 2 ** depth and sets[0] == 0
        assert [bin(x).count("1") for x in sets] == sorted(bin(x).count("1") for x in sets)
    with pytest.raises(psd.PsdError):
        psd.lattice_graph(6)
    assert lib.psd_decode_scratch_bytes(1, 512, 32, 4) > 4 * 512 * 4
    assert lib.psd_decode_scratch_bytes(0, 512, 32, 4) < 0


def test_workspace_and_work_accounting(lib):
    import psd_inputs as inp
    from paper_2605_15609_amd.binding import _Config, _Work
    s = inp.WORKLOADS[3].shape
    cfg = _Config(s.n_layers, s.d_model, s.n_heads, s.n_kv_heads, s.d_head, s.d_ffn, s.vocab, s.mask_id, s.rms_eps, 0, 1,
                  1.0, 512)
    small = lib.psd_workspace_bytes(ctypes.byref(cfg), 1, 512, 32)
    big = lib.psd_workspace_bytes(ctypes.byref(cfg), 4, 512, 32)
    assert 0 < small < big < 2 ** 33
    w = _Work()
    assert lib.psd_forward_work(ctypes.byref(cfg), 4, 512, 32, ctypes.byref(w)) == 0
    # config 3 verify call: ~28.6 TFLOP of layer contractions, 1.036 GB LM-head weights
    assert abs(w.gemm_flops / 28.59e12 - 1) < 0.01
    assert abs(w.attn_flops / 0.55e12 - 1) < 0.01
    assert abs(w.head_bytes / 1.037e9 - 1) < 0.01
    bad = _Config(2, 100, 4, 4, 25, 256, 300, 299, 1e-5, 0, 1, 1.0, 64)
    assert lib.psd_workspace_bytes(ctypes.byref(bad), 1, 32, 8) < 0


def test_the_binding_rejects_tensors_the_library_would_misread(lib):
    """The library reads raw pointers: rotary tables handed over as bf16 would be read as fp32 (garbage, and past
    the end of the tensor).  Model checks dtype and extent of every tensor before psd_create."""
    import numpy as np
    import torch
    import psd_inputs as inp
    from paper_2605_15609_amd import binding as B
    shape = inp.cut_down(inp.WORKLOADS[2].shape, n_layers=1, vocab=512)
    host = inp.draw_model(shape, 64)

    def tensors(rope_dtype=torch.float32, max_seq=64):
        mat = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(torch.bfloat16)
        vec = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(torch.float32)
        t = {"tok_emb": mat(host.tok_emb), "lm_head": mat(host.lm_head), "final_norm": vec(host.final_norm),
             "rope_cos": torch.from_numpy(host.rope_cos[:max_seq]).to(rope_dtype), "rope_sin": torch.from_numpy(host.rope_sin[:max_seq]).to(rope_dtype)}
        lt = {k: (None if v is None else (mat(v) if v.ndim == 2 else vec(v))) for k, v in host.layers[0].items()}
        B.pack_qkv(lt)
        return t, [lt]

    t, layers = tensors(rope_dtype=torch.bfloat16)
    with pytest.raises(B.PsdError, match="rope_cos"):
        B.Model(shape, 64, t, layers, device="cpu")
    t, layers = tensors(max_seq=32)                 # tables shorter than max_seq
    with pytest.raises(B.PsdError, match="rope_cos"):
        B.Model(shape, 64, t, layers, device="cpu")
    t, layers = tensors()
    layers[0]["wo"] = layers[0]["wo"].float()        # a matrix in the wrong dtype
    with pytest.raises(B.PsdError, match="layer 0 wo"):
        B.Model(shape, 64, t, layers, device="cpu")


def _no_gpu_model(psd, lib, d_model, d_ffn):
    """A Model without a handle or device: what the binding computes before the library call."""
    from paper_2605_15609_amd import binding as B
    m = object.__new__(psd.Model)
    m.lib, m.handle = lib, None
    m.cfg = B._Config(2, d_model, 8, 8, 64, d_ffn, 5000, 4999, 1e-5, 0, 1, 1.0, 4096, 1)
    return m


def test_prefill_of_an_empty_batch_is_refused_by_the_library(lib):
    import torch
    import paper_2605_15609_amd as psd
    m = _no_gpu_model(psd, lib, 512, 1408)
    for shape, n_prompt, L in (((0, 64), 32, 16), ((1, 64), 32, 0), ((1, 64), 32, -16)):
        with pytest.raises(psd.PsdError):
            psd.psd_kv_prefill(m, torch.zeros(shape, dtype=torch.int32), n_prompt, L, None)


def test_prefill_workspace_is_bounded_and_falls_back_to_one_block(lib, monkeypatch):
    import types
    import torch
    import paper_2605_15609_amd as psd
    from paper_2605_15609_amd import binding as B
    for d, f in ((512, 1408), (4096, 12288)):
        m = _no_gpu_model(psd, lib, d, f)
        for batch, n_prompt, L in ((1, 0, 16), (1, 16, 16), (1, 4080, 48), (3, 1024, 32), (16, 4096, 64), (500, 64, 64)):
            rows = B._prefill_rows(m, batch, n_prompt, L)
            assert rows % L == 0 and L <= rows <= max(L, n_prompt)
            need = lib.psd_workspace_bytes(ctypes.byref(m.cfg), batch, rows, L)
            assert need > 0 and (rows == L or (need <= B.PREFILL_WORKSPACE and batch * rows <= B.PREFILL_ROWS))
    # an allocation that fails: one block at a time, as small as the call ever was
    seen, passed = [], []

    def workspace(n_bytes):
        seen.append(n_bytes)
        if len(seen) == 1:
            raise torch.cuda.OutOfMemoryError("no memory")
        return torch.empty(1, dtype=torch.uint8)

    m = _no_gpu_model(psd, lib, 512, 1408)
    m.workspace = workspace
    m.lib = types.SimpleNamespace(psd_workspace_bytes=lib.psd_workspace_bytes, psd_kv_prefill=lambda *a: passed.append(a[-2]) or 0)
    monkeypatch.setattr(B, "_stream", lambda: None)
    cache = types.SimpleNamespace(mem=torch.empty(1, dtype=torch.uint8), capacity=64)
    psd.psd_kv_prefill(m, torch.zeros((1, 64), dtype=torch.int32), 64, 16, cache)
    assert seen[1] < seen[0] and passed == [seen[1]] == [lib.psd_workspace_bytes(ctypes.byref(m.cfg), 1, 16, 16)]


def test_head_plan(lib):
    """129 - 192 hidden rows: a second column of tiles, which fetches the matrix again, only where both columns together are one round of the 256
    CUs.  Up to 192 rows the ids of a tile do not depend on the number of rows (the order in which a row's exponentials are added)."""
    ids, width = ctypes.c_int32(), ctypes.c_int32()
    for vocab in (100, 5000, 16384, 16385, 32000, 50304, 65024, 65025, 73728, 128256, 256000):
        for d in (64, 512, 1536, 2048, 4096, 8192):
            seen = set()
            for rows in (1, 32, 33, 64, 65, 128, 129, 160, 192):
                assert lib.psd_debug_head_plan(rows, vocab, d, ctypes.byref(ids), ctypes.byref(width)) in (0, 1)
                seen.add(ids.value)
                tiles, columns = -(-vocab // ids.value), -(-rows // width.value)
                if rows > 128:
                    assert columns == 1 or tiles * columns <= 256, (vocab, d, rows)
            assert len(seen) == 1
    assert lib.psd_debug_head_plan(0, 5000, 512, ctypes.byref(ids), ctypes.byref(width)) < 0


def test_head_plan_of_many_rows(lib):
    """Above 192 hidden rows: tiles of 256 rows only where they give more than half of the 256 CUs work."""
    ids, width = ctypes.c_int32(), ctypes.c_int32()
    widths = set()
    for vocab in (100, 4096, 8192, 16000, 32768, 32769, 50304, 126464, 152064):
        for rows in (193, 256, 257, 384, 768, 8192):
            assert lib.psd_debug_head_plan(rows, vocab, 4096, ctypes.byref(ids), ctypes.byref(width)) == 0
            widths.add(width.value)
            assert width.value == (256 if -(-vocab // 256) * -(-rows // 256) > 128 else 128), (vocab, rows)
    assert widths == {128, 256}


def test_head_plan_of_narrow_models(lib):
    """65 - 128 rows, up to 1536 wide: tiles that share a CU where one tile to a CU would leave less than half of the CUs with a second one."""
    ids, width = ctypes.c_int32(), ctypes.c_int32()
    for vocab in (65025, 65536, 65537, 73728, 98304, 98305, 128256):
        for d in (64, 1536, 1600, 2048):
            for rows in (65, 128):
                assert lib.psd_debug_head_plan(rows, vocab, d, ctypes.byref(ids), ctypes.byref(width)) in (0, 1)
                assert width.value == (64 if d <= 1536 and 65536 < vocab <= 98304 else 128), (vocab, d, rows)


def test_read_ahead_is_for_launches_of_up_to_2048_rows(lib):
    """The rows of a contraction's last launch decide: a cut may leave it few of many (6684 x 12288 SwiGLU: 540 rows, 128 CUs to spare)."""
    rows, cols, cut, ahead = ctypes.c_int64(), ctypes.c_int64(), 0, 0
    for M in (160, 512, 768, 1024, 1671, 2048, 2049, 2304, 4000, 5000, 6143, 6144, 6684, 8192, 20480):
        for nout, kin, epi in ((12288, 4096, 3), (4096, 12288, 2), (4096, 4096, 2), (18944, 3584, 3), (3584, 18944, 2), (12288, 4096, 0), (4608, 3584, 1)):
            wgs = lib.psd_debug_gemm_ahead(M, nout, kin, epi)
            assert lib.psd_debug_gemm_cut(M, nout, kin, epi, ctypes.byref(rows), ctypes.byref(cols)) == 0
            assert 0 <= wgs < 256 and (wgs == 0 or 0 < M - rows.value <= 2048), (M, nout, kin, epi)
            cut += wgs > 0 and rows.value > 0
            ahead += wgs > 0
    assert cut >= 1 and ahead >= 10
    assert lib.psd_debug_gemm_ahead(6684, 12288, 4096, 3) == 128


def test_read_ahead_leaves_the_last_level_cache_to_the_launch(lib):
    """Where the last round of tiles fetches so many weights itself that 200 MB would be exceeded, nothing is read ahead; a short last round fetches few."""
    for M, nout, kin, epi in ((136, 6144, 24576, 2), (136, 18432, 6144, 0), (384, 14336, 4096, 3), (136, 18432, 7168, 3)):
        assert lib.psd_debug_gemm_ahead(M, nout, kin, epi) == 0, (M, nout, kin, epi)
    for M, nout, kin, epi in ((136, 4096, 12288, 2), (136, 2048, 8192, 2), (768, 18944, 3584, 3), (768, 25600, 5120, 3)):
        assert lib.psd_debug_gemm_ahead(M, nout, kin, epi) > 0, (M, nout, kin, epi)


def test_a_contraction_in_two_launches_has_a_number_of_its_own(lib):
    """Not that of the tile it would run on in one launch; its name gives both tiles."""
    rows, cols = ctypes.c_int64(), ctypes.c_int64()
    count, seen = lib.psd_kernel_gemm_tile_count(), 0
    tiles = [lib.psd_kernel_gemm_tile_name(t).decode() for t in range(count)]
    assert len(set(tiles)) == count
    for M in (200, 512, 1000, 1024, 1671, 2048, 5000, 6144, 6684, 20480):
        for nout, kin, epi in ((12288, 4096, 3), (4096, 12288, 2), (4096, 4096, 2), (18944, 3584, 3), (3584, 18944, 2), (12288, 4096, 0)):
            assert lib.psd_debug_gemm_cut(M, nout, kin, epi, ctypes.byref(rows), ctypes.byref(cols)) == 0
            number = lib.psd_debug_gemm_plan(M, nout, kin, epi, None)
            name = lib.psd_kernel_gemm_tile_name(number).decode()
            if rows.value or cols.value:
                seen += 1
                assert number > count and name.startswith("two launches, ")
                assert any(name == f"two launches, {a} and {b}" for a in tiles[:2] for b in tiles), name
            else:
                assert 0 <= number < count and name == tiles[number]
            if kin == 4096:
                assert lib.psd_kernel_gemm_tile(M, nout, epi) == number
    assert seen >= 5


@pytest.mark.parametrize("shape,rows,into_cache,fused", [
    ((4608, 3584, 128, 4096), (16, 32, 64, 96), (0, 1), 0), ((4608, 3584, 128, 4096), (112, 128, 144, 512), (0, 1), 1),     # 28 / 4 heads
    ((6144, 4096, 128, 5120), (16, 96), (0, 1), 0), ((7168, 5120, 128, 6144), (32, 96), (0, 1), 0), ((10240, 8192, 128, 9216), (16, 64), (0, 1), 0),
    ((12288, 4096, 128, 8192), (80, 96), (0, 1), 1), ((12288, 4096, 128, 8192), (16, 64), (0,), 0), ((15360, 5120, 128, 10240), (80, 96), (1,), 1),
    ((3072, 1024, 64, 2048), (16, 96), (0, 1), 1), ((1536, 512, 64, 1024), (16, 96), (0, 1), 1), ((5120, 4096, 64, 4608), (48, 96), (0, 1), 1),
    ((18432, 6144, 64, 12288), (16, 48, 64), (0,), 0), ((9216, 6144, 64, 7680), (80, 96), (0, 1), 1)])
def test_few_rows_of_the_qkv_projection_take_the_faster_form(lib, shape, rows, into_cache, fused):
    """As measured on both forms; what is within a microsecond or two of level is not listed."""
    nout, kin, d_head, v_start = shape
    for M in rows:
        for cache in into_cache:
            assert lib.psd_debug_qkv_fused(M, nout, kin, d_head, v_start, 16, cache) == fused, (M, cache)
