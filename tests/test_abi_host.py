"""Host-only checks of the C ABI: the library loads, exports what include/dlm.h declares, and rejects bad arguments
before touching the GPU (no compute call is made here)."""
import ctypes as C
import os
import re

import numpy as np
import pytest
import torch

from paper_2604_15750_amd import api

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "dlm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dlm_\w+|block_boundary|select_parallel)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    L = api.lib()
    names = _declared()
    assert {"dlm_step", "block_boundary", "select_parallel", "dlm_model_create", "dlm_state_create"} <= set(names)
    for n in names:
        assert hasattr(L, n), n
    assert sorted(api.EXPORTS) == names


def test_struct_layouts_match_header():
    assert C.sizeof(api.dlm_config) == 11 * 4
    assert C.sizeof(api.dlm_weights) == 9 * 8
    assert C.sizeof(api.dlm_step_desc) == 8 + 18 * 8
    assert C.sizeof(api.dlm_boundary_params) == 20 and C.sizeof(api.dlm_select_params) == 16


def _err():
    return api.lib().dlm_last_error().decode()


def test_block_boundary_argument_errors():
    L = api.lib()
    one = C.c_void_p(16)  # never dereferenced: validation fails first
    p = api.dlm_boundary_params(1.2, 8, 1, 0, 0)
    z = (C.c_int32 * 1)(0)
    off = (C.c_int32 * 1)(4)
    call = lambda I=one, H=one, o=off, n=1, pp=p, Lo=one: L.block_boundary(I, H, z, o, None, n, C.byref(pp), Lo, None, None, None)
    assert call(I=None) == -1 and "null" in _err()
    assert call(Lo=None) == -1
    assert call(n=0) == -1
    assert call(n=33) == -3
    assert call(o=(C.c_int32 * 1)(0)) == -3 and "window" in _err()
    assert call(o=(C.c_int32 * 1)(257)) == -3
    for bad in (api.dlm_boundary_params(0.0, 8, 1, 0, 0), api.dlm_boundary_params(1.2, 0, 1, 0, 0),
                api.dlm_boundary_params(1.2, 8, -1, 0, 0), api.dlm_boundary_params(1.2, 8, 1, 4, 0),
                api.dlm_boundary_params(1.2, 8, 1, 0, 2)):
        assert call(pp=bad) == -1


def test_select_parallel_argument_errors():
    L = api.lib()
    one = C.c_void_p(16)
    p = api.dlm_select_params(0.8, 0.95, -16.0, 0)
    z = (C.c_int32 * 1)(0)
    bl = (C.c_int32 * 1)(8)

    def call(logits=one, vocab=100, dtype=1, n=1, pp=p, blen=bl, sel=one):
        return L.select_parallel(logits, vocab, dtype, one, one, one, one, z, z, blen, n, 99, C.byref(pp), 1, sel, one, None, None)

    assert call(logits=None) == -1 and call(sel=None) == -1
    assert call(n=0) == -1 and call(n=40) == -3
    assert call(dtype=2) == -1 and call(vocab=1) == -1
    assert call(pp=api.dlm_select_params(0.9, 0.8, -16.0, 0)) == -1 and "tau_high" in _err()
    assert call(pp=api.dlm_select_params(0.8, 0.95, -16.0, 3)) == -1
    assert call(blen=(C.c_int32 * 1)(257)) == -3 and call(blen=(C.c_int32 * 1)(-1)) == -3


def test_model_and_component_argument_errors():
    L = api.lib()
    one = C.c_void_p(16)
    h = C.c_void_p()
    cfg = api.dlm_config(2, 128, 4, 4, 32, 384, 1024, 1023, 0, 1e-5, 10000.0)
    assert L.dlm_model_create(C.byref(cfg), None, None, C.byref(h)) == -1
    w = api.dlm_weights()
    assert L.dlm_model_create(C.byref(cfg), C.byref(w), None, C.byref(h)) == -1 and "null weight" in _err()
    for field, val, code in (("dtype", 5, -1), ("head_dim", 48, -2), ("n_kv_heads", 3, -2), ("mask_id", 1024, -1), ("vocab", 1, -2)):
        bad = api.dlm_config(2, 128, 4, 4, 32, 384, 1024, 1023, 0, 1e-5, 10000.0)
        setattr(bad, field, val)
        assert L.dlm_model_create(C.byref(bad), C.byref(w), None, C.byref(h)) == code, field
    bf = api.dlm_config(2, 128, 4, 4, 32, 392, 1024, 1023, 1, 1e-5, 10000.0)  # d_ffn not a multiple of 32
    assert L.dlm_model_create(C.byref(bf), C.byref(w), None, C.byref(h)) == -2
    assert L.dlm_state_create(None, 1, 1, 1, 1, C.byref(h)) == -1
    assert L.dlm_step(None, None, None) == -1
    assert L.dlm_state_reset(None, 0) == -1 and L.dlm_state_kv_len(None, 0) == -1
    assert L.dlm_vocab_stats(None, None, None, 1, 8, 0, 7, one, one, one, one, one, one, one, 1 << 20, None) == -1
    assert L.dlm_vocab_stats(one, None, None, 0, 8, 0, 7, one, one, one, one, one, one, one, 1 << 20, None) == -3
    assert L.dlm_vocab_stats(one, None, None, 4, 8, 0, 7, one, one, one, one, one, one, one, 8, None) == -3 and "workspace" in _err()
    assert L.dlm_vocab_stats(one, None, None, 4, 8, 0, 8, one, one, one, one, one, one, one, 1 << 20, None) == -1
    # the entry point that allocates nothing: same checks, and a row limit set by its file-scope scratch
    assert L.dlm_vocab_stats_static(None, None, None, 1, 8, 0, 7, one, one, one, one, one, one, None) == -1
    assert L.dlm_vocab_stats_static(one, None, None, 0, 8, 0, 7, one, one, one, one, one, one, None) == -3
    assert L.dlm_vocab_stats_static(one, None, None, 4097, 8, 0, 7, one, one, one, one, one, one, None) == -3 and "4096" in _err()
    assert L.dlm_vocab_stats_static(one, None, None, 4, 8, 0, 8, one, one, one, one, one, one, None) == -1
    assert L.dlm_gemm_nt(one, one, one, 4, 48, 64, 1, None) == -2
    assert L.dlm_gemm_nt(one, None, one, 4, 64, 64, 1, None) == -1
    assert L.dlm_attention(one, one, one, one, 4, 4, 4, 3, 32, 0, None) == -2
    assert L.dlm_attention(one, one, one, one, 4, 4, 4, 2, 48, 0, None) == -2
    assert L.dlm_vocab_stats_workspace(0) == 0 and L.dlm_vocab_stats_workspace(64) > 0


def test_committed_traffic_summary_feeds_the_bench_line():
    """bench.py takes roofline.traffic of the default workload from the committed counter summary: it must hold both figures, and
    they must be within a few per cent of the kernel's algorithmic bytes (more would mean re-reads from HBM)."""
    import sys
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench
    t = bench.traffic_from_profile("llada8b_p256_g256")
    algorithmic = 2 * 24576 * 4096  # the gate/up weights of the 8B shape, bf16
    assert t is not None and 0.98 * algorithmic < t < 1.10 * algorithmic


@pytest.mark.parametrize("v", [[], [7], (0, -1, 2**31 - 1), list(range(64)), np.arange(5), np.arange(3, dtype=np.int16), torch.arange(4), [3.7, 2],
                               [True, False], [2**31 + 5, 2**40 + 1], np.array([1.5, 2.5]), torch.tensor([1.5, 2.0])])
def test_packed_host_arrays(v):
    """The bytes handed to the two decisions are those of a ctypes int32 array, for whatever that accepts; None stays None."""
    assert api._packed(v) == bytes(api._ints(v))
    assert api._packed(None) is None


def test_current_stream_without_torchs_private_query(monkeypatch):
    class Stream:
        cuda_stream = 0x1234
    monkeypatch.setattr(api, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", Stream)
    assert api._stream() == 0x1234


# ---- launch rules (host arithmetic) ---------------------------------------------------------------
@pytest.mark.parametrize("hd", [32, 64, 128])
@pytest.mark.parametrize("n_q", [1, 4, 16, 28, 32, 64])
def test_attention_takes_a_second_query_tile_only_where_a_span_has_one(n_q, hd):
    for n_seqs in (1, 2, 3, 4, 5, 8, 16, 24, 32):
        for rows in (1, 8, 15, 16, 17, 31, 32, 33, 37, 48, 64, 100, 512, 3072):
            p, tiles = api.plan_attention(rows, n_seqs, n_q, hd), (rows + 15) // 16
            assert p["tiles"] <= tiles, (n_seqs, rows, p)
            assert p["waves"] in (4, 8) and p["shares"] in ({32: (1,), 64: (1, 2), 128: (1, 4)}[hd])
            if p["shares"] == 4 and tiles > 1:  # a narrow pass: two tiles exactly where one would leave a second workgroup per compute unit
                assert (p["tiles"] == 2) == (tiles * n_q * n_seqs * 4 > 256)
            if p["waves"] == 4:
                assert p["tiles"] == min(tiles, 2)
    # spans of one tile: 3 sequences x 32 heads, 3 and 4 x 28 are more than 256 workgroups of one tile
    assert api.plan_attention(16, 3, 32, 128)["tiles"] == api.plan_attention(8, 4, 28, 128)["tiles"] == 1
    assert api.plan_attention(37, 1, 32, 128) == dict(waves=8, shares=4, tiles=2)


def test_attention_pairs_tiles_of_a_middling_pass_only_into_one_round():
    """Eight wavefronts and no shares: two tiles a workgroup where one each would be more than the chip's 256 and two are not."""
    for n_q in (4, 16, 28, 30, 32):
        for n_seqs in range(1, 33):
            for rows in range(1, 260, 3):
                p, tiles = api.plan_attention(rows, n_seqs, n_q, 128), (rows + 15) // 16
                if p["waves"] == 8 and p["shares"] == 1:
                    assert (p["tiles"] == 2) == (tiles > 1 and tiles * n_q * n_seqs > 256 and (tiles + 1) // 2 * n_q * n_seqs <= 256), (rows, n_seqs, n_q)
    assert api.plan_attention(40, 5, 32, 128)["tiles"] == api.plan_attention(72, 3, 32, 128)["tiles"] == 1
    assert api.plan_attention(48, 4, 32, 128)["tiles"] == api.plan_attention(240, 1, 32, 128)["tiles"] == 2


@pytest.mark.parametrize("dt,vec", [(torch.bfloat16, 8), (torch.float32, 4)])
def test_whole_row_statistics_only_where_they_save_a_merge_and_read_in_vectors(dt, vec):
    whole = set()
    for rows in (1, 8, 64, 95, 96, 97, 128, 135, 136, 137, 192, 255, 256, 257, 384, 3072):
        for vocab in (2, 8, 1000, 1001, 1024, 2048, 2056, 4096, 4104, 8199, 16640, 126463, 126464, 152064):
            p = api.plan_vocab_stats(rows, vocab, dt)
            assert p["threads"] in (256, 1024) and 1 <= p["chunks"] <= 32
            if vocab % vec or vocab <= 512 * vec:  # one scalar load in flight per lane; or one chunk, nothing to merge
                assert p["threads"] == 256, (rows, vocab)
            if vocab <= 512 * vec:
                assert p["chunks"] == 1
            if p["threads"] == 1024:
                assert p["chunks"] == 1
                whole.add(rows)
    assert whole == {136, 137, 192, 255, 256}


LAYER_SHAPES = [(12288, 4096, "qkv"), (4096, 4096, "resid"), (24576, 4096, "swiglu"), (4096, 12288, "resid"),  # an 8B model's layer
                (4608, 3584, "qkv"), (3584, 3584, "resid"), (37888, 3584, "swiglu"), (3584, 18944, "resid")]   # a 7B one's, grouped-query


@pytest.mark.parametrize("N,K,epi", LAYER_SHAPES)
def test_no_k_split_beyond_one_round_of_workgroups(N, K, epi):
    """A K split is there to fill idle compute units: its workgroups are never more than the 256 of them, at any row count, and where
    the order of a wide pass's sums asks for two parts of K beyond that, one workgroup keeps both.  Narrow matrices whose tiles fit
    one round of any kind take one."""
    for M in range(1, 3073, 7):
        p = api.plan_gemm(M, N, K, epi)
        assert p["splits"] == 1 or p["workgroups"] <= 256, (M, p)
        assert p["splits"] == p["k_parts"] or (p["splits"], p["k_parts"]) == (1, 2)
        if p["kernel"] == "macro" and N <= 4608 and M <= 2048:
            assert p["workgroups"] <= 256, (M, p)


def test_gated_launches_take_fewer_rounds_where_the_estimates_are_close():
    for M in (481, 500, 512):  # two rounds of 256 x 192, not three of 128 x 256
        p = api.plan_gemm(M, 37888, 3584, "swiglu")
        assert (p["rows"], p["cols"], p["workgroups"]) == (256, 192, 396), (M, p)


def test_paired_column_tiles_leave_the_skinny_kernel_at_17_rows():
    """Beyond 16 rows the skinny kernel is built for single column tiles only."""
    for M in (17, 24, 32, 33, 48, 49, 64, 65, 200, 384):
        for N in list(range(32, 60000, 32 * 17)) + [8192, 8224, 12288, 24576, 37888, 4608]:
            for K in (32, 512, 3584, 8192, 18944):
                for epi in ("qkv", "swiglu", "resid", "sum"):
                    p = api.plan_gemm(M, N, K, epi)
                    assert p["kernel"] != "skinny" or p["cols"] == 16, (M, N, K, epi)


@pytest.mark.parametrize("epi", ["direct", "sum", "qkv", "swiglu", "resid"])
def test_widest_tiles_serve_single_row_blocks(epi):
    """64 and 128 x 320: plain products whose rows are one block of such a tile, whatever the planner's estimates of the others."""
    seen = 0
    for N, K in ((152064, 3584), (66400, 416), (150336, 4096), (37888, 3584), (8192, 4096)):
        for M in range(1, 700, 3):
            p = api.plan_gemm(M, N, K, epi)
            if p["kernel"] == "macro" and p["cols"] == 320 and p["rows"] > 32:
                assert epi in ("direct", "sum") and M <= p["rows"] and p["workgroups"] == -(-N // 320), (M, N, K, p)
                seen += 1
    assert seen or epi not in ("direct", "sum")


def test_shapes_of_the_gpu_tests_reach_the_kernels_they_are_there_for():
    """A retuned planner must not leave a variant without a test."""
    import test_gpu_kernels as k
    import test_gpu_step as st
    tiles = set()
    for (M, N, K), want in k.MACRO_TILE_SHAPES:
        p = api.plan_gemm(M, N, K, "sum")
        assert (p["kernel"], p["rows"], p["cols"], p["splits"]) == ("macro", *want), ((M, N, K), p)
        tiles.add(want[:2])
    for (M, N, K), want in k.MID_SHAPES:
        p = api.plan_gemm(M, N, K, "sum")
        assert (p["kernel"], p["rows"], p["cols"], p["splits"]) == ("mid", *want), ((M, N, K), p)
    for s in k.BEYOND_MID:
        assert api.plan_gemm(*s, "sum")["kernel"] == "macro"
    for V, L, want in st.HEAD_TILES:
        p = api.plan_gemm(L, V, 256, "stats")
        assert (p["rows"], p["cols"]) == want, (V, L, p)
        tiles.add(want)
    for epi, want, M, dims in st.EPILOGUE_TILES:
        assert st.epilogue_tile(epi, M, dims) == want, (epi, M, dims)
    # single row blocks of more than 128 columns have instantiations of their own, which read W past the memory-side cache (the head's
    # products are tested as plain ones)
    alone = {("direct", want[:2]) for (M, _, _), want in k.MACRO_TILE_SHAPES if M <= want[0]} | {("stats", want) for _, L, want in st.HEAD_TILES if L <= want[0]} | \
        {(epi, want) for epi, want, M, _ in st.EPILOGUE_TILES if M <= want[0]}
    # every tile that any row count of a few shapes is given
    used = set()
    for N, K, epi in LAYER_SHAPES + [(126464, 4096, "direct"), (152064, 3584, "direct"), (126464, 4096, "stats"), (152064, 3584, "stats")]:
        for M in range(1, 65 if epi == "stats" else 3073, 5):
            p = api.plan_gemm(M, N, K, epi)
            if p["kernel"] == "macro":
                used.add((p["rows"], p["cols"]))
                assert M > p["rows"] or p["cols"] <= 128 or (epi, (p["rows"], p["cols"])) in alone, (epi, p)
    assert used <= tiles, used - tiles


def test_launch_rule_argument_errors():
    L = api.lib()
    out = (C.c_int32 * 7)()
    assert L.dlm_plan_gemm(8, 64, 64, 3, None) == -1 and L.dlm_plan_gemm(8, 64, 64, 6, out) == -1
    assert L.dlm_plan_gemm(8, 48, 64, 3, out) == -2 and L.dlm_plan_gemm(0, 64, 64, 3, out) == -2
    assert L.dlm_plan_vocab_stats(8, 1024, 0, None) == -1 and L.dlm_plan_vocab_stats(8, 1024, 2, out) == -1
    assert L.dlm_plan_vocab_stats(0, 1024, 0, out) == -2 and L.dlm_plan_vocab_stats(8, 1, 0, out) == -2
    assert L.dlm_plan_attention(8, 1, 32, 128, None) == -1
    assert L.dlm_plan_attention(0, 1, 32, 128, out) == -2 and L.dlm_plan_attention(8, 1, 32, 48, out) == -2
