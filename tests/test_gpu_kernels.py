"""Parity of each HIP kernel (through the C ABI) against the CPU oracle, element by element.

Tolerances:
  bf16 GEMM / attention   2e-2 * max(|ref| over the row, sigma)  (the bound for bf16 logits)
  fp32 GEMM / attention   1e-4 * max(|ref| over the row)          (fp32 accumulation over K <= 4096)
  fp32 statistics         1e-5 * max(1, |ref|), KL additionally 1e-5 * sum p |log p - log p'|
  decisions               exact where the oracle's margin exceeds 1e-4 (boundary) / 1e-5 (selection)
"""
import numpy as np
import pytest
import torch

from oracle import boundary as o_boundary
from oracle import forward as o_fwd
from oracle import select as o_select
from oracle import stats as o_stats
from paper_2604_15750_amd import api, inputs

pytestmark = pytest.mark.gpu


def _np(t):
    return inputs.tensor_to_numpy(t)


def _rowtol(ref, rel, floor=0.0):
    return rel * np.maximum(np.abs(ref).max(axis=-1, keepdims=True), floor)


# ---- GEMM ----------------------------------------------------------------------------------------
@pytest.mark.parametrize("M,N,K", [(1, 32, 32), (7, 64, 96), (16, 128, 128), (64, 4096, 4096), (100, 160, 4096 + 64),
                                   (192, 1024, 1536), (300, 96, 512), (33, 12288, 256),
                                   # 65 .. 160 rows: the mid kernel (every row-tile count; wide matrices with 128- and 96-column groups and a ragged
                                   # last group; narrow ones with and without a K split; k ranges that leave wavefronts idle)
                                   (65, 4096, 4096), (81, 24576, 512), (97, 4096, 1024), (112, 12288, 2048), (113, 4096, 12288),
                                   (136, 12288, 4096), (150, 8224, 1024), (160, 4096, 4096), (80, 126464, 64), (144, 64, 96),
                                   (161, 4096, 4096), (200, 1024, 2048), (225, 4096, 12288), (256, 4096, 512),
                                   (17, 16384, 256), (19, 4128, 416), (47, 8192, 480), (64, 4128, 3584), (40, 24576, 1024), (33, 4096, 8192), (64, 256, 12288), (8, 4608, 3584), (16, 6144, 512),
                                   # more than 256 rows: the macro-tile kernel (ragged rows, column tails, both weight packings, short K)
                                   (257, 4096, 4096), (513, 8224, 1024), (700, 160, 4096 + 64), (1100, 640, 64), (384, 12288, 32),
                                   # ... with 192 x 192 tiles
                                   (368, 24576, 256), (700, 12288, 128)])
def test_gemm_bf16(device, M, N, K):
    g = torch.Generator(device="cpu").manual_seed(M * 7 + N + K)
    x = torch.randn(M, K, generator=g).to(torch.bfloat16).to(device)
    w = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16).to(device)
    y = api.dlm_gemm_nt(x, w)
    torch.cuda.synchronize()
    ref = o_fwd.matmul_nt(_np(x), _np(w))
    got = o_fwd.widen(_np(y))
    assert (np.abs(got - ref) <= _rowtol(ref, 2e-2, 0.05 * np.sqrt(K))).all(), np.abs(got - ref).max()
    # the output is the bf16 rounding of an fp32 accumulation: far tighter on average
    assert np.abs(got - ref).mean() <= 4e-3 * np.abs(ref).mean() + 1e-6


# One shape for every tile the macro GEMM's planner has for more than 32 rows, each with a ragged last row block, a ragged last
# column block, an odd number of k-tiles (13: more than the pipeline has stages) and rows that are no multiple of 16; and K splits
# of three and four ways, whose workgroups hand their partial tiles to the last arriver, run twice (the tickets reset themselves).
# Each with the tile and the split that it is there for.  (The statistics epilogue's tiles: test_statistics_of_every_head_tile.)
MACRO_TILE_SHAPES = [
    ((209, 96, 416), (64, 64, 1)), ((97, 8320, 416), (64, 96, 1)), ((17, 32864, 416), (64, 160, 1)), ((259, 10976, 416), (64, 256, 1)),
    ((130, 12224, 416), (96, 128, 1)), ((259, 16608, 416), (96, 256, 1)), ((70, 12704, 416), (128, 64, 1)), ((129, 8704, 416), (128, 96, 1)),
    ((97, 24768, 416), (128, 128, 1)), ((68, 33088, 416), (128, 160, 1)), ((17, 40992, 416), (128, 192, 1)), ((199, 24672, 416), (128, 256, 1)),
    ((129, 24928, 416), (160, 128, 1)), ((291, 16448, 416), (160, 192, 1)), ((133, 16448, 416), (192, 96, 1)), ((164, 24896, 416), (192, 160, 1)),
    ((161, 41024, 416), (192, 192, 1)), ((387, 16640, 416), (256, 192, 1)), ((257, 24608, 416), (256, 256, 1)),
    ((97, 66400, 416), (128, 320, 1)),
    # ... in a single row block, where most copies of W are non-temporal
    ((19, 49216, 416), (32, 256, 1)), ((19, 65632, 2592), (32, 320, 1)), ((51, 49184, 416), (64, 256, 1)), ((51, 65632, 2592), (64, 320, 1)),
    ((83, 49184, 416), (96, 256, 1)), ((115, 49184, 416), (128, 256, 1)), ((147, 40992, 416), (160, 192, 1)), ((243, 32800, 416), (256, 192, 1)),
    ((243, 49184, 416), (256, 256, 1)),
    ((300, 160, 4128), (64, 64, 3)), ((264, 96, 4128), (64, 64, 4)), ((290, 4064, 8224), (96, 128, 2))]
# ... and the mid kernel's: (rows, columns of a group, split); both sides of every row count at which choose_kernel leaves it
MID_SHAPES = [
    ((17, 16480, 416), (32, 96, 1)), ((17, 24768, 416), (32, 128, 1)), ((64, 24608, 512), (64, 128, 1)), ((48, 24544, 512), (48, 96, 1)),
    ((65, 12288, 256), (80, 48, 1)), ((80, 12288, 256), (80, 48, 1)), ((81, 12288, 256), (96, 48, 1)), ((96, 12256, 416), (96, 48, 1)),
    ((128, 4096, 8224), (128, 64, 4)), ((208, 4096, 992), (208, 32, 1))]
BEYOND_MID = [(97, 12288, 256), (129, 4096, 8224), (209, 4096, 992)]


@pytest.mark.parametrize("M,N,K", [s for s, _ in MACRO_TILE_SHAPES + MID_SHAPES] + BEYOND_MID)
def test_gemm_macro_tiles(device, M, N, K):
    g = torch.Generator(device="cpu").manual_seed(M + N + K)
    x = torch.randn(M, K, generator=g).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16)
    xd, wd = x.to(device), w.to(device)
    y = api.dlm_gemm_nt(xd, wd)
    again = api.dlm_gemm_nt(xd, wd)
    torch.cuda.synchronize()
    ref = o_fwd.matmul_nt(_np(x), _np(w))
    got = o_fwd.widen(_np(y))
    # bf16 rounding of an fp32 sum of exact products (half converts these values exactly): 2^-9 relative, plus K roundings of
    # 2^-24 of partial sums that grow like the result's scale
    bound = 2.0 ** -8 * np.abs(ref) + K * 2.0 ** -24 * 0.05 * np.sqrt(K)
    assert (np.abs(got - ref) <= bound).all(), (np.abs(got - ref) / bound).max()
    assert torch.equal(y, again)


@pytest.mark.parametrize("rows,N,K", [((512, 1345), 4096, 12288), ((796,), 384, 2080), ((653,), 5504, 3616)])
def test_gemm_k_in_two_parts(device, rows, N, K):
    """K summed in two parts by two workgroups or by one: the same order, so the rows that two launches share are equal bit for bit.
    The narrow shapes have an odd number of k-tiles, most of which the first part gets.  Bound as in test_gemm_macro_tiles."""
    g = torch.Generator(device=device).manual_seed(N + K)
    x = torch.randn(max(rows), K, generator=g, device=device).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g, device=device) * 0.05).to(torch.bfloat16)
    ref = torch.cat([x.double() @ w[lo:lo + 512].double().t() for lo in range(0, N, 512)], -1)
    got = []
    for M in rows:
        p = api.plan_gemm(M, N, K, "sum")
        assert p["kernel"] == "macro" and p["k_parts"] == 2 and p["splits"] == (2 if M == 512 else 1), p
        y = api.dlm_gemm_nt(x[:M].contiguous(), w)
        torch.cuda.synchronize()
        assert ((y.double() - ref[:M]).abs() <= 2.0 ** -8 * ref[:M].abs() + K * 2.0 ** -24 * 0.05 * K ** 0.5).all()
        got.append(y)
    assert all(torch.equal(y[:rows[0]], got[0]) for y in got)


@pytest.mark.parametrize("M", [8, 100, 300])
def test_gemm_operand_conversion_at_the_ends_of_halfs_range(device, M):
    """A bf16 model's matrix-core operands are IEEE half.  Weights far below half's smallest normal number (2^-14) land on its
    subnormal grid: each keeps an absolute error of at most 2^-25.  Activations beyond half's largest number saturate at
    +-65504 instead of becoming infinite.  Everything in between converts exactly (covered by test_gemm_bf16)."""
    N, K = 256, 512
    g = torch.Generator(device="cpu").manual_seed(M)
    x = torch.randn(M, K, generator=g).to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g) * 2.0 ** -17).to(torch.bfloat16)  # most of them subnormal in half, many below its resolution
    y = api.dlm_gemm_nt(x.to(device), w.to(device))
    torch.cuda.synchronize()
    ref = o_fwd.matmul_nt(_np(x), _np(w))
    got = o_fwd.widen(_np(y))
    bound = 2.0 ** -25 * np.abs(o_fwd.widen(_np(x))).sum(-1, keepdims=True) + 2.0 ** -8 * np.abs(ref) + 1e-12
    assert (np.abs(got - ref) <= bound).all(), (np.abs(got - ref) / bound).max()
    assert np.abs(ref).max() > 0 and np.abs(got).max() > 0.25 * np.abs(ref).max()  # (not flushed to zero)
    # saturation: one activation per row far beyond 65504
    x2 = x.clone()
    x2[:, 3] = 3.0e5
    w2 = (torch.randn(N, K, generator=g) * 0.05).to(torch.bfloat16)
    y2 = api.dlm_gemm_nt(x2.to(device), w2.to(device))
    torch.cuda.synchronize()
    got2 = o_fwd.widen(_np(y2))
    assert np.isfinite(got2).all()
    xc = o_fwd.widen(_np(x2)).clip(-65504.0, 65504.0)
    ref2 = xc @ o_fwd.widen(_np(w2)).T
    assert (np.abs(got2 - ref2) <= _rowtol(ref2, 2e-2)).all()


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (5, 7, 3), (64, 128, 128), (130, 1024, 384), (67, 384, 129)])
def test_gemm_f32(device, M, N, K):
    g = torch.Generator(device="cpu").manual_seed(M + N + K)
    x = torch.randn(M, K, generator=g).to(device)
    w = torch.randn(N, K, generator=g).to(device)
    y = api.dlm_gemm_nt(x, w)
    torch.cuda.synchronize()
    ref = o_fwd.matmul_nt(_np(x), _np(w))
    assert (np.abs(_np(y) - ref) <= _rowtol(ref, 1e-5, 1.0)).all()


# ---- attention -----------------------------------------------------------------------------------
@pytest.mark.parametrize("dt,A,T,nq,nkv,hd", [
    ("f32", 1, 1, 1, 1, 32), ("f32", 8, 72, 4, 4, 32), ("f32", 37, 101, 4, 2, 64), ("f32", 64, 320, 8, 2, 128),
    ("bf16", 8, 264, 4, 4, 128), ("bf16", 64, 320, 8, 8, 128), ("bf16", 50, 700, 28, 4, 128), ("bf16", 192, 448, 4, 1, 128),
    # head dims of 64 and 32 (a head's output dims split over two workgroups / not split), and enough (tile, head) pairs that
    # nothing is split (4 x 32, 40 x 16)
    ("bf16", 24, 300, 4, 2, 64), ("bf16", 9, 77, 8, 8, 32), ("bf16", 64, 200, 32, 8, 128), ("bf16", 640, 640, 16, 4, 128),
])
def test_attention(device, dt, A, T, nq, nkv, hd):
    tdt = torch.float32 if dt == "f32" else torch.bfloat16
    g = torch.Generator(device="cpu").manual_seed(A * 3 + T)
    q = (torch.randn(A, nq, hd, generator=g) * 1.5).to(tdt).to(device)
    k = (torch.randn(T, nkv, hd, generator=g) * 1.5).to(tdt).to(device)
    v = torch.randn(T, nkv, hd, generator=g).to(tdt).to(device)
    out = api.dlm_attention(q, k, v)
    torch.cuda.synchronize()
    ref = o_fwd.attention(_np(q), _np(k), _np(v))
    got = o_fwd.widen(_np(out))
    tol = 1e-5 if dt == "f32" else 2e-2
    assert (np.abs(got - ref) <= tol * np.maximum(np.abs(ref).max(-1, keepdims=True), 0.1)).all(), np.abs(got - ref).max()


# Two query tiles per workgroup: narrow (split output dims) and wide, each head dim, an odd number of tiles (a workgroup whose second
# tile does not exist), a last tile with one row, key counts at the ends of a 32-key block and fewer blocks than wavefronts.
@pytest.mark.parametrize("A,T,nq,nkv,hd", [(49, 33, 28, 4, 128), (64, 31, 28, 4, 128), (33, 64, 30, 30, 128), (520, 97, 16, 4, 128), (513, 32, 16, 16, 128),
                                           (520, 65, 16, 8, 64), (529, 95, 16, 16, 32), (515, 1, 16, 2, 64)])
def test_attention_pairs_of_query_tiles(device, A, T, nq, nkv, hd):
    g = torch.Generator(device="cpu").manual_seed(A + T + nq)
    q = (torch.randn(A, nq, hd, generator=g) * 1.5).to(torch.bfloat16)
    k = (torch.randn(T, nkv, hd, generator=g) * 1.5).to(torch.bfloat16)
    v = torch.randn(T, nkv, hd, generator=g).to(torch.bfloat16)
    out = api.dlm_attention(q.to(device), k.to(device), v.to(device))
    torch.cuda.synchronize()
    ref = o_fwd.attention(_np(q), _np(k), _np(v))
    got = o_fwd.widen(_np(out))
    # the output rounded to bf16 (2^-9), the probabilities to half (2^-12 each, weighted by them) and fp32 sums
    bound = 2.0 ** -8 * np.abs(ref) + 2.0 ** -11 * float(v.abs().max())
    assert (np.abs(got - ref) <= bound).all(), (np.abs(got - ref) / bound).max()


# ... of eight wavefronts, where one tile each would leave a second workgroup per compute unit: each head dim, odd tiles, fewer key
# blocks than wavefronts, the last of them with one key
@pytest.mark.parametrize("A,T,nq,nkv,hd", [(161, 97, 28, 4, 128), (152, 792, 28, 4, 128), (145, 257, 30, 10, 64), (257, 33, 16, 16, 32)])
def test_attention_pairs_of_query_tiles_with_eight_wavefronts(device, A, T, nq, nkv, hd):
    assert api.plan_attention(A, 1, nq, hd) == dict(waves=8, shares=1, tiles=2)
    test_attention_pairs_of_query_tiles(device, A, T, nq, nkv, hd)


# ---- vocabulary statistics -------------------------------------------------------------------------
def _check_stats(got, ref, z64, zp64, mask_id):
    for key in ("max_logit", "lse", "entropy", "conf"):
        r = ref[key]
        assert (np.abs(got[key].cpu().numpy() - r) <= 1e-5 * np.maximum(1.0, np.abs(r))).all(), key
    assert (got["argmax"].cpu().numpy() == ref["argmax"]).all()
    if zp64 is not None:
        logp, _, _ = o_stats.log_softmax_masked(z64, mask_id)
        logq, _, _ = o_stats.log_softmax_masked(zp64, mask_id)
        keep = np.arange(z64.shape[1]) != mask_id
        spread = np.sum(np.exp(logp[:, keep]) * np.abs(logp[:, keep] - logq[:, keep]), axis=-1)
        r = ref["kl"]
        assert (np.abs(got["kl"].cpu().numpy() - r) <= 1e-5 * np.maximum(1.0, np.abs(r)) + 1e-5 * spread).all()
    else:
        assert (got["kl"].cpu().numpy() == 0).all()


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,V,mask_id", [(1, 8, 7), (3, 1024, 1023), (5, 1001, 17), (64, 126464, 126463), (300, 4096, 0), (9, 152064, 152063)])
@pytest.mark.parametrize("with_prev", [False, True])
def test_vocab_stats(device, dt, rows, V, mask_id, with_prev):
    tdt = torch.float32 if dt == "f32" else torch.bfloat16
    z = torch.from_numpy(inputs.peaked_logits(rows, V, rows + V, [(0, min(5, V - 2), 30.0)])).to(tdt)
    z[:, mask_id] = 50.0  # a huge logit on the mask token must not matter
    if rows > 2:
        z[2, :] = 1.25  # a flat row: argmax ties go to the lowest id
    zp = None
    if with_prev:
        zp = (z.float() + 0.5 * torch.from_numpy(inputs.peaked_logits(rows, V, 99 + rows))).to(tdt)
        if rows > 1:
            zp[1] = z[1]  # identical rows: KL = 0
    got = api.dlm_vocab_stats(z.to(device), mask_id, None if zp is None else zp.to(device))
    torch.cuda.synchronize()
    z64 = o_fwd.widen(_np(z))
    zp64 = None if zp is None else o_fwd.widen(_np(zp))
    ref = o_stats.vocab_stats(z64, mask_id, zp64)
    _check_stats(got, ref, z64, zp64, mask_id)
    if with_prev and rows > 1:
        assert abs(got["kl"][1].item()) <= 1e-6
    if with_prev:  # the previous rows' log-sum-exp handed in (what dlm_step keeps with the retained logits) instead of recomputed
        lse_prev = api.dlm_vocab_stats(zp.to(device), mask_id)["lse"]
        got2 = api.dlm_vocab_stats(z.to(device), mask_id, zp.to(device), prev_lse=lse_prev)
        torch.cuda.synchronize()
        _check_stats(got2, ref, z64, zp64, mask_id)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,V", [(95, 16640), (96, 16640), (97, 8199), (256, 32776), (257, 32776),
                                    (135, 16640), (136, 16640), (137, 8199), (136, 4104), (160, 4096)])
def test_vocab_stats_whole_rows(device, dt, rows, V):
    """The edges of the row counts at which one workgroup takes a whole row; vocabularies with whole trips, a ragged end, and no
    16-byte vectors; the mask token in the first, a middle and the last trip.  Tolerances as test_vocab_stats derives them."""
    tdt = torch.float32 if dt == "f32" else torch.bfloat16
    z = torch.from_numpy(inputs.peaked_logits(rows, V, rows + V, [(rows - 1, V - 2, 30.0)])).to(tdt)
    zp = (z.float() + 0.5 * torch.from_numpy(inputs.peaked_logits(rows, V, 99 + rows))).to(tdt)
    for mask_id, prev in ((0, zp), (V // 2, None), (V - 1, zp)):
        zm = z.clone()
        zm[:, mask_id] = 50.0
        got = api.dlm_vocab_stats(zm.to(device), mask_id, None if prev is None else prev.to(device))
        torch.cuda.synchronize()
        z64, zp64 = o_fwd.widen(_np(zm)), None if prev is None else o_fwd.widen(_np(prev))
        _check_stats(got, o_stats.vocab_stats(z64, mask_id, zp64), z64, zp64, mask_id)


# ... and many rows, a workgroup of 256 threads per chunk: chunks of whole trips, with a ragged end of one vector, of less than a
# trip, and without vectors
@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("rows,V", [(351, 12296), (352, 12288), (353, 12296), (352, 8199), (1023, 4104), (1024, 8200)])
def test_vocab_stats_whole_rows_of_many(device, dt, rows, V):
    test_vocab_stats_whole_rows(device, dt, rows, V)


def _walked_kl_sum(x, threads, chunks, vec):
    """Sum of the columns of x [rows, V] in the order of the streamed statistics, in fp32: a row is cut into `chunks` runs of whole strides
    (`threads` lanes of `vec` consecutive columns); a lane adds its columns of a chunk one by one; 64 lanes are added by a butterfly
    (32, 16, .. 1 apart), the wavefronts of a workgroup in order, and the chunks by a butterfly of 64 places again."""
    rows, V = x.shape
    stride = threads * vec
    chunk = -(-(-(-V // chunks)) // stride) * stride
    n = -(-V // chunk)
    wide = np.zeros((rows, n * chunk), np.float32)  # (columns past the end add zeros)
    wide[:, :V] = x
    wide = wide.reshape(rows, n, chunk // stride, threads, vec)
    lanes = np.zeros((rows, n, threads), np.float32)
    for s in range(chunk // stride):
        for i in range(vec):
            lanes = lanes + wide[:, :, s, :, i]

    def butterfly(v):
        for o in (32, 16, 8, 4, 2, 1):
            v = v + v[..., np.arange(64) ^ o]
        return v[..., 0]

    waves = butterfly(lanes.reshape(rows, n, threads // 64, 64))
    parts = waves[..., 0]
    for w in range(1, threads // 64):
        parts = parts + waves[..., w]
    if n == 1:
        return parts[:, 0]
    return butterfly(np.concatenate([parts, np.zeros((rows, 64 - n), np.float32)], axis=1))


@pytest.mark.parametrize("dt,rows,V", [("bf16", 2, 126464), ("bf16", 200, 126464), ("bf16", 340, 126464), ("bf16", 352, 126464), ("bf16", 400, 126464),
                                       ("bf16", 600, 126464), ("bf16", 1100, 126464), ("bf16", 1600, 126464), ("bf16", 352, 12296),
                                       ("f32", 3, 30000), ("f32", 150, 30000), ("f32", 360, 30000), ("f32", 1030, 30000), ("f32", 1700, 30000),
                                       # five workgroups of 256 threads on each compute unit, six, more than six; fp32: six, seven, more
                                       ("bf16", 1280, 4096), ("bf16", 1281, 4096), ("bf16", 384, 126464), ("bf16", 1537, 8200),
                                       ("f32", 768, 30000), ("f32", 350, 30000), ("f32", 1793, 2048)])
def test_order_of_the_streamed_sums(device, dt, rows, V):
    """KL is w / s - lse + lse' with w = sum e^(z - m) (z - z').  On a flat row every exponential is one and s a whole number, so that w is a
    plain fp32 sum whose value says in which order it was taken; values of z' whose sum cancels make that show.  Bit for bit."""
    tdt, vec = (torch.bfloat16, 8) if dt == "bf16" else (torch.float32, 4)
    g = torch.Generator(device="cpu").manual_seed(rows + V)
    base = (torch.randn(3, V, generator=g) * 1.0e6).to(tdt)
    z = torch.full((rows, V), 1.25, dtype=tdt, device=device)
    zp = base.to(device)[torch.arange(rows, device=device) % 3]
    mask_id = V // 3
    got = api.dlm_vocab_stats(z, mask_id, zp, prev_lse=torch.zeros(rows, device=device))
    torch.cuda.synchronize()
    x = np.float32(1.25) - base.float().numpy()
    x[:, mask_id] = 0.0
    # a workgroup of 1024 threads per row at 136 .. 256 rows, else chunks of 256 threads for about 1536 workgroups
    threads, chunks = (1024, 1) if 136 <= rows <= 256 else (256, max(1, min(-(-1536 // rows), -(-V // (512 * vec)), 32)))
    w = _walked_kl_sum(x, threads, chunks, vec)
    lse = _np(got["lse"])
    want = (w / np.float32(V - 1))[np.arange(rows) % 3] - lse
    assert (_np(got["kl"]) == want).all(), np.abs(_np(got["kl"]) - want).max()


# Whole rows with the next trip's loads in flight and without: bf16 from 153 rows on (193 where the previous rows' log-sum-exp is
# recomputed) and fp32 with any previous row, or from 201 rows on, wait for each trip.  Whole trips and ragged ends, one and an even and an odd number of them
@pytest.mark.parametrize("dt,few,rows", [("bf16", 152, 153), ("bf16", 136, 256), ("bf16", 192, 193), ("f32", 200, 201), ("f32", 136, 256)])
@pytest.mark.parametrize("V", [16384, 24584, 50000, 65536])
def test_whole_rows_a_trip_ahead_or_not(device, dt, few, rows, V):
    """A row's values are the same bits by either kernel, compared or not, wherever the mask token lies; and a sample against 64 bits."""
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(rows + V)
    z = (torch.randn(rows, V, generator=g, device=device) * 4).to(tdt)
    zp = (z.float() + 0.5 * torch.randn(rows, V, generator=g, device=device)).to(tdt)
    at = [0, few // 2, few - 1]
    for mask_id in (0, V // 2, V - 1):
        lse_prev = api.dlm_vocab_stats(zp, mask_id)["lse"]
        for prev, lse in ((None, None), (zp, lse_prev), (zp, None)):
            head = lambda t: None if t is None else t[:few].contiguous()  # noqa: E731
            part, got = api.dlm_vocab_stats(z[:few], mask_id, head(prev), prev_lse=head(lse)), api.dlm_vocab_stats(z, mask_id, prev, prev_lse=lse)
            torch.cuda.synchronize()
            for k, v in part.items():
                assert torch.equal(got[k][:few], v), (mask_id, k)
            z64, zp64 = o_fwd.widen(_np(z[at])), None if prev is None else o_fwd.widen(_np(zp[at]))
            _check_stats({k: v[at] for k, v in got.items()}, o_stats.vocab_stats(z64, mask_id, zp64), z64, zp64, mask_id)


@pytest.mark.parametrize("dt,rows,few", [("bf16", 360, 345), ("bf16", 500, 384), ("f32", 383, 308)])
@pytest.mark.parametrize("own_lse", [True, False])
def test_vocab_stats_of_many_rows_at_a_real_vocabulary(device, dt, rows, few, own_lse):
    """126464 tokens, compared with a previous row whose log-sum-exp is given or recomputed: a sample of rows against 64 bits, and every row
    bit for bit as in a call with fewer rows that are cut into as many chunks."""
    V, mask_id, tdt = 126464, 126463, torch.bfloat16 if dt == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(rows)
    z = (torch.randn(rows, V, generator=g, device=device) * 4).to(tdt)
    zp = (z.float() + 0.5 * torch.randn(rows, V, generator=g, device=device)).to(tdt)
    lse_prev = None if own_lse else api.dlm_vocab_stats(zp, mask_id)["lse"]
    got = api.dlm_vocab_stats(z, mask_id, zp, prev_lse=lse_prev)
    part = api.dlm_vocab_stats(z[:few], mask_id, zp[:few], prev_lse=None if own_lse else lse_prev[:few].contiguous())
    torch.cuda.synchronize()
    for k, v in part.items():
        assert torch.equal(got[k][:few], v), k
    at = [0, 1, 63, few - 1, few, rows - 1]
    z64, zp64 = o_fwd.widen(_np(z[at])), o_fwd.widen(_np(zp[at]))
    _check_stats({k: v[at] for k, v in got.items()}, o_stats.vocab_stats(z64, mask_id, zp64), z64, zp64, mask_id)


# ---- block_boundary ----------------------------------------------------------------------------------
@pytest.mark.parametrize("norm_mode", [0, 1, 2, 3])
@pytest.mark.parametrize("rule", [0, 1])
def test_block_boundary(device, norm_mode, rule):
    rng = np.random.default_rng(norm_mode * 2 + rule)
    for trial in range(6):
        n = int(rng.integers(1, 17))
        Ws = [int(rng.choice([1, 2, 5, 31, 64, 65, 128, 200, 256])) for _ in range(n)]
        off = np.concatenate([[0], np.cumsum(Ws)])
        I = (rng.exponential(0.3, off[-1]) * np.exp(-rng.uniform(0, 3, off[-1]))).astype(np.float32)
        H = rng.uniform(0.1, 6.0, off[-1]).astype(np.float32)
        if trial == 0:
            I[off[0]:off[1]] = 0.0  # identical steps in the first window
        cold = [int(rng.random() < 0.2) for _ in range(n)]
        lam = float(np.float32(rng.choice([0.6, 0.9, 1.0, 1.2, 1.6])))
        l_min, r = int(rng.integers(1, 12)), int(rng.integers(0, 4))
        L = torch.empty(n, dtype=torch.int32, device=device)
        S = torch.empty(int(off[-1]), dtype=torch.float32, device=device)
        mg = torch.empty(n, dtype=torch.float32, device=device)
        api.block_boundary(torch.from_numpy(I).to(device), torch.from_numpy(H).to(device), off[:-1].tolist(), Ws, L, lam, l_min, r, norm_mode,
                           rule, cold=cold, S_out=S, margin_out=mg)
        torch.cuda.synchronize()
        L, S, mg = L.cpu().numpy(), S.cpu().numpy(), mg.cpu().numpy()
        for b in range(n):
            sl = slice(off[b], off[b + 1])
            Lr, Sr, mr = o_boundary.block_boundary(I[sl], H[sl], lam, l_min, r, norm_mode, rule, cold_start=bool(cold[b]))
            assert (np.abs(S[sl] - Sr) <= 1e-5 * np.maximum(1.0, np.abs(Sr))).all()
            if mr > 1e-4:
                assert L[b] == Lr, (b, Ws[b], L[b], Lr, mr)
            assert min(l_min, Ws[b]) <= L[b] <= Ws[b]
            if np.isfinite(mr):
                assert abs(mg[b] - mr) <= 1e-5 * max(1.0, mr)


# Calls whose windows all fit one wavefront, which have a kernel of their own, and the first that does not: every normalisation and rule;
# a window that never crosses, one that does at once, one in between, identical steps
@pytest.mark.parametrize("norm_mode", [0, 1, 2, 3])
@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("Ws", [[1], [64, 64], [63, 64, 2], [32, 33, 64, 64, 64, 64, 5], [64, 65]])
def test_block_boundary_of_short_windows(device, norm_mode, rule, Ws):
    rng = np.random.default_rng(norm_mode * 2 + rule + 16 * len(Ws))
    n, off = len(Ws), np.concatenate([[0], np.cumsum(Ws)])
    I, H = rng.exponential(0.3, off[-1]).astype(np.float32), rng.uniform(0.1, 6.0, off[-1]).astype(np.float32)
    for b in range(n):  # S = I~ - lambda H~: how much larger than H the signal I is decides where it falls below zero
        sl = slice(off[b], off[b + 1])
        if b % 4 == 1:
            I[sl] = 2 * H[sl] + 1
        elif b % 4 == 2:
            I[sl] = H[sl] / 4
        elif b % 4 == 3:
            I[sl] = 0.5
    crossed = []
    for lam, l_min, r, cold in ((0.6, 1, 0, None), (0.9, 8, 1, [b % 5 == 4 for b in range(n)]), (1.6, 3, 3, None)):
        lam = float(np.float32(lam))
        L, S, mg = (torch.empty(k, dtype=t, device=device) for k, t in ((n, torch.int32), (int(off[-1]), torch.float32), (n, torch.float32)))
        api.block_boundary(torch.from_numpy(I).to(device), torch.from_numpy(H).to(device), off[:-1].tolist(), Ws, L, lam, l_min, r, norm_mode,
                           rule, cold=cold, S_out=S, margin_out=mg)
        torch.cuda.synchronize()
        for b in range(n):
            sl = slice(off[b], off[b + 1])
            Lr, Sr, mr = o_boundary.block_boundary(I[sl], H[sl], lam, l_min, r, norm_mode, rule, cold_start=bool(cold and cold[b]))
            # (S is an fp64 result rounded to fp32)
            assert (np.abs(_np(S)[sl] - Sr) <= 2.0 ** -23 * np.maximum(1.0, np.abs(Sr))).all(), (b, np.abs(_np(S)[sl] - Sr).max())
            if mr > 1e-9:
                assert L[b].item() == Lr, (b, Ws[b], L[b].item(), Lr, mr)
            if np.isfinite(mr):
                assert abs(mg[b].item() - mr) <= 2.0 ** -23 * max(1.0, mr) + 1e-9
            crossed.append(Lr < Ws[b])
    assert (any(crossed) and not all(crossed)) or Ws == [1]


# ---- select_parallel -----------------------------------------------------------------------------------
def _select_case(rng, L, V, dt):
    peaks = []
    for r in range(L):
        if rng.random() < 0.7:
            peaks.append((r, int(rng.integers(0, 6)), float(rng.uniform(4, 16))))
        if rng.random() < 0.5:
            peaks.append((r, int(rng.integers(0, 6)), float(rng.uniform(6, 12))))
    z = torch.from_numpy(inputs.peaked_logits(L, V, int(rng.integers(1 << 30)), peaks, sigma=2.0))
    return z.to(torch.float32 if dt == "f32" else torch.bfloat16)


@pytest.mark.parametrize("dt", ["f32", "bf16"])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_select_parallel(device, dt, mode):
    rng = np.random.default_rng(17 + mode)
    V, mask_id = 512, 511
    fired = dict(multi=0, fallback=0, dropped=0)
    for trial in range(12):
        n = int(rng.integers(1, 9))
        lens = [int(rng.choice([0, 1, 3, 8, 32, 64, 100, 256])) for _ in range(n)]
        pad = [int(rng.integers(0, 5)) for _ in range(n)]  # unrelated rows between blocks
        row_start, rows = [], 0
        for b in range(n):
            rows += pad[b]
            row_start.append(rows)
            rows += lens[b]
        rows = max(rows, 1)
        z = _select_case(rng, rows, V, dt)
        tokens = np.where(rng.random(rows) < 0.75, mask_id, 5).astype(np.int32)
        z64 = o_fwd.widen(_np(z))
        st = api.dlm_vocab_stats(z.to(device), mask_id)
        tok_d = torch.from_numpy(tokens).to(device)
        sel = torch.zeros(rows, dtype=torch.uint8, device=device)
        nsel = torch.empty(n, dtype=torch.int32, device=device)
        mg = torch.empty(n, dtype=torch.float32, device=device)
        tl, th, gm = float(np.float32(0.6)), float(np.float32(0.93)), float(np.float32(rng.choice([-4.0, -8.0, -16.0])))
        api.select_parallel(z.to(device), st["lse"], st["conf"], st["argmax"], tok_d, row_start, row_start, lens, mask_id, tl, th, gm,
                            mode, sel, nsel, apply_tokens=True, margin_out=mg)
        torch.cuda.synchronize()
        lse, conf, yh = st["lse"].cpu().numpy(), st["conf"].cpu().numpy(), st["argmax"].cpu().numpy()
        sel, nsel, mg, tok_after = sel.cpu().numpy(), nsel.cpu().numpy(), mg.cpu().numpy(), tok_d.cpu().numpy()
        expect_tok = tokens.copy()
        for b in range(n):
            sl = slice(row_start[b], row_start[b] + lens[b])
            ref, mr = o_select.select_parallel(z64[sl], lse[sl], conf[sl], yh[sl], tokens[sl] == mask_id, tl, th, gm, mode)
            if mr > 1e-5:
                assert (sel[sl].astype(bool) == ref).all(), (trial, b, lens[b], mr)
                assert nsel[b] == ref.sum()
                expect_tok[sl] = np.where(ref, yh[sl], tokens[sl])
                assert (tok_after[sl] == expect_tok[sl]).all()  # Eq. 2
                if np.isfinite(mr):
                    assert abs(mg[b] - mr) <= 1e-5 * max(1.0, mr) + 2e-6 * 20
            E = tokens[sl] == mask_id
            pool = E & (conf[sl] >= tl)
            fired["multi"] += int(ref.sum() > 1)
            fired["fallback"] += int(E.any() and not pool.any())
            fired["dropped"] += int((pool & ~ref).any())
        # rows outside every block are untouched
        outside = np.ones(rows, dtype=bool)
        for b in range(n):
            outside[row_start[b]: row_start[b] + lens[b]] = False
        assert (tok_after[outside] == tokens[outside]).all() and (sel[outside] == 0).all()
    assert fired["multi"] > 3 or mode == 2
    if mode == 0:
        assert fired["fallback"] > 0 and fired["dropped"] > 3, fired


# The rules without pair scores at the edges of the kernels' block sizes, beside a short and an empty block; confidences in ties
@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("L", [32, 33, 64, 65, 128, 129, 255, 256])
def test_select_parallel_without_pairs(device, mode, L):
    rng = np.random.default_rng(L + mode)
    V, mask_id, lens = 64, 63, [L, 5, 0]
    rows = sum(lens)
    conf = (rng.integers(1, 40, rows) / 41.0).astype(np.float32)
    y = rng.integers(0, V - 1, rows).astype(np.int32)
    tokens = np.where(rng.random(rows) < 0.7, mask_id, 5).astype(np.int32)
    tokens[0] = tokens[L] = mask_id
    high = float(np.float32(0.503))
    z = torch.zeros(rows, V, device=device)
    d = lambda x: torch.from_numpy(x.copy()).to(device)  # noqa: E731
    tok, sel, nsel = d(tokens), torch.zeros(rows, dtype=torch.uint8, device=device), torch.empty(3, dtype=torch.int32, device=device)
    api.select_parallel(z, torch.zeros(rows, device=device), d(conf), d(y), tok, [0, L, 0], [0, L, 0], lens, mask_id, 0.1, high, 0.0, mode, sel, nsel)
    torch.cuda.synchronize()
    for b, at in ((0, 0), (1, L)):
        sl = slice(at, at + lens[b])
        ref, _ = o_select.select_parallel(np.zeros((lens[b], V)), np.zeros(lens[b]), conf[sl], y[sl], tokens[sl] == mask_id, 0.1, high, 0.0, mode)
        assert (_np(sel)[sl].astype(bool) == ref).all() and nsel[b].item() == ref.sum(), b
        assert (_np(tok)[sl] == np.where(ref, y[sl], tokens[sl])).all()
    assert nsel[2].item() == 0


@pytest.mark.parametrize("L", [2, 31, 32, 33, 63, 64, 65, 255, 256])
def test_select_parallel_chain_of_conflicts(device, L):
    """Every row conflicts with its two neighbours and the confidences descend along the block: the greedy walk takes every other
    row, each decision depending on the one before it - the longest chain of rounds the kernel can meet, at the row counts
    where its bit words, wavefronts and workgroup sizes end."""
    V, mask_id = 1024, 1023
    z = torch.full((L, V), -10.0)
    y = torch.arange(L)
    z[y, y] = 30.0 - torch.arange(L) * 0.05
    z[y[1:], y[:-1]] = 16.0
    z[y[:-1], y[1:]] = 16.0
    conf = (0.9 - torch.arange(L) * 0.001).to(torch.float32)
    lse = torch.full((L,), 30.0)
    z64 = z.double().numpy()
    ref, margin = o_select.select_parallel(z64, lse.numpy(), conf.numpy(), y.numpy(), np.ones(L, dtype=bool), 0.5, 0.95, -30.0, 0)
    assert ref.sum() == (L + 1) // 2 and margin > 1e-5
    tok = torch.full((L,), mask_id, dtype=torch.int32, device=device)
    sel = torch.zeros(L, dtype=torch.uint8, device=device)
    nsel = torch.empty(1, dtype=torch.int32, device=device)
    mg = torch.empty(1, dtype=torch.float32, device=device)
    api.select_parallel(z.to(device), lse.to(device), conf.to(device), y.to(torch.int32).to(device), tok, [0], [0], [L], mask_id, 0.5, 0.95, -30.0, 0,
                        sel, nsel, margin_out=mg)
    torch.cuda.synchronize()
    assert (sel.cpu().numpy().astype(bool) == ref).all() and int(nsel) == ref.sum()
    assert abs(float(mg) - margin) <= 1e-6
    assert (tok.cpu().numpy() == np.where(ref, y.numpy(), mask_id)).all()


# ---- streams ---------------------------------------------------------------------------------------
def test_calls_run_on_the_current_stream(device, monkeypatch):
    """Both ways to ask for the current stream name it, inside and outside a stream context."""
    side = torch.cuda.Stream()
    for raw in (api._raw_stream, None):
        monkeypatch.setattr(api, "_raw_stream", raw)
        assert api._stream() == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(side):
            assert api._stream() == side.cuda_stream != torch.cuda.default_stream().cuda_stream


# ---- measurement helpers --------------------------------------------------------------------------
def test_probes_report_plausible_rates(device):
    """The two probes bench.py quotes rooflines against: a plain streaming read reaches most of, and no more than, the
    published 8 TB/s; the matrix-core loop (operands of pseudo-random values: power-limited) a good part of, and no more
    than, the published 2.5 PFLOP/s."""
    buf = torch.empty(1 << 30, dtype=torch.uint8, device=device)
    gbs = api.probe_hbm_read(buf, reps=5)
    tf = api.probe_mfma(reps=2)
    assert 3000 < gbs < 8000, gbs
    assert 1000 < tf < 2600, tf
    with pytest.raises(api.DlmError):
        api.probe_hbm_read(torch.empty(1 << 20, dtype=torch.uint8, device=device))
