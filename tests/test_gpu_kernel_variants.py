"""The kernel variants a call may be routed to, each at the sizes where it can go wrong: edges of tiles, remainders, the
smallest and largest of its range.  References in float64; tolerances are bounds derived from the operand types."""
import contextlib
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
U32 = 2.0 ** -24  # half a unit in the last place of a 24-bit significand


@pytest.fixture(scope="module")
def H():
    from paper_2110_08633_amd import hydra
    return hydra


@contextlib.contextmanager
def launched(H):
    """Yields a dict that holds, after the block, the launches per kernel name of what ran in it."""
    from paper_2110_08633_amd import runtime as R
    sess = R.Session(1 << 20, flags=H.FLAG_TIMING)
    names = {}
    try:
        yield names
        torch.cuda.synchronize()
        names.update({k["name"]: k["launches"] for k in H.hydra_kernel_stats(sess.ctx)})
    finally:
        sess.close()


def randn(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(*shape, generator=g, device="cuda")


def stored(x, ld, shift):
    """x in a buffer with leading dimension ld that starts shift elements past a 256-byte boundary; the gap between the
    rows is NaN.  Returns the matrix view."""
    buf = torch.full((x.shape[0] * ld + shift,), float("nan"), dtype=x.dtype, device="cuda")
    v = buf[shift:].view(x.shape[0], ld)
    v[:, :x.shape[1]] = x
    return v


# M, N, K, extra leading dimension, element shift.  16-byte loads: all of K, M, N, leading dimensions and shift multiples
# of 4; else 4-byte loads.  From 640 64x64 tiles on those are used, below 32x32 tiles.
F32_CASES = [(1, 1, 1, 0, 0), (33, 31, 7, 1, 0), (32, 32, 64, 0, 0), (36, 28, 68, 4, 0), (64, 96, 4, 0, 1),
             (100, 52, 129, 0, 0), (1604, 1700, 36, 4, 0), (1664, 1600, 32, 0, 0), (1601, 1663, 33, 3, 2),
             (2, 3, 5, 7340040, 0)]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K,extra,shift", F32_CASES)
def test_gemm_f32_variants(H, ta, tb, M, N, K, extra, shift):
    A, B, resid = randn(M + K, M, K), randn(N + K + 1, K, N), randn(M + N + 2, M, N)
    As, Bs = A.t().contiguous() if ta else A, B if tb else B.t().contiguous()
    dA, dB = stored(As, As.shape[1] + extra, shift), stored(Bs, Bs.shape[1] + extra, shift)
    ldc = N + (extra if extra < 100 else 0)
    out = torch.full((M, ldc), 7.0, device="cuda")
    H.hydra_op_gemm(0, ta, tb, M, N, K, 0.5, dA, As.shape[1] + extra, dB, Bs.shape[1] + extra, None,
                    stored(resid, ldc, 0), out, None, ldc)
    torch.cuda.synchronize()
    ref = 0.5 * (A.double() @ B.double()) + resid.double()
    # a sum of K products in any order, its scaling and the residual: each of the K + 2 roundings is at most U32 of the
    # sum of magnitudes
    bound = (K + 2) * U32 * (0.5 * (A.double().abs() @ B.double().abs()) + resid.double().abs())
    assert ((out[:, :N].double() - ref).abs() <= bound).all()
    assert (out[:, N:] == 7.0).all()


def test_gemm_f32_wide_operands_large_result(H):
    """Leading dimensions beyond a 32-bit byte offset, with enough tiles for 64x64 ones (32x32 tiles would exceed a launch's
    threads from 1.7e10 results on)."""
    test_gemm_f32_variants(H, 1, 1, 1700, 1604, 12, 7340040, 0)


# bf16 products, one matrix each, with ragged last rows, columns and contractions (shorter than a slice, one step into the
# next slice, an odd length); EVERY_SHAPE below takes every tile shape
PLAIN_CASES = [(1, 1, 8), (33, 40, 72), (201, 2304, 768), (520, 264, 200), (513, 1024, 1001), (2050, 776, 2056),
               (1100, 1608, 600), (900, 3300, 776), (1030, 4104, 1000), (2000, 3000, 520), (1000, 6408, 1608),
               (4100, 4104, 72), (1000, 16392, 4096)]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", PLAIN_CASES)
def test_gemm_bf16_tile_shapes(H, ta, tb, M, N, K):
    r8 = lambda n: (n + 7) // 8 * 8
    if not (ta and tb):
        K = r8(K)  # a contraction-contiguous operand is read in chunks of eight steps
    A, B = randn(M + K, M, K).bfloat16(), randn(N + K + 1, K, N).bfloat16()
    bias, resid = randn(N, N), randn(M + N + 2, M, N)
    As, Bs = A.t().contiguous() if ta else A, B if tb else B.t().contiguous()
    lda, ldb, ldc = r8(As.shape[1]) + 8, r8(Bs.shape[1]), N + 1
    dA, dB = stored(As, lda, 0), stored(Bs, ldb, 8)
    if M * N * K < 1 << 30:  # once with everything the epilogue can do, unaligned; large ones plain and aligned
        out, act = torch.full((M, ldc), 7.0, device="cuda"), torch.full((M, ldc), 7.0, device="cuda").bfloat16()
        H.hydra_op_gemm(1, ta, tb, M, N, K, 0.5, dA, lda, dB, ldb, bias, stored(resid, ldc, 0), out, act, ldc)
        ref = 0.5 * (A.double() @ B.double()) + bias.double() + resid.double()
        mag = 0.5 * (A.double().abs() @ B.double().abs()) + bias.double().abs() + resid.double().abs()
        assert (out[:, N:] == 7.0).all() and (act[:, N:] == 7.0).all()
        out, act = out[:, :N], act[:, :N]
        # bf16 copy: half a unit in the last place of 8 bits on top
        assert ((act.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * (K + 4) * U32 * mag).all()
    else:
        out = torch.empty((M, N), device="cuda")
        H.hydra_op_gemm(1, ta, tb, M, N, K, 1.0, dA, lda, dB, ldb, None, None, out, None, N)
        ref, mag = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    # products of bf16 values are exact in fp32; each of the K + 4 additions and scalings errs by at most a unit in the
    # last place of the sum of magnitudes (the matrix instruction may truncate)
    assert ((out.double() - ref).abs() <= 2 * (K + 4) * U32 * mag).all()


# the smallest products of several tiles, ragged on every side, for which the launcher takes a tile shape: per shape one for
# both operands contraction-contiguous, one for one of each kind, one for both strided.  (The CPU suite holds this table
# against the choice as well.)
EVERY_SHAPE = {
    "256x256": ((908, 14548, 200), (641, 13668, 136), (649, 18632, 131)),
    "128x256": ((325, 16392, 264), (260, 16420, 136), (387, 16364, 1293)),
    "128x192": ((194, 18568, 200), (194, 16388, 136), (8778, 516, 901)),
    "128x128": ((130, 10916, 136), (130, 10916, 136), (193, 11748, 133)),
    "128x64": ((2643, 68, 136), (5442, 132, 136), (6977, 388, 133)),
    "64x96": ((131, 7748, 136), (129, 5444, 136), (8934, 264, 525)),
    "64x64": ((66, 68, 136), (66, 68, 136), (66, 68, 131)),
    "64x64k2": ((66, 68, 328), (66, 4452, 136), (66, 5076, 131)),
    "128x64k2": ((8217, 100, 2904), (129, 8180, 392), (193, 8104, 325)),
    "64x96k2": ((66, 8344, 1160), (131, 7596, 136), (5335, 264, 131)),
    "128x128x2": (None, None, (195, 16484, 131)),
}
SHAPE_CASES = [(shape, layout, *dims[i]) for shape, dims in EVERY_SHAPE.items()
               for layout, i in (("nt", 0), ("nn", 1), ("tt", 1), ("tn", 2)) if dims[i]]
# a single, partly empty row or column of tiles
SHAPE_CASES += [("256x256", "nt", 200, 58084, 216), ("256x256", "nt", 58084, 200, 216), ("256x256", "nn", 200, 45660, 72),
                ("256x256", "tn", 200, 44395, 67), ("128x256", "nt", 100, 49156, 272), ("128x192", "nt", 100, 34580, 264),
                ("128x128", "nt", 100, 16504, 72)]


@pytest.mark.parametrize("shape,layout,M,N,K", SHAPE_CASES)
def test_gemm_bf16_every_tile_shape(H, shape, layout, M, N, K):
    ta, tb = layout[0] == "t", layout[1] == "n"
    r8 = lambda n: (n + 7) // 8 * 8
    A, B, bias, resid = randn(M + K, M, K).bfloat16(), randn(N + K + 1, K, N).bfloat16(), randn(N, N), randn(M + N + 2, M, N + 1)
    As, Bs = A.t().contiguous() if ta else A, B if tb else B.t().contiguous()
    dA, dB = stored(As, r8(As.shape[1]), 0), stored(Bs, r8(Bs.shape[1]) + 8, 0)
    prod, mag = A.double() @ B.double(), A.double().abs() @ B.double().abs()
    # aligned rows: two results, nothing added; then rows off the 16-byte grid with everything a caller can add
    out, act = torch.empty(M, N, device="cuda"), torch.empty(M, N, device="cuda").bfloat16()
    with launched(H) as names:
        H.hydra_op_gemm(1, ta, tb, M, N, K, 1.0, dA, dA.shape[1], dB, dB.shape[1], None, None, out, act, N)
    assert list(names) == [f"gemm_bf16_{shape}_{layout}"], names
    # as in test_gemm_bf16_tile_shapes
    assert ((out.double() - prod).abs() <= 2 * (K + 4) * U32 * mag).all()
    assert ((act.double() - prod).abs() <= 2.0 ** -8 * prod.abs() + 2 * (K + 4) * U32 * mag).all()
    out, act = torch.full((M, N + 1), 7.0, device="cuda"), torch.full((M, N + 1), 7.0, device="cuda").bfloat16()
    H.hydra_op_gemm(1, ta, tb, M, N, K, 0.5, dA, dA.shape[1], dB, dB.shape[1], bias, resid, out, act, N + 1)
    prod = 0.5 * prod + bias.double() + resid[:, :N].double()
    mag = 0.5 * mag + bias.double().abs() + resid[:, :N].double().abs()
    assert ((out[:, :N].double() - prod).abs() <= 2 * (K + 4) * U32 * mag).all()
    assert ((act[:, :N].double() - prod).abs() <= 2.0 ** -8 * prod.abs() + 2 * (K + 4) * U32 * mag).all()
    assert (out[:, N:] == 7.0).all() and (act[:, N:] == 7.0).all()


# the shapes whose wavefront groups exchange partial sums through LDS, and others, while a second stream keeps the device busy
@pytest.mark.parametrize("shape,layout,M,N,K", [("64x64k2", "nt", 201, 2304, 768), ("128x64k2", "nn", 1100, 1608, 600),
                                                ("64x96k2", "nt", 2048, 768, 2304), ("64x96k2", "tn", 2048, 768, 2304),
                                                ("128x64k2", "tn", 1100, 1608, 600), ("256x256", "nt", 1024, 12288, 1024),
                                                ("128x128x2", "tn", 1000, 6408, 1608)])
def test_gemm_bf16_repeats_bitwise_under_concurrency(H, shape, layout, M, N, K):
    ta, tb = layout[0] == "t", layout[1] == "n"
    A, B = randn(M + K, *((K, (M + 7) // 8 * 8) if ta else (M, K))).bfloat16(), randn(N + K + 1, *((K, N) if tb else (N, K))).bfloat16()
    run = lambda o, s: H.hydra_op_gemm(1, ta, tb, M, N, K, 1.0, A, A.shape[1], B, B.shape[1], None, None, o, None, N, s)
    big, bigC = randn(5, 4096, 4096).bfloat16(), torch.empty(4096, 4096, device="cuda")
    outs = [torch.zeros(M, N, device="cuda") for _ in range(12)]
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with launched(H) as names:
        run(outs[0], None)
    assert list(names) == [f"gemm_bf16_{shape}_{layout}"], names
    for o in outs:
        H.hydra_op_gemm(1, 0, 0, 4096, 4096, 4096, 1.0, big, 4096, big, 4096, None, None, bigC, None, 4096, s2)
        run(o, s1)
    torch.cuda.synchronize()
    a, b = (A[:, :M].t() if ta else A).double(), (B if tb else B.t()).double()
    assert ((outs[0].double() - a @ b).abs() <= 2 * (K + 4) * U32 * (a.abs() @ b.abs())).all()
    for o in outs[1:]:
        assert torch.equal(o, outs[0])


# leading dimensions beyond what the single-product kernel addresses: the register-staged kernel, with two and with four
# slices in flight and each of its tiles
@pytest.mark.parametrize("layout,M,N,K,wide", [("nt", 70, 90, 200, "ab"), ("nt", 130, 90, 1608, "a"), ("nn", 70, 90, 1608, "a"),
                                               ("nn", 50, 90, 1608, "a"), ("tt", 70, 90, 72, "ab"), ("tn", 70, 90, 72, "ab"),
                                               ("tn", 5800, 5801, 70, "a"), ("tn", 70, 90, 1544, "a")])
def test_gemm_bf16_wide_leading_dimensions(H, layout, M, N, K, wide):
    ta, tb, W = layout[0] == "t", layout[1] == "n", 4000008
    r8 = lambda n: (n + 7) // 8 * 8
    A, B = randn(M + K, M, K).bfloat16(), randn(N + K + 1, K, N).bfloat16()
    As, Bs = A.t().contiguous() if ta else A, B if tb else B.t().contiguous()
    dA, dB = stored(As, W if "a" in wide else r8(As.shape[1]), 0), stored(Bs, W if "b" in wide else r8(Bs.shape[1]), 0)
    out = torch.full((M, N + 1), 7.0, device="cuda")
    with launched(H) as names:
        H.hydra_op_gemm(1, ta, tb, M, N, K, 1.0, dA, dA.shape[1], dB, dB.shape[1], None, None, out, None, N + 1)
    assert [n.startswith("gemm_bf16_staged") for n in names] == [True], names
    # as in test_gemm_bf16_tile_shapes
    assert ((out[:, :N].double() - A.double() @ B.double()).abs()
            <= 2 * (K + 4) * U32 * (A.double().abs() @ B.double().abs())).all()
    assert (out[:, N:] == 7.0).all()


# the weight gradients of a block in one launch: block widths and token counts for which it takes each tile shape
GROUP_CASES = {"256x256": (672, 7312, 8), "128x256": (160, 15760, 1368), "128x192": (160, 10896, 776), "128x128": (96, 12080, 72),
               "128x64": (288, 4808, 200), "64x96": (96, 8712, 920), "64x64": (32, 64, 8), "64x64k2": (32, 6280, 8),
               "128x64k2": (96, 7904, 328), "64x96k2": (96, 6352, 136), "128x128x2": (96, 12040, 8)}


def one_block_step(H, d, F, M):
    """One bf16 training step of a one-block model: every gradient against the oracle; returns the launches per kernel name."""
    import synth_inputs as SI
    from oracle import decoder as D
    from paper_2110_08633_amd import runtime as R
    from tests.parity_utils import assert_close
    cfg = SI.small_cfg(L=1, d=d, H=d // 8, F=F, V=64, T=8, B=M // 8, dtype="bf16")
    W = SI.make_weights(cfg, 3)
    tok, tgt = SI.make_batch(cfg, 5)
    P = D.cast_params(W, np.float64)
    ref = D.train_step(P, D.zeros_like_params(P), D.zeros_like_params(P), tok, tgt, cfg, 1e-3, 1)
    sess = R.Session(R.arena_bytes_for([cfg], 3), max_slots=2, flags=H.FLAG_TIMING)
    got = sess.train_step_manual(sess.add_model(cfg, W, 1e-3), tok, tgt)
    H.hydra_sync(sess.ctx)
    names = {k["name"]: k["launches"] for k in H.hydra_kernel_stats(sess.ctx)}
    sess.close()
    for n, g in ref["grads"].items():
        assert_close(got["grads"][n], g, 2e-2, n)  # the suite's tolerance of the bf16 path
    return names


@pytest.mark.parametrize("shape", GROUP_CASES)
def test_grouped_weight_gradients_of_every_tile_shape(H, shape):
    assert one_block_step(H, *GROUP_CASES[shape]).get(f"gemm_bf16_{shape}_tn_group") == 1


# the MLP's products with GELU and its derivative in their write-out: width, hidden width and tokens for which both take a
# tile shape
@pytest.mark.parametrize("shape,d,F,M", [("256x256", 200, 4744, 2960), ("128x256", 264, 3512, 1736), ("128x192", 264, 3600, 1048),
                                         ("128x128", 72, 1224, 1552), ("128x64", 72, 72, 136), ("64x96", 72, 10896, 136),
                                         ("64x64", 136, 72, 72), ("64x64k2", 72, 456, 1544), ("64x96k2", 1160, 2736, 328)])
def test_gelu_epilogues_of_the_tile_shapes(H, shape, d, F, M):
    assert one_block_step(H, d, F, M).get(f"gemm_bf16_{shape}_nt", 0) >= 2  # forward and backward


# a contraction of one slice or less: which of the two kernels takes it depends on layout, tiles and rows; M, N, K, layout,
# extra leading dimension of the result, whether the register-staged kernel is expected
ONE_SLICE = [(512, 512, 64, "nt", 0, True), (1000, 1000, 64, "nt", 0, True), (8, 768, 40, "nt", 0, True), (8, 768, 64, "nt", 1, False),
             (1000, 1001, 64, "nt", 0, False), (2049, 4100, 8, "nn", 0, True), (1000, 1000, 64, "nn", 0, False),
             (1024, 4096, 64, "tn", 0, True), (1601, 6400, 40, "tt", 0, True), (768, 2304, 64, "tn", 0, False),
             (1024, 4096, 65, "tn", 0, False), (1000, 1000, 72, "nt", 0, False), (4099, 1003, 24, "tn", 0, False)]


@pytest.mark.parametrize("M,N,K,layout,ext,staged", ONE_SLICE)
def test_gemm_bf16_one_slice(H, M, N, K, layout, ext, staged):
    ta, tb = layout[0] == "t", layout[1] == "n"
    r8 = lambda n: (n + 7) // 8 * 8
    A, B, resid = randn(M + K, M, K).bfloat16(), randn(N + K + 1, K, N).bfloat16(), randn(M + N + 2, M, N + ext)
    As, Bs = A.t().contiguous() if ta else A, B if tb else B.t().contiguous()
    dA, dB = stored(As, r8(As.shape[1]), 0), stored(Bs, r8(Bs.shape[1]), 0)
    out, act = torch.full((M, N + ext), 7.0, device="cuda"), torch.full((M, N + ext), 7.0, device="cuda").bfloat16()
    with launched(H) as names:
        H.hydra_op_gemm(1, ta, tb, M, N, K, 1.0, dA, dA.shape[1], dB, dB.shape[1], None, resid, out, act, N + ext)
    assert [n.startswith("gemm_bf16_staged") for n in names] == [staged], names
    ref = A.double() @ B.double() + resid[:, :N].double()
    mag = A.double().abs() @ B.double().abs() + resid[:, :N].double().abs()
    # as in test_gemm_bf16_tile_shapes
    assert ((out[:, :N].double() - ref).abs() <= 2 * (K + 4) * U32 * mag).all()
    assert ((act[:, :N].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * (K + 4) * U32 * mag).all()
    assert (out[:, N:] == 7.0).all() and (act[:, N:] == 7.0).all()


def test_scores_of_many_pairs_take_128x64_tiles(H):
    """Attention at a head width without a fused kernel: the batched score products (both operands contraction-contiguous)
    keep the faster 128x64 tiles also when there are thousands of them."""
    from paper_2110_08633_amd import runtime as R
    cfg = dict(L=1, d=512, H=16, F=512, V=64, T=512, B=8, k=1, dtype="bf16")
    sess = R.Session(R.arena_bytes_for([cfg], 2), max_slots=2, flags=H.FLAG_TIMING)
    n = H.hydra_model_layout(H.model_desc(cfg, 1e-4)).n_params
    host = [np.zeros(n, np.float32) for _ in range(3)]
    pinned = [torch.from_numpy(h).pin_memory().numpy() for h in host]
    rec = sess.add_model(cfg, None, 1e-4, host=tuple(pinned))
    tok = np.zeros((cfg["B"], cfg["T"]), np.int32)
    sess.train_step_manual(rec, tok, tok)
    H.hydra_sync(sess.ctx)
    names = {k["name"]: k["launches"] for k in H.hydra_kernel_stats(sess.ctx)}
    sess.close()
    # forward, recomputation and dP
    assert names.get("gemm_bf16_staged_x64_nt") == 3 and "gemm_bf16_staged_128x128_nt" not in names, names


# one group of wavefronts per block (short sequences, or many row blocks) and two (few row blocks); last tiles and row
# blocks partly empty; an odd number of tiles for two groups to share; peaked scores, for which the running maximum moves
ATT_CASES = [(1, 1, 8, 64, 1.0), (2, 3, 72, 128, 1.0), (1, 3, 256, 64, 1.0), (1, 2, 264, 64, 6.0), (3, 5, 328, 128, 1.0),
             (1, 7, 1000, 64, 1.0), (1, 2, 1096, 128, 6.0), (9, 13, 584, 64, 1.0), (5, 17, 776, 128, 1.0),
             (7, 16, 520, 64, 6.0)]


@pytest.mark.parametrize("B,Hn,T,dh,peak", ATT_CASES)
def test_attention_variants(H, B, Hn, T, dh, peak):
    d = Hn * dh
    qkv = randn(B * T + Hn, B * T, 3 * d)
    qkv[:, :d] *= peak
    qkv, d_o = qkv.bfloat16(), randn(T + dh, B * T, d).bfloat16()
    o, dqkv = (torch.full((B * T + 1, n * d), 7.0, device="cuda").bfloat16() for n in (1, 3))  # a row past the end
    lse, dsum = (torch.empty(B * Hn * T, device="cuda") for _ in range(2))
    H.hydra_op_attention_fwd(qkv, o, lse, B, Hn, T, dh)
    H.hydra_op_attention_bwd(qkv, o, d_o, lse, dsum, dqkv, B, Hn, T, dh)
    torch.cuda.synchronize()
    assert (o[-1] == 7.0).all() and (dqkv[-1] == 7.0).all()
    x = qkv.double().requires_grad_()
    q, k, v = (x[:, j * d:(j + 1) * d].reshape(B, T, Hn, dh).transpose(1, 2) for j in range(3))
    s = (q @ k.transpose(2, 3).contiguous()) / dh ** 0.5
    s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    ref_lse = torch.logsumexp(s, -1)
    p = torch.exp(s - ref_lse[..., None])
    ref = (p @ v).transpose(1, 2).reshape(B * T, d)
    mag = (p @ v.abs()).transpose(1, 2).reshape(B * T, d).detach()
    ref.backward(d_o.double())
    ref = ref.detach()
    # the result is rounded to 8 bits and so is every probability (half a unit each); 2^-12 for the exponentials' and the
    # sums' fp32 rounding
    assert ((o[:-1].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + (2.0 ** -8 + 2.0 ** -12) * mag).all()
    # scores are sums of dh products
    tol = (dh + 8) * U32 * (q.abs().amax() * k.abs().amax()).detach() * dh ** 0.5 + 1e-5
    assert ((lse.double() - ref_lse.detach().reshape(-1)).abs() <= tol).all()
    # gradients: the operands p, dS and dP's input o are rounded to 8 bits, 2^-9 / sqrt(3) rms each; D = sum dO * O and the
    # differences dP - D can double that
    for j in range(3):
        g, r = dqkv[:-1, j * d:(j + 1) * d].double(), x.grad[:, j * d:(j + 1) * d]
        assert (g - r).norm() <= 2.0 ** -7 * r.norm() + 1e-12
    # and element by element on the scale of what was added (a late key's gradient is a thousandth of the tensor's norm):
    # p and dS are rounded to 8 bits, dS = p (dP - D) / sqrt(dh) carries the error of D's input o, the result is rounded
    # once more; 2^-11 for fp32 sums and exponentials on either side
    heads = lambda t: t.reshape(B, T, Hn, dh).transpose(1, 2)
    q, k, v, p, g_o = q.detach(), k.detach(), v.detach(), p.detach(), heads(d_o.double())
    dP, D = g_o @ v.transpose(2, 3).contiguous(), (g_o * heads(ref)).sum(-1, keepdim=True)
    d_err = (g_o.abs() * heads(2.0 ** -8 * ref.abs() + (2.0 ** -8 + 2.0 ** -12) * mag)).sum(-1, keepdim=True)
    fp32 = 2.0 ** -11 * (g_o.abs() @ v.abs().transpose(2, 3).contiguous() + (g_o * heads(ref)).abs().sum(-1, keepdim=True))
    ds_err = p * (2.0 ** -8 * (dP - D).abs() + d_err + fp32) / dh ** 0.5
    bounds = (ds_err @ k.abs(), ds_err.transpose(2, 3).contiguous() @ q.abs(),
              (2.0 ** -8 + 2.0 ** -11) * (p.transpose(2, 3).contiguous() @ g_o.abs()))
    for j, b in enumerate(bounds):
        g, r = heads(dqkv[:-1, j * d:(j + 1) * d].double()), heads(x.grad[:, j * d:(j + 1) * d])
        assert ((g - r).abs() <= 2.0 ** -8 * r.abs() + b).all(), "qkv"[j]
        last = slice((T - 1) // 32 * 32, T)  # what a wavefront owns of the end of the sequence would fail as zeros
        assert (r.abs() > 2.0 ** -8 * r.abs() + b)[:, :, last].any(), "qkv"[j]


def test_attention_more_blocks_than_a_row_of_the_grid_holds(H):
    B, T, dh = (1 << 24) + 3, 8, 64
    one = randn(1, T, 3 * dh).bfloat16()
    qkv = one.repeat(B, 1)
    o, lse = torch.zeros(B, T * dh, device="cuda").bfloat16(), torch.zeros(B, T, device="cuda")
    H.hydra_op_attention_fwd(qkv, o, lse, B, 1, T, dh)
    torch.cuda.synchronize()
    del qkv
    o1, lse1 = torch.zeros(1, T * dh, device="cuda").bfloat16(), torch.zeros(1, T, device="cuda")
    H.hydra_op_attention_fwd(one, o1, lse1, 1, 1, T, dh)
    assert torch.equal(lse, lse1.expand(B, T))
    for part in o.split(1 << 20):
        assert torch.equal(part, o1.expand_as(part))
    del o
    torch.cuda.empty_cache()


# a score of -inf (here by overflow: finite operands, a product beyond fp32) weighs nothing, in whichever group of
# wavefronts and at whichever place of its tile it falls - also where it is all a row sees of a tile (keys 0..63, or the
# diagonal key of row 64 + 128 i, which opens the second group's first tile)
@pytest.mark.parametrize("B,Hn,T,dh", [(1, 2, 328, 64), (1, 1, 264, 128), (40, 16, 264, 64), (1, 1, 136, 128)])
@pytest.mark.parametrize("keys", [(64, 65), (192, 193), (0, 64), (0, 128)])
def test_attention_scores_of_minus_infinity(H, B, Hn, T, dh, keys):
    d = Hn * dh
    keys = slice(min(keys[0], T - 1), min(keys[1], T))
    qkv = randn(T + dh, B * T, 3 * d).bfloat16().view(B, T, 3, Hn, dh)
    qkv[:, :, 0, :, 0], qkv[:, :, 1, :, 0] = 2.0 ** 66, 0.0
    qkv[:, keys, 1, :, 0] = -2.0 ** 66
    o, lse = torch.empty(B * T, d, device="cuda").bfloat16(), torch.empty(B * Hn * T, device="cuda")
    H.hydra_op_attention_fwd(qkv, o, lse, B, Hn, T, dh)
    torch.cuda.synchronize()
    q, k, v = (qkv[:, :, j].double().transpose(1, 2) for j in range(3))
    s = (q @ k.transpose(2, 3).contiguous()) / dh ** 0.5
    s[..., keys] = float("-inf")
    s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    ref_lse = torch.logsumexp(s, -1, keepdim=True)
    p = torch.exp(s - ref_lse)
    seen = torch.isfinite(ref_lse[0, 0, :, 0])  # rows that see a key with a finite score
    ref, mag = (p @ v)[:, :, seen], (p @ v.abs())[:, :, seen]
    got = o.view(B, T, Hn, dh).transpose(1, 2)[:, :, seen].double()
    # as in test_attention_variants
    assert ((got - ref).abs() <= 2.0 ** -8 * ref.abs() + (2.0 ** -8 + 2.0 ** -12) * mag).all()
    assert (lse.view(B, Hn, T)[..., seen].double() - ref_lse[:, :, seen, 0]).abs().max() < 1e-3


# tensors that start off the 16-byte grid (by one element, by eight bytes): the same bits as from aligned ones
@pytest.mark.parametrize("shift", [1, 4])
@pytest.mark.parametrize("B,Hn,T,dh", [(1, 1, 8, 64), (2, 3, 72, 128), (1, 2, 200, 64), (9, 13, 584, 64), (5, 21, 584, 128),
                                       (3, 5, 328, 128), (1, 7, 1000, 64)])
def test_attention_unaligned_tensors(H, B, Hn, T, dh, shift):
    d, n = Hn * dh, B * T
    qkv, d_o = randn(T + dh, n, 3 * d).bfloat16(), randn(T + dh + 1, n, d).bfloat16()

    def run(shift):
        def at(x):
            buf = torch.full((x.numel() + shift + 8,), 7.0, device="cuda").bfloat16()
            buf[shift:shift + x.numel()] = x.reshape(-1)
            return buf, buf[shift:shift + x.numel()]
        bufs = [at(x) for x in (qkv, d_o, torch.zeros_like(d_o), torch.zeros_like(qkv))]
        q, g, o, dq = (v for _, v in bufs)
        lse, dsum = (torch.zeros(B * Hn * T, device="cuda") for _ in range(2))
        H.hydra_op_attention_fwd(q, o, lse, B, Hn, T, dh)
        H.hydra_op_attention_bwd(q, o, g, lse, dsum, dq, B, Hn, T, dh)
        torch.cuda.synchronize()
        assert all((b[:shift] == 7.0).all() and (b[-8:] == 7.0).all() for b, _ in bufs)
        return o, dq, lse, dsum

    for a, b in zip(run(0), run(shift)):
        assert torch.equal(a, b)


# every register width of the one-pass LayerNorm backward (1 to 8 float4 per lane), row counts around its block of 8 rows,
# more than 512 partial rows for the column sums
@pytest.mark.parametrize("M,d", [(1, 4), (7, 252), (8, 512), (9, 764), (17, 1024), (4100, 1028), (23, 1532), (15, 1792),
                                 (33, 2048)])
def test_layernorm_bwd_widths(H, M, d):
    x, dy, dres = randn(M + d, M, d) * 2 + 0.5, randn(M, M, d), randn(d, M, d)
    gamma = randn(d + 1, d) * 0.1 + 1
    mean = x.mean(1)
    rstd = 1 / torch.sqrt(x.var(1, unbiased=False) + 1e-5)
    dx, dxh = torch.empty_like(x), torch.empty_like(x, dtype=torch.bfloat16)
    cols = [torch.empty(d, device="cuda") for _ in range(3)]
    H.hydra_op_layernorm_bwd(dy, x, mean, rstd, gamma, dres, dx, dxh, *cols, torch.empty(3 * d * ((M + 7) // 8), device="cuda"),
                             M, d)
    torch.cuda.synchronize()
    xh = (x.double() - mean.double()[:, None]) * rstd.double()[:, None]
    h = dy.double() * gamma.double()
    part = h - h.mean(1, keepdim=True) - xh * (h * xh).mean(1, keepdim=True)
    ref = rstd.double()[:, None] * part + dres.double()
    # a dozen roundings of values no larger than the terms' magnitudes
    mag = rstd.double()[:, None] * (h.abs() + h.abs().mean(1, keepdim=True) + xh.abs() * (h * xh).abs().mean(1, keepdim=True))
    assert ((dx.double() - ref).abs() <= (d / 64 + 16) * U32 * (mag + dres.double().abs())).all()
    assert (dxh == dx.bfloat16()).all()
    for got, v in zip(cols, (dy.double() * xh, dy.double(), dx.double())):
        # eight rows in fp32, the rest in 64 bits; xhat itself carries three roundings
        assert ((got.double() - v.sum(0)).abs() <= 14 * U32 * v.abs().sum(0) + 4 * U32 * dy.double().abs().sum(0)).all()


def test_layernorm_bwd_more_blocks_than_a_row_of_the_grid_holds(H):
    M, d = 67200003, 4
    x, dy = randn(1, M, d), randn(2, M, d)
    gamma = randn(3, d) * 0.1 + 1
    mean = x.mean(1)
    rstd = 1 / torch.sqrt(((x - mean[:, None]) ** 2).mean(1) + 1e-5)
    dx, cols = torch.full((M + 1, d), 7.0, device="cuda"), [torch.empty(d, device="cuda") for _ in range(3)]
    H.hydra_op_layernorm_bwd(dy, x, mean, rstd, gamma, None, dx, None, *cols, torch.empty(3 * d * ((M + 7) // 8), device="cuda"),
                             M, d)
    torch.cuda.synchronize()
    assert (dx[-1] == 7.0).all()
    xh = (x - mean[:, None]) * rstd[:, None]
    h = dy * gamma
    part = h - h.mean(1, keepdim=True) - xh * (h * xh).mean(1, keepdim=True)
    mag = h.abs() + h.abs().mean(1, keepdim=True) + xh.abs() * (h * xh).abs().mean(1, keepdim=True)
    # a dozen roundings on either side
    assert ((dx[:-1] - rstd[:, None] * part).abs() <= 32 * U32 * rstd[:, None] * mag).all()
    for got, v in zip(cols, (dy * xh, dy, dx[:-1])):
        # eight rows in fp32, the rest in 64 bits; xhat itself carries three roundings on either side
        assert ((got.double() - v.sum(0, dtype=torch.float64)).abs() <= 20 * U32 * v.abs().sum(0, dtype=torch.float64)).all()


# bf16 cross-entropy: rows, columns, leading dimension.  256 threads hold a row of up to 8192 columns, 512 up to 32768, 1024
# up to 65536, and from 2049 on where there are no more than 256 rows; from 192 MB of logits on they are read past the cache
@pytest.mark.parametrize("M,V,ld", [(3, 1, 4), (5, 1021, 1024), (5, 1025, 1028), (5, 2049, 2052), (5, 4097, 4100), (5, 8193, 8196),
                                    (5, 16385, 16388), (5, 32769, 32772), (5, 53249, 53252), (5, 65536, 65536),
                                    (12100, 3999, 4096), (5900, 8190, 8192), (2940, 16384, 16384), (1470, 32760, 32768),
                                    (910, 53240, 53248), (740, 65000, 65024), (257, 2049, 2052), (257, 4097, 4100), (257, 8193, 8196),
                                    (257, 16385, 16388)])
def test_cross_entropy_rows(H, M, V, ld):
    z = stored(randn(V, M, V) * 2, ld, 0)
    tgt = torch.randint(0, V, (M,), device="cuda", dtype=torch.int32)
    tgt[-1] = -1
    if V > 4:
        tgt[0], tgt[1] = 3, V - 1
        z[0, 4] = z[0, V - 1] = -float("inf")
        z[2, V // 2] = float("nan")
    row, dl = torch.full((M,), 7.0, device="cuda"), torch.full((M, ld), 7.0, device="cuda").bfloat16()
    H.hydra_op_cross_entropy(1, z, tgt, row, dl, M, V, ld, 0.25)
    if V > 4:
        assert torch.isnan(row[2]) and torch.isnan(dl[2, :V]).all()
        z[2] = 0.0
        row[2] = float(np.log(V))
    keep = (tgt >= 0).nonzero()[:, 0]
    for r in range(0, len(keep), 256):  # some rows at a time: 64-bit copies of all would be large
        i = keep[r:r + 256]
        x, t = z[i, :V].double(), tgt[i].long()[:, None]
        lse = torch.logsumexp(x, 1, keepdim=True)
        p = torch.exp(x - lse)
        one = torch.zeros_like(p).scatter_(1, t, 1.0)
        ref, got = 0.25 * (p - one), dl[i, :V].double()
        # half a unit of 8 bits of the result; 2^-20 of what is subtracted: exponential (two units of 24 bits), the sum (a few,
        # its terms are added in a tree), reciprocal and two products, with a factor of two in reserve
        ok = (got - ref).abs() <= 2.0 ** -8 * ref.abs() + 0.25 * 2.0 ** -20 * (p + one)
        assert (ok | (i == 2)[:, None]).all() if V > 4 else ok.all()
        loss = (lse - x.gather(1, t))[:, 0]
        assert ((row[i].double() - loss).abs() <= 2.0 ** -20 * (1 + lse[:, 0].abs() + x.abs().nan_to_num(posinf=0).amax(1))).all()
    if V > 4:
        dl[2] = 0.0  # (the pad of a row with a NaN is NaN too)
    assert (dl[keep][:, V:] == 0).all() and (dl[-1] == 0).all() and row[-1] == 0


# a target far above the rest: gradients below 2^-126 keep their bits in bf16, and a small loss is as exact as the sum it is the
# logarithm of
@pytest.mark.parametrize("M", [3, 300])
@pytest.mark.parametrize("V,ld", [(1021, 1024), (4097, 4100), (12001, 12004), (30001, 30004), (50257, 50260)])
def test_cross_entropy_of_a_dominant_target(H, M, V, ld):
    z = torch.empty(M, V, device="cuda")
    z[::2] = -87.0 - 5.0 * torch.rand(V, generator=torch.Generator("cuda").manual_seed(V), device="cuda")
    z[1::2] = -float(np.log(2.0 * V)) - torch.rand(V, generator=torch.Generator("cuda").manual_seed(V + 1), device="cuda")
    tgt = torch.arange(M, device="cuda", dtype=torch.int32) % V
    z[torch.arange(M), tgt.long()] = 0.0
    row, dl = torch.full((M,), 7.0, device="cuda"), torch.full((M, ld), 7.0, device="cuda").bfloat16()
    H.hydra_op_cross_entropy(1, stored(z, ld, 0), tgt, row, dl, M, V, ld, 1.0)
    row, got, x, t = row.cpu().double(), dl.cpu()[:, :V].float().double(), z.cpu().double(), tgt.cpu().long()[:, None]
    ref = torch.exp(x - torch.logsumexp(x, 1, keepdim=True)).scatter_(1, t, 0.0)
    got = got.scatter(1, t, 0.0)
    # half a unit of bf16, whose subnormals are 2^-133 apart, and what the fp32 value it is rounded from is off by
    assert ((got - ref).abs() <= 2.0 ** -134 * (1 + 2.0 ** -10) + 2.0 ** -8 * ref).all()
    assert (ref[::2] < 2.0 ** -125).all() and (got[::2].sum(1) > 0).all()
    # relative error of the sum: exponential (2), at most 16 + 2 + 6 + 16 additions on a term's way; the logarithm's own (2)
    loss = torch.log1p(torch.exp(x).scatter_(1, t, 0.0).sum(1))
    assert ((row - loss).abs() <= 42 * U32 + 2 * U32 * loss).all()


# every block form of the fused attention kernels, forward and backward (their indices in the tables, which the CPU suite holds
# against the choice): row blocks, tiles and groups partly empty
ATT_FORM_CASES = [(9, 13, 1000, 64, 0, 0), (8, 11, 1000, 64, 0, 0), (9, 13, 776, 64, 0, 0), (25, 8, 520, 64, 1, 1), (1, 1, 8, 64, 1, 1), (40, 16, 264, 64, 1, 1), (9, 13, 136, 64, 2, 1),
                  (5, 7, 136, 64, 2, 2), (9, 13, 584, 64, 0, 0), (7, 11, 456, 64, 2, 2), (3, 8, 56, 64, 1, 0), (1, 1, 136, 64, 2, 3), (1, 1, 200, 64, 3, 3), (1, 1, 520, 64, 4, 3),
                  (1, 3, 1096, 64, 4, 3), (9, 7, 584, 128, 0, 0), (9, 13, 328, 128, 0, 0), (1, 1, 8, 128, 1, 1), (9, 13, 72, 128, 1, 1),
                  (1, 1, 136, 128, 2, 2), (5, 7, 520, 128, 2, 2)]


@pytest.mark.parametrize("B,Hn,T,dh", [c[:4] for c in ATT_FORM_CASES])
def test_attention_every_form(H, B, Hn, T, dh):
    test_attention_variants(H, B, Hn, T, dh, 1.0)
    test_attention_variants(H, B, Hn, T, dh, 6.0)
    if 64 < T <= 328:  # groups whose tiles show a row only scores of -inf; tensors off the 16-byte grid
        test_attention_scores_of_minus_infinity(H, B, Hn, T, dh, (0, 64))
        test_attention_unaligned_tensors(H, B, Hn, T, dh, 1)


# every block form of the backward pass in every way its parts are launched (0 two launches, 1 one, 2 one after a launch that sums
# D, 3 and 4 the same with the parts' blocks mixed; the CPU suite holds the table against the choice): partly empty row blocks,
# tiles and groups
ATT_BWD_CASES = [(1, 1, 40, 64, 0, 1), (11, 5, 888, 64, 0, 1), (40, 8, 232, 64, 0, 2), (40, 13, 40, 64, 0, 2), (1, 1, 8, 64, 1, 1),
                 (1, 2, 88, 64, 1, 1), (11, 13, 200, 64, 1, 1), (5, 7, 136, 64, 2, 1), (11, 5, 584, 64, 2, 2), (1, 2, 104, 64, 3, 1),
                 (1, 1, 1000, 64, 3, 1), (40, 13, 200, 128, 0, 0), (11, 13, 232, 128, 0, 2), (1, 2, 8, 128, 1, 1), (3, 5, 32, 128, 1, 1),
                 (1, 3, 72, 128, 1, 2), (29, 25, 40, 128, 1, 0), (2, 1, 104, 128, 2, 2), (1, 3, 1000, 128, 2, 2),
                 (89, 3, 1200, 64, 0, 0), (129, 32, 16, 64, 1, 0), (47, 32, 400, 64, 1, 0), (1, 16, 3416, 64, 0, 3), (1, 24, 2816, 64, 0, 4),
                 (49, 17, 72, 64, 1, 4), (1, 8, 2136, 64, 2, 3), (1, 8, 4144, 64, 2, 4), (1, 16, 4208, 128, 0, 4), (3, 5, 40, 128, 1, 4),
                 (100, 13, 56, 128, 1, 4), (2, 8, 2128, 128, 2, 4)]


@pytest.mark.parametrize("B,Hn,T,dh", [c[:4] for c in ATT_BWD_CASES])
def test_attention_backward_launches(H, B, Hn, T, dh):
    test_attention_variants(H, B, Hn, T, dh, 1.0)
    test_attention_unaligned_tensors(H, B, Hn, T, dh, 1)
    d = Hn * dh
    qkv, o, d_o = randn(T, B * T, 3 * d).bfloat16(), randn(dh, B * T, d).bfloat16(), randn(B, B * T, d).bfloat16()
    lse, dsum = torch.ones(B * Hn * T, device="cuda"), torch.full((B * Hn * T + 8,), 7.0, device="cuda")
    H.hydra_op_attention_bwd(qkv, o, d_o, lse, dsum, torch.empty_like(qkv), B, Hn, T, dh)
    x = (o.double() * d_o.double()).view(B, T, Hn, dh).transpose(1, 2)
    # at most dh additions on a product's way to the sum
    assert ((dsum[:-8].double() - x.sum(-1).reshape(-1)).abs() <= dh * U32 * x.abs().sum(-1).reshape(-1)).all()
    assert (dsum[-8:] == 7.0).all()


def test_attention_backward_more_samples_than_a_grid_column(H):
    B, T, dh = 32768 + 5, 56, 128
    one = [randn(T + n, T, n * dh).bfloat16() for n in (3, 1)]
    qkv, d_o = (x.repeat(B, 1) for x in one)

    def run(qkv, d_o, B):
        o, dqkv = torch.zeros_like(d_o), torch.zeros_like(qkv)
        lse, dsum = (torch.zeros(B * T, device="cuda") for _ in range(2))
        H.hydra_op_attention_fwd(qkv, o, lse, B, 1, T, dh)
        H.hydra_op_attention_bwd(qkv, o, d_o, lse, dsum, dqkv, B, 1, T, dh)
        torch.cuda.synchronize()
        return dqkv.view(B, -1), dsum.view(B, -1)

    got = run(qkv, d_o, B)
    for g in got:  # the first sample's as the others', and right
        assert torch.equal(g, g[:1].expand_as(g))
    for g, r in zip(got, run(*one, 1)):
        assert (g[0].double() - r[0].double()).norm() <= 2.0 ** -8 * r[0].double().norm()


# a row whose weight sits almost wholly on one of its first 128 keys: that weight is exact in every form, so the result is off
# by its own rounding only
@pytest.mark.parametrize("B,Hn,T,dh", [c[:4] for c in ATT_FORM_CASES if c[2] >= 136])
def test_attention_heaviest_weight_is_exact(H, B, Hn, T, dh):
    n = B * T
    qkv = torch.zeros(B, T, 3, Hn, dh, device="cuda")
    qkv[:, :, 2] = randn(T, B, T, Hn, dh)
    g = torch.Generator("cuda").manual_seed(T + dh)
    # score of a row's key 0: 0, of one key: 4.6 to 5.4 (e^5.4 = 221 stays below the 2^8 that would move any reference), others -8
    qkv[:, :, 0, :, 0] = (4.6 + 0.8 * torch.rand(B, T, Hn, generator=g, device="cuda")) * dh ** 0.5
    qkv[:, :, 0, :, 1] = dh ** 0.5
    qkv[:, 1:, 1, :, 1] = -8.0
    for heavy in (17, 33, 64, 70, 95, 96, 127):
        x = qkv.clone()
        x[:, heavy, 1, :, 0], x[:, heavy, 1, :, 1] = 1.0, 0.0
        x = x.bfloat16()
        o, lse = torch.empty(n, Hn * dh, device="cuda").bfloat16(), torch.empty(B * Hn * T, device="cuda")
        H.hydra_op_attention_fwd(x, o, lse, B, Hn, T, dh)
        q, k, v = (x[:, :, j].double().transpose(1, 2) for j in range(3))
        s = (q[:, :, heavy:] @ k.transpose(2, 3).contiguous()) / dh ** 0.5
        s = s.masked_fill(torch.ones(T, T, dtype=torch.bool, device="cuda").triu(1)[heavy:], float("-inf"))
        ref = torch.softmax(s, -1) @ v
        got = o.view(B, T, Hn, dh).transpose(1, 2)[:, :, heavy:].double()
        # the other weights are 1.5 % at most and rounded to 8 bits themselves (2^-9 of them); were the heavy one rounded, its
        # 0.29 units of 1 / 100 to 1 / 221 would come on top of the result's rounding: 1.2 to 1.4 times as much
        assert (got - ref).norm() <= 1.02 * (ref.bfloat16().double() - ref).norm(), heavy


# products with few tiles: every tile shape in every layout, ragged on every side, with contractions that leave most of the
# eight wavefronts a slice, end within a slice, or are long (the CPU suite holds this table against the choice)
SPLIT_CASES = [("64x32w8", "nt", 387, 900, 392), ("64x32w8", "nn", 387, 900, 712), ("64x32w8", "tt", 387, 900, 456),
               ("64x32w8", "tn", 100, 2052, 391), ("64x32w8", "tn", 900, 516, 5121), ("48x32w8", "nt", 259, 900, 392),
               ("48x32w8", "nn", 100, 2052, 392), ("48x32w8", "tt", 259, 900, 392), ("48x32w8", "tn", 259, 900, 385),
               ("48x32w8", "nt", 900, 388, 5128), ("32x32w8", "nt", 49, 2052, 392), ("32x32w8", "nn", 49, 2052, 392),
               ("32x32w8", "tt", 49, 2052, 456), ("32x32w8", "tn", 49, 2052, 391), ("32x32w8", "nn", 520, 388, 5128),
               ("16x32w8", "nt", 17, 196, 392), ("16x32w8", "nn", 17, 388, 392), ("16x32w8", "tt", 387, 20, 392),
               ("16x32w8", "tn", 17, 516, 385), ("16x32w8", "tt", 2000, 52, 5128), ("16x16w8", "nt", 9, 20, 392),
               ("16x16w8", "nn", 9, 20, 456), ("16x16w8", "tt", 9, 20, 520), ("16x16w8", "tn", 9, 20, 385),
               ("16x16w8", "nt", 520, 100, 5128), ("16x16w8", "tn", 520, 100, 5121), ("64x64k2", "nt", 387, 1300, 1160),
               ("64x64k2", "tn", 195, 2052, 1293)]


@pytest.mark.parametrize("shape,layout,M,N,K", SPLIT_CASES)
def test_gemm_bf16_few_tiles(H, shape, layout, M, N, K):
    test_gemm_bf16_every_tile_shape(H, shape, layout, M, N, K)


@pytest.mark.parametrize("shape,layout,M,N,K", [("64x32w8", "nt", 387, 900, 392), ("48x32w8", "tn", 259, 904, 385),
                                                ("32x32w8", "nt", 49, 2052, 392), ("16x32w8", "tn", 17, 520, 385),
                                                ("16x16w8", "tn", 9, 24, 385)])
def test_gemm_bf16_few_tiles_repeats_bitwise_under_concurrency(H, shape, layout, M, N, K):
    test_gemm_bf16_repeats_bitwise_under_concurrency(H, shape, layout, M, N, K)


# width, hidden width and tokens of a block whose two MLP products with GELU and its derivative, and no other of its products,
# take a shape (the CPU suite holds this table against the choice)
GELU_SPLIT_CASES = [("64x32w8", 384, 4104, 56), ("48x32w8", 384, 4104, 40), ("32x32w8", 384, 4104, 24), ("16x32w8", 648, 72, 200),
                    ("16x16w8", 384, 8, 104)]


@pytest.mark.parametrize("shape,d,F,M", GELU_SPLIT_CASES)
def test_gelu_epilogues_of_few_tiles(H, shape, d, F, M):
    assert one_block_step(H, d, F, M).get(f"gemm_bf16_{shape}_nt", 0) == 3  # forward, its recomputation and backward


# long contractions whose halves are multiplied by a workgroup each: tiles and columns partly empty, halves of unequal length, the
# last slice partly empty (the CPU suite holds this table against the choice)
HALVES_CASES = [("128x128", 3414, 385, 11284), ("128x128", 1500, 1100, 10241), ("128x192", 2292, 918, 10243),
                ("128x192", 2045, 1511, 12445), ("128x256", 2787, 1055, 11525), ("128x256", 1823, 1581, 12087)]


@pytest.mark.parametrize("shape,M,N,K", HALVES_CASES)
def test_gemm_bf16_in_halves(H, shape, M, N, K):
    r8 = lambda n: (n + 7) // 8 * 8
    A, B = torch.zeros(M, r8(K) + 8, device="cuda").bfloat16(), torch.full((K, r8(N) + 8), float("nan"), device="cuda").bfloat16()
    A[:, :K], B[:, :N] = randn(M, M, K).bfloat16(), randn(N, K, N).bfloat16()
    A[:, r8(K):] = float("nan")
    a, b = A[:, :K].double(), B[:, :N].double()
    prod, mag = 0.5 * (a @ b), 0.5 * (a.abs() @ b.abs())
    outs = [torch.full((M, N + 3), 7.0, device="cuda") for _ in range(4)]
    with launched(H) as names:
        for o in outs:
            H.hydra_op_gemm(1, 0, 1, M, N, K, 0.5, A, A.shape[1], B, B.shape[1], None, None, o, None, N + 3)
    assert names == {f"gemm_bf16_{shape}_halves_nn": 4}, names
    for o in outs:
        assert torch.equal(o, outs[0]) and (o[:, N:] == 7.0).all()
    # as in test_gemm_bf16_tile_shapes
    assert ((outs[0][:, :N].double() - prod).abs() <= 2 * (K + 4) * U32 * mag).all()
    # what a caller adds, a bf16 result, results in host memory: whole
    resid, bias = randn(3, M, N), randn(4, N)
    act, host = torch.empty(M, N, device="cuda").bfloat16(), torch.empty(M, N, pin_memory=True)
    for args, want in (((bias, None, outs[0], None), prod + bias.double()), ((None, resid, outs[0], None), prod + resid.double()),
                       ((None, None, None, act), prod), ((None, None, host, None), prod)):
        o = args[2] if args[2] is not None else args[3]
        o = o if o is not outs[0] else torch.empty(M, N, device="cuda")
        with launched(H) as names:
            H.hydra_op_gemm(1, 0, 1, M, N, K, 0.5, A, A.shape[1], B, B.shape[1], *args[:2], *((None, o) if args[2] is None else (o, None)), N)
        assert not any("halves" in n for n in names), names
        assert (o.cuda().double() - want).norm() <= 2.0 ** -8 * want.norm()


def test_gemm_bf16_halves_are_not_added_to_fine_grained_memory(H):
    hip, (_, M, N, K) = H.lib, HALVES_CASES[1]  # (the runtime that the library is linked to)
    mem = C.c_void_p()
    assert hip.hipExtMallocWithFlags(C.byref(mem), C.c_size_t(4 * M * N), C.c_uint(1)) == 0  # hipDeviceMallocFinegrained

    class Result:
        def data_ptr(self):
            return mem.value

    A, B = randn(1, M, (K + 7) // 8 * 8).bfloat16(), randn(2, K, (N + 7) // 8 * 8).bfloat16()
    got, whole = torch.empty(M, N, device="cuda"), torch.empty(M, N, device="cuda")
    with launched(H) as names:
        H.hydra_op_gemm(1, 0, 1, M, N, K, 1.0, A, A.shape[1], B, B.shape[1], None, None, Result(), None, N)
    assert names and not any("halves" in n for n in names), names
    torch.cuda.synchronize()
    assert hip.hipMemcpy(C.c_void_p(got.data_ptr()), mem, C.c_size_t(4 * M * N), C.c_int(3)) == 0
    torch.cuda.synchronize()
    H.hydra_op_gemm(1, 0, 1, M, N, K, 1.0, A, A.shape[1], B, B.shape[1], None, torch.zeros(M, N, device="cuda"), whole, None, N)
    assert torch.equal(got, whole)


def test_gemm_bf16_in_halves_under_concurrency(H):
    test_gemm_bf16_repeats_bitwise_under_concurrency(H, "128x128_halves", "nn", 1500, 1096, 10248)


# large products of contraction-strided operands (at least 128 tiles of 256x256): the shapes with slices of 32 steps, an odd and
# an even number of them, the last one partly empty, and the others that large_tn may choose (the CPU suite holds this table
# against the choice); then the weight gradients of a block in one launch
LARGE_TN_CASES = [("256x256", 641, 17132, 257), ("256x256", 641, 17132, 289), ("128x256x2", 1300, 17864, 257),
                  ("128x256x2", 1300, 17864, 289), ("128x192", 515, 18352, 257), ("128x128x2", 515, 10788, 257),
                  ("128x256", 515, 12496, 257)]


@pytest.mark.parametrize("shape,M,N,K", LARGE_TN_CASES)
def test_gemm_bf16_large_weight_gradients(H, shape, M, N, K):
    test_gemm_bf16_every_tile_shape(H, shape, "tn", M, N, K)


@pytest.mark.parametrize("shape,M,N,K", [("256x256", 641, 17136, 257), ("128x256x2", 1300, 17864, 257)])
def test_gemm_bf16_large_weight_gradients_repeat_bitwise_under_concurrency(H, shape, M, N, K):
    test_gemm_bf16_repeats_bitwise_under_concurrency(H, shape, "tn", M, N, K)


# large products of contraction-contiguous operands (more than one round of 256x256 tiles, a short contraction): the shapes that
# large_nt takes instead of the one that all products would (the CPU suite holds this table against both)
LARGE_NT_CASES = [("256x256", 658, 39020, 136), ("256x256", 648, 33892, 328), ("128x256", 328, 33332, 520), ("128x192", 394, 35764, 328)]


@pytest.mark.parametrize("shape,M,N,K", LARGE_NT_CASES)
def test_gemm_bf16_large_products_of_short_contractions(H, shape, M, N, K):
    test_gemm_bf16_every_tile_shape(H, shape, "nt", M, N, K)


# a group that four launches were once estimated to be faster for (they take 1.2 times as long)
def test_weight_gradients_of_a_block_stay_together(H):
    names = one_block_step(H, 1160, 4640, 776)
    assert sum(n for name, n in names.items() if name.endswith("_tn_group")) == 1, names


@pytest.mark.parametrize("shape,d,F,M", [("256x256", 1160, 2744, 264), ("128x256x2", 1544, 4480, 264)])
def test_grouped_large_weight_gradients(H, shape, d, F, M):
    assert one_block_step(H, d, F, M).get(f"gemm_bf16_{shape}_tn_group") == 1
