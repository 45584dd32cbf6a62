"""Per-kernel parity on the GPU: each HIP kernel (through the op C-ABI) against
the oracle's building block on the same seeded inputs, at sizes spanning
several tiles with ragged tails."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import announce, host, max_rel, nans, rnd, to_dev, torch_dev, zeros

pytestmark = pytest.mark.gpu

NT, NN, TN = 0, 1, 2
E_STORE, E_GELU, E_RESID, E_GELUBWD, E_F32 = range(5)
TOL = {"bf16": 1e-2, "f32": 2e-5}


def _dt(s):
    return 1 if s == "bf16" else 0


def _ref_product(layout, A, B):
    if layout == NT:
        return oracle.linear(A, B)
    if layout == NN:
        return oracle.linear(A, B.T)
    return oracle.linear(A.T, B.T)


GEMM_SHAPES = {
    # bf16: 64x64 tiles, or the general kernel where N % 8 != 0 (test_gemm_large_kernels has
    # the large ones); fp32: the 32x32 kernel.  K pipelines: 1 to 3 tiles, ragged last tiles,
    # several passes
    NT: [(300, 200, 256), (1, 8, 8), (129, 257, 72), (512, 384, 1280), (700, 520, 200),
         (1030, 588, 64), (600, 300, 24), (520, 264, 96), (515, 260, 168), (520, 264, 264),
         (530, 256, 1000)],
    NN: [(300, 200, 256), (129, 264, 72), (77, 8, 520), (600, 264, 136), (777, 1032, 1280),
         (530, 280, 40)],
    TN: [(200, 264, 333), (8, 16, 1), (136, 128, 1000), (520, 264, 1000), (1280, 600, 77),
         (512, 256, 5), (600, 392, 63), (600, 392, 250), (520, 264, 291),
         (1280, 1176, 700)],
}


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", [NT, NN, TN])
def test_gemm_layouts(dtype, layout):
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng = np.random.default_rng(10 * layout + len(dtype))
    for (M, N, K) in GEMM_SHAPES[layout]:
        if dtype == "f32" and layout != TN and K % 4:
            continue
        announce(f"gemm {dtype} layout={layout} M={M} N={N} K={K}")
        A = rnd(rng, (K, M) if layout == TN else (M, K), dtype)
        B = rnd(rng, (N, K) if layout == NT else (K, N), dtype)
        ref = _ref_product(layout, A, B)
        C = nans((M, N), "f32")
        mp.op_gemm(_dt(dtype), layout, E_F32, M, N, K, to_dev(A, dtype), A.shape[1],
                   to_dev(B, dtype), B.shape[1], C, N)
        torch.cuda.synchronize()
        err = max_rel(host(C), ref)
        assert err < (2e-5 if dtype == "f32" else 1e-5), (M, N, K, err)


@pytest.mark.parametrize("layout", [NT, NN])
@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 333, 264, 192), ("f32", 333, 264, 192),
                                         ("bf16", 700, 392, 256), ("bf16", 530, 300, 64),
                                         ("bf16", 1100, 520, 360)])
def test_gemm_epilogues(dtype, M, N, K, layout):
    """Fused epilogues of 64x64 tiles (bf16) and of the 32x32 kernel (fp32); (530, 300) has
    N % 8 != 0 (rows that break 16-byte alignment), which the dispatcher sends to the general
    kernel.  NN takes the weight as [K][N].  (test_gemm_epilogues_by_kernel has the other
    kernels.)"""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng = np.random.default_rng(7)
    A, B, bias = rnd(rng, (M, K), dtype), rnd(rng, (N, K), dtype, 0.1), rnd(rng, (N,), dtype)
    dA, db = to_dev(A, dtype), to_dev(bias, dtype)
    if layout == NT:
        dB, ldb = to_dev(B, dtype), K
    else:   # [K][N] in rows padded to a multiple of 8 (a K-major operand's stride rule)
        ldb = (N + 7) // 8 * 8
        BT = np.zeros((K, ldb), np.float32)
        BT[:, :N] = B.T
        dB = to_dev(BT, dtype)
    pre = oracle.linear(A, B, bias)
    # store with bias
    announce(f"gemm epilogue store {dtype} layout={layout}")
    C = nans((M, N), dtype)
    mp.op_gemm(_dt(dtype), layout, E_STORE, M, N, K, dA, K, dB, ldb, C, N, bias=db)
    assert max_rel(host(C), pre) < TOL[dtype]
    # GELU, with GELU' of the pre-activation stored for the backward
    announce(f"gemm epilogue gelu {dtype} layout={layout}")
    C, C2 = nans((M, N), dtype), nans((M, N), dtype)
    mp.op_gemm(_dt(dtype), layout, E_GELU, M, N, K, dA, K, dB, ldb, C, N, bias=db, C2=C2, ldc2=N)
    assert max_rel(host(C2), oracle.gelu_grad(pre)) < TOL[dtype]
    assert max_rel(host(C), oracle.gelu(pre)) < TOL[dtype]
    # residual update in place (aux aliases C)
    announce(f"gemm epilogue resid {dtype} layout={layout}")
    R = rng.standard_normal((M, N)).astype(np.float32)
    C = to_dev(R, "f32")
    mp.op_gemm(_dt(dtype), layout, E_RESID, M, N, K, dA, K, dB, ldb, C, N, bias=db, aux=C, ld_aux=N)
    assert max_rel(host(C), R + pre) < 2e-5
    # GELU backward: acc * aux, aux = GELU'(u) as the forward epilogue stores it
    announce(f"gemm epilogue gelu-bwd {dtype} layout={layout}")
    U = rnd(rng, (M, N), dtype)
    Gd = oracle.gelu_grad(U).astype(np.float32)
    C = nans((M, N), dtype)
    mp.op_gemm(_dt(dtype), layout, E_GELUBWD, M, N, K, dA, K, dB, ldb, C, N, aux=to_dev(Gd, dtype),
               ld_aux=N)
    assert max_rel(host(C), oracle.linear(A, B) * oracle.gelu_grad(U)) < TOL[dtype]
    # fp32 accumulate (beta = 1)
    announce(f"gemm epilogue f32 accumulate {dtype} layout={layout}")
    C = to_dev(R, "f32")
    mp.op_gemm(_dt(dtype), layout, E_F32, M, N, K, dA, K, dB, ldb, C, N, beta=1)
    assert max_rel(host(C), R + oracle.linear(A, B)) < 2e-5


@pytest.mark.parametrize("dtype,M,N,K,kps", [("bf16", 136, 264, 1000, 256),
                                              ("f32", 136, 264, 1000, 256),
                                              ("bf16", 520, 264, 1000, 256),
                                              ("bf16", 1280, 768, 3000, 1024)])
@pytest.mark.parametrize("ldo_pad", [0, 3])
def test_gemm_split_k(dtype, M, N, K, kps, ldo_pad):
    """The weight-gradient route of the backward: the TN GEMM writes one fp32 partial per K
    split, and the split-K reduction adds the partials, in split order, into a d_weights
    block that already holds a value (Accumulate).  Checked against the oracle's Linear
    backward, dW = dY^T X.  ldo_pad = 0 takes the four-column reduction, 3 the
    one-column one (a row stride that is not a multiple of 4)."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng = np.random.default_rng(3 + M)
    announce(f"gemm split-k {dtype} M={M} N={N} K={K} kps={kps} ldo_pad={ldo_pad}")
    A, B = rnd(rng, (K, M), dtype), rnd(rng, (K, N), dtype)
    splits = (K + kps - 1) // kps
    part = nans((splits, M, N), "f32")
    mp.op_gemm(_dt(dtype), TN, E_F32, M, N, K, to_dev(A, dtype), M, to_dev(B, dtype), N, part, N,
               k_per_split=kps, split_stride=M * N)
    got = host(part)
    for s in range(splits):
        sl = slice(s * kps, min(K, (s + 1) * kps))
        _, ref_s, _ = oracle.linear_bwd(A[sl], B[sl], np.zeros((M, N)))
        assert max_rel(got[s], ref_s) < 2e-5, s
    # reduce into an accumulating target
    ldo = N + ldo_pad
    base = rng.standard_normal((M, ldo)).astype(np.float32)
    out = to_dev(base, "f32")
    mp.op_splitk_reduce(part, splits, M, N, out, ldo)
    res = host(out)
    _, ref, _ = oracle.linear_bwd(A, B, np.zeros((M, N)))
    assert max_rel(res[:, :N], base[:, :N] + ref) < 2e-5
    np.testing.assert_array_equal(res[:, N:], base[:, N:])   # the stride's pad untouched
    # the two reduction paths add in the same order: bitwise the same sums
    if ldo_pad:
        out4 = to_dev(base[:, :N], "f32")
        mp.op_splitk_reduce(part, splits, M, N, out4, N)
        np.testing.assert_array_equal(host(out4), res[:, :N])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [128, 1024, 1280])
def test_layernorm_fwd_bwd(dtype, n):
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng = np.random.default_rng(n)
    rows = 333
    announce(f"layernorm {dtype} n={n}")
    X = (rng.standard_normal((rows, n)) * 3 + 1).astype(np.float32)
    g, b = rnd(rng, (n,), dtype, 0.1, 1.0), rnd(rng, (n,), dtype, 0.1)
    Y = nans((rows, n), dtype)
    mean, rstd = nans((rows,), "f32"), nans((rows,), "f32")
    dX_ = to_dev(X, "f32")
    mp.op_layernorm_fwd(_dt(dtype), dX_, rows, n, to_dev(g, dtype), to_dev(b, dtype), 1e-6, Y,
                        mean, rstd)
    ry, rmu, rrs = oracle.layernorm(X, g, b, 1e-6)
    assert max_rel(host(Y), ry) < TOL[dtype]
    assert max_rel(host(mean), rmu) < 1e-5 and max_rel(host(rstd), rrs) < 1e-5
    dY = rng.standard_normal((rows, n)).astype(np.float32)
    dres = rng.standard_normal((rows, n)).astype(np.float32)
    dX, dXt = nans((rows, n), "f32"), nans((rows, n), dtype)
    gg, gb = to_dev(np.ones(n), "f32"), to_dev(np.zeros(n), "f32")
    gc = to_dev(np.full(n, 2.0), "f32")
    scratch = torch.empty(mp.op_scratch_bytes(rows, 1, n, 0), dtype=torch.uint8, device=dev)
    mp.op_layernorm_bwd(_dt(dtype), to_dev(dY, "f32"), dX_, mean, rstd, to_dev(g, dtype), rows, n,
                        to_dev(dres, "f32"), dX, dXt, gg, gb, scratch, colsum_dx=gc)
    rdx, rdg, rdb = oracle.layernorm_bwd(dY, X, g, rmu, rrs)
    assert max_rel(host(dX), rdx + dres) < 1e-4
    assert max_rel(host(dXt), rdx + dres) < TOL[dtype]
    assert max_rel(host(gg), 1 + rdg) < 1e-4 and max_rel(host(gb), rdb) < 1e-4
    # the fused column sums of dX, accumulated onto 2 (the bias-gradient Accumulate)
    assert max_rel(host(gc), 2.0 + (rdx + dres).sum(axis=0)) < 1e-4
    # without colsum_dx, and without dX (affine gradients only), nothing else changes
    gg2, gb2 = to_dev(np.zeros(n), "f32"), to_dev(np.zeros(n), "f32")
    mp.op_layernorm_bwd(_dt(dtype), to_dev(dY, "f32"), dX_, mean, rstd, to_dev(g, dtype), rows, n,
                        None, None, None, gg2, gb2, scratch)
    assert max_rel(host(gg2), rdg) < 1e-4 and max_rel(host(gb2), rdb) < 1e-4


@pytest.mark.parametrize("dtype,heads,d", [("bf16", 16, 80), ("bf16", 4, 64), ("f32", 4, 32)])
def test_rope(dtype, heads, d):
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    grid = np.array([[1, 6, 8], [2, 4, 4], [1, 96, 2]], np.int32)
    N = int((grid[:, 0] * grid[:, 1] * grid[:, 2]).sum())
    announce(f"rope {dtype} heads={heads} d={d} N={N}")
    rng = np.random.default_rng(d)
    h = heads * d
    qkv = rnd(rng, (N, 3 * h), dtype)
    t = to_dev(qkv, dtype)
    scratch = torch.empty(mp.op_scratch_bytes(N, heads, h, 3), dtype=torch.uint8, device=dev)
    mp.op_rope(_dt(dtype), t, N, heads, d, grid, 10000.0, 0, scratch)
    py, px = oracle.positions(grid)
    got = host(t)
    for part in (0, 1):
        ref = oracle.rope2d(qkv[:, part * h:(part + 1) * h], heads, d, py, px)
        assert max_rel(got[:, part * h:(part + 1) * h], ref) < TOL[dtype]
    np.testing.assert_array_equal(got[:, 2 * h:], qkv[:, 2 * h:])    # v untouched
    mp.op_rope(_dt(dtype), t, N, heads, d, grid, 10000.0, 1, scratch)
    assert max_rel(host(t), qkv) < 2 * TOL[dtype]


# segment lengths: empty-ish, sub-tile, exact tiles, ragged tails, and long segments that
# run the pipelined steady state over several loop passes (1000 = 16 key tiles)
ATTN_LENS = [1, 5, 64, 127, 128, 129, 300, 16, 1000, 705]


def test_attention_longest_segments():
    """The longest segments the workloads hold: a 1344 x 1344 image (9,216 patches) and a
    ragged 8,229-row segment, d = 80, forward and backward against the oracle.  Many key
    tiles per query test the lazily moved softmax offset and the long accumulations."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    lens = [9216, 8229]
    heads, d = 2, 80
    h = heads * d
    rng = np.random.default_rng(77)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    N = int(cu[-1])
    announce(f"attention longest segments {lens} heads={heads} d={d}")
    qkv = rnd(rng, (N, 3 * h), "bf16", 1.5)
    q, k, v = qkv[:, :h], qkv[:, h:2 * h], qkv[:, 2 * h:]
    tq = to_dev(qkv, "bf16")
    o, lse = nans((N, h), "bf16"), nans((heads, N), "f32")
    scratch = torch.empty(mp.op_scratch_bytes(N, heads, h, len(lens)), dtype=torch.uint8,
                          device=dev)
    mp.op_attention_fwd(_dt("bf16"), tq, N, heads, d, cu, o, lse, scratch)
    dO = rnd(rng, (N, h), "bf16")
    dqkv = nans((N, 3 * h), "bf16")
    mp.op_attention_bwd(_dt("bf16"), tq, o, to_dev(dO, "bf16"), lse, N, heads, d, cu, dqkv,
                        scratch)
    got_o, got_lse, got = host(o), host(lse), host(dqkv)
    ro, rlse = oracle.attention(q, k, v, cu, heads, d)
    assert max_rel(got_o, ro) < 2e-2
    assert max_rel(got_lse, rlse.T) < 1e-3
    rdq, rdk, rdv = oracle.attention_bwd(q, k, v, ro, dO, rlse, cu, heads, d)
    for name, sl, ref in (("dq", slice(0, h), rdq), ("dk", slice(h, 2 * h), rdk),
                          ("dv", slice(2 * h, 3 * h), rdv)):
        err = max_rel(got[:, sl], ref)
        print(f"longest segments {name}: max-rel {err:.2e}")
        assert err < 2e-2, (name, err)


@pytest.mark.parametrize("dtype,heads,d", [("bf16", 2, 80), ("bf16", 2, 64), ("bf16", 3, 32),
                                           ("f32", 2, 32)])
def test_attention_fwd_bwd(dtype, heads, d):
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng = np.random.default_rng(d + heads)
    cu = np.concatenate([[0], np.cumsum(ATTN_LENS)]).astype(np.int32)
    N = int(cu[-1])
    h = heads * d
    announce(f"attention {dtype} heads={heads} d={d} N={N}")
    qkv = rnd(rng, (N, 3 * h), dtype, 1.5)
    q, k, v = qkv[:, :h], qkv[:, h:2 * h], qkv[:, 2 * h:]
    ro, rlse = oracle.attention(q, k, v, cu, heads, d)
    tq = to_dev(qkv, dtype)
    o, lse = nans((N, h), dtype), nans((heads, N), "f32")
    scratch = torch.empty(mp.op_scratch_bytes(N, heads, h, len(ATTN_LENS)), dtype=torch.uint8,
                          device=dev)
    mp.op_attention_fwd(_dt(dtype), tq, N, heads, d, cu, o, lse, scratch)
    tol = 2e-2 if dtype == "bf16" else 1e-5
    assert max_rel(host(o), ro) < tol
    assert max_rel(host(lse), rlse.T) < (1e-3 if dtype == "bf16" else 1e-5)
    announce(f"attention bwd {dtype} heads={heads} d={d} N={N}")
    dO = rnd(rng, (N, h), dtype)
    rdq, rdk, rdv = oracle.attention_bwd(q, k, v, ro, dO, rlse, cu, heads, d)
    dqkv = nans((N, 3 * h), dtype)
    mp.op_attention_bwd(_dt(dtype), tq, o, to_dev(dO, dtype), lse, N, heads, d, cu, dqkv, scratch)
    got = host(dqkv)
    for name, sl, ref in (("dq", slice(0, h), rdq), ("dk", slice(h, 2 * h), rdk),
                          ("dv", slice(2 * h, 3 * h), rdv)):
        err = max_rel(got[:, sl], ref)
        assert err < (2e-2 if dtype == "bf16" else 1e-5), (name, err)


@pytest.mark.parametrize("heads,d", [(3, 32), (2, 64), (1, 80)])
def test_attention_f32_tile_edges(heads, d):
    """The fp32 attention kernels work on 16-row tiles dealt to four waves: segments of one
    row, of a row more or less than one to five tiles (waves with no tile, with one, with two)
    and across the 128-row work item, against the oracle.  1e-5 is some fifty roundings of
    2^-24, more than the longest chain of a 145-row segment adds up to."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    lens = [1, 15, 16, 17, 47, 49, 63, 64, 65, 80, 127, 145]
    rng = np.random.default_rng(100 + d)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    N, h = int(cu[-1]), heads * d
    announce(f"fp32 attention tile edges heads={heads} d={d} N={N}")
    qkv, dO = rnd(rng, (N, 3 * h), "f32", 1.5), rnd(rng, (N, h), "f32")
    q, k, v = qkv[:, :h], qkv[:, h:2 * h], qkv[:, 2 * h:]
    ro, rlse = oracle.attention(q, k, v, cu, heads, d)
    ref = oracle.attention_bwd(q, k, v, ro, dO, rlse, cu, heads, d)
    o, lse, dqkv = nans((N, h), "f32"), nans((heads, N), "f32"), nans((N, 3 * h), "f32")
    scratch = torch.empty(mp.op_scratch_bytes(N, heads, h, len(lens)), dtype=torch.uint8,
                          device=dev)
    tq = to_dev(qkv, "f32")
    mp.op_attention_fwd(0, tq, N, heads, d, cu, o, lse, scratch)
    mp.op_attention_bwd(0, tq, o, to_dev(dO, "f32"), lse, N, heads, d, cu, dqkv, scratch)
    got = host(dqkv)
    errs = [max_rel(host(o), ro), max_rel(host(lse), rlse.T)]
    errs += [max_rel(got[:, i * h:(i + 1) * h], ref[i]) for i in range(3)]
    assert max(errs) < 1e-5, errs


@pytest.mark.parametrize("d", [32, 64, 80])
def test_attention_bf16_half_items(d):
    """Micro-batches of up to 256 (work item, head) pairs deal each pair to two blocks of 64
    rows: segments at the edges of 16, 64 and 128 rows on that path against the oracle, and
    the same segments ten times over (360 pairs, a block per pair) bit for bit, since a
    row's value may not depend on what shares its micro-batch."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    lens, heads = [1, 15, 16, 17, 63, 64, 65, 79, 127, 128, 129, 145, 193, 256], 2
    h, n = heads * d, sum(lens)
    rng = np.random.default_rng(60 + d)
    qkv, dO = rnd(rng, (n, 3 * h), "bf16", 1.5), rnd(rng, (n, h), "bf16")
    out = []
    for reps in (1, 10):
        cu = np.concatenate([[0], np.cumsum(lens * reps)]).astype(np.int32)
        N = n * reps
        announce(f"bf16 attention half items d={d} N={N}")
        o, lse, dqkv = nans((N, h), "bf16"), nans((heads, N), "f32"), nans((N, 3 * h), "bf16")
        scratch = torch.empty(mp.op_scratch_bytes(N, heads, h, len(lens) * reps),
                              dtype=torch.uint8, device=dev)
        tq, tdo = to_dev(np.tile(qkv, (reps, 1)), "bf16"), to_dev(np.tile(dO, (reps, 1)), "bf16")
        mp.op_attention_fwd(_dt("bf16"), tq, N, heads, d, cu, o, lse, scratch)
        mp.op_attention_bwd(_dt("bf16"), tq, o, tdo, lse, N, heads, d, cu, dqkv, scratch)
        out.append([host(o), host(lse).T, host(dqkv)])
    for one, ten in zip(*out):
        assert np.array_equal(np.tile(one, (10, 1)), ten)
    q, k, v = qkv[:, :h], qkv[:, h:2 * h], qkv[:, 2 * h:]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ro, rlse = oracle.attention(q, k, v, cu, heads, d)
    ref = oracle.attention_bwd(q, k, v, ro, dO, rlse, cu, heads, d)
    o, lse, got = out[0]
    errs = [max_rel(o, ro)] + [max_rel(got[:, i * h:(i + 1) * h], ref[i]) for i in range(3)]
    assert max(errs) < 2e-2, errs
    assert max_rel(lse, rlse) < 1e-3


@pytest.mark.parametrize("layout", [NT, NN, TN])
def test_gemm_f32_tiles(layout):
    """fp32 products at the edges of the 32x32 kernel (a K of less than one 16-deep step, of
    one to five steps over the four waves, odd remainders, one row or column more or less than
    a tile), split over K, and just past the tile count from which the 128x128 kernel runs
    (1,430 x 1,424: 144 tiles).  2e-5: the bound of the other fp32 products here."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng = np.random.default_rng(40 + layout)
    for (M, N, K, kps) in [(1, 4, 4, 0), (32, 32, 16, 0), (33, 31, 20, 0), (31, 36, 60, 0),
                           (64, 33, 64, 0), (65, 64, 68, 0), (40, 100, 260, 0),
                           (36, 40, 200, 64), (1430, 1424, 36, 0)]:
        if layout == TN:
            M, K = (M + 3) // 4 * 4, K + (1 if K > 4 else 0)
        announce(f"gemm f32 tiles layout={layout} M={M} N={N} K={K} kps={kps}")
        A = rnd(rng, (K, M) if layout == TN else (M, K), "f32")
        ldb = K if layout == NT else (N + 3) // 4 * 4
        B = rnd(rng, (N if layout == NT else K, ldb), "f32")
        ref = _ref_product(layout, A, B if layout == NT else B[:, :N])
        splits = -(-K // kps) if kps else 1
        C = nans((splits, M, N), "f32")
        mp.op_gemm(0, layout, E_F32, M, N, K, to_dev(A, "f32"), A.shape[1], to_dev(B, "f32"),
                   ldb, C, N, k_per_split=kps, split_stride=M * N)
        assert max_rel(host(C).sum(0), ref) < 2e-5, (M, N, K)


@pytest.mark.parametrize("layout", [NT, NN, TN])
def test_gemm_bf16_small_tiles(layout):
    """bf16 products of few tiles, nearly all on 64x64 ones: K of less than one 64-deep tile,
    with an odd remainder, of a ring's depth more or less.  Rows are the same bits as those of
    a taller product (200 and 1,400 rows alone and within 6,000, which run 128x128 tiles for NT
    and the large ones for NN; test_gemm_bf16_rows_have_one_value has all four)."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng = np.random.default_rng(60 + layout)
    for (M, N, K) in [(1, 8, 8), (64, 64, 64), (65, 72, 136), (63, 56, 200), (200, 136, 264),
                      (128, 128, 320), (130, 264, 456), (1408, 1280, 648), (2560, 1280, 136)]:
        M = (M + 7) // 8 * 8 if layout == TN else M
        announce(f"gemm bf16 small tiles layout={layout} M={M} N={N} K={K}")
        A = rnd(rng, (K, M) if layout == TN else (M, K), "bf16")
        B = rnd(rng, (N, K) if layout == NT else (K, N), "bf16")
        C = nans((M, N), "f32")
        mp.op_gemm(1, layout, E_F32, M, N, K, to_dev(A, "bf16"), A.shape[1], to_dev(B, "bf16"),
                   B.shape[1], C, N)
        assert max_rel(host(C), _ref_product(layout, A, B)) < 1e-5, (M, N, K)
    if layout == TN:
        return
    M, N, K = 6000, 1280, 1000
    announce(f"gemm bf16 rows of a taller product layout={layout}")
    dA, dB = to_dev(rnd(rng, (M, K), "bf16"), "bf16"), to_dev(
        rnd(rng, (N, K) if layout == NT else (K, N), "bf16"), "bf16")
    out = []
    for rows in (M, 1400, 200):
        C = nans((rows, N), "f32")
        mp.op_gemm(1, layout, E_F32, rows, N, K, dA, K, dB, dB.shape[1], C, N)
        out.append(C)
    assert all(torch.equal(out[0][:c.shape[0]], c) for c in out[1:])


@pytest.mark.parametrize("rows", [1, 4, 60, 66, 2048, 2052, 5000])
def test_affine_gradient_partials(rows):
    """The LayerNorm affine gradients are reduced from one partial row per block: 1, a wave's
    share more or less, 512 (the most that one launch takes), 513 and 1,024 partial rows.
    Sums of up to 5,000 fp32 terms in any order: 1e-5 of the largest."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng, n = np.random.default_rng(rows), 132
    announce(f"affine gradient partials rows={rows}")
    X, dY = rng.standard_normal((2, rows, n)).astype(np.float32)
    mean, rstd = X.mean(1), 1 / np.sqrt(X.astype(np.float64).var(1) + 1e-6)
    gg, gb = to_dev(np.ones(n), "f32"), to_dev(np.zeros(n), "f32")
    scratch = torch.empty(mp.op_scratch_bytes(rows, 1, n, 0), dtype=torch.uint8, device=dev)
    tm, tr = to_dev(mean, "f32"), to_dev(rstd, "f32")
    mp.op_layernorm_bwd(0, to_dev(dY, "f32"), to_dev(X, "f32"), tm, tr, to_dev(np.ones(n), "f32"),
                        rows, n, None, None, None, gg, gb, scratch)
    xhat = (X - host(tm)[:, None]) * host(tr)[:, None]
    assert max_rel(host(gg), 1 + (dY * xhat).sum(0)) < 1e-5
    assert max_rel(host(gb), dY.astype(np.float64).sum(0)) < 1e-5


def test_attention_f32_scores_of_minus_infinity():
    """Scores that overflow to -inf have weight 0 and leave the others' softmax alone, also
    where one wave of the fp32 forward (tiles w, w + 4, ... of 16 keys) meets nothing else:
    all of wave 1's keys, wave 2's first tile and one key of wave 3 here.  Against the oracle,
    which holds the scores in 64 bits; 1e-5 as for the other fp32 attention tests."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    heads, d, N = 2, 32, 200
    h = heads * d
    rng = np.random.default_rng(5)
    announce(f"fp32 attention with scores of -inf heads={heads} d={d} N={N}")
    qkv, dO = rnd(rng, (N, 3 * h), "f32", 1.5), rnd(rng, (N, h), "f32")
    first = np.arange(heads) * d                       # component 0 of each head
    keys = [j for j in range(N) if j // 16 % 4 == 1 or j // 16 == 2 or j == 50]
    qkv[:, first] = 1e20
    qkv[:, h + first] = 0.0
    qkv[np.ix_(keys, h + first)] = -1e20               # 1e20 * -1e20 overflows
    q, k, v = qkv[:, :h], qkv[:, h:2 * h], qkv[:, 2 * h:]
    cu = np.array([0, N], np.int32)
    ro, rlse = oracle.attention(q, k, v, cu, heads, d)
    ref = oracle.attention_bwd(q, k, v, ro, dO, rlse, cu, heads, d)
    o, lse, dqkv = nans((N, h), "f32"), nans((heads, N), "f32"), nans((N, 3 * h), "f32")
    scratch = torch.empty(mp.op_scratch_bytes(N, heads, h, 1), dtype=torch.uint8, device=dev)
    tq = to_dev(qkv, "f32")
    mp.op_attention_fwd(0, tq, N, heads, d, cu, o, lse, scratch)
    mp.op_attention_bwd(0, tq, o, to_dev(dO, "f32"), lse, N, heads, d, cu, dqkv, scratch)
    got = host(dqkv)
    rest = np.setdiff1d(np.arange(h), first)           # (dK's component 0 is 1e20 times dS)
    errs = [max_rel(host(o), ro), max_rel(host(lse), rlse.T), max_rel(got[:, :h], ref[0]),
            max_rel(got[:, h + rest], ref[1][:, rest]), max_rel(got[:, 2 * h:], ref[2])]
    assert max(errs) < 1e-5, errs


@pytest.mark.parametrize("layout", [NT, NN])
@pytest.mark.parametrize("N,K", [(1280, 1000), (392, 68), (388, 20)])
def test_gemm_f32_rows_of_a_taller_product(layout, N, K):
    """6,000 rows run the 128x128 kernel, 1,400 and 200 of them the 32x32 one (up to 128 tiles
    of 128x128); both add K in the same order, so the rows are the same bits: with K of whole
    and ragged quarters of 16-deep steps, and of fewer steps than quarters."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    rng, M = np.random.default_rng(K), 6000
    announce(f"gemm f32 rows of a taller product layout={layout} N={N} K={K}")
    A, B = rnd(rng, (M, K), "f32"), rnd(rng, (N, K) if layout == NT else (K, N), "f32")
    dA, dB, bias = to_dev(A, "f32"), to_dev(B, "f32"), to_dev(rnd(rng, (N,), "f32"), "f32")
    for epi in (E_F32, E_GELU):
        out = []
        for rows in (M, 1400, 200):
            C = nans((rows, N), "f32")
            mp.op_gemm(0, layout, epi, rows, N, K, dA, K, dB, dB.shape[1], C, N,
                       bias=None if epi == E_F32 else bias)
            out.append(C)
        if epi == E_F32:
            assert max_rel(host(out[0]), _ref_product(layout, A, B)) < 2e-5
        assert all(torch.equal(out[0][:c.shape[0]], c) for c in out[1:]), epi


@pytest.mark.parametrize("dtype,N", [("f32", 131200), ("bf16", 1048640)])
def test_attention_more_blocks_than_one_launch(dtype, N):
    """One-row segments of 16 heads, more (segment, head) pairs than blocks of 256 threads fit
    into one launch of 2^32 threads: 2,099,200 pairs of eight blocks (fp32), 16,778,240 of one
    (bf16).  A row alone attends to itself: O is V to the bit, dV is dO to the type's rounding
    (2^-8 of up to 6, and of the weight's own), and dQ, dK are the rounding of a zero
    (dP - delta, 32 terms of up to 30 in two orders, times |k| <= 6: below 1e-4)."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    heads, d = 16, 32
    h = heads * d
    announce(f"{dtype} attention over {N} one-row segments, {heads} heads")
    gen = torch.Generator(device=dev).manual_seed(1)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    qkv = torch.randn((N, 3 * h), device=dev, generator=gen, dtype=t)
    dO = torch.randn((N, h), device=dev, generator=gen, dtype=t)
    o, lse, dqkv = nans((N, h), dtype), nans((heads, N), "f32"), nans((N, 3 * h), dtype)
    scratch = torch.empty(mp.op_scratch_bytes(N, heads, h, N), dtype=torch.uint8, device=dev)
    cu = np.arange(N + 1, dtype=np.int32)
    mp.op_attention_fwd(_dt(dtype), qkv, N, heads, d, cu, o, lse, scratch)
    mp.op_attention_bwd(_dt(dtype), qkv, o, dO, lse, N, heads, d, cu, dqkv, scratch)
    torch.cuda.synchronize()
    assert torch.equal(o, qkv[:, 2 * h:])
    assert (dqkv[:, 2 * h:] - dO).abs().max() < (6e-2 if dtype == "bf16" else 1e-4)
    assert dqkv[:, :2 * h].abs().max() < 1e-4


@pytest.mark.parametrize("d", [32, 80])
def test_attention_f32_at_any_float(d):
    """The fp32 attention takes tensors that start at any float: the same bits as for tensors
    on 16 bytes."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    lens, heads = [65, 17, 145], 2
    N, h = sum(lens), heads * d
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    announce(f"fp32 attention d={d} on tensors one to three floats off 16 bytes")
    gen = torch.Generator(device=dev).manual_seed(d)
    f32 = dict(dtype=torch.float32, device=dev)
    qkv, dO = (torch.randn((N, n), generator=gen, **f32) for n in (3 * h, h))
    scratch = torch.empty(mp.op_scratch_bytes(N, heads, h, 3), dtype=torch.uint8, device=dev)
    outs = []
    for off in range(4):
        def at(t):
            out = torch.full((t.numel() + 4,), float("nan"), **f32)[off:off + t.numel()]
            return out.view(t.shape).copy_(t)
        tq, tdo, o, dqkv = at(qkv), at(dO), at(torch.empty_like(dO)), at(torch.empty_like(qkv))
        lse = nans((heads, N), "f32")
        mp.op_attention_fwd(0, tq, N, heads, d, cu, o, lse, scratch)
        mp.op_attention_bwd(0, tq, o, tdo, lse, N, heads, d, cu, dqkv, scratch)
        outs.append((o, lse, dqkv))
    torch.cuda.synchronize()
    assert torch.isfinite(outs[0][2]).all()
    assert all(torch.equal(a, b) for out in outs[1:] for a, b in zip(outs[0], out))


# ---- one kernel at a time: the sizes below name the kernel that runs them, and
# ---- gemm_kernel has to agree ---------------------------------------------------------

def _dev_max_rel(x, ref):
    """max |x - ref| / max |ref| on the device, NaN if either side holds one"""
    return float((x.double() - ref).abs().max() / ref.abs().max())


def _gemm_operands(layout, dtype, M, N, K, seed):
    """Device operands of a product (rows of a K-major B padded to 8) and, in float64, A and B
    as [M][K] and [K][N]."""
    torch, dev = torch_dev()
    gen = torch.Generator(device=dev).manual_seed(seed)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    ldb = K if layout == NT else (N + 7) // 8 * 8
    A = torch.randn((K, M) if layout == TN else (M, K), device=dev, generator=gen).to(t)
    B = torch.randn((N if layout == NT else K, ldb), device=dev, generator=gen).to(t)
    A64, B64 = A.double(), B.double()
    return A, B, ldb, A64.T if layout == TN else A64, B64.T if layout == NT else B64[:, :N]


@pytest.mark.parametrize("layout,M,N,Ks", [
    (NT, 4100, 4360, (8, 64, 72, 136, 200, 264, 328, 520, 1000)),
    (NN, 5000, 2056, (8, 40, 64, 72, 136, 200, 264, 328, 520, 1000)),
    (TN, 2056, 2312, (1, 5, 63, 64, 77, 128, 250, 291, 700))])
def test_gemm_large_kernels(layout, M, N, Ks):
    """The large bf16 kernels on ragged M, N and K: less than a K tile, one to three, ragged
    last ones, several passes.  Against the product of the same values in float64; 1e-5 as for
    the other fp32 outputs."""
    import paper_2607_03229_amd as mp
    torch_dev()   # (torch's HIP runtime is loaded before the library)
    for K in Ks:
        assert mp.gemm_kernel(1, layout, E_F32, M, N, K) == "large"
        announce(f"gemm large kernel layout={layout} M={M} N={N} K={K}")
        A, B, ldb, A64, B64 = _gemm_operands(layout, "bf16", M, N, K, K)
        C = nans((M, N), "f32")
        mp.op_gemm(1, layout, E_F32, M, N, K, A, A.shape[1], B, ldb, C, N)
        assert _dev_max_rel(C, A64 @ B64) < 1e-5, K


@pytest.mark.parametrize("kernel,dtype,layout,M,N,K", [
    ("large", "bf16", NT, 4100, 4360, 200), ("large", "bf16", NN, 5000, 2056, 136),
    ("large", "bf16", NN, 5000, 2056, 1000),
    ("64x128", "bf16", NT, 645, 2040, 2040), ("64x128", "bf16", NN, 645, 2040, 2040),
    ("128x128", "bf16", NT, 1100, 2040, 2040), ("128x128", "bf16", NN, 1100, 2040, 2040),
    ("general", "bf16", NT, 1100, 1026, 200), ("general", "bf16", NN, 1100, 1026, 200),
    ("general", "f32", NT, 1430, 1426, 100), ("general", "f32", NN, 1430, 1426, 100),
    ("general", "f32", NN, 2050, 1283, 388)])
def test_gemm_epilogues_by_kernel(kernel, dtype, layout, M, N, K):
    """Every epilogue of each kernel that test_gemm_epilogues' sizes don't reach, with the
    bounds of that test, against float64."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    dt, tol = _dt(dtype), TOL[dtype]
    A, B, ldb, A64, _ = _gemm_operands(layout, dtype, M, N, K, M)
    t = A.dtype
    B = (B.float() * 0.1).to(t)
    B64 = B.double().T if layout == NT else B.double()[:, :N]
    gen = torch.Generator(device=dev).manual_seed(1)
    bias = torch.randn(N, device=dev, generator=gen).to(t)
    acc = A64 @ B64
    u = acc + bias.double()
    phi = torch.special.ndtr(u)
    dgelu = phi + u * torch.exp(-0.5 * u * u) / np.sqrt(2 * np.pi)

    def go(epi, C, **kw):
        assert mp.gemm_kernel(dt, layout, epi, M, N, K) == kernel
        announce(f"{kernel} {dtype} layout={layout} M={M} N={N} K={K} epilogue {epi}")
        mp.op_gemm(dt, layout, epi, M, N, K, A, A.shape[1], B, ldb, C, N, **kw)
        return C

    assert _dev_max_rel(go(E_STORE, nans((M, N), dtype), bias=bias), u) < tol
    C2 = nans((M, N), dtype)
    assert _dev_max_rel(go(E_GELU, nans((M, N), dtype), bias=bias, C2=C2, ldc2=N), u * phi) < tol
    assert _dev_max_rel(C2, dgelu) < tol
    assert _dev_max_rel(go(E_GELU, nans((M, N), dtype), bias=bias), u * phi) < tol
    R = torch.randn((M, N), device=dev, generator=gen, dtype=torch.float32)
    assert _dev_max_rel(go(E_RESID, R.clone(), bias=bias, aux=R, ld_aux=N), R.double() + u) < 2e-5
    C = R.clone()   # in place
    assert _dev_max_rel(go(E_RESID, C, bias=bias, aux=C, ld_aux=N), R.double() + u) < 2e-5
    assert _dev_max_rel(go(E_RESID, nans((M, N), "f32"), bias=bias), u) < 2e-5
    G = torch.rand((M, N), device=dev, generator=gen).to(t)
    assert _dev_max_rel(go(E_GELUBWD, nans((M, N), dtype), aux=G, ld_aux=N),
                        acc * G.double()) < tol
    assert _dev_max_rel(go(E_F32, R.clone(), beta=1), R.double() + acc) < 2e-5


@pytest.mark.parametrize("kernel,dtype,layout,M,N,K,kps", [
    ("large", "bf16", NT, 4100, 4360, 200, 128), ("large", "bf16", NN, 5000, 2056, 200, 64),
    ("large", "bf16", TN, 1040, 1032, 4100, 1088), ("general", "f32", TN, 700, 700, 1001, 256),
    ("general", "f32", NN, 700, 700, 1000, 256), ("general", "f32", NT, 700, 700, 1000, 256),
    ("f32_32x32", "f32", NN, 333, 264, 1000, 320)])
def test_gemm_split_k_by_kernel(kernel, dtype, layout, M, N, K, kps):
    """K splits, each against its own range of K in float64."""
    import paper_2607_03229_amd as mp
    torch_dev()
    assert mp.gemm_kernel(_dt(dtype), layout, E_F32, M, N, K, kps) == kernel
    announce(f"split k {kernel} {dtype} layout={layout} M={M} N={N} K={K} kps={kps}")
    A, B, ldb, A64, B64 = _gemm_operands(layout, dtype, M, N, K, kps)
    splits = -(-K // kps)
    part = nans((splits, M, N), "f32")
    mp.op_gemm(_dt(dtype), layout, E_F32, M, N, K, A, A.shape[1], B, ldb, part, N,
               k_per_split=kps, split_stride=M * N)
    for s in range(splits):
        sl = slice(s * kps, min(K, (s + 1) * kps))
        assert _dev_max_rel(part[s], A64[:, sl] @ B64[sl]) < 2e-5, s


@pytest.mark.parametrize("layout", [NT, NN])
def test_gemm_bf16_rows_have_one_value(layout):
    """5,000 rows run the large kernel, 1,100 of them 128x128 tiles, 645 64x128 and 200 64x64
    (with K of 32 tiles less 8): the same bits from all four, plain, with GELU and with the
    residual, as an item's rows may not change with what shares its micro-batch."""
    import paper_2607_03229_amd as mp
    torch, dev = torch_dev()
    N = K = 2040
    A, B, ldb, _, _ = _gemm_operands(layout, "bf16", 5000, N, K, 3)
    B = (B.float() * 0.1).to(B.dtype)
    gen = torch.Generator(device=dev).manual_seed(2)
    bias = torch.randn(N, device=dev, generator=gen).to(B.dtype)
    R = torch.randn((5000, N), device=dev, generator=gen, dtype=torch.float32)
    for epi in (E_STORE, E_GELU, E_RESID, E_F32):
        out = []
        for rows, kernel in ((5000, "large"), (1100, "128x128"), (645, "64x128"), (200, "64x64")):
            assert mp.gemm_kernel(1, layout, epi, rows, N, K) == kernel
            announce(f"{kernel} layout={layout} epilogue {epi}, {rows} rows")
            C = nans((rows, N), "f32" if epi in (E_RESID, E_F32) else "bf16")
            mp.op_gemm(1, layout, epi, rows, N, K, A, A.shape[1], B, ldb, C, N,
                       bias=None if epi == E_F32 else bias,
                       aux=R if epi == E_RESID else None, ld_aux=N)
            out.append(C)
        assert torch.isfinite(out[0]).all()
        assert all(torch.equal(out[0][:c.shape[0]], c) for c in out[1:]), epi
