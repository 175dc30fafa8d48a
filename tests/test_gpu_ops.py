"""Parity of the single HIP operations against the CPU oracle, through the C ABI.

Tolerances (max |got - ref| / max |ref| per tensor): 1e-4 in fp32, 2e-2 in bf16.
The oracle is fed the values the kernel is fed (bf16-rounded where bf16)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import stage_oracle as so
from paper_2503_01328_amd import binding as po
from paper_2503_01328_amd import inputs as syn
from paper_2503_01328_amd.harness import check_parity, max_rel_err

pytestmark = pytest.mark.gpu

DT = {"f32": (po.PO_F32, torch.float32, 1e-4), "bf16": (po.PO_BF16, torch.bfloat16, 2e-2)}


def _dev(a, tdt, dev):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(dev).to(tdt).contiguous()


def _rand(rng, shape, dtype, scale=1.0, shift=0.0):
    a = (rng.standard_normal(shape) * scale + shift).astype(np.float32)
    return syn.round_to_bf16(a) if dtype == "bf16" else a


def _np(t):
    return t.to(torch.float32).cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,h", [(1, 64), (7, 256), (130, 1024), (33, 5120), (5, 2048), (3, 3584), (4, 8192)])
def test_layernorm_forward_and_backward(gpu_device, dtype, rows, h):
    code, tdt, tol = DT[dtype]
    rng = np.random.default_rng(rows * 1000 + h)
    x = _rand(rng, (rows, h), dtype, 2.0, 0.5)
    g = _rand(rng, (h,), dtype, 0.1, 1.0)
    b = _rand(rng, (h,), dtype, 0.1)
    dn = _rand(rng, (rows, h), dtype)
    dres = _rand(rng, (rows, h), dtype)
    xd, gd, bd, dnd, dresd = (_dev(a, tdt, gpu_device) for a in (x, g, b, dn, dres))
    y = torch.empty_like(xd)
    po.po_op_layernorm_forward(code, xd, gd, bd, y, rows, h, 1e-5)
    ref, cache = so.layernorm_forward(x.astype(np.float64), g.astype(np.float64), b.astype(np.float64), 1e-5)
    assert max_rel_err(_np(y), ref) < tol
    ws = torch.empty(po.po_op_layernorm_backward_workspace(rows, h) // 4, dtype=torch.float32, device=gpu_device)
    dx = torch.empty_like(xd)
    dg0 = rng.standard_normal(h).astype(np.float32)
    db0 = rng.standard_normal(h).astype(np.float32)
    dg, db = torch.from_numpy(dg0).to(gpu_device), torch.from_numpy(db0).to(gpu_device)
    po.po_op_layernorm_backward(code, dnd, xd, gd, dresd, dx, dg, db, ws, rows, h, 1e-5)
    rdx, rdg, rdb = so.layernorm_backward(dn.astype(np.float64), cache, g.astype(np.float64))
    assert max_rel_err(_np(dx), rdx + dres) < tol
    assert max_rel_err(_np(dg) - dg0, rdg) < max(tol, 1e-4)  # fp32 accumulators added into existing values
    assert max_rel_err(_np(db) - db0, rdb) < max(tol, 1e-4)
    # without a residual
    po.po_op_layernorm_backward(code, dnd, xd, gd, None, dx, dg, db, ws, rows, h, 1e-5)
    assert max_rel_err(_np(dx), rdx) < tol


GEMM_SHAPES_GENERIC = [(1, 1, 1), (5, 7, 3), (64, 64, 16), (70, 130, 45), (128, 256, 256)]


def _gemm_case(gpu_device, dtype, ta, tb, M, N, K, epilogue, force_generic):
    code, tdt, tol = DT[dtype]
    rng = np.random.default_rng(M * 7 + N * 3 + K + ta * 2 + tb)
    A = _rand(rng, (K, M) if ta else (M, K), dtype)
    B = _rand(rng, (N, K) if tb else (K, N), dtype, 0.05)
    Ad, Bd = _dev(A, tdt, gpu_device), _dev(B, tdt, gpu_device)
    a64 = (A.T if ta else A).astype(np.float64)
    b64 = (B.T if tb else B).astype(np.float64)
    ref = a64 @ b64
    lda, ldb = A.shape[1], B.shape[1]
    kw = dict(force_generic=force_generic)
    if epilogue == "plain":
        out = torch.empty(M, N, dtype=tdt, device=gpu_device)
        po.po_op_gemm(code, ta, tb, M, N, K, Ad, lda, Bd, ldb, out=out, **kw)
        assert max_rel_err(_np(out), ref) < tol
    elif epilogue == "bias_residual":
        bias = _rand(rng, (N,), dtype)
        res = _rand(rng, (M, N), dtype)
        out = torch.empty(M, N, dtype=tdt, device=gpu_device)
        po.po_op_gemm(code, ta, tb, M, N, K, Ad, lda, Bd, ldb, bias=_dev(bias, tdt, gpu_device),
                      residual=_dev(res, tdt, gpu_device), out=out, **kw)
        assert max_rel_err(_np(out), ref + bias + res) < tol
    elif epilogue == "bias_gelu":
        bias = _rand(rng, (N,), dtype)
        out = torch.empty(M, N, dtype=tdt, device=gpu_device)
        g = torch.empty(M, N, dtype=tdt, device=gpu_device)
        po.po_op_gemm(code, ta, tb, M, N, K, Ad, lda, Bd, ldb, bias=_dev(bias, tdt, gpu_device), out=out,
                      gelu_out=g, **kw)
        assert max_rel_err(_np(out), ref + bias) < tol
        assert max_rel_err(_np(g), so.gelu(_np(out).astype(np.float64))) < tol  # gelu of the stored (rounded) u
    elif epilogue == "gelu_backward":
        u = _rand(rng, (M, N), dtype, 1.5)
        out = torch.empty(M, N, dtype=tdt, device=gpu_device)
        g = torch.empty(M, N, dtype=tdt, device=gpu_device)
        po.po_op_gemm(code, ta, tb, M, N, K, Ad, lda, Bd, ldb, out=out, gelu_out=g,
                      gelu_u=_dev(u, tdt, gpu_device), **kw)
        assert max_rel_err(_np(out), ref * so.gelu_derivative(u.astype(np.float64))) < tol
        assert max_rel_err(_np(g), so.gelu(u.astype(np.float64))) < tol
    elif epilogue == "accumulate":
        acc0 = rng.standard_normal((M, N)).astype(np.float32)
        acc = torch.from_numpy(acc0).to(gpu_device)
        po.po_op_gemm(code, ta, tb, M, N, K, Ad, lda, Bd, ldb, acc_f32=acc, **kw)
        assert max_rel_err(_np(acc) - acc0, ref) < max(tol, 2e-4)
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", GEMM_SHAPES_GENERIC)
def test_gemm_generic_all_forms(gpu_device, dtype, ta, tb, shape):
    _gemm_case(gpu_device, dtype, ta, tb, *shape, "plain", 1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("epilogue", ["bias_residual", "bias_gelu", "gelu_backward", "accumulate"])
def test_gemm_generic_epilogues(gpu_device, dtype, epilogue):
    _gemm_case(gpu_device, dtype, 0, 0, 70, 130, 45, epilogue, 1)


# MFMA path: 128-tiles (M, N multiples of 128), 256-tiles (>= 192 tiles of 256 x 256) and 256 x 192 tiles (N a
# multiple of 192 and a round of them cheaper), K multiple of 64 (one, two, three and many slices)
MFMA_SHAPES = [(128, 128, 64), (256, 384, 192), (384, 128, 1024), (4096, 3328, 128), (2048, 6144, 64),
               (4096, 3072, 192), (4096, 6144, 128), (2048, 6144, 512)]


def test_gemm_mfma_shapes_cover_every_tile():
    assert {po.po_op_gemm_tile(M, N) for M, N, _ in MFMA_SHAPES} == {(128, 128), (256, 256), (256, 192)}


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("shape", MFMA_SHAPES)
def test_gemm_mfma_all_forms(gpu_device, ta, tb, shape):
    _gemm_case(gpu_device, "bf16", ta, tb, *shape, "plain", 0)


@pytest.mark.parametrize("epilogue", ["bias_residual", "bias_gelu", "gelu_backward", "accumulate"])
@pytest.mark.parametrize("shape", [(256, 384, 192), (4096, 3328, 128), (2048, 6144, 192)])
def test_gemm_mfma_epilogues(gpu_device, epilogue, shape):
    form = {"accumulate": (1, 0), "gelu_backward": (0, 1)}.get(epilogue, (0, 0))
    _gemm_case(gpu_device, "bf16", *form, *shape, epilogue, 0)


# the kernel for fp32 and for bf16 results of any size: one row, tiles that end inside, K with a remainder, and result
# sizes on both sides of the lines between its forms (32 x 32 and 64 x 64 tiles, 8, 4, 2 and 1 waves); a multiple of 8
# in N, and in whichever of M and K is contiguous, is what its 16-byte loads need.  (1100, 1032, 320) and the last two are, in bf16, results
# whose large tiles (128 x 128, 256 x 192, 256 x 256) end inside; the three between are, in fp32, results of more tiles of
# 16 x 16 than one round and few enough of 32 x 32, of eight and four waves.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (40, 24, 520), (1, 64, 72), (33, 200, 1096), (1000, 520, 264),
                                   (1000, 520, 1160), (1032, 2008, 72), (2056, 2008, 328), (1100, 1032, 320),
                                   (200, 520, 264), (200, 520, 520), (680, 576, 72), (1733, 6152, 128), (1733, 8200, 128)])
def test_gemm_small_edges(gpu_device, dtype, ta, tb, M, N, K):
    """Against the product in fp64.  K sums of fp32 products each round by at most 2^-24 of a partial sum, independent of
    each other: 2^-24 sqrt(K) relative (2-norm) is generous; a bf16 result (8 significant bits) adds its own rounding,
    at most 2^-8 of every element and so of the norm."""
    code, tdt, _ = DT[dtype]
    if ta:
        M = 8 * -(-M // 8)
    g = torch.Generator(device=gpu_device)
    g.manual_seed(M + N + K + ta)
    # operands followed by NaNs: what lies past an operand's end must not reach the result
    def rand(rows, cols):
        t = torch.full((rows * cols + 70000,), float("nan"), dtype=tdt, device=gpu_device)
        t[:rows * cols] = torch.randn(rows * cols, generator=g, device=gpu_device).to(tdt)
        return t[:rows * cols].view(rows, cols)
    A, B = rand(*((K, M) if ta else (M, K))), rand(*((N, K) if tb else (K, N)))
    bias, res, u = rand(1, N)[0], rand(M, N), rand(M, N)
    a64, b64 = (A.t() if ta else A).double(), (B.t() if tb else B).double()
    ref = a64 @ b64
    rel = lambda got, want: float((got.double() - want).norm() / want.norm())
    sums = 2.0 ** -24 * K ** 0.5
    tol = sums + 2.0 ** -23 + (2.0 ** -8 if dtype == "bf16" else 0.0)
    call = lambda **kw: po.po_op_gemm(code, ta, tb, M, N, K, A, A.shape[1], B, B.shape[1], **kw)
    out, gel = torch.empty(M, N, dtype=tdt, device=gpu_device), torch.empty(M, N, dtype=tdt, device=gpu_device)
    call(out=out, bias=bias, residual=res)
    assert rel(out, ref + bias.double() + res.double()) < tol
    call(out=out, bias=bias, gelu_out=gel)
    assert rel(out, ref + bias.double()) < tol
    gelu = lambda x: torch.nn.functional.gelu(x, approximate="tanh")
    assert rel(gel, gelu(out.double())) < tol + 2e-6  # the gate's exp2 and reciprocal: 1 ulp each of values near one
    ud = u.double().requires_grad_()
    gelu(ud).sum().backward()
    call(out=out, gelu_u=u, gelu_out=gel)
    assert rel(out, ref * ud.grad) < tol + 2e-6 and rel(gel, gelu(u.double())) < tol + 2e-6
    acc = torch.ones(M, N, device=gpu_device)
    call(acc_f32=acc)
    assert rel(acc, ref + 1.0) < sums + 2.0 ** -23


# fp32 results of up to 256 tiles of 16 x 16 and one more row of tiles: less than a tile, fewer chunks of 32 k than waves, more than
# the waves have stages, K that ends inside a chunk.
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(4, 4, 4), (16, 20, 36), (100, 72, 252), (36, 48, 1024), (20, 32, 1060), (40, 36, 4108),
                                   (256, 256, 260), (260, 256, 1156)])
def test_gemm_f32_tiles_of_16(gpu_device, ta, tb, M, N, K):
    """Against fp64 as above: 2^-24 sqrt(K) for the sums, 2^-23 for the epilogue's additions."""
    g = torch.Generator(device=gpu_device)
    g.manual_seed(M + N + K + 2 * ta + tb)
    def rand(rows, cols):  # followed by NaNs
        t = torch.full((rows * cols + 5000,), float("nan"), device=gpu_device)
        t[:rows * cols] = torch.randn(rows * cols, generator=g, device=gpu_device)
        return t[:rows * cols].view(rows, cols)
    A, B, bias = rand(*((K, M) if ta else (M, K))), rand(*((N, K) if tb else (K, N))), rand(1, N)[0]
    ref = (A.t() if ta else A).double().contiguous() @ (B.t() if tb else B).double().contiguous()
    tol = 2.0 ** -24 * K ** 0.5 + 2.0 ** -23
    out, acc = torch.full((M + 4, N), 7.0, device=gpu_device), torch.ones(M, N, device=gpu_device)
    po.po_op_gemm(po.PO_F32, ta, tb, M, N, K, A, A.shape[1], B, B.shape[1], out=out, bias=bias)
    po.po_op_gemm(po.PO_F32, ta, tb, M, N, K, A, A.shape[1], B, B.shape[1], acc_f32=acc)
    assert (out[M:] == 7).all()
    for got, want in ((out[:M], ref + bias.double()), (acc, ref + 1.0)):
        assert (got.double() - want).norm() < tol * want.norm()


# Equal rows of A give equal rows of the result, whichever tile they lie in and whichever XCD works on it: whole tiles of 128, 256
# and 256 x 192, tiles that end inside, and both sizes of small tiles, forward, input-gradient and weight-gradient layouts.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(2048, 2048, 2048), (1736, 2048, 8192), (4096, 4096, 4096), (4096, 3072, 4096),
                                   (104, 1024, 1024), (520, 1536, 1024)])
def test_gemm_row_does_not_depend_on_its_place(gpu_device, dtype, ta, tb, M, N, K):
    code, tdt, _ = DT[dtype]
    g = torch.Generator(device=gpu_device)
    g.manual_seed(M + N + K)
    rand = lambda *size: torch.randn(*size, generator=g, device=gpu_device).to(tdt)
    row, B = rand(K), rand(*((N, K) if tb else (K, N)))
    A = row[:, None].repeat(1, M) if ta else row.repeat(M, 1)
    out = torch.zeros(M, N, dtype=torch.float32 if ta else tdt, device=gpu_device)
    po.po_op_gemm(code, ta, tb, M, N, K, A, A.shape[1], B, B.shape[1], **{"acc_f32" if ta else "out": out})
    assert torch.equal(out, out[:1].expand(M, N))


# fp32 results of more tiles than one round of 32 x 32 ones: 128 x 64, 64 x 64 and 32 x 64 tiles (two groups of waves, never for
# one chunk of K) with one chunk (32) and part of one, as many as there are stages, one more, a first and a second half, chunks
# that leave a group without a last one, a K that ends inside a chunk and one that ends with it, results that end inside a tile
# and with it, and rows of operands that are longer than what is used of them.
F32_TILES = {2: [(1028, 964, 20), (1028, 1088, 32), (1024, 1088, 64), (1028, 964, 100), (1028, 964, 132), (1028, 964, 292)],
             1: [(964, 964, 28), (1024, 1024, 32), (964, 964, 60), (964, 964, 100), (960, 1024, 128), (964, 964, 132), (964, 964, 292)],
             0: [(484, 1020, 36), (512, 1024, 64), (484, 1020, 100), (548, 572, 132), (548, 572, 160), (484, 1020, 224), (544, 576, 516)],
             None: [(960, 964, 4), (1028, 964, 4)]}  # so short a K stays with the vector kernel


def test_gemm_f32_tiles_cover_every_tile():
    form = po.lib["_ZN2po13gemm_f32_formEiPKiS1_i"]
    form.restype, form.argtypes = ctypes.c_int, [ctypes.c_int, ctypes.POINTER(ctypes.c_int), ctypes.POINTER(ctypes.c_int), ctypes.c_int]
    for want in (0, 1, 2):
        for M, N, K in F32_TILES[want]:
            assert form(1, ctypes.c_int(M), ctypes.c_int(N), K) == want, (M, N, K)
    # the weight gradients of a layer (QKV, output projection, FC1, FC2) in one launch: the fp32 stages of
    # test_grouped_weight_gradients_of_any_shape
    four = lambda *v: (ctypes.c_int * 4)(*v)
    group = lambda h, f, seq: form(4, four(h, h, h, f), four(3 * h, h, f, h), seq)
    assert [group(192, 768, 200), group(512, 1536, 37), group(1024, 2048, 300), group(384, 1536, 100)] == [0, 1, 1, 2]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [shape for shapes in F32_TILES.values() for shape in shapes])
def test_gemm_f32_tiles(gpu_device, ta, tb, M, N, K):
    """Bounds as in test_gemm_small_edges."""
    g = torch.Generator(device=gpu_device)
    g.manual_seed(M + N + K + ta)
    def rand(rows, cols):  # NaNs between the rows and behind the last one
        t = torch.full((rows * (cols + 8) + 70000,), float("nan"), device=gpu_device)[:rows * (cols + 8)].view(rows, cols + 8)
        t[:, :cols] = torch.randn(rows, cols, generator=g, device=gpu_device)
        return t[:, :cols]
    A, B = rand(*((K, M) if ta else (M, K))), rand(*((N, K) if tb else (K, N)))
    ref = (A.t() if ta else A).double() @ (B.t() if tb else B).double()
    sums = 2.0 ** -24 * K ** 0.5 + 2.0 ** -23
    got = torch.full((M, N), 7.0, device=gpu_device)
    bias = torch.randn(N, generator=g, device=gpu_device)
    po.po_op_gemm(po.PO_F32, ta, tb, M, N, K, A, A.stride(0), B, B.stride(0), bias=bias, out=got)
    assert (got.double() - ref - bias.double()).norm() < sums * (ref + bias.double()).norm()
    po.po_op_gemm(po.PO_F32, ta, tb, M, N, K, A, A.stride(0), B, B.stride(0), acc_f32=got)
    assert (got.double() - 2 * ref - bias.double()).norm() < 2 * sums * (2 * ref + bias.double()).norm()
    acc = [torch.zeros(M, N, device=gpu_device) for _ in range(2)]
    for generic in (0, 1):  # the matrix cores add in another order
        po.po_op_gemm(po.PO_F32, ta, tb, M, N, K, A, A.stride(0), B, B.stride(0), acc_f32=acc[generic], force_generic=generic)
    assert torch.equal(acc[0], acc[1]) == ((M, N, K) in F32_TILES[None])


# The length of fp32 chains of additions: each of the three tiles, K that ends with a chunk of 32 and inside one.
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K,chains", [(640, 512, 1024, 8), (780, 640, 2560, 4), (1024, 1024, 1024, 4), (2056, 2008, 328, 4),
                                          (1024, 4096, 1024, 4), (2004, 2936, 788, 4), (2048, 2048, 8192, 4)])
def test_gemm_f32_sums_in_short_chains(gpu_device, ta, tb, M, N, K, chains):
    """A chain of n additions of equal terms of random sign leaves the sum of n roundings, the i-th of sqrt(i) terms: n / sqrt(2)
    roundings of a term, over its chains sqrt(K n / 2), and relative to the sum of K terms sqrt(n / 2), n = K / chains.  The
    additions of the chains' sums add sqrt(chains / 2).  A rounding is 2^-24 of the value at most and 0.42 of that (root of the
    mean square) over values of any size; 0.5 leaves a fifth.  Half as many chains are 1.4 times as far off."""
    g = torch.Generator(device=gpu_device)
    g.manual_seed(M + N + K + ta)
    rand = lambda *size: torch.randn(*size, generator=g, device=gpu_device)
    A, B = rand(*((K, M) if ta else (M, K))), rand(*((N, K) if tb else (K, N)))
    got = torch.zeros(M, N, device=gpu_device)
    po.po_op_gemm(po.PO_F32, ta, tb, M, N, K, A, A.shape[1], B, B.shape[1], acc_f32=got)
    ref = (A.t() if ta else A).double() @ (B.t() if tb else B).double()
    assert (got.double() - ref).norm() < 0.5 * 2.0 ** -24 * (K / chains / 2 + chains / 2) ** 0.5 * ref.norm()


# Short K under many tiles stays with the vector kernel, bit for bit; on the other side of the line the order of the sums is
# another one.
@pytest.mark.parametrize("dtype,ta,M,N,K,vector", [("f32", 1, 1024, 512, 16, 1), ("f32", 1, 1024, 512, 20, 0),
                                                   ("f32", 1, 448, 1024, 16, 0), ("f32", 0, 520, 1000, 12, 1),
                                                   ("f32", 1, 4096, 4096, 32, 1), ("f32", 1, 4096, 2048, 40, 1),
                                                   ("f32", 1, 4096, 2048, 52, 0), ("f32", 1, 4096, 1984, 40, 0),
                                                   ("bf16", 0, 2048, 2056, 16, 1), ("bf16", 0, 2048, 2056, 24, 0)])
def test_gemm_of_short_k_runs_on_the_vector_kernel(gpu_device, dtype, ta, M, N, K, vector):
    code, tdt, _ = DT[dtype]
    g = torch.Generator(device=gpu_device)
    g.manual_seed(M + N + K)
    A = torch.randn(*((K, M) if ta else (M, K)), generator=g, device=gpu_device).to(tdt)
    B = torch.randn(K, N, generator=g, device=gpu_device).to(tdt)
    out = [torch.zeros(M, N, device=gpu_device) for _ in range(2)]
    for generic in (1, 0):  # accumulated: fp32 results in either type
        po.po_op_gemm(code, ta, 0, M, N, K, A, A.shape[1], B, N, acc_f32=out[generic], force_generic=generic)
    assert torch.equal(out[0], out[1]) == bool(vector)
    want = (A.double().t().contiguous() if ta else A.double()) @ B.double()
    assert (out[0].double() - want).norm() < (2.0 ** -24 * K ** 0.5 + 2.0 ** -23) * want.norm()


# a GeLU backward is multiplied onto the sum of product, bias and residual: one row, few tiles, and results whose large tiles
# end inside, whose kernel has no such epilogue and leaves these calls to the small tiles
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1, 64, 64), (200, 200, 128), (905, 4096, 1088), (1733, 8200, 128)])
@pytest.mark.parametrize("with_bias,with_residual", [(1, 0), (0, 1), (1, 1)])
def test_gemm_gelu_backward_of_a_sum(gpu_device, tb, M, N, K, with_bias, with_residual):
    g = torch.Generator(device=gpu_device)
    g.manual_seed(M + N + K)
    rand = lambda *size: torch.randn(*size, generator=g, device=gpu_device).bfloat16()
    A, B = rand(M, K), rand(*((N, K) if tb else (K, N)))
    bias, res, u = 8 * rand(N), 8 * rand(M, N), rand(M, N)
    ud = u.double().requires_grad_()
    torch.nn.functional.gelu(ud, approximate="tanh").sum().backward()
    ref = A.double() @ (B.double().t().contiguous() if tb else B.double())
    ref = (ref + with_bias * bias.double() + with_residual * res.double()) * ud.grad
    out, gel = torch.empty_like(u), torch.empty_like(u)
    po.po_op_gemm(po.PO_BF16, 0, tb, M, N, K, A, K, B, B.shape[1], out=out, gelu_out=gel, gelu_u=u,
                  bias=bias if with_bias else None, residual=res if with_residual else None)
    # the rounding of the result to bf16 (2^-8 of it at most); the fp32 sums and the slope are far below
    assert float((out.double() - ref).norm() / ref.norm()) < 2.0 ** -8


def test_gemm_grouped_equals_single_launches_and_the_oracle(gpu_device):
    """Four weight-gradient products of different shapes in one launch: each accumulator equals, bit for bit, what
    the single launch of that product leaves, and the fp64 product within the bf16 tolerance.  Tile counts
    8 + 24 + 4 + 257 = 293 make two rounds, the second one ragged."""
    rng = np.random.default_rng(11)
    shapes = [(512, 1024, 192), (2048, 768, 64), (256, 1024, 128), (256, 65792, 64)]
    probs, single, refs, acc0s = [], [], [], []
    for M, N, K in shapes:
        A = _rand(rng, (K, M), "bf16")
        B = _rand(rng, (K, N), "bf16", 0.05)
        acc0 = rng.standard_normal((M, N)).astype(np.float32)
        Ad, Bd = _dev(A, torch.bfloat16, gpu_device), _dev(B, torch.bfloat16, gpu_device)
        acc = torch.from_numpy(acc0).to(gpu_device)
        alone = torch.from_numpy(acc0).to(gpu_device)
        po.po_op_gemm(po.PO_BF16, 1, 0, M, N, K, Ad, M, Bd, N, acc_f32=alone)
        probs.append((M, N, K, Ad, M, Bd, N, acc, N))
        single.append(alone)
        refs.append(A.T.astype(np.float64) @ B.astype(np.float64))
        acc0s.append(acc0)
    po.po_op_gemm_grouped(probs)
    torch.cuda.synchronize()
    for p, alone, ref, acc0 in zip(probs, single, refs, acc0s):
        assert torch.equal(p[7], alone)
        assert max_rel_err(_np(p[7]) - acc0, ref) < 2e-2
    # one problem alone, fewer tiles than compute units
    M, N, K = 256, 512, 64
    A = _rand(rng, (K, M), "bf16")
    B = _rand(rng, (K, N), "bf16")
    acc = torch.zeros(M, N, device=gpu_device)
    po.po_op_gemm_grouped([(M, N, K, _dev(A, torch.bfloat16, gpu_device), M, _dev(B, torch.bfloat16, gpu_device), N,
                            acc, N)])
    assert max_rel_err(_np(acc), A.T.astype(np.float64) @ B.astype(np.float64)) < 2e-2
    with pytest.raises(po.PipeOffloadError):  # 384 is no multiple of 256
        po.po_op_gemm_grouped([(384, 512, 64, acc, 384, acc, 512, acc, 512)])
    with pytest.raises(po.PipeOffloadError):
        po.po_op_gemm_grouped([(256, 512, 64, acc, 256, acc, 512, acc, 512)] * 5)


def test_gemm_rejects_bad_arguments(gpu_device):
    a = torch.zeros(64, 64, device=gpu_device)
    with pytest.raises(po.PipeOffloadError):
        po.po_op_gemm(po.PO_F32, 0, 0, 64, 64, 64, a, 32, a, 64, out=a)  # lda too small
    with pytest.raises(po.PipeOffloadError):
        po.po_op_gemm(po.PO_F32, 0, 0, 64, 64, 64, a, 64, a, 64)  # no output
    with pytest.raises(po.PipeOffloadError):
        po.po_op_gemm(9, 0, 0, 64, 64, 64, a, 64, a, 64, out=a)  # bad dtype
    with pytest.raises(po.PipeOffloadError):
        po.po_op_gemm(po.PO_F32, 0, 0, 0, 64, 64, a, 64, a, 64, out=a)  # empty


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("s,h,a", [(1, 64, 1), (5, 64, 2), (64, 128, 2), (65, 256, 4), (200, 256, 2), (130, 512, 2)])
@pytest.mark.parametrize("force_generic", [1, 0])
def test_attention_forward_and_backward(gpu_device, dtype, s, h, a, force_generic):
    _attention_case(gpu_device, dtype, s, h, a, force_generic)


# the fp32 matrix-core kernels: every head size, tiles of 32 rows that end inside, fewer tiles than waves, one row,
# key/value heads shared by groups
@pytest.mark.parametrize("s,h,a,akv", [(1, 32, 1, 1), (31, 64, 1, 1), (33, 192, 2, 1), (97, 256, 2, 2), (160, 128, 4, 2),
                                       (161, 512, 4, 1), (300, 192, 3, 3)])
def test_attention_f32(gpu_device, s, h, a, akv):
    _attention_case(gpu_device, "f32", s, h, a, 0, akv)


# more than 256 forward blocks that all find a place at once (their order turns round there, the last row of 256 partly
# filled), and the head sizes of which one block fills a CU's LDS
@pytest.mark.parametrize("s,h,a,akv", [(545, 512, 16, 16), (1057, 512, 8, 2), (550, 1152, 12, 12), (290, 2560, 20, 4)])
def test_attention_f32_many_blocks(gpu_device, s, h, a, akv):
    _attention_case(gpu_device, "f32", s, h, a, 0, akv)


@pytest.mark.parametrize("s,dh,a", [(1, 64, 1), (33, 32, 3), (70, 96, 2), (50, 128, 5)])
@pytest.mark.parametrize("offset", [0, 1])
def test_attention_f32_backward_takes_any_output_alignment(gpu_device, s, dh, a, offset):
    """delta by whole vectors, or element by element where o is not 16-byte aligned; every product and addition rounds by
    at most 2^-24 of what it yields, dh products in all."""
    h = a * dh
    g = torch.Generator(device=gpu_device)
    g.manual_seed(s + dh)
    rand = lambda *n: torch.randn(*n, generator=g, device=gpu_device)
    qkv, d_o, o = rand(s, 3 * h), rand(s, h), rand(s * h + 4)[offset:offset + s * h].view(s, h)
    lse, delta, dqkv = torch.zeros(a, s, device=gpu_device), torch.empty(a, s, device=gpu_device), torch.empty_like(qkv)
    po.po_op_attention_backward(po.PO_F32, qkv, o, lse, d_o, dqkv, delta, s, h, a)
    terms = (o.double() * d_o.double()).view(s, a, dh)
    assert ((delta.t().double() - terms.sum(2)).abs() <= dh * 2.0 ** -24 * terms.abs().sum(2)).all()


@pytest.mark.parametrize("dh", [32, 64, 96, 128])
def test_attention_f32_delta_is_a_tree_of_additions(gpu_device, dh):
    """Every level of a tree of additions leaves, over all its nodes, one rounding of the whole sum: sqrt(levels) in all, one level
    for the products.  A rounding is 2^-24 of the value at most, and at most half of that as the root of the mean square over a
    sum's values of any size and sign (1 / sqrt(3) of it at the lower end of a binade, half as much at the upper)."""
    s, a = 2048, 16
    h = a * dh
    g = torch.Generator(device=gpu_device)
    g.manual_seed(dh)
    rand = lambda *n: torch.randn(*n, generator=g, device=gpu_device)
    qkv, d_o, o = rand(s, 3 * h), rand(s, h), rand(s, h)
    lse, delta, dqkv = torch.full((a, s), 9.0, device=gpu_device), torch.empty(a, s, device=gpu_device), torch.empty_like(qkv)
    po.po_op_attention_backward(po.PO_F32, qkv, o, lse, d_o, dqkv, delta, s, h, a)
    want = (o.double() * d_o.double()).view(s, a, dh).sum(2).t()
    assert (delta.double() - want).norm() < 0.5 * 2.0 ** -24 * (1 + np.log2(dh)) ** 0.5 * want.norm()


# bf16 shapes (rows, head size, heads, key/value heads) past the lines to the blocks of 32 rows and not so many that the forward
# takes 256 rows a block, or the backward four waves: forward blocks of 128 rows whose two groups of waves split the keys, eight-wave
# backward blocks.  Whole tiles; sequences that end inside one; and backward passes alone, over groups.
TWO_GROUPS = dict(whole=[(128, 64, 120, 120), (256, 128, 48, 48), (384, 64, 40, 40), (640, 64, 27, 27)],
                  ragged=[(63, 64, 220, 110), (65, 128, 150, 150), (127, 64, 120, 60), (129, 128, 96, 96), (191, 64, 80, 80),
                          (193, 128, 68, 17), (255, 64, 64, 64), (700, 128, 28, 7)],
                  precision=[(200, 64, 100, 100), (200, 128, 100, 100), (300, 64, 60, 60)],
                  infinite=[(300, 64, 100, 100), (300, 128, 100, 100)],
                  nonfinite=[(200, 64, 100, 100), (200, 128, 100, 50)])
EIGHT_WAVES = dict(ragged=[(200, 64, 64, 16), (130, 128, 72, 12), (257, 64, 45, 5), (65, 128, 112, 14), (300, 128, 45, 5),
                           (200, 64, 52, 26), (131, 128, 72, 24), (70, 64, 110, 22)],
                   whole=[(256, 64, 40, 10), (256, 128, 40, 20)])


def test_attention_shapes_reach_the_128_row_blocks():
    """Host logic: which of the two kinds of blocks a shape goes to, with and without partial results of its groups."""
    forward, backward = (po.lib[n] for n in ("_ZN2po31attention_few_forward_is_fasterEiiii",
                                             "_ZN2po32attention_few_backward_is_fasterEiiiii"))
    forward.restype = backward.restype = ctypes.c_bool
    for s, dh, a, akv in sum(TWO_GROUPS.values(), []):
        assert s > 51 and not forward(s, a * dh, a, akv) and a * -(-s // 256) < 256, (s, dh, a, akv)
    for s, dh, a, akv in sum([*TWO_GROUPS.values(), *EIGHT_WAVES.values()], []):
        assert a * -(-s // 128) <= (768 if s % 128 else 256), (s, dh, a, akv)
        for heads_a_block in range(1, a // akv + 1):
            assert not backward(s, a * dh, a, akv, heads_a_block), (s, dh, a, akv)


# shapes the matrix-core kernels take: head size 64 / 128, s a multiple of 128; the last two of the first six
# are large enough in (s / 256) * heads to select the forward kernel's 256-row blocks (both head sizes)
@pytest.mark.parametrize("s,h,a", [(128, 128, 2), (256, 256, 2), (384, 128, 1), (640, 192, 3), (512, 16384, 256),
                                   (512, 32768, 256), *[(s, dh * a, a) for s, dh, a, _ in TWO_GROUPS["whole"]]])
def test_attention_mfma(gpu_device, s, h, a):
    _attention_case(gpu_device, "bf16", s, h, a, 0)


# bf16 sequences that end inside a tile, both head sizes: one row, ends around 64 and 128 rows, a last key block with one
# query tile, 256-row forward blocks, key/value heads shared by groups; in blocks of 32 rows and in those of 128.  What lies behind the tensors is NaN and must not be read, what lies behind the results must stay.
# 2^-8 for o: half of it is the rounding of o, P enters with 16 bits.
@pytest.mark.parametrize("s,h,a,akv", [(1, 128, 1, 1), (1, 64, 1, 1), (63, 128, 2, 1), (65, 256, 2, 2), (127, 256, 4, 2),
                                       (129, 128, 1, 1), (191, 64, 1, 1), (193, 512, 4, 1), (255, 256, 4, 4),
                                       (300, 16384, 128, 128), (300, 8192, 128, 2), (700, 1024, 8, 2),
                                       *[(s, dh * a, a, akv) for s, dh, a, akv in TWO_GROUPS["ragged"]]])
def test_attention_ragged_bf16(gpu_device, s, h, a, akv):
    rng = np.random.default_rng(s + h + a)
    dh, hkv, group = h // a, h // a * akv, a // akv
    pad = lambda *size, t=torch.bfloat16: torch.full(size, float("nan"), dtype=t, device=gpu_device)
    qkv, d_o = _rand(rng, (s, h + 2 * hkv), "bf16"), _rand(rng, (s, h), "bf16")
    qd, dod, o, dqkv = pad(s + 130, h + 2 * hkv), pad(s + 130, h), pad(s + 130, h), pad(s + 130, h + 2 * hkv)
    lse, delta = pad(a * s + 200, t=torch.float32), pad(a * s + 200, t=torch.float32)
    qd[:s], dod[:s] = torch.from_numpy(qkv).to(gpu_device), torch.from_numpy(d_o).to(gpu_device)
    po.po_op_attention_forward(po.PO_BF16, qd, o, lse, s, h, a, n_kv_heads=akv)
    po.po_op_attention_backward(po.PO_BF16, qd, o, lse, dod, dqkv, delta, s, h, a, n_kv_heads=akv)
    for t, n in ((o, s), (dqkv, s), (lse, a * s), (delta, a * s)):
        assert not torch.isnan(t[:n]).any() and torch.isnan(t[n:]).all()
    # the same in 64 bits, head by head
    q, k, v = (torch.from_numpy(x).to(gpu_device).double() for x in (qkv[:, :h], qkv[:, h:h + hkv], qkv[:, h + hkv:]))
    g = dod[:s].double()
    future = torch.ones(s, s, dtype=torch.bool, device=gpu_device).triu(1)
    ro, rq, rk, rv = torch.zeros_like(g), torch.zeros_like(g), torch.zeros_like(k), torch.zeros_like(k)
    for t in range(a):
        c, ck = slice(t * dh, (t + 1) * dh), slice(t // group * dh, (t // group + 1) * dh)
        sc = (q[:, c] @ k[:, ck].T.contiguous() / np.sqrt(dh)).masked_fill(future, -np.inf)
        p = torch.softmax(sc, 1)
        ro[:, c] = p @ v[:, ck]
        ds = p * (g[:, c] @ v[:, ck].T.contiguous() - (g[:, c] * ro[:, c]).sum(1, keepdim=True)) / np.sqrt(dh)
        rq[:, c] = ds @ k[:, ck]
        rk[:, ck] += ds.T.contiguous() @ q[:, c]
        rv[:, ck] += p.T.contiguous() @ g[:, c]
        assert (lse[t * s:(t + 1) * s] - torch.logsumexp(sc, 1)).abs().max() < 1e-5 * max(1.0, lse[:a * s].abs().max())
    assert max_rel_err(_np(o[:s]), ro.cpu().numpy()) < 2.0 ** -8
    got = _np(dqkv[:s])
    for name, mine, ref in (("dQ", got[:, :h], rq), ("dK", got[:, h:h + hkv], rk), ("dV", got[:, h + hkv:], rv)):
        check_parity(mine, ref.cpu().numpy(), 2e-2, name)


# P and dS enter the products with all 24 bits.  Rows of q come in pairs (2 i, 2 i + 1) and keys in pairs (2 j, 2 j + 1) whose
# scores differ by 2^-11 / sqrt(dh) in the odd rows only, and everything P or dS is multiplied with has alternating
# signs: results are differences of probabilities that agree in 14 bits.  With 16 bits they are 1.5 to 16 % off, with 24
# below 0.1 %; the rounding of a result to bf16 is 2^-9, lse and score sums add less than that again.  2, 100 and 400 heads: blocks of
# 32 rows, of 128 rows and eight waves, of 256 rows and four.
@pytest.mark.parametrize("generic", [0, 1])
@pytest.mark.parametrize("a", [2, 100, 400])
@pytest.mark.parametrize("dh", [64, 128])
def test_attention_ragged_bf16_keeps_probabilities_in_fp32(gpu_device, dh, a, generic):
    s, h = 200, a * dh
    i = torch.arange(s, dtype=torch.float64, device=gpu_device)
    odd, sign, pair = i % 2, 1 - 2 * (i % 2), i // 2
    q, k, v, g = (torch.zeros(s, dh, dtype=torch.float64, device=gpu_device) for _ in range(4))
    q[:, 0], q[:, 2], q[:, 5] = odd, sign, 1
    k[:, 0], k[:, 1], k[:, 5] = sign * 2.0 ** -11, sign, (-0.37 * (pair % 13)).bfloat16().double()
    v[:, 3], v[:, 4] = 1, sign
    g[:, 0], g[:, 3] = sign, 1  # dP = 1
    lse_in = (0.3 + 0.013 * pair).float()  # the same for both rows of a pair
    sc = (q @ k.T.contiguous() / dh ** 0.5).masked_fill(torch.ones(s, s, dtype=torch.bool, device=gpu_device).triu(1), -np.inf)
    p, pb = torch.softmax(sc, 1), torch.exp(sc - lse_in.double()[:, None])
    every = lambda x: x.bfloat16().repeat(1, a).contiguous()
    qkv = torch.cat([every(q), every(k), every(v)], 1).contiguous()
    o, lse = torch.empty(s, h, dtype=torch.bfloat16, device=gpu_device), torch.empty(a, s, device=gpu_device)
    po.po_op_attention_forward(po.PO_BF16, qkv, o, lse, s, h, a, generic)
    dqkv, delta = torch.empty_like(qkv), torch.empty(a, s, device=gpu_device)
    po.po_op_attention_backward(po.PO_BF16, qkv, torch.zeros_like(o), lse_in.repeat(a, 1).contiguous(), every(g), dqkv,
                                delta, s, h, a, generic)
    def check(got, column, want, rows):  # every head holds the same
        got = got.double().view(s, a, dh)[rows, :, column]
        assert ((got - want[rows, None]) / want[rows, None]).abs().max() < 2.0 ** -7
    odd_rows, even_rows = slice(1, None, 2), slice(0, None, 2)
    check(o, 4, p @ sign, odd_rows)
    check(dqkv[:, :h], 1, pb @ sign / dh ** 0.5, odd_rows)
    check(dqkv[:, h:2 * h], 2, pb.T.contiguous() @ sign / dh ** 0.5, even_rows)
    check(dqkv[:, 2 * h:], 0, pb.T.contiguous() @ sign, even_rows)


# Keys no row may attend to, by scores of -inf: a whole tile of them, the first or one that starts a wave's or a group's
# share of the tiles, adds nothing.  (Row i of a query of ones against keys of -inf; rows that see no other key are NaN.)
@pytest.mark.parametrize("first,last", [(0, 40), (0, 64), (32, 64), (64, 128), (96, 160)])
@pytest.mark.parametrize("dtype,s,dh,a", [("f32", 200, 64, 2), ("f32", 200, 128, 1), ("bf16", 300, 64, 2),
                                          ("bf16", 300, 128, 400),
                                          *[("bf16", s, dh, a) for s, dh, a, _ in TWO_GROUPS["infinite"]]])
def test_attention_keys_of_minus_infinity_add_nothing(gpu_device, dtype, s, dh, a, first, last):
    code, tdt, _ = DT[dtype]
    h = a * dh
    g = torch.Generator(device=gpu_device)
    g.manual_seed(first + last + s)
    qkv = torch.randn(s, 3 * h, generator=g, device=gpu_device).to(tdt)
    qkv[:, :h] = 1
    qkv[first:last, h:2 * h] = float("-inf")
    o, lse = torch.empty(s, h, dtype=tdt, device=gpu_device), torch.empty(a, s, device=gpu_device)
    po.po_op_attention_forward(code, qkv, o, lse, s, h, a)
    k, v = qkv[:, h:h + dh].double(), qkv[:, 2 * h:2 * h + dh].double()
    sc = (k.sum(1) / dh ** 0.5).expand(s, s).masked_fill(torch.ones(s, s, dtype=torch.bool, device=gpu_device).triu(1), -np.inf)
    want, sees = torch.softmax(sc, 1) @ v, slice(0 if first else last, s)
    assert (o[sees, :dh].double() - want[sees]).norm() < (2.0 ** -8 if dtype == "bf16" else 1e-6) * want[sees].norm()
    assert (lse[0, sees] - torch.logsumexp(sc, 1)[sees]).abs().max() < 1e-5
    assert not torch.isfinite(o[:sees.start]).any() and not torch.isfinite(lse[:, :sees.start]).any()


def _attention_64(qkv, d_o, o, lse, dh, a, akv):
    """o and lse in 64 bits, and the gradients that follow in 64 bits from the given o and lse."""
    s, h, hkv, group = len(qkv), a * dh, akv * dh, a // akv
    q, k, v = (x.double() for x in (qkv[:, :h], qkv[:, h:h + hkv], qkv[:, h + hkv:]))
    want = dict(o=torch.zeros_like(d_o, dtype=torch.float64), lse=torch.zeros_like(lse, dtype=torch.float64),
                dqkv=torch.zeros_like(qkv, dtype=torch.float64))
    future = torch.ones(s, s, dtype=torch.bool, device=qkv.device).triu(1)
    for t in range(a):
        c, ck = slice(t * dh, (t + 1) * dh), slice(t // group * dh, (t // group + 1) * dh)
        sc = (q[:, c] @ k[:, ck].T.contiguous() / dh ** 0.5).masked_fill(future, -np.inf)
        want["o"][:, c], want["lse"][t] = torch.softmax(sc, 1) @ v[:, ck], torch.logsumexp(sc, 1)
        p, up = torch.exp(sc - lse[t].double()[:, None]), d_o[:, c].double()
        ds = p * (up @ v[:, ck].T.contiguous() - (up * o[:, c].double()).sum(1, keepdim=True)) / dh ** 0.5
        want["dqkv"][:, c] = ds @ k[:, ck]
        want["dqkv"][:, h:h + hkv][:, ck] += ds.T.contiguous() @ q[:, c]
        want["dqkv"][:, h + hkv:][:, ck] += p.T.contiguous() @ up
    return want


# Blocks of 32 rows: one tile and less, ends around a tile, more tiles than a block's waves have stages (8 x 2 with heads of 64,
# 4 x 2 or 8 with heads of 128), groups, and both sides of the lines to the 128-row blocks.  Against 64 bits: P, dS and the results
# are rounded to bf16 (2^-9 each); what lies behind the results stays.
@pytest.mark.parametrize("s,dh,a,akv", [(128, 64, 2, 2), (640, 64, 4, 1), (512, 64, 30, 30), (512, 64, 31, 31), (20, 64, 3, 3),
                                        (44, 64, 2, 1), (97, 64, 8, 1), (545, 64, 4, 2), (777, 64, 25, 25), (128, 128, 2, 2),
                                        (512, 128, 4, 2), (384, 128, 23, 23), (384, 128, 24, 24), (384, 128, 31, 31),
                                        (384, 128, 32, 32), (31, 128, 2, 1),
                                        (65, 128, 3, 3), (300, 128, 4, 1), (129, 128, 70, 70), (512, 64, 18, 18),
                                        (512, 64, 29, 29), (384, 128, 22, 22)])
def test_attention_blocks_of_32_rows(gpu_device, s, dh, a, akv):
    h, hkv = a * dh, akv * dh
    g = torch.Generator(device=gpu_device)
    g.manual_seed(s + dh + a)
    bf = lambda *size: torch.randn(*size, generator=g, device=gpu_device).bfloat16()
    qkv, d_o = bf(s, h + 2 * hkv), bf(s, h)
    o, dqkv = (torch.full((s + 40, n), 7.0, dtype=torch.bfloat16, device=gpu_device) for n in (h, h + 2 * hkv))
    lse, delta = torch.full((a * s + 40,), 7.0, device=gpu_device), torch.empty(a, s, device=gpu_device)
    po.po_op_attention_forward(po.PO_BF16, qkv, o, lse, s, h, a, n_kv_heads=akv)
    po.po_op_attention_backward(po.PO_BF16, qkv, o, lse, d_o, dqkv, delta, s, h, a, n_kv_heads=akv)
    assert (o[s:] == 7).all() and (dqkv[s:] == 7).all() and (lse[a * s:] == 7).all()
    want = _attention_64(qkv, d_o, o[:s], lse[:a * s].view(a, s), dh, a, akv)
    err = lambda got, ref: ((got.double() - ref).norm() / ref.norm()).item()
    assert err(o[:s], want["o"]) < 2.0 ** -8 and (lse[:a * s].view(a, s) - want["lse"]).abs().max() < 1e-5
    for part in (slice(0, h), slice(h, h + hkv), slice(h + hkv, h + 2 * hkv)):
        assert err(dqkv[:s, part], want["dqkv"][:, part]) < 2.0 ** -7, part


# Row sums of many tiles, scaled again between tiles and in the merge of the waves, at scores of deviation 6 where the maximum moves:
# lse is an fp32 number near that maximum, and its own rounding is the largest part of its error (2^-25 at most, root mean square; the
# other parts, the maximum in units of the exponent, the constants, log l, are each below that).
@pytest.mark.parametrize("s,dh,a", [(2048, 128, 2), (1500, 128, 3), (4096, 128, 1), (1024, 64, 8), (777, 64, 10)])
def test_attention_blocks_of_32_rows_lse_is_exact_to_a_rounding(gpu_device, s, dh, a):
    h, err = a * dh, [0.0, 0.0]
    for seed in range(3):
        g = torch.Generator(device=gpu_device)
        g.manual_seed(s + a + seed)
        qkv = (2.5 * torch.randn(s, 3 * h, generator=g, device=gpu_device)).bfloat16()
        o, lse = torch.empty(s, h, dtype=torch.bfloat16, device=gpu_device), torch.empty(a, s, device=gpu_device)
        po.po_op_attention_forward(po.PO_BF16, qkv, o, lse, s, h, a)
        want = _attention_64(qkv, torch.zeros_like(o), o, lse, dh, a, a)["lse"]
        err[0] += float((lse.double() - want).square().sum())
        err[1] += float(want.square().sum())
    assert err[0] ** 0.5 < 2.0 ** -24 * err[1] ** 0.5


# Short sequences stay with the vector kernels, bit for bit; one row more and a call goes to the matrix cores (the bf16
# backward always does).
@pytest.mark.parametrize("dtype,dh,forward,backward", [("f32", 32, 4, 6), ("f32", 64, 9, 12), ("f32", 96, 13, 18),
                                                       ("f32", 128, 18, 24), ("bf16", 64, 43, 0), ("bf16", 128, 51, 0)])
def test_attention_of_few_rows_runs_on_the_vector_kernels(gpu_device, dtype, dh, forward, backward):
    code, tdt, _ = DT[dtype]
    a, akv = 4, 2
    h, hkv = a * dh, akv * dh
    g = torch.Generator(device=gpu_device)
    g.manual_seed(dh)
    for s in sorted({1, forward, forward + 1, backward, backward + 1} - {0}):
        qkv = torch.randn(s, h + 2 * hkv, generator=g, device=gpu_device).to(tdt)
        d_o = torch.randn(s, h, generator=g, device=gpu_device).to(tdt)
        o, lse, grad = ([torch.zeros(*size, dtype=t, device=gpu_device) for _ in range(2)]
                        for size, t in (((s, h), tdt), ((a, s), torch.float32), ((s, h + 2 * hkv), tdt)))
        delta = torch.empty(a, s, device=gpu_device)
        for generic in (1, 0):
            po.po_op_attention_forward(code, qkv, o[generic], lse[generic], s, h, a, generic, n_kv_heads=akv)
        for generic in (1, 0):
            po.po_op_attention_backward(code, qkv, o[1], lse[1], d_o, grad[generic], delta, s, h, a, generic,
                                        n_kv_heads=akv)
        assert (torch.equal(o[0], o[1]) and torch.equal(lse[0], lse[1])) == (s <= forward), s
        if backward:
            assert torch.equal(grad[0], grad[1]) == (s <= backward), s


# The workspace of a ragged grouped backward: fp32 partials of two query heads, or of the group's next divisor, inside [s, 2h]
# bf16.  Groups of 4, 6, 8 (two heads each), 9 (three), and of 2, 3, 5, which have no such divisor; both head sizes; first blocks of
# 32 rows, then 800 blocks of four waves, then blocks of eight.  Nothing behind the workspace is written, an
# unaligned one is not used.  2^-8: the rounding of the results to bf16.
@pytest.mark.parametrize("s,dh,a,akv,parts", [(200, 64, 8, 2, 2), (130, 128, 6, 1, 3), (257, 64, 9, 1, 3), (65, 128, 16, 2, 4),
                                              (300, 128, 9, 1, 3), (200, 64, 4, 2, 0), (131, 128, 6, 2, 0), (70, 64, 5, 1, 0),
                                              (130, 64, 800, 200, 2),
                                              *[(*shape, parts) for shape, parts in
                                                zip(EIGHT_WAVES["ragged"], (2, 3, 3, 4, 3, 0, 0, 0), strict=True)]])
def test_attention_ragged_bf16_group_partials(gpu_device, s, dh, a, akv, parts):
    h, hkv = a * dh, akv * dh
    g = torch.Generator(device=gpu_device)
    g.manual_seed(s + a)
    qkv = torch.randn(s, h + 2 * hkv, generator=g, device=gpu_device).bfloat16()
    d_o = torch.randn(s, h, generator=g, device=gpu_device).bfloat16()
    o, lse, delta = torch.empty_like(d_o), torch.empty(a, s, device=gpu_device), torch.empty(a, s, device=gpu_device)
    po.po_op_attention_forward(po.PO_BF16, qkv, o, lse, s, h, a, n_kv_heads=akv)
    want = _attention_64(qkv, d_o, o, lse, dh, a, akv)["dqkv"]
    for offset in (0, 4):
        room = torch.full((s * 2 * h + 4096,), float("nan"), dtype=torch.bfloat16, device=gpu_device)
        work, dqkv = room[offset:], torch.full_like(qkv, float("nan"))
        po.po_op_attention_backward(po.PO_BF16, qkv, o, lse, d_o, dqkv, delta, s, h, a, n_kv_heads=akv, partials=work)
        for part in (slice(0, h), slice(h, h + hkv), slice(h + hkv, h + 2 * hkv)):
            assert (dqkv[:, part].double() - want[:, part]).norm() < 2.0 ** -8 * want[:, part].norm()
        used = 0 if offset else s * 2 * parts * hkv  # floats
        assert not torch.isnan(room[:2 * used].view(torch.float32)).any() and torch.isnan(room[2 * used:]).all()


# What the matrix-core kernels put in place of the vector kernels is no further from the truth: 2-norm errors against 64 bits,
# the backward from the same o and lse.  A twentieth is what such an error differs by between two draws of the inputs.
@pytest.mark.parametrize("dtype,s,dh,a,akv", [("f32", 100, 64, 64, 64), ("f32", 333, 32, 64, 64), ("f32", 333, 96, 32, 32),
                                              ("f32", 777, 128, 24, 8), ("bf16", 1733, 128, 16, 16),
                                              ("bf16", 300, 128, 40, 40), ("bf16", 300, 64, 32, 8),
                                              *[("bf16", *shape) for shape in TWO_GROUPS["precision"]]])
def test_attention_errors_are_no_larger_than_the_vector_kernels(gpu_device, dtype, s, dh, a, akv):
    code, tdt, _ = DT[dtype]
    h, hkv = a * dh, akv * dh
    g = torch.Generator(device=gpu_device)
    g.manual_seed(s)
    qkv = torch.randn(s, h + 2 * hkv, generator=g, device=gpu_device).to(tdt)
    d_o = torch.randn(s, h, generator=g, device=gpu_device).to(tdt)
    got = [dict(o=torch.empty_like(d_o), lse=torch.empty(a, s, device=gpu_device), dqkv=torch.empty_like(qkv)) for _ in range(2)]
    for generic in (1, 0):
        po.po_op_attention_forward(code, qkv, got[generic]["o"], got[generic]["lse"], s, h, a, generic, n_kv_heads=akv)
    o, lse, delta = got[1]["o"], got[1]["lse"], torch.empty(a, s, device=gpu_device)
    for generic in (1, 0):
        po.po_op_attention_backward(code, qkv, o, lse, d_o, got[generic]["dqkv"], delta, s, h, a, generic, n_kv_heads=akv)
    want = _attention_64(qkv, d_o, o, lse, dh, a, akv)
    parts = dict(dq=slice(0, h), dk=slice(h, h + hkv), dv=slice(h + hkv, h + 2 * hkv))
    for name in ("o", "lse", *parts):
        pick = lambda r: r["dqkv"][:, parts[name]] if name in parts else r[name]
        err = [float((pick(r).double() - pick(want)).norm()) for r in got]
        assert err[0] <= 1.05 * err[1], (name, err)


def _nonfinite_inputs(gpu_device, dtype, s, dh, a, akv, where, value, row):
    _, tdt, _ = DT[dtype]
    g = torch.Generator(device=gpu_device)
    g.manual_seed(s + dh + a + row)
    h, hkv = a * dh, akv * dh
    qkv = torch.randn(s, h + 2 * hkv, generator=g, device=gpu_device).to(tdt)
    d_o = torch.randn(s, h, generator=g, device=gpu_device).to(tdt)
    first, last = {"k": (h, h + hkv), "v": (h + hkv, h + 2 * hkv), "qkv": (0, h + 2 * hkv), "d_o": (0, h)}[where]
    (d_o if where == "d_o" else qkv)[row, first:last] = value
    return qkv, d_o


# A non-finite row among the keys, the values, a whole token or the upstream gradient: what lies behind a row may not
# reach it.  Compared with the vector kernels, which never read a key behind the row; row: the first, inside the first
# tile, around tile ends, the last of the sequence.  2 and 4, 100 and 400 heads: blocks of 32 rows, of 128 rows and eight waves, of 256
# rows and four waves in the bf16 kernels.
NONFINITE = [("f32", 200, 32, 2, 2), ("f32", 97, 64, 2, 1), ("f32", 128, 96, 1, 1), ("f32", 200, 128, 2, 2),
             ("f32", 512, 64, 4, 4), ("bf16", 200, 64, 2, 2), ("bf16", 200, 128, 4, 2), ("bf16", 300, 64, 400, 400),
             ("bf16", 300, 128, 400, 400), *[("bf16", *shape) for shape in TWO_GROUPS["nonfinite"]]]


@pytest.mark.parametrize("where", ["k", "v", "qkv", "d_o"])
@pytest.mark.parametrize("dtype,s,dh,a,akv", NONFINITE)
def test_attention_non_finite_rows_stay_where_they_are(gpu_device, dtype, s, dh, a, akv, where):
    code, tdt, _ = DT[dtype]
    h, hkv = a * dh, akv * dh
    for value, row in ((float("nan"), s - 1), (float("inf"), 63), (float("nan"), 64), (float("-inf"), 17), (float("inf"), 0)):
        qkv, d_o = _nonfinite_inputs(gpu_device, dtype, s, dh, a, akv, where, value, row)
        o, lse = [torch.full((s, h), 7.0, dtype=tdt, device=gpu_device) for _ in range(2)], \
                 [torch.full((a, s), 7.0, device=gpu_device) for _ in range(2)]
        dqkv = [torch.full((s, h + 2 * hkv), 7.0, dtype=tdt, device=gpu_device) for _ in range(2)]
        delta = torch.empty(a, s, device=gpu_device)
        for generic in (1, 0):
            po.po_op_attention_forward(code, qkv, o[generic], lse[generic], s, h, a, generic, n_kv_heads=akv)
        for generic in (1, 0):  # both from the same forward results
            po.po_op_attention_backward(code, qkv, o[1], lse[1], d_o, dqkv[generic], delta, s, h, a, generic,
                                        n_kv_heads=akv)
        same = lambda x, y: torch.equal(torch.isfinite(x), torch.isfinite(y))
        what = (where, value, row)
        assert same(o[0], o[1]) and same(lse[0], lse[1]), what
        assert same(dqkv[0][:, :h], dqkv[1][:, :h]), what
        # dK and dV of a key: the vector kernel lets a row of its 64-row block before it through, the others at most that
        ok = torch.isfinite(dqkv[1])
        assert torch.isfinite(dqkv[0][ok]).all(), what
        close = lambda x, y: (x - y).double().norm() <= (2.0 ** -6 if dtype == "bf16" else 1e-4) * y.double().norm()
        okf = torch.isfinite(o[1])
        assert close(o[0][okf], o[1][okf]) and close(dqkv[0][ok], dqkv[1][ok]), what


def _attention_case(gpu_device, dtype, s, h, a, force_generic, akv=0, with_partials=False):
    code, tdt, tol = DT[dtype]
    rng = np.random.default_rng(s * 31 + h + a + 7 * akv)
    dh = h // a
    hkv = (akv or a) * dh
    group = a // (akv or a)
    qkv = _rand(rng, (s, h + 2 * hkv), dtype)
    d_o = _rand(rng, (s, h), dtype)
    qd, dod = _dev(qkv, tdt, gpu_device), _dev(d_o, tdt, gpu_device)
    o = torch.empty(s, h, dtype=tdt, device=gpu_device)
    lse = torch.empty(a, s, dtype=torch.float32, device=gpu_device)
    po.po_op_attention_forward(code, qd, o, lse, s, h, a, force_generic, n_kv_heads=akv)
    q64 = qkv.astype(np.float64)
    q, k, v = q64[:, :h], q64[:, h:h + hkv], q64[:, h + hkv:]
    ro, probs = so.attention_forward(q, k, v, a)
    assert max_rel_err(_np(o), ro) < tol
    # log-sum-exp of the scaled, masked scores: a plain definition
    for t in range(a):
        kt = k[:, (t // group) * dh:(t // group + 1) * dh]
        sc = (q[:, t * dh:(t + 1) * dh] @ kt.T) / np.sqrt(dh)
        sc = np.where(np.triu(np.ones((s, s), dtype=bool), 1), -np.inf, sc)
        ref_lse = np.log(np.exp(sc - sc.max(1, keepdims=True)).sum(1)) + sc.max(1)
        assert np.abs(_np(lse[t]) - ref_lse).max() < 1e-3 * max(1.0, np.abs(ref_lse).max())
    dqkv = torch.empty(s, h + 2 * hkv, dtype=tdt, device=gpu_device)
    delta = torch.empty(a, s, dtype=torch.float32, device=gpu_device)
    partials = torch.empty(s, 2 * h, dtype=tdt, device=gpu_device) if with_partials else None
    po.po_op_attention_backward(code, qd, o, lse, dod, dqkv, delta, s, h, a, force_generic, n_kv_heads=akv,
                                partials=partials)
    rdq, rdk, rdv = so.attention_backward(d_o.astype(np.float64), q, k, v, probs, a)
    got = _np(dqkv)
    check_parity(got[:, :h], rdq, tol, "dQ")
    check_parity(got[:, h:h + hkv], rdk, tol, "dK")
    check_parity(got[:, h + hkv:], rdv, tol, "dV")


# grouped-query attention: key/value heads shared by groups of query heads
@pytest.mark.parametrize("dtype,s,h,a,akv,force_generic", [
    ("f32", 37, 128, 4, 2, 1), ("f32", 70, 192, 6, 1, 1), ("bf16", 130, 256, 4, 2, 1),
    ("bf16", 128, 256, 4, 2, 0), ("bf16", 384, 512, 4, 1, 0), ("bf16", 256, 512, 8, 2, 0),
    ("bf16", 640, 768, 6, 3, 0), ("bf16", 512, 1024, 16, 4, 0), ("bf16", 256, 256, 4, 4, 0),
    *[("bf16", s, dh * a, a, akv, 0) for s, dh, a, akv in EIGHT_WAVES["whole"]],
    # 17 row blocks x 16 heads: more dQ blocks than CUs but fewer dK/dV blocks, so without the workspace the two
    # backward kernels have different block forms and go out as two launches; with it, as one launch of four-wave blocks
    ("bf16", 2176, 1024, 16, 2, 0)])
@pytest.mark.parametrize("with_partials", [False, True], ids=["direct", "per-head-then-sum"])
def test_grouped_query_attention(gpu_device, dtype, s, h, a, akv, force_generic, with_partials):
    _attention_case(gpu_device, dtype, s, h, a, force_generic, akv, with_partials)


def test_grouped_query_attention_rejects_bad_groups(gpu_device):
    t = torch.zeros(128, 3 * 256, dtype=torch.bfloat16, device=gpu_device)
    o = torch.zeros(128, 256, dtype=torch.bfloat16, device=gpu_device)
    lse = torch.zeros(4, 128, device=gpu_device)
    with pytest.raises(po.PipeOffloadError):
        po.po_op_attention_forward(po.PO_BF16, t, o, lse, 128, 256, 4, 0, n_kv_heads=3)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,n", [(1, 2), (37, 130), (300, 1024)])
def test_colsum_accumulate(gpu_device, dtype, rows, n):
    code, tdt, tol = DT[dtype]
    rng = np.random.default_rng(rows + n)
    x = _rand(rng, (rows, n), dtype)
    acc0 = rng.standard_normal(n).astype(np.float32)
    acc = torch.from_numpy(acc0).to(gpu_device)
    ws = torch.empty(po.po_op_colsum_workspace(rows, n) // 4, dtype=torch.float32, device=gpu_device)
    po.po_op_colsum_accumulate(code, _dev(x, tdt, gpu_device), acc, ws, rows, n)
    assert max_rel_err(_np(acc) - acc0, x.astype(np.float64).sum(0)) < 1e-4


# one launch over all rows (up to 512; bf16 up to 256 blocks of 64 columns) and the two of more: rows that leave lanes, waves and
# a lane's one, two or four rows without work, a last block of few columns, rows that are no whole vectors
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,h", [(1, 8), (63, 72), (65, 72), (129, 200), (511, 64), (512, 136), (513, 136), (30, 16384), (30, 16392)])
def test_column_reductions_of_few_rows(gpu_device, dtype, rows, h):
    """Against fp64.  Each sum has `rows` terms, which no order of additions rounds by more than rows * 2^-24 of their
    magnitudes' sum; a LayerNorm gain's terms are off by the statistics' rounding too, 2^-20 of theirs."""
    code, tdt, _ = DT[dtype]
    g = torch.Generator(device=gpu_device)
    g.manual_seed(rows + h)
    rand = lambda *n: torch.randn(*n, generator=g, device=gpu_device).to(tdt)
    x, dn, dres, gain = rand(rows, h), rand(rows, h), rand(rows, h), rand(h)
    words = max(po.po_op_layernorm_backward_workspace(rows, h), po.po_op_colsum_workspace(rows, h)) // 4
    ws = torch.full((words,), float("nan"), device=gpu_device)
    out = torch.zeros(3, h, device=gpu_device)
    po.po_op_colsum_accumulate(code, dn, out[0], ws, rows, h)
    po.po_op_layernorm_backward(code, dn, x, gain, dres, torch.empty_like(x), out[1], out[2], ws, rows, h, 1e-5)
    d64, x64 = dn.double(), x.double()
    xhat = (x64 - x64.mean(1, keepdim=True)) / (x64.var(1, keepdim=True, unbiased=False) + 1e-5).sqrt()
    for got, terms, extra in ((out[0], d64, 0.0), (out[2], d64, 0.0), (out[1], d64 * xhat, 2.0 ** -20)):
        bound = (rows * 2.0 ** -24 + extra) * (terms.abs().sum(0) + d64.abs().sum(0))
        assert ((got.double() - terms.sum(0)).abs() <= bound).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,h", [(100, 26624), (520, 4096), (1024, 4096), (3000, 4096)])
def test_layernorm_gain_gradient_rounds_no_more_than_a_plain_order(gpu_device, dtype, rows, h):
    """Against fp64, beside the same terms added in fp32 in a plain order: chunks of some 32 rows in four chains each, the chunks in
    four chains.  Orders of the same quality differ by chance, over 4 x h columns by 1 / sqrt(8 h): half a percent at most; two
    percent is four times that."""
    code, tdt, _ = DT[dtype]
    err = [0.0, 0.0]
    chunks = max(1, min(64, -(-rows // 32)))
    per_chunk = -(-rows // chunks)
    def four_chains(t):  # along the first dimension
        acc = torch.zeros(4, *t.shape[1:], device=gpu_device)
        for i in range(0, t.shape[0], 4):
            n = min(4, t.shape[0] - i)
            acc[:n] += t[i:i + n]
        return ((acc[0] + acc[1]) + acc[2]) + acc[3]
    for seed in range(4):
        g = torch.Generator(device=gpu_device)
        g.manual_seed(rows + h + seed)
        rand = lambda *n: torch.randn(*n, generator=g, device=gpu_device).to(tdt)
        x, dn, dres, gain = rand(rows, h), rand(rows, h), rand(rows, h), rand(h)
        ws = torch.empty(po.po_op_layernorm_backward_workspace(rows, h) // 4, device=gpu_device)
        out = torch.zeros(2, h, device=gpu_device)
        po.po_op_layernorm_backward(code, dn, x, gain, dres, torch.empty_like(x), out[0], out[1], ws, rows, h, 1e-5)
        mean = x.double().mean(1, keepdim=True)
        rstd = (x.double().var(1, keepdim=True, unbiased=False) + 1e-5).rsqrt()
        want = (dn.double() * (x.double() - mean) * rstd).sum(0)
        mean32, rstd32 = ws[:2 * rows].view(rows, 2).split(1, 1)  # the kernel's, whose own rounding is not in question
        terms = dn.float() * (x.float() - mean32) * rstd32
        plain = four_chains(torch.stack([four_chains(t) for t in terms.split(per_chunk)]))
        for k, got in enumerate((out[0], plain)):
            err[k] += float((got.double() - want).square().sum())
    assert err[0] ** 0.5 <= 1.02 * err[1] ** 0.5


def test_pack_unpack_roundtrip_is_bit_exact(gpu_device):
    rng = np.random.default_rng(0)
    sizes = [16, 4096 + 16, 0, 1 << 20, 48, 3 * 16384 + 32]  # bytes, multiples of 16, one empty
    segs = [torch.from_numpy(rng.integers(0, 256, size=n, dtype=np.uint8)).to(gpu_device) for n in sizes]
    total = sum(sizes)
    packed = torch.zeros(total, dtype=torch.uint8, device=gpu_device)
    po.po_op_pack([(t if t.numel() else 0, n) for t, n in zip(segs, sizes)], packed)
    want = np.concatenate([t.cpu().numpy() for t in segs])
    assert np.array_equal(packed.cpu().numpy(), want)  # byte-exact: oracle = concatenation
    outs = [torch.zeros_like(t) for t in segs]
    po.po_op_unpack([(t if t.numel() else 0, n) for t, n in zip(outs, sizes)], packed)
    for a, b in zip(outs, segs):
        assert torch.equal(a, b)
    with pytest.raises(po.PipeOffloadError):
        po.po_op_pack([(segs[0], 8)], packed)  # not a multiple of 16
    po.po_op_pack([], packed)  # empty is a no-op


# ---- dropout with regenerated masks ------------------------------------------------------------------------------
# the last five: one vector per row, widths between the block widths of the kernel that takes whole vectors, one row
@pytest.mark.parametrize("rows,cols,p,seed,layer,site,mb", [(37, 130, 0.1, 1234, 0, 0, 0), (64, 256, 0.25, 2 ** 40 + 7, 3, 1, 5),
                                                            (5, 7, 0.5, 1, 11, 0, 2), (300, 1024, 0.9, 99, 1, 1, 31),
                                                            (9, 8, 0.3, 5, 2, 0, 1), (129, 264, 0.2, 6, 0, 1, 3),
                                                            (33, 1288, 0.4, 7, 1, 0, 0), (3, 2056, 0.6, 8, 5, 1, 9),
                                                            (1, 5120, 0.1, 9, 0, 0, 4)])
def test_dropout_mask_is_the_oracle_mask_bit_for_bit(gpu_device, rows, cols, p, seed, layer, site, mb):
    p = float(np.float32(p))  # the probability the library sees is the fp32 value
    x = torch.ones(rows, cols, dtype=torch.float32, device=gpu_device)
    out = torch.empty_like(x)
    po.po_op_dropout(po.PO_F32, x, out, rows, cols, p, seed, layer, site, mb)
    keep = so.dropout_keep_mask(seed, layer, site, mb, rows, cols, p)
    got = _np(out)
    assert np.array_equal(got != 0, keep)
    assert np.all(got[keep] == np.float32(1.0 / (1.0 - p)))
    # bf16 values through the same mask
    rng = np.random.default_rng(rows)
    v = _rand(rng, (rows, cols), "bf16")
    xb = _dev(v, torch.bfloat16, gpu_device)
    ob = torch.empty_like(xb)
    po.po_op_dropout(po.PO_BF16, xb, ob, rows, cols, p, seed, layer, site, mb)
    assert max_rel_err(_np(ob), v.astype(np.float64) * keep / (1.0 - p)) < 1e-2
    # the same from and to addresses that are no multiple of 16 bytes
    buf = torch.zeros(2, rows * cols + 1, dtype=torch.bfloat16, device=gpu_device)
    buf[0, 1:] = xb.view(-1)
    if buf[0, 1:].data_ptr() % 16:
        po.po_op_dropout(po.PO_BF16, buf[0, 1:], buf[1, 1:], rows, cols, p, seed, layer, site, mb)
        assert torch.equal(buf[1, 1:].view(rows, cols), ob)
