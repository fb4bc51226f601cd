"""Parity of each HIP kernel with the oracle's function for the same step, element by element, on
seeded inputs spanning several tiles and ragged tails.  All calls go through the C ABI."""
import math

import numpy as np
import pytest
import torch

from oracle import prism_oracle as O
from paper_2510_15620_amd import binding as B
from paper_2510_15620_amd import workloads as W
from tests.helpers import fp32_tile, gemm_plan, head_plan, oracle_model, oracle_weights

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _rand(shape, dtype, seed, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(*shape, generator=g) * scale).to(dtype)


def _f64(t):
    return t.detach().cpu().to(torch.float64).numpy()


def _tol(dtype):
    return dict(rtol=2e-5, atol=2e-5) if dtype == torch.float32 else dict(rtol=1.2e-2, atol=1e-2)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_embed(dtype):
    table = _rand((300, 256), dtype, 1)
    tok = torch.randint(0, 300, (777,), generator=torch.Generator().manual_seed(2), dtype=torch.int32)
    X = torch.empty(777, 256, dtype=torch.float32, device=DEV)
    B.op_embed(tok.to(DEV), table.to(DEV), X)
    assert np.array_equal(X.cpu().numpy().astype(np.float64), O.embed(tok.numpy(), _f64(table)))


SIXTEEN = [torch.bfloat16, torch.float16]
EPS16 = {torch.bfloat16: 2.0 ** -8, torch.float16: 2.0 ** -11}      # half an ulp, relative
OPERAND = {torch.bfloat16: "bf16", torch.float16: "f16"}
WHOLE_CALL_ERROR = {torch.bfloat16: 9e-3, torch.float16: 2e-3}      # of the largest score; four times the largest measured over the cases


@pytest.mark.parametrize("dtype,hidden", [(torch.float32, 256), (torch.float32, 192), (torch.bfloat16, 4096), (torch.bfloat16, 512),
                                          (torch.float16, 4096), (torch.float16, 1024)])
def test_rmsnorm(dtype, hidden):
    X = _rand((333, hidden), torch.float32, 3, 2.5)
    g = (1 + _rand((hidden,), torch.float32, 4, 0.1)).to(dtype)
    out = torch.empty(333, hidden, dtype=dtype, device=DEV)
    B.op_rmsnorm(X.to(DEV), g.to(DEV), 1e-6, out)
    ref = O.rmsnorm(_f64(X), _f64(g), 1e-6)
    tol = dict(rtol=1e-5, atol=1e-6) if dtype == torch.float32 else dict(rtol=EPS16[dtype] * 1.01, atol=1e-6)
    np.testing.assert_allclose(_f64(out), ref, **tol)


GEMM_SHAPES = [  # M, N (rows of W), K
    (1, 64, 64), (77, 200, 128), (300, 384, 256), (513, 1024, 192), (1000, 2560, 1408), (4100, 6144, 1024),
]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_RESIDUAL, B.EPI_SWIGLU])
@pytest.mark.parametrize("shape", GEMM_SHAPES)
def test_gemm(dtype, epi, shape):
    M, N, K = shape
    if dtype == torch.float32:
        K += 3; N += 2                                   # the fp32 kernel takes any shape
    A = _rand((M, K), dtype, 10 + M, 1.0)
    Wt = _rand((N, K), dtype, 20 + N, 1.0 / math.sqrt(K))
    ref = _f64(A) @ _f64(Wt).T
    if epi == B.EPI_STORE:
        out = torch.zeros(M, N, dtype=dtype, device=DEV)
    elif epi == B.EPI_RESIDUAL:
        X0 = _rand((M, N), torch.float32, 30, 1.0)
        out = X0.to(DEV).clone()
        ref = _f64(X0) + ref
    else:
        F = N // 2
        out = torch.zeros(M, F, dtype=dtype, device=DEV)
        ref = O.silu(ref[:, :F]) * ref[:, F:]
    B.op_gemm(epi, A.to(DEV), Wt.to(DEV), out)
    torch.cuda.synchronize()
    if dtype == torch.float32:
        np.testing.assert_allclose(_f64(out), ref, rtol=1e-4, atol=1e-4)
    elif epi == B.EPI_RESIDUAL:
        np.testing.assert_allclose(_f64(out), ref, rtol=1e-4, atol=1e-4)       # fp32 accumulate, fp32 out
    else:
        np.testing.assert_allclose(_f64(out), ref, rtol=EPS16[dtype] * 1.01, atol=2e-3 * EPS16[dtype] * 256)    # one 16-bit rounding of the result


def _gemm_16_case(dtype, epi, M, N, K):
    A = _rand((M, K), dtype, 10 + M + K, 1.0)
    Wt = _rand((N, K), dtype, 20 + N + K, 1.0 / math.sqrt(K))
    ref = _f64(A) @ _f64(Wt).T
    if epi == B.EPI_RESIDUAL:
        X0 = _rand((M, N), torch.float32, 30, 1.0)
        out = X0.to(DEV).clone()
        ref = _f64(X0) + ref
    elif epi == B.EPI_SWIGLU:
        out = torch.zeros(M, N // 2, dtype=dtype, device=DEV)
        ref = O.silu(ref[:, :N // 2]) * ref[:, N // 2:]
    else:
        out = torch.zeros(M, N, dtype=dtype, device=DEV)
    B.op_gemm(epi, A.to(DEV), Wt.to(DEV), out)
    torch.cuda.synchronize()
    if epi == B.EPI_RESIDUAL:
        np.testing.assert_allclose(_f64(out), ref, rtol=1e-4, atol=1e-4)
    else:
        np.testing.assert_allclose(_f64(out), ref, rtol=EPS16[dtype] * 1.01, atol=2e-3 * EPS16[dtype] * 256)


@pytest.mark.parametrize("dtype", SIXTEEN)
def test_gemm_16_swiglu_over_the_range_of_the_gate(dtype):
    """Gates with the factor 1 + e^-g from 1 to just below the largest fp32 number, on whole and cut column tiles.  The result
    is one 16-bit rounding of gate / (1 + e^-gate) * up with an fp32 exponential, whose argument's rounding is worth up to
    |gate| 2^-24 of it, some 2^-17 at the largest; below the smallest normal number of the type, half a unit there."""
    gates = torch.tensor([-88.5, -88.25, -88.0, -87.5, -87.0, -80.0, -16.5, -3.25, -0.5, 0.0, 0.5, 3.25, 16.5, 90.0], dtype=dtype)
    K, F, ups = 64, 40, torch.tensor([1.0, -3.0, 0.25, 512.0], dtype=dtype)
    A, Wt = torch.zeros(len(gates), K, dtype=dtype), torch.zeros(2 * F, K, dtype=dtype)
    A[:, 0], A[:, 1] = gates, 1.0
    Wt[:F, 0] = 1.0
    Wt[F:, 1] = ups.repeat(F // len(ups))
    out = torch.full((len(gates), F), 7.0, dtype=dtype, device=DEV)
    B.op_gemm(B.EPI_SWIGLU, A.to(DEV), Wt.to(DEV), out)
    g, u = _f64(gates)[:, None], _f64(Wt[F:, 1])[None]
    ref = g / (1.0 + np.exp(-g)) * u
    tiny = torch.finfo(dtype).tiny
    np.testing.assert_array_less(np.abs(_f64(out) - ref), (EPS16[dtype] + 2.0 ** -16) * np.maximum(np.abs(ref), tiny) + 1e-45)


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_RESIDUAL, B.EPI_SWIGLU])
@pytest.mark.parametrize("K", [64, 128, 192, 320, 448])
def test_gemm_16_big_tile_with_few_and_odd_slice_counts(dtype, epi, K):
    """4100 x 6144 outputs are 17 x 24 tiles of 256 x 256 (SwiGLU: 17 x 24 of 256 x 128), enough for the launcher to pick
    the big tile, whose K loop is unrolled over six 64-deep slices: 1, 2, 3, 5 and 7 slices exercise exits inside the first
    turn and in the second."""
    assert gemm_plan(4100, 6144, K, epi == B.EPI_SWIGLU)[0][1] == "kTile256"
    _gemm_16_case(dtype, epi, 4100, 6144, K)


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_RESIDUAL, B.EPI_SWIGLU])
def test_gemm_16_big_tile_with_a_ragged_last_column_tile(dtype, epi):
    """N = 6144 + 128: the last column tile of the 256 x 256 path is half outside the matrix (SwiGLU: N / 2 = 3136 =
    24.5 tiles of 128 output columns)."""
    assert gemm_plan(4100, 6144 + 128, 320, epi == B.EPI_SWIGLU)[0][1] == "kTile256"
    _gemm_16_case(dtype, epi, 4100, 6144 + 128, 320)


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_RESIDUAL, B.EPI_SWIGLU])
def test_gemm_16_rows_beyond_whole_rounds_go_to_small_tiles_with_the_same_bits(dtype, epi):
    """2900 x 6144 outputs are 12 x 24 = 288 tiles of 256 x 256: one round of 256 compute units and a few tiles more.  The
    launcher gives the first 10 row tiles (240 tiles, one round) to the big tile and the last 340 rows to a second launch
    with smaller tiles.  Checked against the oracle, and bit for bit against the same rows in launches that take other tiles
    than the whole call took for them."""
    M, N, K, cut = 2900, 6144, 320, 2560
    glu = epi == B.EPI_SWIGLU
    assert gemm_plan(M, N, K, glu) == [(cut, "kTile256"), (M - cut, "kTile128x64")]
    _gemm_16_case(dtype, epi, M, N, K)
    A = _rand((M, K), dtype, 10 + M + K, 1.0).to(DEV)
    Wt = _rand((N, K), dtype, 20 + N + K, 1.0 / math.sqrt(K)).to(DEV)
    cols = N // 2 if glu else N

    def run(lo, hi):
        out = _rand((M, N), torch.float32, 30, 1.0)[lo:hi].to(DEV) if epi == B.EPI_RESIDUAL else torch.zeros(hi - lo, cols, dtype=dtype, device=DEV)
        B.op_gemm(epi, A[lo:hi], Wt, out)
        return out
    whole = run(0, M)
    for lo, hi, kind in ((0, 400, "kTile128x64"), (400, 1100, "kTile128"), (2480, 2560, "kTile64"), (1100, 2900, "kTile256"), (2820, 2900, "kTile64")):
        assert gemm_plan(hi - lo, N, K, glu) == [(hi - lo, kind)]
        assert torch.equal(run(lo, hi), whole[lo:hi]), (lo, hi)


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("epi", [B.EPI_RESIDUAL, B.EPI_SWIGLU])
@pytest.mark.parametrize("slices", range(1, 14))
def test_gemm_16_big_tile_at_every_place_of_its_ring(dtype, epi, slices):
    """The big tile's loop is unrolled over the six slices after which its three stages of A and two of W stand alike: 1 to 13
    slices end it at every place of the first two turns.  Bit for bit against the same rows in a launch of smaller tiles, which
    have rings of their own (and are compared to fp64 below); the last rows and columns are ragged."""
    M, N, K, glu = 4100, 6144 + 8, 64 * slices, epi == B.EPI_SWIGLU
    assert gemm_plan(M, N, K, glu)[0][1] == "kTile256"
    A = _rand((M, K), dtype, 91 + K, 1.0).to(DEV)
    Wt = _rand((N, K), dtype, 92 + K, 1.0 / math.sqrt(K)).to(DEV)
    X0 = _rand((M, N // 2 if glu else N), torch.float32 if not glu else dtype, 93, 1.0).to(DEV)
    whole = X0.clone()
    B.op_gemm(epi, A, Wt, whole)
    for lo, hi in ((0, 300), (2000, 2300), (3900, 4100)):
        assert all(k != "kTile256" for _, k in gemm_plan(hi - lo, N, K, glu))
        part = X0[lo:hi].clone()
        B.op_gemm(epi, A[lo:hi], Wt, part)
        assert torch.equal(part, whole[lo:hi]), (lo, hi)


# Per tile: its loop, (SwiGLU?, rows, N, 64-deep slices) of launches that take it.  The slices end a launch, within what the
# launcher gives the tile, at every place of the unrolled ring in its first and second turn (test_tile_plan.py checks that against
# the loops' generator; the big tile has a test of its own above); rows and N leave the last tiles ragged.  SwiGLU pairs two
# 32-column tiles in a wave, so the 32-wide tiles have none.
TILE_LAUNCHES = {
    "kTile256": ("256", [(g, 2001, 6152, k) for g in (False, True) for k in (1, 2, 3)]),
    "kTile128": ("128x128_2", [(g, 4101, 1000, k) for g in (False, True) for k in (1, 2, 3, 4, 5)]),
    "kTile128Deep": ("128x128_4", [(g, 9001, 200, k) for g in (False, True) for k in (6, 7, 8, 9, 10, 11)]),
    "kTile128x64": ("128x64_3", [(False, 9001, 200, k) for k in (1, 2, 3, 4, 5)] + [(False, 2601, 392, k) for k in (6, 7)] + [(True, 9001, 200, k) for k in (1, 2, 3, 4)] + [(True, 9001, 72, k) for k in (5, 6)]),
    "kTile64": ("64x64_5", [(False, 65, 4104, k) for k in range(3, 11)] + [(False, 1, 40, 1), (False, 33, 40, 2)] + [(True, 33, 40, k) for k in range(1, 11)]),
    "kTile32x64": ("32x64_4", [(False, 129, 6152, k) for k in (3, 4, 5, 6, 7, 8)] + [(True, 33, 40, k) for k in (11, 12, 13, 14)]),
    "kTile64x32": ("64x32_7", [(False, 33, 72, k) for k in range(3, 13)] + [(False, 33, 4104, k) for k in range(13, 29)]),
    "kTile32": ("32x32_9", [(False, 33, 72, k) for k in range(16, 37)] + [(False, 1, 1000, 16), (False, 65, 1000, 48)]),
}


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("kind,epi", [(k, e) for k, (_, launches) in TILE_LAUNCHES.items()
                                      for e in (B.EPI_STORE, B.EPI_RESIDUAL, B.EPI_SWIGLU, B.EPI_STORE_F32)
                                      if any(l[0] == (e == B.EPI_SWIGLU) for l in launches)])
def test_gemm_16_every_tile_size_gives_a_row_the_same_bits(dtype, epi, kind):
    """Every tile against fp64, and bit for bit against the same rows inside a taller launch that takes other tiles.  Products of
    16-bit operands are exact in fp32, so |error| of a sum of K of them is at most K 2^-24 sum |a w|; a 16-bit result is rounded
    once more (SwiGLU: as in the fp32 test)."""
    glu = epi == B.EPI_SWIGLU
    for _, M, N, slices in [l for l in TILE_LAUNCHES[kind][1] if l[0] == glu]:
        K, case = 64 * slices, (M, N, slices)
        assert gemm_plan(M, N, K, glu) == [(M, kind)], case
        tall = next((t for t in (100, 300, 500, 900, 2000, 4000, 8000, 12000, 17000, 24000, 40000, 80000) if t > M and kind not in [k for _, k in gemm_plan(t, N, K, glu)]), None)
        assert tall is not None, case
        A = _rand((tall, K), dtype, 71 + K, 1.0).to(DEV)
        Wt = _rand((N, K), dtype, 72 + N + K, 1.0 / math.sqrt(K)).to(DEV)
        X0 = _rand((tall, N), torch.float32, 73, 1.0).to(DEV) if epi == B.EPI_RESIDUAL else None

        def run(rows):
            if epi == B.EPI_RESIDUAL:
                out = X0[:rows].clone()
            else:
                out = torch.full((rows, N // 2 if glu else N), 7.0, dtype=torch.float32 if epi == B.EPI_STORE_F32 else dtype, device=DEV)
            B.op_gemm(epi, A[:rows], Wt, out)
            return out
        got = run(M)
        assert torch.equal(got, run(tall)[:M]), case
        a, w = A[:M].double(), Wt.double().t().contiguous()
        ref, mag = a @ w, a.abs() @ w.abs()
        bound = K * 2.0 ** -24 * mag
        if epi == B.EPI_RESIDUAL:
            ref = ref + X0[:M].double()
            bound = bound + 2.0 ** -23 * (X0[:M].double().abs() + mag)
        if glu:
            gt, up, bg, bu = ref[:, :N // 2], ref[:, N // 2:], bound[:, :N // 2], bound[:, N // 2:]
            ref = torch.nn.functional.silu(gt) * up
            bound = 1.1 * bg * up.abs() + gt.abs() * bu + bg * bu + 2.0 ** -20 * ref.abs()
        if epi in (B.EPI_STORE, B.EPI_SWIGLU):
            bound = bound * (1 + EPS16[dtype]) + EPS16[dtype] * ref.abs() + 2.0 ** -25          # 2^-25: half a unit of subnormal half
        assert ((got.double() - ref).abs() <= bound + 1e-30).all(), case


@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_RESIDUAL, B.EPI_SWIGLU])
@pytest.mark.parametrize("N,K", [(200, 64), (200, 68), (202, 688), (198, 67), (1376, 256), (2, 1)])
def test_gemm_fp32_tiles(epi, N, K):
    """fp32 on the matrix instruction: the two smallest tiles (SwiGLU: 32 x 64 and 64 x 32), rows of 16-byte aligned and other
    lengths, slices cut off by K, columns cut off by N.  Against fp64: |error| of a K-term fp32 sum of products is at most
    K 2^-24 sum |a w| (SwiGLU: of each factor, plus the exponential's and two products' roundings); and rows do not
    depend on how many are computed with them."""
    M = 6001
    g = torch.Generator().manual_seed(N * 1000 + K)
    A, Wt = torch.randn(M, K, generator=g), torch.randn(N, K, generator=g) / math.sqrt(K)
    X0 = torch.randn(M, N, generator=g)
    a, w, cols = A.to(DEV), Wt.to(DEV), N // 2 if epi == B.EPI_SWIGLU else N

    def run(rows):
        out = X0[:rows].to(DEV) if epi == B.EPI_RESIDUAL else torch.full((rows, cols), 7.0, device=DEV)
        B.op_gemm(epi, a[:rows], w, out)
        return out
    whole = run(M)
    ref, mag = A.double() @ Wt.double().T, A.double().abs() @ Wt.double().abs().T
    bound = (K + 2) * 2.0 ** -24 * mag
    if epi == B.EPI_RESIDUAL:
        ref, bound = ref + X0.double(), bound + 2.0 ** -23 * (X0.double().abs() + mag)
    if epi == B.EPI_SWIGLU:
        gt, up, bg, bu = ref[:, :cols], ref[:, cols:], bound[:, :cols], bound[:, cols:]
        ref = torch.nn.functional.silu(gt) * up
        bound = 1.1 * bg * up.abs() + gt.abs() * bu + bg * bu + 2.0 ** -20 * ref.abs()      # |silu'| < 1.1, |silu(x)| <= |x|
    assert ((whole.cpu().double() - ref).abs() <= bound + 1e-30).all()
    for rows in (1, 31, 33, 354, 1000):
        assert torch.equal(run(rows), whole[:rows]), rows


@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_RESIDUAL, B.EPI_SWIGLU])
@pytest.mark.parametrize("M,N,K,tile", [(3001, 1378, 130, (64, 32)), (6001, 1378, 128, (64, 32)), (4201, 1378, 100, (64, 64)), (20001, 1378, 130, (128, 64)),
                                        (20001, 1378, 132, (128, 64)), (20001, 2018, 260, (128, 128)), (20001, 2018, 270, (128, 128))])
def test_gemm_fp32_larger_tiles(epi, M, N, K, tile):
    """The larger tiles (taken by the number of rounds each needs), with ragged rows, columns and K, rows of 16-byte aligned and other
    lengths.  Every tile sums in the same order, so rows at the start, the middle and the end equal, bit for bit, the same rows in
    calls of at most 200, which take smaller tiles, those of 32 the smallest, and are compared to fp64 above."""
    glu = epi == B.EPI_SWIGLU
    assert fp32_tile(M, N, K, glu) == tile and fp32_tile(32, N, K, glu) == ((32, 64) if glu else (32, 32))
    g = torch.Generator().manual_seed(M + N + K)
    A, Wt = torch.randn(M, K, generator=g).to(DEV), (torch.randn(N, K, generator=g) / math.sqrt(K)).to(DEV)
    X0 = torch.randn(M, N // 2 if glu else N, generator=g).to(DEV)
    whole = X0.clone()
    B.op_gemm(epi, A, Wt, whole)
    for lo in (0, 1984, M // 64 * 64 - 128, M - 33):
        for rows in (32, 200):
            part = X0[lo:lo + rows].clone()
            B.op_gemm(epi, A[lo:lo + rows], Wt, part)
            assert torch.equal(part, whole[lo:lo + rows]), (lo, rows)


@pytest.mark.parametrize("epi,N", [(B.EPI_STORE, 8), (B.EPI_RESIDUAL, 8), (B.EPI_SWIGLU, 4)])
def test_gemm_fp32_row_panels(epi, N):
    """More rows than one grid covers (65535 blocks of 32): the launcher cuts the call into panels of 2 097 120 rows.  Bound as
    above, for 4 products."""
    K, M = 4, 65535 * 32 + 700
    g = torch.Generator(device=DEV).manual_seed(5)
    A, Wt = torch.randn(M, K, device=DEV, generator=g), torch.randn(N, K, device=DEV, generator=g)
    cols = N // 2 if epi == B.EPI_SWIGLU else N
    X0 = torch.randn(M, cols, device=DEV, generator=g)
    out = X0.clone()
    B.op_gemm(epi, A, Wt, out)
    prod = (A.double()[:, None, :] * Wt.double()[None]).unbind(2)
    ref, mag = sum(prod), sum(p.abs() for p in prod)
    bound = (K + 2) * 2.0 ** -24 * mag
    if epi == B.EPI_RESIDUAL:
        ref, bound = ref + X0.double(), bound + 2.0 ** -23 * (X0.double().abs() + mag)
    if epi == B.EPI_SWIGLU:
        gt, up, bg, bu = ref[:, :cols], ref[:, cols:], bound[:, :cols], bound[:, cols:]
        ref = torch.nn.functional.silu(gt) * up
        bound = 1.1 * bg * up.abs() + gt.abs() * bu + bg * bu + 2.0 ** -20 * ref.abs()
    assert ((out.double() - ref).abs() <= bound + 1e-30).all()


@pytest.mark.parametrize("dtype", SIXTEEN)
def test_gemm_16_fp32_output(dtype):
    M, N, K = 700, 6144, 1024
    A, Wt = _rand((M, K), dtype, 5), _rand((N, K), dtype, 6, 1.0 / math.sqrt(K))
    out = torch.zeros(M, N, dtype=torch.float32, device=DEV)
    B.op_gemm(B.EPI_STORE_F32, A.to(DEV), Wt.to(DEV), out)
    np.testing.assert_allclose(_f64(out), _f64(A) @ _f64(Wt).T, rtol=1e-4, atol=1e-4)


def test_gemm_16_row_panels_beyond_4gib():
    """A has more than 4 GiB of bytes: the launcher cuts it into row panels (the kernel addresses with 32-bit offsets).
    Sampled rows on both sides of the cut against the oracle's plain product."""
    K, N = 12288, 512
    M = ((1 << 32) // (K * 2) // 256 + 3) * 256                  # three row tiles past the first panel
    g = torch.Generator(device=DEV).manual_seed(7)
    A = torch.randn(M, K, device=DEV, generator=g, dtype=torch.float32).to(torch.float16)
    Wt = (torch.randn(N, K, device=DEV, generator=g, dtype=torch.float32) / math.sqrt(K)).to(torch.float16)
    out = torch.zeros(M, N, dtype=torch.float32, device=DEV)
    B.op_gemm(B.EPI_STORE_F32, A, Wt, out)
    torch.cuda.synchronize()
    cut = (1 << 32) // (K * 2) // 256 * 256
    rows = [0, 1, 255, cut - 1, cut, cut + 1, cut + 300, M - 1]
    ref = _f64(A[rows]) @ _f64(Wt).T
    np.testing.assert_allclose(_f64(out[rows]), ref, rtol=1e-4, atol=1e-4)
    assert out.abs().sum(dim=1).min().item() > 0                 # no row was left unwritten


def _vt_layout(lens):
    """Column of every token in the transposed V buffer: sequences start at multiples of 64; within every group of 16
    positions the columns follow the order 0-3, 8-11, 4-7, 12-15 (the header's prism_vt_column_of_key)."""
    col0 = np.concatenate([[0], np.cumsum([(l + 63) // 64 * 64 for l in lens])]).astype(np.int32)
    vt_col = np.concatenate([col0[i] + B.vt_column_of_key(np.arange(l)) for i, l in enumerate(lens)]).astype(np.int32)
    return col0[:-1], vt_col, int(col0[-1])


@pytest.mark.parametrize("dtype,nq,nkv,hd", [(torch.float32, 4, 2, 64), (torch.float32, 6, 3, 32), (torch.bfloat16, 8, 2, 128),
                                             (torch.float16, 8, 2, 128)])
@pytest.mark.parametrize("qk_norm", [True, False])
def test_qkv_finish(dtype, nq, nkv, hd, qk_norm):
    lens = [5, 130, 1, 64, 299]
    T = sum(lens)
    pos = np.concatenate([np.arange(l) for l in lens]).astype(np.int32)
    QKV = _rand((T, (nq + 2 * nkv) * hd), torch.float32, 40, 1.5)
    gq, gk = (1 + _rand((hd,), torch.float32, 41, 0.1)).to(dtype), (1 + _rand((hd,), torch.float32, 42, 0.1)).to(dtype)
    x = _f64(QKV).reshape(T, nq + 2 * nkv, hd)
    q, k, v = x[:, :nq], x[:, nq:nq + nkv], x[:, nq + nkv:]
    if qk_norm:
        q, k = O.rmsnorm(q, _f64(gq), 1e-6), O.rmsnorm(k, _f64(gk), 1e-6)
    q, k = O.rope(q, pos, 1e6), O.rope(k, pos, 1e6)
    d = QKV.to(DEV).clone()
    dpos = torch.from_numpy(pos).to(DEV)
    if dtype == torch.float32:
        B.op_qkv_finish(B.DTYPE_FP32, d, dpos, 512, gq.to(DEV), gk.to(DEV), nq, nkv, hd, 1e-6, 1e6, qk_norm)
        ref = np.concatenate([q, k, v], axis=1).reshape(T, -1)
        np.testing.assert_allclose(_f64(d), ref, rtol=1e-5, atol=2e-5)
        return
    col0, vt_col, ncol = _vt_layout(lens)
    QK = torch.zeros(T, (nq + nkv) * hd, dtype=dtype, device=DEV)
    Vt = torch.zeros(nkv, hd, ncol, dtype=torch.float16, device=DEV)
    B.op_qkv_finish(B._dt(QK), d, dpos, 512, gq.to(DEV), gk.to(DEV), nq, nkv, hd, 1e-6, 1e6, qk_norm,
                    QK, Vt, torch.from_numpy(vt_col).to(DEV), ncol)
    ref_qk = np.concatenate([q, k], axis=1).reshape(T, -1)
    got = _f64(QK)
    # one rounding to bf16 of a value computed in fp32: within one bf16 ulp of the oracle's rounded value,
    # and equal to it except where fp32 arithmetic lands on the other side of a rounding boundary
    np.testing.assert_allclose(got, ref_qk, rtol=EPS16[dtype] * 1.01, atol=1e-6)
    assert np.mean(got != O.round_operand(ref_qk, OPERAND[dtype])) < 0.02
    vt = _f64(Vt)
    ref_v = np.transpose(O.round_operand(v, OPERAND[dtype]), (1, 2, 0))
    diff = np.abs(vt[:, :, vt_col] - ref_v)
    # exact (rounding + layout), except that half cannot hold bf16 values below 2^-17 exactly
    assert diff.max() <= 2.0 ** -25 and np.all(diff[np.abs(ref_v) >= 2.0 ** -14] == 0), (diff.max(), int((diff > 0).sum()))
    pad = np.setdiff1d(np.arange(ncol), vt_col)
    assert (vt[:, :, pad] == 0).all()


def _off_by_one(t):
    """The same values in a buffer that starts one element behind an aligned address."""
    b = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:].view(t.shape)
    b.copy_(t)
    assert b.data_ptr() % 8 != 0
    return b


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("qk_norm", [True, False])
@pytest.mark.parametrize("moved", ["QKV", "QK", "gains"])
def test_qkv_finish_of_unaligned_buffers_has_the_same_bits(dtype, qk_norm, moved):
    """Head size 128 goes value by value through two kernels where a buffer does not allow 16- and 8-byte accesses."""
    nq, nkv, hd, lens = 8, 2, 128, [5, 130, 1, 64, 299]
    T = sum(lens)
    pos = torch.from_numpy(np.concatenate([np.arange(l) for l in lens]).astype(np.int32)).to(DEV)
    col0, vt_col, ncol = _vt_layout(lens)
    QKV = _rand((T, (nq + 2 * nkv) * hd), torch.float32, 43, 1.5).to(DEV)
    gq, gk = ((1 + _rand((hd,), torch.float32, seed, 0.1)).to(dtype).to(DEV) for seed in (41, 42))
    QK, Vt = torch.zeros(T, (nq + nkv) * hd, dtype=dtype, device=DEV), torch.zeros(nkv, hd, ncol, dtype=torch.float16, device=DEV)
    QK2, Vt2 = _off_by_one(QK) if moved == "QK" else QK.clone(), Vt.clone()
    run = lambda x, a, b, qk, vt: B.op_qkv_finish(B._dt(QK), x, pos, 512, a, b, nq, nkv, hd, 1e-6, 1e6, qk_norm, qk, vt,
                                                  torch.from_numpy(vt_col).to(DEV), ncol)
    run(QKV, gq, gk, QK, Vt)
    run(_off_by_one(QKV) if moved == "QKV" else QKV, *((_off_by_one(gq), _off_by_one(gk)) if moved == "gains" else (gq, gk)), QK2, Vt2)
    assert torch.equal(QK, QK2) and torch.equal(Vt, Vt2)


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("qk_norm", [True, False])
@pytest.mark.parametrize("nq,H,lens,kinds", [
    (32, 256, [700, 1, 1024, 64, 911], ["kHead128"]),
    (32, 1024, [1000, 1, 1024, 64, 1024, 887, 1000], ["kHead256"]),
    (32, 1024, [700, 1, 1024, 64, 911, 7], ["kHead256", "kHead64"]),
    (24, 1024, [900, 1, 1024, 64, 1024, 487], ["kHead256", "kHead128Deep"]),
    (24, 1024, [900, 1, 1024, 64, 1024, 1024, 63], ["kHead256", "kHead128"])])
def test_qkv_project_fused(dtype, qk_norm, nq, H, lens, kinds):
    """Projection + norm + RoPE + V transposition in one kernel against the oracle's separate steps, several row
    tiles with a ragged last one, and against the unfused device path: the 256-row tile alone, with a second launch of
    each smaller tile for the remaining rows, and a smaller tile alone."""
    nkv, hd = 8, 128
    assert [k for _, k in head_plan(sum(lens), nq, nkv, H)] == kinds
    T = sum(lens)
    pos = np.concatenate([np.arange(l) for l in lens]).astype(np.int32)
    Xn, Wt = _rand((T, H), dtype, 50), _rand(((nq + 2 * nkv) * hd, H), dtype, 51, 1.0 / math.sqrt(H))
    gq, gk = (1 + _rand((hd,), torch.float32, 52, 0.1)).to(dtype), (1 + _rand((hd,), torch.float32, 53, 0.1)).to(dtype)
    x = (_f64(Xn) @ _f64(Wt).T).reshape(T, nq + 2 * nkv, hd)
    q, k, v = x[:, :nq], x[:, nq:nq + nkv], x[:, nq + nkv:]
    if qk_norm:
        q, k = O.rmsnorm(q, _f64(gq), 1e-6), O.rmsnorm(k, _f64(gk), 1e-6)
    q, k = O.rope(q, pos, 1e6), O.rope(k, pos, 1e6)
    col0, vt_col, ncol = _vt_layout(lens)
    dpos, dcol = torch.from_numpy(pos).to(DEV), torch.from_numpy(vt_col).to(DEV)
    QK = torch.zeros(T, (nq + nkv) * hd, dtype=dtype, device=DEV)
    Vt = torch.zeros(nkv, hd, ncol, dtype=torch.float16, device=DEV)
    B.op_qkv_project(Xn.to(DEV), Wt.to(DEV), dpos, 1024, gq.to(DEV), gk.to(DEV), nq, nkv, hd, 1e-6, 1e6, qk_norm, QK, Vt, dcol, ncol)
    ref_qk = np.concatenate([q, k], axis=1).reshape(T, -1)
    got = _f64(QK)
    # fp32 accumulation over H products, fp32 norm and rotation, then ONE 16-bit rounding
    atol = 2e-6 * H / 256                                    # the fp32 sums' share, for values near zero: grows with their length
    np.testing.assert_allclose(got, ref_qk, rtol=EPS16[dtype] * 1.01, atol=atol)
    assert np.mean(got != O.round_operand(ref_qk, OPERAND[dtype])) < 0.02
    vt = _f64(Vt)
    ref_v = np.transpose(v, (1, 2, 0))
    np.testing.assert_allclose(vt[:, :, vt_col], ref_v, rtol=EPS16[dtype] * 1.01, atol=atol)
    pad = np.setdiff1d(np.arange(ncol), vt_col)
    assert (vt[:, :, pad] == 0).all()
    # the unfused device path: one order of every sum, so the same bits
    QKV = torch.zeros(T, (nq + 2 * nkv) * hd, dtype=torch.float32, device=DEV)
    B.op_gemm(B.EPI_STORE_F32, Xn.to(DEV), Wt.to(DEV), QKV)
    QK2, Vt2 = torch.zeros_like(QK), torch.zeros_like(Vt)
    B.op_qkv_finish(B._dt(QK), QKV, dpos, 1024, gq.to(DEV), gk.to(DEV), nq, nkv, hd, 1e-6, 1e6, qk_norm, QK2, Vt2, dcol, ncol)
    assert torch.equal(Vt, Vt2) and torch.equal(QK, QK2)


def test_qkv_project_rejects_small_problems():
    Xn, Wt = torch.zeros(100, 256, dtype=torch.float16, device=DEV), torch.zeros(48 * 128, 256, dtype=torch.float16, device=DEV)
    z = torch.zeros(128, dtype=torch.float16, device=DEV)
    with pytest.raises(B.PrismError) as e:
        B.op_qkv_project(Xn, Wt, torch.zeros(100, dtype=torch.int32, device=DEV), 16, z, z, 32, 8, 128, 1e-6, 1e6, True,
                         torch.zeros(100, 40 * 128, dtype=torch.float16, device=DEV), torch.zeros(8, 128, 128, dtype=torch.float16, device=DEV),
                         torch.zeros(100, dtype=torch.int32, device=DEV), 128)
    assert e.value.code == B.EUNSUPPORTED


ATTN_CASES = [
    (torch.float32, 4, 2, 64, [1, 17, 64, 100]),
    (torch.float32, 6, 3, 32, [33, 2]),
    (torch.bfloat16, 8, 2, 128, [1, 63, 64, 65, 130, 300]),      # G = 4
    (torch.bfloat16, 16, 8, 128, [200, 129, 31]),                # G = 2
    (torch.bfloat16, 8, 8, 128, [257, 5]),                       # G = 1
    (torch.bfloat16, 8, 1, 128, [97, 32]),                       # G = 8
    (torch.bfloat16, 32, 8, 128, [1024, 700]),                   # the 8B head shape at its sequence length
    (torch.float16, 32, 8, 128, [1024, 700]),
    (torch.float16, 16, 8, 128, [200, 129, 31]),
    (torch.float16, 8, 2, 128, [1, 63, 64, 65, 130, 300]),
]


@pytest.mark.parametrize("dtype,nq,nkv,hd,lens", ATTN_CASES)
def test_attention(dtype, nq, nkv, hd, lens):
    T = sum(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    QKV = _rand((T, (nq + 2 * nkv) * hd), dtype, 50 + T, 1.0)
    out = torch.zeros(T, nq * hd, dtype=dtype, device=DEV)
    x = _f64(QKV).reshape(T, nq + 2 * nkv, hd)
    if dtype == torch.float32:
        B.op_attention(B.DTYPE_FP32, QKV.to(DEV), None, 0, cu, None, nq, nkv, hd, out)
    else:
        col0, vt_col, ncol = _vt_layout(lens)
        QK = QKV[:, :(nq + nkv) * hd].contiguous().to(DEV)
        Vt = torch.zeros(nkv, hd, ncol, dtype=torch.float16)
        Vt[:, :, torch.from_numpy(vt_col.astype(np.int64))] = QKV.view(T, -1, hd)[:, nq + nkv:].permute(1, 2, 0).to(torch.float16)
        B.op_attention(B._dt(QK), QK, Vt.to(DEV), ncol, cu, col0, nq, nkv, hd, out)
    ref = np.concatenate([O.causal_gqa_attention(x[a:b, :nq], x[a:b, nq:nq + nkv], x[a:b, nq + nkv:]).reshape(b - a, -1)
                          for a, b in zip(cu[:-1], cu[1:])])
    # bf16 mode: exact operands, f16 probabilities, fp32 accumulation, one bf16 rounding of the output
    tol = dict(rtol=1e-4, atol=1e-5) if dtype == torch.float32 else dict(rtol=2 ** -8 if dtype == torch.bfloat16 else 2 ** -9, atol=2e-3)
    np.testing.assert_allclose(_f64(out), ref, **tol)


@pytest.mark.parametrize("nq,nkv,hd", [(4, 2, 64), (6, 3, 32), (3, 1, 128), (2, 2, 48)])
def test_attention_fp32_work_items(nq, nkv, hd):
    """fp32 attention by work items (head sizes 32, 64, 128; 48 goes token by token): sequences around the 16-key tiles and the
    64-query items, more than one item per sequence.  A sequence holding infinities and NaN behind its first 20 tokens
    changes neither those nor any other sequence."""
    lens = [1, 15, 16, 17, 63, 64, 65, 200, 333, 40, 31]
    T = sum(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    QKV = _rand((T, (nq + 2 * nkv) * hd), torch.float32, 500 + hd, 1.0)
    x = _f64(QKV).reshape(T, nq + 2 * nkv, hd)
    ref = np.concatenate([O.causal_gqa_attention(x[a:b, :nq], x[a:b, nq:nq + nkv], x[a:b, nq + nkv:]).reshape(b - a, -1)
                          for a, b in zip(cu[:-1], cu[1:])])
    out, again = torch.zeros(T, nq * hd, device=DEV), torch.zeros(T, nq * hd, device=DEV)
    B.op_attention(B.DTYPE_FP32, QKV.to(DEV), None, 0, cu, None, nq, nkv, hd, out)
    np.testing.assert_allclose(_f64(out), ref, rtol=1e-5, atol=2e-6)
    dirty = QKV.clone()
    i = lens.index(200)
    dirty[cu[i] + 20:cu[i + 1]] = torch.tensor([float("nan"), float("inf"), -float("inf"), 1e38]).repeat(180 * QKV.shape[1] // 4).view(180, -1)
    B.op_attention(B.DTYPE_FP32, dirty.to(DEV), None, 0, cu, None, nq, nkv, hd, again)
    clean = torch.ones(T, dtype=torch.bool)
    clean[cu[i] + 20:cu[i + 1]] = False
    assert torch.equal(again.cpu()[clean], out.cpu()[clean])
    assert not torch.isfinite(again.cpu()[cu[i + 1] - 1]).any()


@pytest.mark.parametrize("hd", [32, 64, 128, 48])
@pytest.mark.parametrize("n_blocked", [15, 16, 20, 64, 70])
@pytest.mark.parametrize("by", ["infinite keys", "overflow"])
def test_attention_fp32_scores_of_minus_infinity(hd, n_blocked, by):
    """The first n_blocked keys of a sequence score -inf, through infinities in K or through an overflow of finite q . k: they
    weigh nothing, and a query that sees a finite score has the softmax over the finite ones, also where all keys of its
    first tiles (16 keys each) are blocked.  A query without any finite score has 0 / 0, as by the definition."""
    nq, nkv, L, other = 4, 2, 150, 30
    QKV = _rand((L + other, (nq + 2 * nkv) * hd), torch.float32, 700 + hd + n_blocked, 1.0)
    x = QKV.view(L + other, nq + 2 * nkv, hd)
    x[:, :nq] = x[:, :nq].abs() + 0.1
    x[:n_blocked, nq:nq + nkv] = -math.inf
    ref = [O.causal_gqa_attention(_f64(s[:, :nq]), np.maximum(_f64(s[:, nq:nq + nkv]), -1e30), _f64(s[:, nq + nkv:])).reshape(len(s), -1)
           for s in (x[:L], x[L:])]                          # -1e30: the same weights of zero beside scores of order one
    if by == "overflow":
        x[:, :nq] *= 16
        x[n_blocked:, nq:nq + nkv] /= 16
        x[:n_blocked, nq:nq + nkv] = -3e38
    out = torch.zeros(L + other, nq * hd, device=DEV)
    B.op_attention(B.DTYPE_FP32, QKV.to(DEV), None, 0, np.array([0, L, L + other], np.int32), None, nq, nkv, hd, out)
    got = _f64(out)
    assert np.isnan(got[:n_blocked]).all()
    np.testing.assert_allclose(got[n_blocked:L], ref[0][n_blocked:], rtol=1e-5, atol=2e-6)
    np.testing.assert_allclose(got[L:], ref[1], rtol=1e-5, atol=2e-6)


@pytest.mark.parametrize("moved", ["QKV", "out"])
def test_attention_fp32_of_unaligned_buffers(moved):
    """Buffers that do not allow 16-byte accesses go token by token, at the tolerance of the work items."""
    nq, nkv, hd, lens = 4, 2, 64, [1, 17, 64, 100]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    QKV = _rand((sum(lens), (nq + 2 * nkv) * hd), torch.float32, 60, 1.0)
    x = _f64(QKV).reshape(-1, nq + 2 * nkv, hd)
    ref = np.concatenate([O.causal_gqa_attention(x[a:b, :nq], x[a:b, nq:nq + nkv], x[a:b, nq + nkv:]).reshape(b - a, -1)
                          for a, b in zip(cu[:-1], cu[1:])])
    dev, out = QKV.to(DEV), torch.zeros(sum(lens), nq * hd, device=DEV)
    dev, out = (_off_by_one(dev), out) if moved == "QKV" else (dev, _off_by_one(out))
    B.op_attention(B.DTYPE_FP32, dev, None, 0, cu, None, nq, nkv, hd, out)
    np.testing.assert_allclose(_f64(out), ref, rtol=1e-5, atol=2e-6)


@pytest.mark.parametrize("hd", [64, 48])
def test_attention_fp32_sequences_that_start_behind_token_zero(hd):
    """cu_seqlens[0] > 0, with work items (head size 64) and with positions token by token (48): the sequences are what they
    are when they start at token 0, to the bit, and a token in front of them attends to itself, so its output is its value."""
    nq, nkv, lens, skip = 4, 2, [70, 1, 33], 37
    T = sum(lens)
    QKV = _rand((skip + T, (nq + 2 * nkv) * hd), torch.float32, 800 + hd, 1.0)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    front, behind = torch.zeros(T, nq * hd, device=DEV), torch.zeros(skip + T, nq * hd, device=DEV)
    B.op_attention(B.DTYPE_FP32, QKV[skip:].contiguous().to(DEV), None, 0, cu, None, nq, nkv, hd, front)
    B.op_attention(B.DTYPE_FP32, QKV.to(DEV), None, 0, cu + skip, None, nq, nkv, hd, behind)
    assert torch.equal(behind[skip:], front)
    v = QKV.view(skip + T, nq + 2 * nkv, hd)[:skip, nq + nkv:].repeat_interleave(nq // nkv, dim=1)
    assert torch.equal(behind[:skip].cpu(), v.reshape(skip, -1))


@pytest.mark.parametrize("dtype,nq,nkv,hd", [(torch.float32, 2, 1, 64), (torch.float16, 4, 2, 128), (torch.bfloat16, 8, 1, 128)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 256])
def test_attention_by_sequences_and_by_list(dtype, nq, nkv, hd, n):
    """Up to 256 sequences travel in the launch's arguments, searched 64 at a time; 257 and more go by a list of work items.
    The n sequences have the same bits alone and at the front of a longer call, of one block of queries and of several."""
    lens = np.array([1 + (i * 37) % 150 for i in range(257)])
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col0, vt_col, ncol = _vt_layout(lens)
    QKV = _rand((int(cu[-1]), (nq + 2 * nkv) * hd), dtype, 91, 1.0).to(DEV)
    QK, Vt = QKV, None
    if dtype != torch.float32:
        QK = QKV[:, :(nq + nkv) * hd].contiguous()
        Vt = torch.zeros(nkv, hd, ncol, dtype=torch.float16, device=DEV)
        Vt[:, :, torch.from_numpy(vt_col.astype(np.int64)).to(DEV)] = QKV.view(len(QKV), -1, hd)[:, nq + nkv:].permute(1, 2, 0).to(torch.float16)
    code = B.DTYPE_FP32 if Vt is None else B._dt(QK)
    few, many = (torch.zeros(len(QKV), nq * hd, dtype=dtype, device=DEV) for _ in range(2))
    B.op_attention(code, QK, Vt, ncol, cu[:n + 1], col0[:n], nq, nkv, hd, few)
    B.op_attention(code, QK, Vt, ncol, cu, col0, nq, nkv, hd, many)
    T = int(cu[n])
    assert torch.equal(few[:T], many[:T]) and not few[T:].any()
    assert many.float().abs().sum(1).min() > 0


@pytest.mark.parametrize("hd", [32, 64, 128])
@pytest.mark.parametrize("lens", [[8192, 1, 64, 65, 4097, 130], [16, 17, 32, 33, 48, 49], [200] * 5 + [64] * 3 + [129]])
def test_attention_fp32_longest_first_and_by_list(hd, lens):
    """Work items dealt longest first (up to 128 blocks of a sequence, searched 64 at a time; tiles in turn in two sets of registers,
    odd and even numbers of them) against the list, which a call takes whose first sequence starts behind token 0, to the bit."""
    nq, nkv = 2, 1
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    QKV = _rand((1 + sum(lens), (nq + 2 * nkv) * hd), torch.float32, 810 + hd, 1.0).to(DEV)
    levels, by_list = torch.zeros(sum(lens), nq * hd, device=DEV), torch.zeros(1 + sum(lens), nq * hd, device=DEV)
    B.op_attention(B.DTYPE_FP32, QKV[1:].contiguous(), None, 0, cu, None, nq, nkv, hd, levels)
    B.op_attention(B.DTYPE_FP32, QKV, None, 0, cu + 1, None, nq, nkv, hd, by_list)
    assert torch.equal(levels, by_list[1:]) and levels.abs().sum(1).min() > 0


@pytest.mark.parametrize("nq,nkv,hd,n,longest_first", [(16, 8, 32, 136, True), (16, 8, 32, 137, False), (16, 8, 64, 68, True), (16, 8, 64, 69, False),
                                                       (16, 8, 128, 34, True), (16, 8, 128, 35, False), (12, 6, 128, 180, True), (12, 6, 128, 183, False),
                                                       (2, 1, 64, 300, True), (16, 16, 64, 300, False)])
def test_attention_fp32_on_both_sides_of_its_order_rule(nq, nkv, hd, n, longest_first):
    """Pools whose K/V lie just below and above the limits between longest first and sequence by sequence, in launch arguments and by list: every
    sequence has the bits that it has in a call of its own."""
    lens = np.array([300 + (i * 37) % 320 for i in range(n)])
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    kv, limit = int(cu[-1]) * nkv * hd * 8, 512e6 if nq <= 12 else 128e6
    assert (kv <= limit) == longest_first and (n == 300 or abs(kv / limit - 1) < 0.05)
    QKV = torch.randn(int(cu[-1]), (nq + 2 * nkv) * hd, generator=torch.Generator(DEV).manual_seed(n), device=DEV)
    out = torch.zeros(int(cu[-1]), nq * hd, device=DEV)
    B.op_attention(B.DTYPE_FP32, QKV, None, 0, cu, None, nq, nkv, hd, out)
    for i in range(n):
        a, b = int(cu[i]), int(cu[i + 1])
        alone = torch.zeros(b - a, nq * hd, device=DEV)
        B.op_attention(B.DTYPE_FP32, QKV[a:b].clone(), None, 0, np.array([0, b - a], np.int32), None, nq, nkv, hd, alone)
        assert torch.equal(out[a:b], alone), i


def test_fp32_call_on_both_sides_of_the_attention_order_rule():
    """A whole fp32 call whose K/V exceed the limit for longest first, against the same call in chunks that do not."""
    m = W.ModelShape(2, 128, 16, 8, 64, 192, 64, "fp32")
    d = torch.Generator().manual_seed(5)
    draw = lambda *s: torch.randn(*s, generator=d) * 0.05
    layers = [{n: (1 + draw(*s) if len(s) == 1 else draw(*s)).to(DEV) for n, s in W.layer_tensor_shapes(m).items()} for _ in range(2)]
    wt = W.Weights(draw(64, 128).to(DEV), layers, (1 + draw(128)).to(DEV))
    r = np.random.RandomState(4)
    q, cands = r.randint(0, 64, 9).astype(np.int32), [r.randint(0, 64, 200 + (i * 53) % 480).astype(np.int32) for i in range(80)]
    T = sum(len(c) + len(q) for c in cands)
    assert T * 8 * 64 * 8 > 128e6
    scores = []
    for chunk in (0, 16):
        p = B.Prism(m, wt, chunk_cands=chunk)
        _, _, rep = p.select(q, cands, len(cands))
        p.destroy()
        scores.append(rep.scores[-1])
    assert np.array_equal(scores[0], scores[1]) and len(set(scores[0])) == len(cands)


@pytest.mark.parametrize("nq,nkv", [(1, 1), (16, 8), (32, 8)])
@pytest.mark.parametrize("T", [1, 3, 65])
def test_qkv_finish_16_evaluates_the_tables_rotations(nq, nkv, T):
    """The one-launch kernel (a part of a round of heads, one, more than one; tokens that fill no workgroup) against the kernels
    that read the table, to the bit."""
    hd, dtype = 128, torch.float16
    pos = torch.arange(4096 - T, 4096, dtype=torch.int32, device=DEV)
    col = torch.from_numpy(B.vt_column_of_key(np.arange(T, dtype=np.int32))).to(DEV)
    QKV = _rand((T, (nq + 2 * nkv) * hd), torch.float32, 44, 1.5).to(DEV)
    g = (1 + _rand((hd,), torch.float32, 41, 0.1)).to(dtype).to(DEV)
    got = []
    for x in (QKV, _off_by_one(QKV)):
        QK, Vt = torch.zeros(T, (nq + nkv) * hd, dtype=dtype, device=DEV), torch.zeros(nkv, hd, 128, dtype=torch.float16, device=DEV)
        B.op_qkv_finish(B._dt(QK), x, pos, 4096, g, g, nq, nkv, hd, 1e-6, 1e6, True, QK, Vt, col, 128)
        got.append((QK, Vt))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("nq,nkv,T", [(1, 1, 8191), (1, 1, 8192), (2, 1, 8193), (4, 2, 8207), (5, 1, 8208), (4, 3, 8200)])
def test_qkv_finish_16_of_few_heads_and_many_tokens(nq, nkv, T):
    """From 8192 tokens on a wave takes up to six heads of four tokens: both sides of each limit and workgroups that tokens do not fill,
    against the kernels that read the table, to the bit."""
    hd, dtype, stride = 128, torch.float16, -(-T // 64) * 64
    pos = 4095 - torch.arange(T, dtype=torch.int32, device=DEV) % 4096
    col = torch.from_numpy(B.vt_column_of_key(np.arange(T, dtype=np.int32))).to(DEV)
    QKV = _rand((T, (nq + 2 * nkv) * hd), torch.float32, 45, 1.5).to(DEV)
    gq, gk = ((1 + _rand((hd,), torch.float32, seed, 0.1)).to(dtype).to(DEV) for seed in (41, 42))
    got = []
    for x in (QKV, _off_by_one(QKV)):
        QK, Vt = torch.zeros(T, (nq + nkv) * hd, dtype=dtype, device=DEV), torch.zeros(nkv, hd, stride, dtype=torch.float16, device=DEV)
        B.op_qkv_finish(B._dt(QK), x, pos, 4096, gq, gk, nq, nkv, hd, 1e-6, 1e6, True, QK, Vt, col, stride)
        got.append((QK, Vt))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]) and got[0][0].float().abs().sum(1).min() > 0


def test_attention_refuses_a_transposed_v_stride_beyond_its_32_bit_offsets():
    """The 16-bit kernel addresses the 128 rows of a KV head's V^T with 32-bit byte offsets: a row stride of 2^24 columns
    (128 rows x 2 bytes = 4 GiB) is refused before anything is launched (the buffers here are tiny and never touched)."""
    nq, nkv, hd = 8, 2, 128
    QK = torch.zeros(4, (nq + nkv) * hd, dtype=torch.float16, device=DEV)
    Vt = torch.zeros(nkv, hd, 64, dtype=torch.float16, device=DEV)
    out = torch.zeros(4, nq * hd, dtype=torch.float16, device=DEV)
    with pytest.raises(B.PrismError) as e:
        B.op_attention(B.DTYPE_F16, QK, Vt, 1 << 24, np.array([0, 4], np.int32), np.array([0], np.int32), nq, nkv, hd, out)
    assert e.value.code == B.EUNSUPPORTED


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_score(dtype):
    H, T = 1024, 500
    X = _rand((T, H), torch.float32, 60, 3.0)
    g = (1 + _rand((H,), torch.float32, 61, 0.05)).to(dtype)
    wy, wn = _rand((H,), dtype, 62, 0.02), _rand((H,), dtype, 63, 0.02)
    rows = np.array([0, 17, 499, 250, 17], np.int32)
    s = torch.zeros(len(rows), dtype=torch.float32, device=DEV)
    B.op_score(X.to(DEV), torch.from_numpy(rows).to(DEV), g.to(DEV), wy.to(DEV), wn.to(DEV), 1e-6, s)
    ref = [O.head_score(_f64(X)[r], _f64(g), _f64(wy), _f64(wn), 1e-6) for r in rows]
    np.testing.assert_allclose(_f64(s), ref, rtol=1e-5, atol=2e-6)


def _route_case(scores, K, k, tau):
    s = torch.tensor(scores, dtype=torch.float32)
    fate = torch.full((len(scores),), 9, dtype=torch.int8, device=DEV)
    stats = torch.zeros(4, dtype=torch.float64, device=DEV)
    B.op_route(s.to(DEV), K, k, tau, fate, stats)
    r = O.route(s.numpy().astype(np.float64), K, k, float(np.float32(tau)))
    st = stats.cpu().numpy()
    assert np.array_equal(fate.cpu().numpy(), r.fate), (scores[:8], K, k, tau)
    assert st[0] == r.mean and st[1] == r.std and bool(st[2]) == r.gate and int(st[3]) == r.n_clusters


def test_route_hand_cases_and_degenerate_inputs():
    _route_case([0.1, 5.0, 0.2, 9.0, 5.1, 0.0, 4.9], 2, 3, 0.0)
    _route_case([0.1, 5.0, 0.2, 9.0, 5.1, 0.0, 4.9], 5, 3, 0.0)
    _route_case([1.0, 2.0, 3.0], 3, 3, 0.0)                # n <= K
    _route_case([4.0, 4.0, 4.0, 4.0], 2, 3, 0.0)           # one distinct value
    _route_case([4.0, 4.0, 1.0, 1.0, 1.0], 1, 3, 0.0)      # two distinct values, k = 3
    _route_case([2.0, 1.0, 0.0], 1, 2, 0.0)                # SSE tie between the two splits
    _route_case([1, 2, 3, 4], 2, 3, 0.45)                  # gate closed
    _route_case([1, 2, 3, 4], 2, 3, 0.44)                  # gate open
    _route_case([5.0], 1, 3, 0.0)


@pytest.mark.parametrize("seed", range(12))
def test_route_random_matches_oracle_bit_for_bit(seed):
    r = np.random.default_rng(seed)
    n = int(r.choice([4, 9, 40, 100, 257, 500]))
    k = int(r.integers(2, 6))
    K = int(r.integers(1, n))
    s = r.normal(size=n) * r.choice([0.3, 1.0, 3.0]) + r.choice([0.0, 2.0])
    if seed % 3 == 0:
        s = np.round(s, 1)                                 # many exact duplicates
    _route_case(s.astype(np.float32).tolist(), K, k, float(r.choice([0.0, 0.5])))


def test_route_large_n():
    r = np.random.default_rng(99)
    _route_case(r.normal(size=1500).astype(np.float32).tolist(), 20, 3, 0.0)


def test_compact_and_topk():
    H = 512
    lens = np.array([5, 130, 1, 64, 299, 40], np.int32)
    start = np.concatenate([[0], np.cumsum(lens)])[:-1].astype(np.int32)
    X = _rand((int(lens.sum()), H), torch.float32, 70)
    keep = np.array([1, 0, 1, 1, 0, 1], bool)
    kl = lens[keep]
    dst = np.concatenate([[0], np.cumsum(kl)])[:-1].astype(np.int32)
    Xd = torch.full((int(kl.sum()) + 3, H), 7.0, dtype=torch.float32, device=DEV)
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    B.op_compact(X.to(DEV), Xd, T(start[keep]), T(dst), T(kl))
    ref = np.concatenate([X.numpy()[s:s + l] for s, l in zip(start[keep], kl)])
    assert np.array_equal(Xd.cpu().numpy()[:len(ref)], ref) and (Xd.cpu().numpy()[len(ref):] == 7.0).all()

    s = np.array([0.5, 2.0, -1.0, 2.0, 0.5, 3.5, 2.0], np.float32)
    pos = torch.zeros(4, dtype=torch.int32, device=DEV)
    sc = torch.zeros(4, dtype=torch.float32, device=DEV)
    B.op_topk(T(s), 4, pos, sc)
    order = O.rank_order(s.astype(np.float64))[:4]
    assert pos.cpu().numpy().tolist() == order.tolist() == [5, 1, 3, 6]
    assert np.array_equal(sc.cpu().numpy(), s[order])


@pytest.mark.parametrize("n", [255, 256, 700, 2047, 2048, 4096])
@pytest.mark.parametrize("H", [4, 260])
def test_compact_of_many_sequences(n, H):
    """The launcher gives a sequence 64 workgroups, fewer from 256 sequences and 8 from 2048 on; sequences of none to 40 rows, and
    one of 900, which takes several rounds of its workgroups' pieces."""
    r = np.random.default_rng(n)
    lens = r.integers(0, 41, size=n).astype(np.int32)
    lens[n // 2] = 900
    start = np.concatenate([[0], np.cumsum(lens + 1)])[:-1].astype(np.int32)         # a row between sequences stays behind
    dst = np.concatenate([[0], np.cumsum(lens)])[:-1].astype(np.int32)
    X = _rand((int((lens + 1).sum()), H), torch.float32, 71).to(DEV)
    Xd = torch.full((int(lens.sum()) + 3, H), 7.0, device=DEV)
    T = lambda a: torch.from_numpy(a).to(DEV)
    B.op_compact(X, Xd, T(start), T(dst), T(lens))
    rows = torch.from_numpy(np.concatenate([np.arange(s, s + l) for s, l in zip(start, lens)])).to(DEV)
    assert torch.equal(Xd[:-3], X[rows]) and (Xd[-3:] == 7.0).all()


def _layer_by_entry_points(m, lw, X, cu, dtype):
    """One layer on the fp32 residual X, step by step through the kernel-level entry points."""
    nq, nkv, hd, H, T = m.n_q_heads, m.n_kv_heads, m.head_dim, m.hidden, len(X)
    lens = np.diff(cu)
    pos = torch.from_numpy(np.concatenate([np.arange(l) for l in lens]).astype(np.int32)).to(DEV)
    col0, vt_col, ncol = _vt_layout(lens.tolist())
    new = lambda *shape, dt=dtype: torch.zeros(*shape, dtype=dt, device=DEV)
    w = {k: v.to(dtype).to(DEV) for k, v in lw.items()}
    Xn, QKV, QK, Vt, AO, S = (new(T, H), new(T, (nq + 2 * nkv) * hd, dt=torch.float32), new(T, (nq + nkv) * hd),
                              new(nkv, hd, ncol, dt=torch.float16), new(T, nq * hd), new(T, m.ffn))
    B.op_rmsnorm(X, w["attn_norm"], m.rms_eps, Xn)
    B.op_gemm(B.EPI_STORE_F32, Xn, torch.cat([w["wq"], w["wk"], w["wv"]]), QKV)
    B.op_qkv_finish(B._dt(QK), QKV, pos, int(lens.max()), w["q_norm"], w["k_norm"], nq, nkv, hd, m.rms_eps, m.rope_base, m.qk_norm, QK, Vt,
                    torch.from_numpy(vt_col).to(DEV), ncol)
    B.op_attention(B._dt(QK), QK, Vt, ncol, cu, col0, nq, nkv, hd, AO)
    B.op_gemm(B.EPI_RESIDUAL, AO, w["wo"], X)
    B.op_rmsnorm(X, w["ffn_norm"], m.rms_eps, Xn)
    B.op_gemm(B.EPI_SWIGLU, Xn, torch.cat([w["w_gate"], w["w_up"]]), S)
    B.op_gemm(B.EPI_RESIDUAL, S, w["w_down"], X)


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("nq,nkv,H,lens,kind", [
    (2, 1, 256, [40, 18], "kHead64"), (16, 8, 256, [33, 1, 200], "kHead64"), (1, 1, 64, [70, 5], "kHead64"),
    (32, 8, 192, [300, 70, 1], "kHead128Deep"), (3, 3, 128, [1200, 1, 781], "kHead128Deep"),
    (2, 1, 320, [40, 18], "kHead64"), (2, 1, 384, [40, 18], "kHead64"),              # every place of the rings' second turn
    (32, 8, 256, [300, 70, 1], "kHead128Deep"), (32, 8, 320, [300, 70, 1], "kHead128Deep"), (32, 8, 384, [300, 70, 1], "kHead128Deep"),
    (32, 8, 256, [700, 63], "kHead128"), (1, 1, 320, [4000, 4001, 3900, 5], "kHead128"),
    (8, 8, 1024, [1500, 1, 1024, 64, 1490], "kHead256")])
def test_projection_of_a_whole_call_has_the_bits_of_its_entry_points(dtype, nq, nkv, H, lens, kind):
    """Below 256 big tiles a call's fused q/k/v projection gives the bits of prism_op_gemm + prism_op_qkv_finish, in every tile
    and with an odd number of heads too: two layers of a whole call against the same layers through the entry points, whose
    own steps are tested above.  The second layer's scores see every q, k and v of the first."""
    q = np.arange(7, dtype=np.int32)
    m = W.ModelShape(2, H, nq, nkv, 128, 128, 64, "bf16")
    T = sum(lens) + len(lens) * len(q)
    heads = nq + 2 * nkv
    assert head_plan(T, nq, nkv, H) == [(T, kind)] and (heads % 2 or -(-T // 256) * (heads // 2) < 256)
    d = torch.Generator().manual_seed(9)
    draw = lambda *s, std=0.05: (torch.randn(*s, generator=d) * std).to(torch.bfloat16)
    layers = [{n: ((1 + draw(s[0])).to(torch.bfloat16) if len(s) == 1 else draw(*s)) for n, s in W.layer_tensor_shapes(m).items()} for _ in range(2)]
    embed, final_norm = draw(64, H, std=1.0), (1 + draw(H)).to(torch.bfloat16)
    r = np.random.RandomState(3)
    cands = [r.randint(0, 64, n).astype(np.int32) for n in lens]

    cu = np.concatenate([[0], np.cumsum([len(q) + n for n in lens])]).astype(np.int32)
    X, scores = torch.zeros(T, H, device=DEV), torch.zeros(len(lens), device=DEV)
    B.op_embed(torch.from_numpy(np.concatenate([np.concatenate([q, c]) for c in cands])).to(DEV), embed.to(DEV), X)
    for lw in layers:
        _layer_by_entry_points(m, lw, X, cu, dtype)
    B.op_score(X, torch.from_numpy(cu[1:] - 1).to(DEV), final_norm.to(DEV), embed[1].to(DEV), embed[0].to(DEV), m.rms_eps, scores)

    wt = W.Weights(embed.to(DEV), [{k: v.to(DEV) for k, v in lw.items()} for lw in layers], final_norm.to(DEV))
    for share in (False, True):
        p = B.Prism(m, wt, operand=OPERAND[dtype], share_query=share)
        _, _, rep = p.select(q, cands, len(lens))
        p.destroy()
        assert np.array_equal(rep.scores[-1], scores.cpu().numpy()), share
    if T < 300:                                              # and the whole against fp64: the oracle is slow
        ref = O.select(q, cands, len(lens), oracle_weights(W.Weights(embed, layers, final_norm)), oracle_model(m), checkpoints=[], n_clusters=3,
                       tau=0.0, mode=O.MODE_DROP_ONLY).events[-1]
        err = np.abs(rep.scores[-1][ref.live] - ref.scores).max() / np.abs(ref.scores).max()
        print(f"{dtype} {nq} {nkv} {H}: {err:.2e}")
        assert err < WHOLE_CALL_ERROR[dtype]


HEAD_RING_LAUNCHES = [(16, 8, 1024 + 64 * k, [300, 1, 60], "kHead64") for k in range(6)] + [(32, 8, 2048 + 64 * k, [300, 70, 1], "kHead128Deep") for k in range(5)]


@pytest.mark.parametrize("nq,nkv,H,lens,kind", HEAD_RING_LAUNCHES)
def test_projection_on_the_deep_rings(nq, nkv, H, lens, kind):
    """At most 256 tiles and a long K: rings of 6 and 5 slices, ended at every place (that these launches take them: test_tile_plan.py)."""
    test_projection_of_a_whole_call_has_the_bits_of_its_entry_points(torch.float16, nq, nkv, H, lens, kind)


# (epilogue, tile, rows, N, K slices, rows of the taller launch that it is compared with)
RING_LAUNCHES = [(e, *c) for e in (B.EPI_STORE, B.EPI_RESIDUAL, B.EPI_STORE_F32) for c in (
    ("kTile128x64", 391, 2552, range(32, 38), 2000), ("kTile128Deep", 777, 2552, range(32, 37), 4100))] + [
    (e, "kTile128x64", 391, 4088, range(16, 22), 1500) for e in (B.EPI_STORE, B.EPI_STORE_F32)] + [
    (B.EPI_SWIGLU, "kTile128x64", 200, 6152, range(16, 22), 1500), (B.EPI_SWIGLU, "kTile128Deep", 391, 6152, range(32, 37), 1500)]


@pytest.mark.parametrize("dtype", SIXTEEN)
@pytest.mark.parametrize("epi,kind,M,N,slices,tall", RING_LAUNCHES)
def test_gemm_16_deep_rings_give_a_row_the_same_bits(dtype, epi, kind, M, N, slices, tall):
    """Tiles of 128 rows on their ring for one tile per compute unit, a loop's end at every place of it, ragged last tiles: bit for
    bit the same rows inside a taller launch, which takes the other ring or other tiles (test_tile_plan.py asks the launcher; each of
    those is compared with fp64 above)."""
    glu = epi == B.EPI_SWIGLU
    for k in slices:
        K = 64 * k
        assert gemm_plan(M, N, K, glu) == [(M, kind)]
        A, Wt = _rand((tall, K), dtype, 75, 1.0).to(DEV), _rand((N, K), dtype, 76, 1.0 / math.sqrt(K)).to(DEV)
        X0 = _rand((tall, N), torch.float32, 77, 1.0).to(DEV)

        def run(rows):
            if epi == B.EPI_RESIDUAL:
                out = X0[:rows].clone()
            else:
                out = torch.full((rows, N // 2 if glu else N), 7.0, dtype=torch.float32 if epi == B.EPI_STORE_F32 else dtype, device=DEV)
            B.op_gemm(epi, A[:rows], Wt, out)
            return out
        assert torch.equal(run(M), run(tall)[:M]), k


@pytest.mark.parametrize("n,k", [(2, 2), (3, 8), (64, 8), (127, 4), (128, 8), (129, 8), (130, 2), (513, 5), (1000, 3), (4096, 3)])
@pytest.mark.parametrize("shape", ["normal", "duplicates", "tiny spread", "clusters"])
def test_route_around_its_workgroup_boundary(n, k, shape):
    """One workgroup up to 128 candidates, several launches beyond: the same decisions as the oracle, bit for bit, on scores
    with many ties, with a spread far below their mean (costs that differ in the last bits only) and with clear clusters;
    -0 and 0 tie."""
    r = np.random.default_rng(n * 10 + k)
    s = r.normal(size=n)
    if shape == "duplicates":
        s = np.round(s * 2) / 2 * np.where(r.random(n) < 0.5, 1.0, -1.0)          # -0.0 among them
    elif shape == "tiny spread":
        s = 1000.0 + s * 1e-3
    elif shape == "clusters":
        s = r.choice([-3.0, 0.0, 5.0, 40.0], size=n) + s * 0.01
    _route_case(s.astype(np.float32).tolist(), max(1, n // 5), k, 0.0)


@pytest.mark.parametrize("n,K", [(1, 1), (15, 15), (17, 3), (500, 20), (4096, 4096)])
def test_topk_of_any_pool(n, K):
    s = np.round(np.random.default_rng(n).normal(size=n), 1).astype(np.float32)    # many ties
    pos, sc = torch.zeros(K, dtype=torch.int32, device=DEV), torch.zeros(K, device=DEV)
    B.op_topk(torch.from_numpy(s).to(DEV), K, pos, sc)
    order = O.rank_order(s.astype(np.float64))[:K]
    assert np.array_equal(pos.cpu().numpy(), order) and np.array_equal(sc.cpu().numpy(), s[order])


@pytest.mark.parametrize("n,K", [(1, 1), (17, 17), (300, 40)])
def test_topk_ranks_nan_behind_every_number(n, K):
    """Infinities, zeros of both signs and NaN of both signs among the scores: K different positions, NaN last by position."""
    r = np.random.default_rng(n)
    s = r.choice(np.array([np.inf, -np.inf, 0.0, -0.0, 1.5, -1.5, np.nan, -np.nan, 3e38, -3e38, 1e-45], np.float32), size=n)
    pos, sc = torch.full((K,), -1, dtype=torch.int32, device=DEV), torch.zeros(K, device=DEV)
    B.op_topk(torch.from_numpy(s).to(DEV), K, pos, sc)
    order = np.array(sorted(range(n), key=lambda i: (np.isnan(s[i]), -s[i] if not np.isnan(s[i]) else 0.0, i)))[:K]
    assert np.array_equal(pos.cpu().numpy(), order)
    assert np.array_equal(sc.cpu().numpy().view(np.int32), s[order].view(np.int32))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("T,hidden", [(1, 4), (5, 252), (4095, 256), (4097, 256), (4098, 64), (7, 260)])
def test_rmsnorm_of_short_rows(T, hidden, dtype):
    """A wave per row up to 256 values, one or four rows to a workgroup; 260 values take a workgroup."""
    X, g = _rand((T, hidden), torch.float32, 7, 3.0), (1 + _rand((hidden,), torch.float32, 8, 0.1)).to(dtype)
    out = torch.zeros(T, hidden, dtype=dtype, device=DEV)
    B.op_rmsnorm(X.to(DEV), g.to(DEV), 1e-6, out)
    ref = O.rmsnorm(_f64(X), _f64(g), 1e-6)
    # fp32: sum of 256 squares, reciprocal root, two products; a 16-bit result is rounded once more
    np.testing.assert_allclose(_f64(out), ref, rtol=2e-6 if dtype == torch.float32 else EPS16[dtype] * 1.01, atol=1e-7)


@pytest.mark.parametrize("hd,nq,nkv,T", [(32, 3, 1, 5), (64, 4, 2, 354), (64, 4, 2, 12859), (128, 1, 1, 9001), (48, 2, 1, 77)])
@pytest.mark.parametrize("qk_norm", [True, False])
def test_qk_finish_fp32_head_sizes(hd, nq, nkv, T, qk_norm):
    """fp32 finishing, up to six heads of a token per lane with rotations evaluated in the kernel, other head sizes one at a time by the table:
    against fp64 at the bound of the single-kernel test; v is left as it was."""
    pos = (np.arange(T) % 517).astype(np.int32)
    QKV = _rand((T, (nq + 2 * nkv) * hd), torch.float32, T + hd, 1.5)
    gq, gk = 1 + _rand((hd,), torch.float32, 41, 0.1), 1 + _rand((hd,), torch.float32, 42, 0.1)
    x = _f64(QKV).reshape(T, nq + 2 * nkv, hd)
    q, k = x[:, :nq], x[:, nq:nq + nkv]
    if qk_norm:
        q, k = O.rmsnorm(q, _f64(gq), 1e-6), O.rmsnorm(k, _f64(gk), 1e-6)
    d = QKV.to(DEV).clone()
    B.op_qkv_finish(B.DTYPE_FP32, d, torch.from_numpy(pos).to(DEV), 517, gq.to(DEV), gk.to(DEV), nq, nkv, hd, 1e-6, 1e6, qk_norm)
    ref = np.concatenate([O.rope(q, pos, 1e6), O.rope(k, pos, 1e6), x[:, nq + nkv:]], axis=1).reshape(T, -1)
    np.testing.assert_allclose(_f64(d), ref, rtol=1e-5, atol=2e-5)
    assert torch.equal(d.cpu()[:, (nq + nkv) * hd:], QKV[:, (nq + nkv) * hd:])
