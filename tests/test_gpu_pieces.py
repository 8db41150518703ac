"""The piece-sum kernel of modes 1 and 2 (materialised X, any size and alignment) against plain fp64 torch at the sizes where
it can go wrong, and against the generic fp32 kernel (EXAT_PIPELINED=0) on values outside the range of the piece sums, which
the library hands to that kernel.

Tolerance: three bf16 pieces hold an fp32 value exactly and the products left out are 2^-26, so what remains is the rounding
of the fp32 running sums, as in the fp32 kernels: relative rms error about 2^-24 sqrt(n) / 2.4 per mode, below 1e-6 for the
extents here; two fp16 pieces carry 21 bits (2^-22 per operand and mode).  2e-6 covers both."""
import os

import pytest
import torch

from paper_2311_13693_amd import exat

pytestmark = pytest.mark.gpu
TOL = 2e-6
DT = {"f32": exat.EXAT_F32, "bf16": exat.EXAT_BF16, "f32s": exat.EXAT_F32_SPLIT}


def _problem(I, J, K, L, M, N, P, dtype, seed=5):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    X = rn(K, J, I)
    return (X.to(torch.bfloat16) if dtype == "bf16" else X), rn(P * L, I) * L ** -0.5, rn(P * M, J) * M ** -0.5, rn(P * N, K) * N ** -0.5


def _plan(I, J, K, L, M, N, P, dtype, U, V, W, d=None):
    d = d or (I, J, K)
    plan = exat.Plan(exat.make_desc(I, J, K, L, M, N, P, *d, DT[dtype]))
    plan.set_factors(U, V, W)
    return plan


def _ref(X, U, V, W, L, M, N, P, dtype):
    r = (lambda t: t.to(torch.bfloat16).double()) if dtype == "bf16" else (lambda t: t.double())
    X, U, V, W = X.double(), r(U), r(V), r(W)
    K, J, I = X.shape
    Z = (X.reshape(-1, I) @ U.T).view(K, J, P * L)
    Y = [W[p * N:(p + 1) * N] @ torch.matmul(V[p * M:(p + 1) * M], Z[:, :, p * L:(p + 1) * L].contiguous()).view(K, M * L) for p in range(P)]
    return torch.stack(Y).view(-1)


def _err(Y, R):
    return float((Y.double() - R).norm() / R.norm())


# stacked rows around the tile, quad, wave-column and group boundaries; replicas inside a tile, straddling tiles, whole tiles
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f32s"])
@pytest.mark.parametrize("P,L", [(1, 1), (2, 16), (3, 33), (8, 16), (9, 16), (5, 50), (16, 16), (17, 16), (11, 50), (16, 32), (33, 16), (21, 50), (20, 64)])
def test_row_groups(dtype, P, L):
    I, J, K, M, N = 96, 130, 9, 7, 5
    print("case", dtype, P, L, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    assert _err(plan.compress(X), _ref(X, U, V, W, L, M, N, P, dtype)) <= TOL


# stages, ring slots and chunks: one stage and less, the ring length and around it, fibres around a chunk
@pytest.mark.parametrize("dtype", ["f32", "bf16", "f32s"])
@pytest.mark.parametrize("I,J,M", [(1, 1, 1), (8, 127, 32), (31, 128, 33), (32, 129, 64), (33, 40, 50), (64, 257, 20), (127, 16, 64), (128, 15, 32),
                                   (129, 300, 50), (250, 250, 50), (244, 60, 20), (257, 33, 64), (511, 130, 17)])
@pytest.mark.parametrize("P", [2, 7, 13])   # 4, 2 and 1 wave columns
def test_extents(dtype, I, J, M, P):
    K, L, N = 6, 40, 9
    print("case", dtype, I, J, M, P, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    assert _err(plan.compress(X), _ref(X, U, V, W, L, M, N, P, dtype)) <= TOL


# blocks whose edges are multiples of nothing, one by one; a slab of blocks of half stages in one launch; X not 16-byte aligned
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [(50, 45, 7), (37, 128, 4), (100, 33, 13), (52, 60, 5)])
def test_odd_blocks(dtype, d):
    I, J, K, L, M, N, P = 115, 140, 13, 50, 50, 20, 13
    print("case", dtype, d, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W, d)
    for k in range(0, K, d[2]):
        for j in range(0, J, d[1]):
            for i in range(0, I, d[0]):
                plan.compress_block(X[k:k + d[2], j:j + d[1], i:i + d[0]].contiguous(), i // d[0], j // d[1], k // d[2])
    assert _err(plan.finalize(), _ref(X, U, V, W, L, M, N, P, dtype)) <= TOL


@pytest.mark.parametrize("dtype,dI", [("f32", 16), ("f32", 48), ("bf16", 32), ("f32s", 32)])
@pytest.mark.parametrize("P", [2, 6, 13])
def test_slab_blocks(dtype, dI, P):
    I, J, K, L, M, N = 144 if dI != 32 else 160, 300, 10, 40, 50, 20
    d = (dI, 128, 4)
    print("case", dtype, dI, P, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W, d)
    blocks = [X[k:k + 4, j:j + 128, i:i + dI].contiguous() for k in range(0, K, 4) for j in range(0, J, 128) for i in range(0, I, dI)]
    plan.compress_blocks(blocks, 0, 3, 0, 3)
    assert _err(plan.finalize(), _ref(X, U, V, W, L, M, N, P, dtype)) <= TOL


@pytest.mark.parametrize("dtype,off", [("f32", 1), ("f32", 3), ("bf16", 1), ("bf16", 4), ("f32s", 2)])
def test_unaligned_tensor(dtype, off):
    I, J, K, L, M, N, P = 96, 130, 5, 50, 33, 20, 12
    print("case", dtype, off, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    buf = torch.full((X.numel() + 8,), float("nan"), dtype=X.dtype, device="cuda")
    buf[off:off + X.numel()] = X.view(-1)
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    assert _err(plan.compress(buf[off:]), _ref(X, U, V, W, L, M, N, P, dtype)) <= TOL


# values outside the range of the piece sums: the call is computed with fp32 products, as the generic kernel does
RANGES = {
    "x_tiny": (1e-36, 1.0, 1.0), "x_huge": (1e30, 1.0, 1.0), "u_tiny": (1.0, 1e-30, 1.0), "u_huge": (1.0, 1e15, 1.0), "v_tiny": (1.0, 1.0, 1e-25),
    "v_huge": (1.0, 1.0, 1e10), "z_tiny": (1e-11, 1e-5, 1.0),
}


@pytest.mark.parametrize("P", [2, 7, 13])
@pytest.mark.parametrize("case", list(RANGES) + ["x_inf", "x_max", "x_zero", "one_huge", "bf16_inf"])
def test_value_ranges(case, P):
    I, J, K, L, M, N = 70, 140, 6, 40, 50, 20
    dtype = "bf16" if case.startswith("bf16") else "f32"
    print("case", case, P, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    sx, su, sv = RANGES.get(case, (1.0, 1.0, 1.0))
    X, U, V = X * sx, U * su, V * sv
    if case in ("x_inf", "bf16_inf"):
        X[3, 100, 17] = float("inf")
    elif case == "x_max":
        X[3, 100, 17] = torch.finfo(torch.float32).max / 64
        V.clamp_(-0.5, 0.5)
    elif case == "x_zero":
        X.zero_()
    elif case == "one_huge":
        X[0, 0, 0] = 1e25
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    Y = plan.compress(X)
    os.environ["EXAT_PIPELINED"] = "0"
    try:
        G = plan.compress(X)
    finally:
        os.environ.pop("EXAT_PIPELINED")
    if case == "z_tiny":   # inside the ranges of X and U, and Z as small as they make it: either route
        assert _err(Y, G.double()) <= 2 * TOL
    else:
        assert torch.equal(torch.isnan(Y), torch.isnan(G)) and torch.equal(torch.isinf(Y), torch.isinf(G))
        fin = torch.isfinite(G)
        assert torch.equal(Y[~fin].nan_to_num(0), G[~fin].nan_to_num(0))
        if P == 13:
            assert torch.equal(Y[fin], G[fin])
        else:   # several wave columns: mode 3 adds the same partial results (and zeros) in another order
            assert float((Y[fin].double() - G[fin].double()).norm()) <= TOL * float(G[fin].double().norm())
    # the next call starts with a clean record
    X2, _, _, _ = _problem(I, J, K, L, M, N, P, dtype, seed=6)
    if case in ("x_tiny", "x_huge", "x_inf", "x_max", "x_zero", "one_huge", "bf16_inf"):
        assert _err(plan.compress(X2), _ref(X2, U, V, W, L, M, N, P, dtype)) <= TOL


# mode 3: slabs of k per wave (4 or 16 waves), their remainders, the flush of long slabs into fp64 sums; one and two tiles of m, n
@pytest.mark.parametrize("K", [1, 15, 63, 64, 65, 129, 513, 2041, 2060, 8001])
@pytest.mark.parametrize("P,L,M,N", [(2, 3, 20, 33), (2, 9, 50, 20), (40, 16, 33, 64), (2, 300, 33, 40)])
def test_mode3_slabs(K, P, L, M, N):
    I, J = 8, 9
    print("case", K, P, L, M, N, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, "f32")
    plan = _plan(I, J, K, L, M, N, P, "f32", U, V, W)
    assert _err(plan.compress(X), _ref(X, U, V, W, L, M, N, P, "f32")) <= TOL


# uneven row groups (13, 18 and 19 quads of row tiles): slices dealt in runs to the compute dies, with runs that are empty, short and whole
@pytest.mark.parametrize("K", [1, 9, 70, 257])
@pytest.mark.parametrize("P,L,dtype", [(31, 50, "f32"), (31, 50, "f32s"), (48, 50, "bf16"), (45, 50, "f32")])
def test_slice_runs(P, L, dtype, K):
    I, J, M, N = 288, 130, 9, 7
    print("case", P, L, dtype, K, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    assert _err(plan.compress(X), _ref(X, U, V, W, L, M, N, P, dtype)) <= TOL


# a slab of blocks with values outside the range of the piece sums: the generic kernel behind reads X through the block table too.
# dI of whole and of half stages, a ragged last block along j and k; the same blocks one by one give the expectation (and the next slab
# starts with a clean record).  EXAT_PIPELINED=0 takes every slab apart, that of a split plan as well.
@pytest.mark.parametrize("dtype,dI", [("f32", 32), ("f32", 48), ("bf16", 32), ("f32s", 32)])
@pytest.mark.parametrize("case", ["x_inf", "one_huge", "x_huge", "x_tiny", "u_huge", "v_tiny"])
@pytest.mark.parametrize("P", [2, 13])
def test_slab_value_ranges(dtype, dI, case, P):
    I, J, K, L, M, N = 96, 300, 6, 40, 50, 20
    d = (dI, 128, 4)
    print("case", dtype, dI, case, P, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    sx, su, sv = RANGES.get(case, (1.0, 1.0, 1.0))
    X, U, V = X * sx, U * su, V * sv
    if case == "x_inf":
        X[3, 200, 17] = float("inf")
    elif case == "one_huge":
        X[0, 0, 0] = 1e25
    cut = lambda X: [X[k:k + 4, j:j + 128, i:i + dI].contiguous() for k in range(0, K, 4) for j in range(0, J, 128) for i in range(0, I, dI)]
    nb = (I // dI, 3, 2)

    def one_by_one(X):
        for n, b in enumerate(cut(X)):
            plan.compress_block(b, n % nb[0], n // nb[0] % nb[1], n // (nb[0] * nb[1]))
        return plan.finalize()

    def slab(X):
        plan.compress_blocks(cut(X), 0, nb[1], 0, nb[2])
        return plan.finalize()

    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W, d)
    if dtype == "f32s":   # two fp16 pieces have fp16 range; fp32 products are what the switch asks for
        os.environ["EXAT_PIPELINED"] = "0"
    try:
        G, Y = one_by_one(X), slab(X)
        assert torch.equal(torch.isnan(Y), torch.isnan(G)) and torch.equal(torch.isinf(Y), torch.isinf(G))
        fin = torch.isfinite(G)
        assert torch.equal(Y[~fin].nan_to_num(0), G[~fin].nan_to_num(0))
        assert float((Y[fin].double() - G[fin].double()).norm()) <= 2 * TOL * float(G[fin].double().norm())
        X2 = _problem(I, J, K, L, M, N, P, dtype, seed=6)[0]
        if case[0] == "x" or case == "one_huge":
            assert _err(slab(X2), _ref(X2, U, V, W, L, M, N, P, dtype)) <= TOL
    finally:
        os.environ.pop("EXAT_PIPELINED", None)


# a bf16 chunk is filled up to a multiple of four stages: the stages past the tensor's last one must not bring in what lies behind a row
# tile's U -- other rows (a NaN there belongs to its own replica only), or, in a plan whose last tile is in use (7680 rows), other memory
@pytest.mark.parametrize("P,L", [(3, 32), (7, 40), (120, 64)])
@pytest.mark.parametrize("I", [32, 70, 96, 129])
def test_bf16_stages_past_the_end(P, L, I):
    J, K, M, N, dtype = 40, 3, 7, 5, "bf16"
    print("case", P, L, I, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    bad = torch.full((1 << 20,), float("nan"), device="cuda")   # what the plan's memory may have held before
    torch.cuda.synchronize()
    del bad
    torch.cuda.empty_cache()
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    R = _ref(X, U, V, W, L, M, N, P, dtype)
    assert _err(plan.compress(X), R) <= TOL
    U[P // 2 * L + 5, :] = float("nan")   # one row of the middle replica
    plan.set_factors(U, V, W)
    Y, R = plan.compress(X).view(P, N, M, L), R.view(P, N, M, L)
    ok = torch.ones(P, L, dtype=torch.bool, device="cuda")
    ok[P // 2, 5] = False
    ok = ok[:, None, None, :].expand_as(Y)
    assert torch.isnan(Y[~ok]).all() and _err(Y[ok], R[ok]) <= TOL


def _same_as_generic(call, P):
    """call() on the route the library takes and with fp32 products throughout: the same infinities and NaN, the same values elsewhere"""
    Y = call()
    os.environ["EXAT_PIPELINED"] = "0"
    try:
        G = call()
    finally:
        os.environ.pop("EXAT_PIPELINED")
    assert torch.equal(torch.isnan(Y), torch.isnan(G)) and torch.equal(torch.isinf(Y), torch.isinf(G))
    fin = torch.isfinite(G)
    assert torch.equal(Y[~fin].nan_to_num(0), G[~fin].nan_to_num(0))
    if P == 13:
        assert torch.equal(Y[fin], G[fin])
    else:   # several wave columns: see test_value_ranges
        assert float((Y[fin].double() - G[fin].double()).norm()) <= TOL * float(G[fin].double().norm())
    return G


# NaN and infinities in each operand are noted like any value outside the range
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("P", [2, 7, 13])
@pytest.mark.parametrize("case", ["x_nan", "u_nan", "v_nan", "u_inf", "v_inf"])
def test_non_finite_operands(dtype, case, P):
    I, J, K, L, M, N = 70, 140, 6, 40, 50, 20
    print("case", dtype, case, P, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    bad = float(case[2:])
    if case[0] == "x":
        X[3, 100, 17] = bad
    elif case[0] == "u":
        U[L + 3, 44] = bad
    else:
        V[M + 7, 111] = bad
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    G = _same_as_generic(lambda: plan.compress(X), P)
    if case != "x_nan":   # one row of U or V: the other replicas are what they are without it
        G = G.view(P, N, M, L)
        bad_p = (~torch.isfinite(G)).flatten(1).any(1)
        assert bad_p.tolist() == [p == 1 for p in range(P)]


# generated in fp32: the factors are taken as fp16 pieces, and what lies beyond fp16 becomes an infinity or a NaN of the tile
@pytest.mark.parametrize("R", [5, 40])
@pytest.mark.parametrize("P", [2, 7, 13])
@pytest.mark.parametrize("scale", [(1e5, 1.0, 1.0), (1.0, 1e4, 30.0), (1e30, 1e-20, 1.0)])
def test_generated_factor_range(P, R, scale):
    I, J, K, L, M, N = 70, 140, 6, 40, 50, 20
    print("case", P, R, scale, flush=True)
    _, U, V, W = _problem(I, J, K, L, M, N, P, "f32")
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    A, B, C = [s * torch.randn(R, n, generator=g, device="cuda") for s, n in zip(scale, (I, J, K))]
    gen = exat.make_gen(A, B, C, 77, 0.01)
    plan = _plan(I, J, K, L, M, N, P, "f32", U, V, W)
    G = _same_as_generic(lambda: plan.compress_gen(gen), P)
    X = torch.matmul((C.double()[:, :, None] * B.double()[:, None, :]).reshape(R, -1).T.contiguous(), A.double()).view(K, J, I)
    assert _err(G, _ref(X, U, V, W, L, M, N, P, "f32")) <= TOL   # the noise is below rounding here


# a small part of an operand beside ordinary values, and an output made of that part alone: one replica's U or V, a slice of X that one row of
# W picks.  Small enough that pieces would lose bits (1e-36: error 1e-4 and more), or not (1e-15).
@pytest.mark.parametrize("P", [2, 7, 13])
@pytest.mark.parametrize("scale", [1e-36, 1e-15])
@pytest.mark.parametrize("part", ["u", "v", "x"])
def test_small_part_beside_ordinary(part, scale, P):
    I, J, K, L, M, N = 70, 140, 6, 40, 50, 20
    print("case", part, scale, P, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, "f32")
    if part == "u":
        U[L:2 * L] *= scale
    elif part == "v":
        V[M:2 * M] *= scale
    else:
        X[3] *= scale
        W[N + 4] = 0
        W[N + 4, 3] = 1
    plan = _plan(I, J, K, L, M, N, P, "f32", U, V, W)
    Y, R = plan.compress(X).view(P, N, -1), _ref(X, U, V, W, L, M, N, P, "f32").view(P, N, -1)
    sel = (1, 4) if part == "x" else (1,)
    assert _err(Y[sel], R[sel]) <= TOL and _err(Y, R) <= TOL


# scales that the pieces hold: the call is not computed a second time (the generic kernel adds up in another order)
@pytest.mark.parametrize("sx,su", [(1e-24, 1.0), (1e-15, 1.0), (1e20, 1.0), (1.0, 1e-20), (1.0, 1e10), (1e-12, 1e-7)])
def test_scales_inside_the_range(sx, su):
    I, J, K, L, M, N, P = 70, 140, 6, 40, 50, 20, 13
    print("case", sx, su, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, "f32")
    X, U = X * sx, U * su
    plan = _plan(I, J, K, L, M, N, P, "f32", U, V, W)
    Y = plan.compress(X)
    os.environ["EXAT_PIPELINED"] = "0"
    try:
        G = plan.compress(X)
    finally:
        os.environ.pop("EXAT_PIPELINED")
    assert _err(Y, _ref(X, U, V, W, L, M, N, P, "f32")) <= TOL and not torch.equal(Y, G)


# Rows of Q that stay in LDS over the chunks: row lengths that are odd multiples of 4, that are not (46 to 50 columns for fp32), the longest
# ones and the first ones without room; two chunks and more, a last chunk of one fibre; rows that fill the last group, or not; odd ends in i.
# Up to 128 rows the wave columns' partial rows are added there (up to 20 columns for fp32, 40 for bf16), also of a single chunk.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M", [1, 4, 5, 19, 20, 21, 32, 33, 37, 40, 41, 44, 45, 47, 48, 49, 50, 51, 52, 53, 60, 61])
@pytest.mark.parametrize("I,J,P,L", [(33, 257, 11, 47), (64, 129, 16, 32), (64, 129, 4, 31), (33, 257, 3, 11), (128, 100, 8, 16), (40, 1, 1, 1)])
def test_rows_in_lds(dtype, M, I, J, P, L):
    K, N = 9, 3
    print("case", dtype, M, I, J, P, L, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    R = _ref(X, U, V, W, L, M, N, P, dtype)
    Y = plan.new_y()
    for _ in range(2):   # and again over what the first call left
        Y.fill_(float("nan"))
        assert _err(plan.compress(X, Y), R) <= TOL


# Around the rule for keeping rows of Q in LDS (bf16: three stages, 57000 or 120000 values a slice, the third of four stages cut inside a piece of four;
# fp32: 16000 values a slice): two and three chunks, the last of which writes the sums.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M", [32, 50])
@pytest.mark.parametrize("I,J,K,P,L", [(64, 256, 5, 12, 32), (96, 129, 5, 12, 32), (92, 300, 5, 12, 32), (90, 300, 5, 12, 32), (101, 200, 5, 13, 31),
                                       (152, 384, 130, 12, 32), (148, 384, 130, 12, 32), (64, 250, 130, 12, 32), (62, 250, 130, 12, 32), (400, 304, 5, 25, 20), (392, 300, 5, 25, 20)])
def test_rows_in_lds_rule(dtype, M, I, J, K, P, L):
    N = 3
    print("case", dtype, M, I, J, K, P, L, flush=True)
    X, U, V, W = _problem(I, J, K, L, M, N, P, dtype)
    plan = _plan(I, J, K, L, M, N, P, dtype, U, V, W)
    Y = plan.new_y()
    Y.fill_(float("nan"))
    assert _err(plan.compress(X, Y), _ref(X, U, V, W, L, M, N, P, dtype)) <= TOL
