"""The block generator at odd block edges, ranks and output alignments, element by element against the CPU oracle; nothing is
written outside the block.  Tolerance as in test_gpu_parity: an R-term fp32 multiply-add chain against fp64 rounded once
(R 2^-24 of the largest partial sum), bf16 values on the other side of a rounding boundary by one unit."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import oracle
import workloads as wl
from paper_2311_13693_amd import exat

pytestmark = pytest.mark.gpu


# quads around a wave's 64, fibres around a wave's 8 and a workgroup's 32, blocks that begin and end inside a quad
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("I,J,K,dI,dJ,dK,R,off", [
    (1, 1, 1, 1, 1, 1, 1, 0), (259, 9, 3, 259, 9, 3, 5, 1), (520, 33, 2, 257, 31, 1, 16, 3), (101, 70, 5, 50, 33, 2, 3, 2), (64, 8, 4, 21, 7, 3, 256, 0),
])
def test_gen_block_odd_sizes(dtype, I, J, K, dI, dJ, dK, R, off):
    cfg = wl.small(name="genodd", index=260 + I % 30, I=I, J=J, K=K, R=R, dI=dI, dJ=dJ, dK=dK, dtype=dtype)
    print("case", dtype, I, J, K, dI, dJ, dK, R, off, flush=True)
    A, B, C = wl.cp_factors(cfg)
    desc, gen = gu.desc_of(cfg), gu.gen_of(cfg, A, B, C)
    nb = [-(-n // d) for n, d in ((I, dI), (J, dJ), (K, dK))]
    for blk in {(0, 0, 0), tuple(n - 1 for n in nb), (nb[0] // 2, nb[1] // 2, 0)}:
        lo = [b * d for b, d in zip(blk, (dI, dJ, dK))]
        hi = [min(n, l + d) for n, l, d in zip((I, J, K), lo, (dI, dJ, dK))]
        ext = [h - l for h, l in zip(hi, lo)]
        n = ext[0] * ext[1] * ext[2]
        buf = torch.full((n + 8,), 7.0, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
        exat.gen_block(desc, gen, *blk, buf[off:])
        got = buf.float().cpu().numpy()
        assert np.all(got[:off] == 7.0) and np.all(got[off + n:] == 7.0)
        got = got[off:off + n].reshape(ext, order="F").astype(np.float64)
        want = oracle.gen_box(A, B, C, cfg.seed, cfg.sigma, (lo[0], hi[0], lo[1], hi[1], lo[2], hi[2]), to_bf16=(dtype == "bf16")).astype(np.float64)
        diff = np.abs(got - want)
        if dtype == "f32":
            assert diff.max() <= max(2e-6, R * 2.0 ** -24) * (1.0 + np.abs(want).max())
        else:
            assert np.all(diff <= np.abs(want) * 2.0 ** -7 + 1e-30)


# blocks thin in i or j: quads around every power of two up to 64, fibres around a wave's share, blocks short in i and j and long in k.
# Tolerance: the fp32 chain as above; in bf16 one unit (2^-7) on top of that chain's error, which shows where a sum nearly cancels.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("I,J,K,dI,dJ,dK,R,off", [
    (1, 600, 3, 1, 600, 3, 5, 1), (9, 7, 300, 4, 3, 150, 6, 0), (11, 5, 220, 11, 5, 220, 17, 2), (30, 65, 7, 13, 65, 7, 5, 3), (33, 40, 5, 33, 33, 5, 33, 0),
    (70, 19, 9, 65, 19, 9, 4, 1), (128, 40, 4, 128, 40, 4, 256, 0), (129, 9, 4, 129, 9, 4, 3, 2), (200, 1, 130, 100, 1, 130, 2, 0), (8, 2, 5000, 8, 2, 4097, 1, 0),
    (64, 32, 40, 64, 32, 40, 5, 0), (64, 33, 40, 64, 33, 40, 5, 1), (1030, 3, 21, 517, 3, 21, 7, 3), (256, 8, 9, 256, 8, 9, 2, 0),   # a quarter of the lanes, and longer fibres
])
def test_gen_block_short_fibres(dtype, I, J, K, dI, dJ, dK, R, off):
    cfg = wl.small(name="genthin", index=290 + I % 30, I=I, J=J, K=K, R=R, dI=dI, dJ=dJ, dK=dK, dtype=dtype)
    print("case", dtype, I, J, K, dI, dJ, dK, R, off, flush=True)
    A, B, C = wl.cp_factors(cfg)
    desc, gen = gu.desc_of(cfg), gu.gen_of(cfg, A, B, C)
    for blk in {(0, 0, 0), tuple(-(-n // d) - 1 for n, d in ((I, dI), (J, dJ), (K, dK)))}:
        lo = [b * d for b, d in zip(blk, (dI, dJ, dK))]
        hi = [min(n, l + d) for n, l, d in zip((I, J, K), lo, (dI, dJ, dK))]
        ext = [h - l for h, l in zip(hi, lo)]
        n = ext[0] * ext[1] * ext[2]
        buf = torch.full((n + 8,), 7.0, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
        exat.gen_block(desc, gen, *blk, buf[off:])
        got = buf.float().cpu().numpy()
        assert np.all(got[:off] == 7.0) and np.all(got[off + n:] == 7.0)
        got = got[off:off + n].reshape(ext, order="F").astype(np.float64)
        want = oracle.gen_box(A, B, C, cfg.seed, cfg.sigma, (lo[0], hi[0], lo[1], hi[1], lo[2], hi[2]), to_bf16=(dtype == "bf16")).astype(np.float64)
        chain = max(2e-6, R * 2.0 ** -24) * (1.0 + np.abs(want).max())
        assert np.all(np.abs(got - want) <= chain + (np.abs(want) * 2.0 ** -7 if dtype == "bf16" else 0.0))
