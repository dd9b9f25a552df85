"""Block-sparse x block-sparse product: host segment pointers (CPU) and the HIP kernel against
the oracle (GPU)."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_2407_09453_amd as bsp

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _draw(Ra, Rb, N, seed, da=0.5, db=0.5):
    rng = np.random.default_rng(seed)
    A = oracle.round_to_storage(rng.standard_normal((Ra * 8, N * 8)), "bf16").astype(np.float32)
    B = oracle.round_to_storage(rng.standard_normal((Rb * 8, N * 8)), "bf16").astype(np.float32)
    gamma = (rng.random((Ra, N)) < da).astype(np.uint8)
    omega = (rng.random((Rb, N)) < db).astype(np.uint8)
    return A, gamma, B, omega


def test_segment_pointers_host():
    """seg_ptr[r][s] is where row r's kept blocks with column >= 16 s start: checked against a
    search of the mask itself, on a shape with a ragged last sixteen."""
    A, gamma, _, _ = _draw(5, 3, 37, 1)
    rp, ci, pl = bsp.bsp_pack(A.reshape(40, 1, 1, 37 * 8), gamma, 8, 8, bsp.BSP_BF16)
    seg = bsp.bsp_bcsr_segments(rp, ci, 5, 37)
    assert seg.shape == (5, 4)
    for r in range(5):
        for s in range(4):
            assert seg[r, s] == rp[r] + int(gamma[r, :16 * s].sum())
        assert seg[r, 0] == rp[r] and seg[r, 3] == rp[r + 1]
        for s in range(3):
            cols = ci[seg[r, s]:seg[r, s + 1]]
            assert ((cols >= 16 * s) & (cols < 16 * s + 16)).all()
            assert cols.tolist() == [c for c in range(16 * s, min(16 * s + 16, 37)) if gamma[r, c]]
            for n, c in zip(range(seg[r, s], seg[r, s + 1]), cols):
                blk = oracle.bf16_bits_to_f32(pl[n].reshape(8, 8))
                assert (blk == A[r * 8:(r + 1) * 8, c * 8:(c + 1) * 8]).all()
    with pytest.raises(bsp.BspError) as e:
        bsp.bsp_bcsr_segments(np.array([0, 2, 1], np.int32), ci, 2, 37)
    assert e.value.code == -4


@pytest.mark.gpu
@pytest.mark.parametrize("Ra,Rb,N", [(2, 2, 4), (5, 3, 7), (16, 16, 16), (33, 17, 21), (64, 64, 128), (40, 150, 200)])
def test_spgemm_vs_oracle(Ra, Rb, N):
    import torch
    for da, db in ((0.5, 0.5), (0.1, 0.9), (1.0, 1.0), (0.0, 0.5)):
        A, gamma, B, omega = _draw(Ra, Rb, N, Ra * 100 + N, da, db)
        Am, Bm = bsp.BspMatrix(A, gamma), bsp.BspMatrix(B, omega)
        C = Am.matmul_nt(Bm)
        torch.cuda.synchronize()
        want = oracle.spgemm_nt(A, gamma, B, omega, 8)
        got = C.cpu().numpy().astype(np.float64)
        assert got.shape == want.shape
        scale = np.maximum(np.abs(want), np.sqrt(np.mean(want * want)) + 1e-30)
        # exact bf16 products, fp32 accumulation of at most 8 N terms
        assert (np.abs(got - want) <= 1e-5 * scale + 1e-30).all(), (da, db)
        if da == 0.0:
            assert not got.any()


@pytest.mark.gpu
def test_spgemm_ignores_masked_contents_and_writes_every_element():
    import torch
    A, gamma, B, omega = _draw(9, 7, 11, 5)
    C0 = bsp.BspMatrix(A, gamma).matmul_nt(bsp.BspMatrix(B, omega))
    A2 = np.where(np.kron(gamma, np.ones((8, 8))) > 0, A, np.float32(3e38))
    out = torch.full((72, 56), float("nan"), device="cuda")
    C1 = bsp.BspMatrix(A2, gamma).matmul_nt(bsp.BspMatrix(B, omega), out=out)
    torch.cuda.synchronize()
    assert torch.equal(C0, C1) and not torch.isnan(C1).any()


def _pair_union_product(A, gamma, B, omega):
    """C where a 16 x 16 tile multiplies the block columns that one of its two rows of A and one of
    its two rows of B keep: absent blocks are zeros there, other columns take no part."""
    Ra, N = gamma.shape
    Rb = omega.shape[0]
    Am = np.where(np.kron(gamma, np.ones((8, 8))) > 0, A, 0.0).astype(np.float64)
    Bm = np.where(np.kron(omega, np.ones((8, 8))) > 0, B, 0.0).astype(np.float64)
    C = np.zeros((Ra * 8, Rb * 8))
    with np.errstate(invalid="ignore"):
        for i in range(0, Ra, 2):
            for j in range(0, Rb, 2):
                cols = np.flatnonzero(gamma[i:i + 2].any(0) & omega[j:j + 2].any(0))
                k = (cols[:, None] * 8 + np.arange(8)).ravel()
                C[i * 8:i * 8 + 16, j * 8:j * 8 + 16] = Am[i * 8:i * 8 + 16][:, k] @ Bm[j * 8:j * 8 + 16][:, k].T
    return C


@pytest.mark.gpu
@pytest.mark.parametrize("Ra,Rb,N", [(1, 1, 1), (9, 8, 9), (64, 65, 20), (130, 150, 33), (300, 300, 17), (512, 520, 24)])
def test_spgemm_tiles_and_infinities(Ra, Rb, N):
    """The sizes at which the tiles of the staged product change and end; infinities and NaNs reach
    the elements they are multiplied for and no others."""
    import torch
    A, gamma, B, omega = _draw(Ra, Rb, N, Ra + N, 0.5, 0.5)
    for bad in (False, True):
        if bad:
            rng = np.random.default_rng(N)
            for M, v in ((A, np.inf), (B, -np.inf), (A, np.nan)):
                M[rng.integers(M.shape[0]), rng.integers(M.shape[1])] = v
        out = torch.full((Ra * 8, Rb * 8), float("nan"), device="cuda")
        got = bsp.BspMatrix(A, gamma).matmul_nt(bsp.BspMatrix(B, omega), out=out).cpu().numpy().astype(np.float64)
        want = _pair_union_product(A, gamma, B, omega)
        ok = np.isfinite(want)
        assert (np.isnan(got) == np.isnan(want)).all() and (got[~ok & ~np.isnan(want)] == want[~ok & ~np.isnan(want)]).all()
        scale = np.maximum(np.abs(want[ok]), np.sqrt(np.mean(want[ok] ** 2)) + 1e-30)
        assert (np.abs(got[ok] - want[ok]) <= 1e-5 * scale + 1e-30).all()


PICK = r"""
#include <cstdio>
#include "bsp_spgemm_pick.h"
int main() {
  long checked = 0, wrong = 0, chosen[SP_TILES + 1] = {};
  const double shares[] = {0.02, 0.05, 0.1, 0.2, 0.25, 0.5, 1.0};
  for (long r = 1; r <= 1024; r += r / 3 + 1)
    for (long c = 1; c <= 1024; c += c / 3 + 1)
      for (long n = 1; n <= 4096; n += n / 7 + 1)
        for (double da : shares)
          for (double db : shares) {
            const int t = sp_pick(r, c, n, da, db);
            const double time = sp_time(t, r, c, n, da, db);
            ++checked;
            ++chosen[t];
            // fits, is no slower than the kernel that needs no table, nor than any other tile that fits
            if (t < SP_TILES && (kSpTile[t].ra + kSpTile[t].rb) * (kSpTile[t].nbuf * 1024 + n * 4) > 160 * 1024) ++wrong;
            if (time > sp_time(SP_SELECT, r, c, n, da, db)) ++wrong;
            for (int o = 0; o < SP_TILES; ++o)
              if ((kSpTile[o].ra + kSpTile[o].rb) * (kSpTile[o].nbuf * 1024 + n * 4) <= 160 * 1024 && time > sp_time(o, r, c, n, da, db)) ++wrong;
          }
  for (long n : chosen)
    if (!n) ++wrong;
  // 4096 x 4096 with an inner dimension past the large tiles' tables
  if (sp_pick(512, 512, 1024 / 8 + 2, 0.2, 0.2) != SP_SELECT || sp_pick(512, 512, 2048 / 8, 0.5, 0.5) != SP_TILE_128) ++wrong;
  std::printf("%ld %ld\n", checked, wrong);
}
"""


def test_chosen_tile_fits_and_is_the_fastest_that_does(tmp_path):
    src = tmp_path / "pick.cpp"
    src.write_text(PICK)
    exe = str(tmp_path / "pick")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2407_09453_amd", "csrc"), str(src), "-o", exe], check=True)
    checked, wrong = map(int, subprocess.run([exe], capture_output=True, text=True, check=True).stdout.split())
    assert checked > 10 ** 5 and wrong == 0


@pytest.mark.gpu
@pytest.mark.parametrize("Ra,Rb,N,d,kernel", [
    (250, 250, 40, 0.5, "dense_bf16<2, 4, 4, 2, 8, 3>"), (200, 260, 130, 0.5, "dense_bf16<2, 4, 4, 2, 8, 3>"),
    (300, 260, 81, 1.0, "dense_bf16<4, 4, 2, 4, 6, 3>"), (512, 505, 70, 0.5, "dense_bf16<8, 4, 2, 4, 4, 2>"),
    (40, 150, 200, 0.5, "dense_bf16<2, 2, 2, 2, 4, 4>"), (300, 300, 60, 0.1, "nt_bf16"), (199, 261, 130, 0.1, "nt_bf16"),
    (512, 512, 1040, 0.2, "nt_bf16"), (512, 512, 1040, 0.5, "dense_bf16<2, 4, 4, 2, 8, 3>")])
def test_every_kernel_of_the_product(Ra, Rb, N, d, kernel):
    """Each tile of the staged product and the column-selecting kernel over several of its segments,
    also where the table of the tile that the model likes best does not fit; against fp64."""
    import torch
    from gpu_util import kernels_of
    A, gamma, B, omega = _draw(Ra, Rb, N, Ra + N, d, d)
    gamma[1], omega[2] = 0, 1                      # an empty block row and a full one
    Am, Bm = bsp.BspMatrix(A, gamma), bsp.BspMatrix(B, omega)
    out = torch.full((Ra * 8, Rb * 8), float("nan"), device="cuda")
    ran = kernels_of(lambda: Am.matmul_nt(Bm, out=out))
    assert any(kernel in k for k in ran), ran
    mask = lambda M, g: torch.from_numpy(M).cuda().double() * torch.from_numpy(np.kron(g, np.ones((8, 8), np.uint8))).cuda()
    want = mask(A, gamma) @ mask(B, omega).t().contiguous()
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    assert bool(((out.double() - want).abs() <= 1e-5 * scale).all())


@pytest.mark.gpu
def test_one_nan_costs_little_and_leaves_the_other_rows_alone():
    """What is not finite is computed once more, from a table that is in LDS anyway: the rows without
    it keep their bits, and the product stays within a few times its own time (about 1.5)."""
    import torch
    A, gamma, B, omega = _draw(256, 256, 256, 77)
    gamma[3, 5] = 1
    def product(A):
        Am, Bm = bsp.BspMatrix(A, gamma), bsp.BspMatrix(B, omega)
        C = Am.matmul_nt(Bm)
        best = float("inf")
        for _ in range(5):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(10):
                Am.matmul_nt(Bm, out=C)
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1))
        return C, best
    clean, t_clean = product(A)
    A[3 * 8 + 2, 5 * 8 + 1] = np.nan
    got, t_nan = product(A)
    others = torch.arange(2048, device="cuda") != 26
    assert torch.equal(got[others], clean[others]) and bool(got[26].isnan().any())
    assert t_nan < 4 * t_clean, (t_nan, t_clean)
