"""The three-part section of an fp32 layer's plan (layout: csrc/bsp_plan.h) against the weights that it stands for."""
import numpy as np
import pytest

import paper_2407_09453_amd as bsp
from paper_2407_09453_amd.binding import BSP_F32, bsp_plan_build

# header words of the plan and of the section
TOTAL, NSTRIPS, OFF_X3 = 13, 8, 26
NSTEPS, NSLABS, SLAB, OFF_SLAB, OFF_DESC, OFF_FRAG, USABLE, OFF_SRC = range(8)


def _layer(O, H, K, I, bo, bi, density, seed=0):
    rng = np.random.default_rng(seed)
    W = rng.standard_normal((O, H, K, I)).astype(np.float32)
    gamma = (rng.random((-(-O // bo), -(-I // bi))) < density).astype(np.uint8)
    row_ptr, col_idx, payload = bsp.bsp_pack(W, gamma, bo, bi, BSP_F32)
    keep = np.kron(gamma, np.ones((bo, bi), np.uint8))[:O, :I]
    return W * keep[:, None, None, :], payload, bsp_plan_build(row_ptr, col_idx, payload, O, H, K, I, bo, bi)


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
@pytest.mark.parametrize("O,H,K,I", [(40, 3, 3, 136), (72, 1, 5, 48), (90, 1, 1, 264), (1040, 1, 1, 1032), (522, 1, 1, 2048)])
def test_every_kept_weight_once(O, H, K, I, bo, bi):
    W, payload, plan = _layer(O, H, K, I, bo, bi, 0.4)
    assert plan[OFF_X3] and plan[TOTAL] == plan.size
    sec = plan[plan[OFF_X3]:]
    nsteps, nslabs, slab, nstrips = sec[NSTEPS], sec[NSLABS], sec[SLAB], plan[NSTRIPS]
    assert sec[USABLE] == 1
    first = sec[sec[OFF_SLAB]:][:nstrips * (nslabs + 1)].reshape(nstrips, nslabs + 1)
    desc = sec[sec[OFF_DESC]:][:nsteps * 4].reshape(nsteps, 4)
    direct = sec[OFF_SRC] != 0
    assert direct == (H * K == 1 and O * I > 1 << 20) and direct == (sec[OFF_FRAG] == 0)
    if direct:
        src = sec[sec[OFF_SRC]:].reshape(nsteps, 4, 4, 2)
        flat = payload.reshape(-1)
        frag = np.zeros((nsteps, 4, 16, 8))
        for j in range(16):
            at = src[:, :, j // bo, :]
            for h in range(2):
                for c in range(4):
                    a = at[:, :, h] + j % bo * bi + c
                    frag[:, :, j, 4 * h + c] = np.where(at[:, :, h] < 0, 0.0, flat[np.where(at[:, :, h] < 0, 0, a)])
    else:
        parts = (sec[sec[OFF_FRAG]:].view(np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        frag = parts.reshape(nsteps, 3, 4, 16, 8).sum(1)  # (exact: a weight is the sum of its parts)
    got = np.zeros((nstrips * 16, H, K, I))
    for t in range(nstrips):
        for sl in range(nslabs):
            seen = set()
            for s in range(first[t, sl], first[t, sl + 1]):
                for g in range(4):
                    chunk, th, tw = desc[s, g] & 0xFFFF, desc[s, g] >> 16 & 0xFF, desc[s, g] >> 24
                    if not frag[s, g].any():
                        continue
                    assert (chunk, th, tw) not in seen
                    seen.add((chunk, th, tw))
                    c = sl * slab + chunk * 8
                    got[t * 16:t * 16 + 16, th, tw, c:c + 8] = frag[s, g]
    assert (got[:O] == W).all() and not got[O:].any()


def test_large_1x1_layers_hold_no_weights():
    """Most of them are FC layers, whose kernels read the payload."""
    for O, I in ((1000, 2048), (4096, 1000)):
        _, payload, plan = _layer(O, 1, 1, I, 8, 8, 0.5)
        assert plan.nbytes < payload.nbytes / 4
