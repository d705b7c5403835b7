"""Edges of the kernels and of the rules that pick them: rows at the borders of a tile, contractions of a few
steps, the smallest and largest sizes a variant serves.  Every element against the float64 oracle.

Tolerance: check_close of test_gpu_parity (elementwise 2e-2; normalised maximum 6e-3: one bf16 rounding of the
hidden row and one of the output, 2^-9 each, over fp32 sums)."""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import check_close, f64, moe  # noqa: F401  (moe is a fixture)

pytestmark = pytest.mark.gpu


def block_case(oracle64, counts, H, I, seed):
    """Expert rows laid out directly (no gating), weights, and the oracle's Yp."""
    counts = np.asarray(counts, dtype=np.int64)
    E, P = len(counts), int(counts.sum())
    g = torch.Generator().manual_seed(seed)
    Xp = torch.randn((P, H), generator=g).to(torch.bfloat16)
    Wg = (torch.randn((E, I, H), generator=g) * 0.05).to(torch.bfloat16)
    Wu = (torch.randn((E, I, H), generator=g) * 0.05).to(torch.bfloat16)
    Wd = (torch.randn((E, H, I), generator=g) * 0.05).to(torch.bfloat16)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ref = oracle64.expert_group_forward(0, E, Xp.float().numpy(), off, Wg.float().numpy(), Wu.float().numpy(),
                                        Wd.float().numpy())
    return dict(E=E, P=P, H=H, I=I, ref=ref, Xp=Xp.cuda(), Wg=Wg.cuda(), Wu=Wu.cuda(), Wd=Wd.cuda(),
                off=torch.from_numpy(off).cuda())


def run_blocks(moe, c, policy, cuts=None):
    ws = torch.empty(int(moe.load().moe_expert_workspace_bytes(c["P"], c["I"])), dtype=torch.uint8, device="cuda")
    Yp = torch.full((c["P"], c["H"]), 768.0, dtype=torch.bfloat16, device="cuda")
    for lo, hi in cuts or [(0, c["E"])]:
        moe.moe_expert_group_forward(lo, hi, c["Xp"], c["off"], c["Wg"], c["Wu"], c["Wd"], Yp, ws, policy)
    torch.cuda.synchronize()
    return Yp


# policy -> token rows of its tile
TILE_ROWS = {3: 128, 4: 256, 10: 128, 11: 160}


@pytest.mark.parametrize("H,I", [(64, 320), (192, 64), (448, 576)])     # 1 to 9 K steps: shorter than the ring, and not a multiple of it
@pytest.mark.parametrize("policy", sorted(TILE_ROWS))
def test_single_tile_experts_start_anywhere_in_k(moe, oracle64, policy, H, I):
    # an expert whose rows fit one tile starts its walk over K at a step of its own and wraps around; one row more
    # and it is two tiles that start at step 0
    bm = TILE_ROWS[policy]
    counts = [bm - 1, bm, bm + 1, 1, 0, 31, 32, 33, bm - 32, 64, 2 * bm, 2]
    print(f"[case] single-tile experts policy={policy} H={H} I={I}", flush=True)
    c = block_case(oracle64, counts, H, I, 100 + policy)
    Yp = run_blocks(moe, c, policy)
    check_close(f64(Yp), c["ref"], f"Yp policy {policy}")
    # and the same bits whatever the block cut
    Yc = run_blocks(moe, c, policy, [(5, 12), (0, 2), (2, 5)])
    assert torch.equal(Yp.view(torch.int16), Yc.view(torch.int16))
