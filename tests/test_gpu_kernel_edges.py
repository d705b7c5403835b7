"""Edges of the kernels and of the rules that pick them: rows at the borders of a tile, contractions of a few
steps, the smallest and largest sizes a variant serves.  Every element against the float64 oracle.

Tolerance: check_close of test_gpu_parity (elementwise 2e-2; normalised maximum 6e-3: one bf16 rounding of the
hidden row and one of the output, 2^-9 each, over fp32 sums)."""
import numpy as np
import pytest
import torch

import workloads
from tests.test_launch_routes_host import SHARED_BESIDE, SORT_BESIDE
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


# contractions of up to four steps (the narrow kernel), five (the deepest ring), seven
@pytest.mark.parametrize("H,I", [(64, 64), (128, 192), (320, 448), (448, 320)])
@pytest.mark.parametrize("counts", [
    [0, 1, 31, 32, 33, 63, 64, 65, 0, 0, 2, 5],                 # one, two, three token blocks
    [95, 96, 97, 0, 0, 0, 0, 1, 0, 0, 0, 0],                    # the last row of one pass and the first of two
    [0] * 20 + [191, 192, 193, 0, 289, 0] + [0] * 20,           # two to four passes, blocks dealt unevenly
    [7] * 256,                                                  # four experts in every lane of the prefix
], ids=["blocks", "pass", "passes", "many experts"])
def test_wide_streaming_at_block_and_pass_borders(moe, oracle64, counts, H, I):
    c = block_case(oracle64, counts, H, I, sum(counts) + H)
    print(f"[case] wide streaming, {len(counts)} experts, {c['P']} rows, H={H} I={I}", flush=True)
    Yp = run_blocks(moe, c, 9)
    check_close(f64(Yp), c["ref"], "Yp")
    e = c["E"]
    Yc = run_blocks(moe, c, 9, [(e // 3, e), (0, 1), (1, e // 3)])
    assert torch.equal(Yp.view(torch.int16), Yc.view(torch.int16)), "depends on the block cut"
    # a list in reverse order, its rows read through src_of_row: the same bits
    src = torch.arange(c["P"], dtype=torch.int32, device="cuda")
    ids = torch.arange(e - 1, -1, -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(int(moe.load().moe_expert_workspace_bytes(c["P"], I)), dtype=torch.uint8, device="cuda")
    Yl = torch.full_like(Yp, 768.0)
    moe.moe_expert_list_forward(ids, c["Xp"], src, 1, c["off"], c["Wg"], c["Wu"], c["Wd"], Yl, ws, 9)
    torch.cuda.synchronize()
    assert torch.equal(Yp.view(torch.int16), Yl.view(torch.int16)), "depends on list or gather"


# waves of 64 weight rows at the lines between the kernel's forms: gate/up 384 | 390, 512 | 520, 768 | 780; down 384 | 385, 510 | 516, 768 | 774
@pytest.mark.parametrize("E,H,I", [(24, 320, 512), (39, 320, 320), (32, 320, 512), (26, 320, 640), (32, 384, 768), (26, 320, 960),
                                   (32, 768, 320), (35, 704, 320), (34, 960, 320), (43, 768, 384), (32, 1536, 320), (43, 1152, 320)])
def test_wide_streaming_forms_give_the_same_bits(moe, oracle64, E, H, I):
    print(f"[case] forms of the wide kernel E={E} H={H} I={I}", flush=True)
    pattern = [1, 31, 32, 33, 0, 64, 65, 7, 96, 97, 5, 129, 12, 193, 8, 9]      # one to three blocks, one to four passes
    counts = [pattern[e % len(pattern)] for e in range(E)]
    c = block_case(oracle64, counts, H, I, E + H)
    Yp = run_blocks(moe, c, 9)
    check_close(f64(Yp), c["ref"], "Yp")
    for cuts in ([(e, e + 1) for e in range(E)], [(E // 2, E), (0, E // 2)], [(0, E - 1), (E - 1, E)]):
        Yc = run_blocks(moe, c, 9, cuts)
        assert torch.equal(Yp.view(torch.int16), Yc.view(torch.int16)), f"{len(cuts)} blocks"


@pytest.mark.parametrize("E,rows", [(8, 5), (8, 32), (8, 33), (20, 6), (20, 7), (20, 32), (20, 33), (1, 20)])
@pytest.mark.parametrize("H,I", [(192, 128), (320, 384), (256, 320)])     # contractions for the narrow kernel, the wide one, one each
def test_automatic_choice_around_its_lines(moe, oracle64, E, rows, H, I):
    # mean rows per expert 6 | 7: narrow or wide streaming; 32 | 33: streaming or tiles
    g = torch.Generator().manual_seed(E * 100 + rows)
    cut = torch.sort(torch.randint(0, E * rows + 1, (E - 1,), generator=g)).values.tolist()
    counts = np.diff([0] + cut + [E * rows])
    c = block_case(oracle64, counts, H, I, rows)
    Yp = run_blocks(moe, c, 0)
    check_close(f64(Yp), c["ref"], f"Yp, {E} experts of {rows} rows on average")
    Yc = run_blocks(moe, c, 0, [(e, e + 1) for e in range(E)])
    assert torch.equal(Yp.view(torch.int16), Yc.view(torch.int16))


@pytest.mark.parametrize("T", [12, 56])     # 8 experts, top-2: 3 and 14 rows per expert
def test_block_call_that_hosts_the_shared_experts_on_few_rows(moe, oracle64, T):
    wl = workloads.prefill(seed=77, T=T, H=192, E=8, K=2, I=128, Is=256)
    s, g, d = wl.shape, wl.to("cuda"), wl.f32_numpy()
    ids, w = moe.moe_route(g.x, g.Wr, g.bias, s.K, s.renorm)
    off, src, rowp, _ = moe.moe_permute(ids, g.x, s.E, materialize=False)
    buf = moe.LayerBuffers.allocate(s.T, s.H, s.E, s.K, s.I, s.Is)
    moe.moe_expert_group_forward_fused(0, s.E, g.x, src, s.K, off, g.Wg, g.Wu, g.Wd, g.Wsg, g.Wsu, g.Wsd, g.wgate, buf.Yp,
                                       buf.S_parts, buf.sg, buf.workspace_fused)
    Y = torch.empty_like(buf.Yp)
    moe.moe_expert_group_forward_gather(0, s.E, g.x, src, s.K, off, g.Wg, g.Wu, g.Wd, Y, buf.workspace)
    torch.cuda.synchronize()
    assert torch.equal(Y.view(torch.int16), buf.Yp.view(torch.int16))
    for p in range(s.Is // s.I):
        sl = slice(p * s.I, (p + 1) * s.I)
        S, sg = oracle64.shared_forward(d["x"], d["Wsg"][sl], d["Wsu"][sl], np.ascontiguousarray(d["Wsd"][:, sl]), d["wgate"])
        check_close(f64(buf.S_parts[p]), S, f"shared expert {p}")


# mean rows per expert and tokens at the lines between narrow, wide and separate launches: (64, 65 | 6 rows), (192, 193 | 32 rows)
@pytest.mark.parametrize("T,E,K,n_sets", [(1, 12, 2, 3), (16, 12, 4, 1), (36, 12, 2, 3), (37, 12, 2, 3), (64, 12, 1, 8), (65, 12, 1, 8),
                                          (96, 12, 2, 2), (97, 12, 2, 2), (192, 12, 2, 3), (193, 12, 2, 3), (200, 15, 1, 3), (410, 60, 4, 2)])
@pytest.mark.parametrize("H,I", [(128, 64), (192, 320), (384, 320)])     # narrow, one kernel each, wide where the rows call for it
def test_block_call_that_hosts_the_shared_experts_in_every_launch_form(moe, oracle64, T, E, K, n_sets, H, I):
    print(f"[case] hosted shared experts T={T} E={E} K={K} sets={n_sets} H={H} I={I}", flush=True)
    Is = n_sets * I
    w = workloads.layer_weights(H, E, I, Is, 31 + T, 0.05, 0.1, torch.bfloat16, device="cpu")
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16)
    d, xg = {k: v.cuda() for k, v in w.items()}, x.cuda()
    assert moe.moe_fused_shared_sets(T, H, E, K, I, Is) == n_sets
    ids, _ = moe.moe_route(xg, d["Wr"], None, K, False)
    off, src, rowp, _ = moe.moe_permute(ids, xg, E, materialize=False)
    buf = moe.LayerBuffers.allocate(T, H, E, K, I, Is)
    Y = torch.full_like(buf.Yp, 768.0)
    lo, hi = 1, E - 1       # a block that is not the whole layer
    moe.moe_expert_group_forward_gather(lo, hi, xg, src, K, off, d["Wg"], d["Wu"], d["Wd"], Y, buf.workspace)
    buf.Yp.fill_(768.0)
    buf.S_parts.fill_(768.0)
    moe.moe_expert_group_forward_fused(lo, hi, xg, src, K, off, d["Wg"], d["Wu"], d["Wd"], d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"], buf.Yp,
                                       buf.S_parts, buf.sg, buf.workspace_fused)
    torch.cuda.synchronize()
    assert torch.equal(Y.view(torch.int16), buf.Yp.view(torch.int16))
    f32 = {k: v.float().numpy() for k, v in w.items()}
    for p in range(n_sets):
        sl = slice(p * I, (p + 1) * I)
        S, sg = oracle64.shared_forward(x.float().numpy(), f32["Wsg"][sl], f32["Wsu"][sl], np.ascontiguousarray(f32["Wsd"][:, sl]),
                                        f32["wgate"])
        check_close(f64(buf.S_parts[p]), S, f"shared expert {p}")
    assert np.allclose(buf.sg.cpu().numpy(), sg, rtol=1e-4, atol=1e-5)


@pytest.mark.parametrize("T,H,Is", [(777, 2048, 5632), (600, 64, 1536), (513, 256, 1024), (640, 1024, 256), (700, 1536, 768), (1000, 128, 640),
                                          (129, 512, 1024), (300, 2048, 512), (1100, 3072, 128)])
def test_shared_expert_with_the_down_projection_cut_along_k(moe, oracle64, T, H, Is):
    # the parts that the workspace has room for (at most; K must also divide into them), and none of them
    wl = workloads.qwen_layer(T, 900 + T, H=H, E=4, K=1, I=64, Is=Is, renorm=False)
    g, d = wl.to("cuda"), wl.f32_numpy()
    full = int(moe.load().moe_shared_workspace_bytes(T, H, Is))
    h_only = (T * Is * 2 + 255) // 256 * 256
    if T > 512:
        assert full in (h_only, h_only + 2 * T * H * 4, h_only + 4 * T * H * 4, h_only + 8 * T * H * 4)
    S_ref, sg_ref = oracle64.shared_forward(d["x"], d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"])
    first = None     # beyond 512 tokens: the same bits with room for every part, for some, for none
    for nbytes in sorted({full, h_only, h_only + T * H * 4, min(full, h_only + 2 * T * H * 4)}) if T > 512 else {full}:
        print(f"[case] shared expert T={T} H={H} Is={Is}, workspace {nbytes}", flush=True)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        S = torch.full((T, H), 768.0, dtype=torch.bfloat16, device="cuda")
        sg = torch.full((T,), 768.0, dtype=torch.float32, device="cuda")
        moe.moe_shared_forward(g.x, g.Wsg, g.Wsu, g.Wsd, g.wgate, S, sg, ws)
        torch.cuda.synchronize()
        check_close(f64(S), S_ref, f"S, workspace {nbytes}")
        assert np.allclose(sg.cpu().numpy(), sg_ref, rtol=1e-4, atol=1e-5)
        first = S if first is None else first
        assert torch.equal(S.view(torch.int16), first.view(torch.int16)), f"bits depend on the workspace ({nbytes})"


@pytest.mark.parametrize("T", [1, 16, 17, 31, 32, 33, 65])     # one and two tiles of 16 rows per pass, further passes
@pytest.mark.parametrize("H,Is", [(64, 192), (448, 576)])
def test_shared_expert_streamed_on_request(moe, oracle64, T, H, Is):
    print(f"[case] shared expert streamed T={T} H={H} Is={Is}", flush=True)
    w = workloads.layer_weights(H, 2, 64, Is, T, 0.05, 0.1, torch.bfloat16, device="cpu")
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16)
    d = {k: v.cuda() for k, v in w.items()}
    ws = torch.empty((T * Is * 2 + 255) // 256 * 256, dtype=torch.uint8, device="cuda")
    run = lambda n: moe.moe_shared_forward(x[:n].cuda(), d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"], torch.empty((n, H), dtype=torch.bfloat16,
                                           device="cuda"), torch.empty(n, device="cuda"), ws, 9)[0]
    S, S16 = run(T), run(min(T, 16))
    torch.cuda.synchronize()
    S_ref, _ = oracle64.shared_forward(x.float().numpy(), *[w[k].float().numpy() for k in ("Wsg", "Wsu", "Wsd", "wgate")])
    check_close(f64(S), S_ref, "S")
    assert torch.equal(S[:16].view(torch.int16), S16.view(torch.int16)), "a row depends on the rows of its pass"


@pytest.mark.parametrize("T", [33, 160, 161, 640, 641, 700])     # 1, 2, 4, 5 token tiles of 160 rows and one row more
def test_shared_expert_walk_over_incomplete_tile_groups(moe, oracle64, T):
    wl = workloads.qwen_layer(T, 950 + T, H=128, E=4, K=1, I=64, Is=448, renorm=False)
    g, d = wl.to("cuda"), wl.f32_numpy()
    S_ref, _ = oracle64.shared_forward(d["x"], d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"])
    ws = torch.empty(int(moe.load().moe_shared_workspace_bytes(T, 128, 448)) + 8 * T * 128 * 4, dtype=torch.uint8, device="cuda")
    for policy in (3, 4, 8, 10, 11):
        S = torch.full((T, 128), 768.0, dtype=torch.bfloat16, device="cuda")
        sg = torch.empty(T, dtype=torch.float32, device="cuda")
        moe.moe_shared_forward(g.x, g.Wsg, g.Wsu, g.Wsd, g.wgate, S, sg, ws, policy)
        torch.cuda.synchronize()
        check_close(f64(S), S_ref, f"S, T={T} policy {policy}")


def router_bits(moe, oracle64, T, H, E, K):
    # The batch repeats one token and bias[e] = -(the oracle's fp32 logit of e): every logit becomes exactly 0 when it
    # has the oracle's bits, and ids 0..K-1 win the tie at weight 1/E; one ulp anywhere changes the ids.
    print(f"[case] router variants T={T} H={H} E={E}", flush=True)
    g = torch.Generator().manual_seed(T * 7 + H)
    x = ((torch.rand((1, H), generator=g) - 0.5) * torch.pow(2.0, torch.randint(-8, 9, (1, H), generator=g).float())).to(torch.bfloat16)
    Wr = (torch.randn((E, H), generator=g) * 0.05).to(torch.bfloat16)
    _, _, L = oracle64.route(x.float().numpy(), Wr.float().numpy(), None, K, False, want_logits=True)
    expect = np.tile(np.arange(K, dtype=np.int32), (T, 1))
    for sign in (1.0, -1.0):
        bias = torch.from_numpy(-sign * L[0]).contiguous().cuda()
        ids, w = moe.moe_route(x.repeat(T, 1).cuda(), (Wr * sign).to(torch.bfloat16).cuda(), bias, K, False)
        torch.cuda.synchronize()
        assert np.array_equal(ids.cpu().numpy(), expect), sign
        assert np.allclose(w.cpu().numpy(), 1.0 / E, rtol=1e-6)


@pytest.mark.parametrize("H", [64, 960, 1024, 1088, 1536, 1984, 2048, 3072, 4096])
@pytest.mark.parametrize("T", [1, 255, 256, 257, 511, 512, 513, 1024, 1025, 2049, 4095, 4097])
def test_router_sums_keep_their_order_in_every_variant(moe, oracle64, T, H):
    E, K = (61, 4) if H % 512 else (66, 7)      # ragged last batches of experts
    router_bits(moe, oracle64, T, H, E, K)


# few experts, whose waves work on pairs of token groups; rounds of 8 and of 16 tokens per workgroup (4096 | 4097, 8192 | 8193)
@pytest.mark.parametrize("T,H,E,K", [(1025, 64, 8, 3), (1031, 320, 3, 1), (2049, 1024, 5, 2), (4099, 512, 8, 8), (1024, 64, 8, 3), (1030, 64, 9, 3),
                                     (4096, 2560, 6, 2), (4098, 2112, 6, 2), (8192, 2112, 5, 2), (8193, 4096, 4, 1)])
def test_router_sums_keep_their_order_with_few_experts_and_in_whole_rounds(moe, oracle64, T, H, E, K):
    router_bits(moe, oracle64, T, H, E, K)


@pytest.mark.parametrize("T,H,E,K", [(1, 64, 8, 2), (64, 64, 3, 1), (65, 128, 61, 1), (1023, 64, 256, 1), (257, 192, 60, 4), (341, 64, 256, 3),
                                     (683, 320, 7, 6), (4095, 64, 60, 1), (4096, 64, 1, 1), (4097, 64, 60, 1), (256, 64, 256, 16)])
@pytest.mark.parametrize("hot", [False, True])
def test_sort_of_pairs_at_the_borders_of_its_kernels(moe, oracle64, T, H, E, K, hot):
    # one workgroup up to 1024 pairs (index arrays only), one launch up to 4096, the table beyond; whole numbers and copied rows: exact
    print(f"[case] permute borders T={T} H={H} E={E} K={K} hot={hot}", flush=True)
    rng = np.random.default_rng(T * 3 + E)
    keys = rng.random((T, E))
    if hot:
        keys[:, E // 2] = 2.0      # every token chooses this expert
    ids = np.argsort(-keys, axis=1)[:, :K].astype(np.int32)
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16)
    off_r, src_r, rowp_r = oracle64.permute(ids, E)
    for materialize in (True, False):
        off, src, rowp, Xp = moe.moe_permute(torch.from_numpy(ids).cuda(), x.cuda(), E, materialize=materialize)
        torch.cuda.synchronize()
        assert np.array_equal(off.cpu().numpy(), off_r)
        assert np.array_equal(src.cpu().numpy(), src_r)
        assert np.array_equal(rowp.cpu().numpy(), rowp_r)
        if materialize:
            assert torch.equal(Xp.cpu().view(torch.int16), x[torch.from_numpy(src_r.astype(np.int64)) // K].view(torch.int16))


# Layers whose tiles do not fill the chip twice: 128x128, 128x64, 160- and 128-row tiles for gate/up and down
@pytest.mark.parametrize("counts,H,I", [([40] * 16, 64, 2304), ([60] * 4, 128, 320), ([200] * 8, 64, 1024), ([300, 1, 500, 399], 64, 512),
                                        ([34] * 2, 2048, 64), ([129, 0, 130, 33, 128], 192, 192)])
def test_few_expert_layers_pick_tiles_from_the_whole_layer(moe, oracle64, counts, H, I):
    print(f"[case] few experts counts={counts} H={H} I={I}", flush=True)
    c = block_case(oracle64, counts, H, I, 300 + len(counts))
    Yp = run_blocks(moe, c, 0)
    check_close(f64(Yp), c["ref"], "Yp")
    Yc = run_blocks(moe, c, 0, [(i, i + 1) for i in range(c["E"])])      # the same bits whatever the block cut
    assert torch.equal(Yp.view(torch.int16), Yc.view(torch.int16))


def record_one_calls(monkeypatch):
    """Whether each layer from here on ran as one native call (a sequence that fell back to its steps would pass every
    comparison with them)."""
    from paper_2604_26881_amd import binding
    inner, served = binding._layer_in_one_call, []

    def recorded(*args, **kw):
        served.append(inner(*args, **kw))
        return served[-1]
    monkeypatch.setattr(binding, "_layer_in_one_call", recorded)
    return served


@pytest.mark.parametrize("T", [1, 3, 16, 17, 31, 32, 33])
# sets of I columns of the shared expert: narrower than one, whole, a ragged last one, more than can ride along, none
@pytest.mark.parametrize("H,E,K,I,Is", [(64, 8, 2, 192, 128), (192, 60, 4, 64, 256), (320, 16, 2, 192, 448), (128, 12, 2, 64, 576),
                                        (64, 8, 1, 64, 0)])
@pytest.mark.parametrize("gather,segments", [(False, False), (True, True)])
def test_layer_in_one_call_equals_its_steps(moe, oracle64, monkeypatch, T, H, E, K, I, Is, gather, segments):
    print(f"[case] layer in one call T={T} H={H} E={E} K={K} I={I} Is={Is} gather={gather} segments={segments}", flush=True)
    w = workloads.layer_weights(H, E, I, Is, 11 + T, 0.05, 0.1, torch.bfloat16, device="cpu")
    g = torch.Generator().manual_seed(T * 5 + E)
    x = torch.randn((T, H), generator=g).to(torch.bfloat16)
    cut = [(0, T // 2), (T // 2, T)] if segments else None
    bias = torch.randn((2, E), generator=g) if segments else torch.randn((E,), generator=g)
    d = {k: None if v is None else v.cuda() for k, v in w.items()}
    shared = None if Is == 0 else (d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"])
    seg = moe.segment_offsets(cut, T, "cuda") if segments else None
    run = lambda groups: moe.moe_layer_forward(x.cuda(), d["Wr"], bias.cuda(), d["Wg"], d["Wu"], d["Wd"], shared, K, True,
                                               groups=groups, tenant_rows=cut, fused_gather=gather, seg_offsets=seg)
    served = record_one_calls(monkeypatch)
    one, steps = run(None), run([(0, 1), (1, E)])       # two blocks take the step-by-step sequence
    torch.cuda.synchronize()
    assert served == [True, False]
    for name in ("topk_ids", "topk_w", "expert_offsets", "src_of_row", "row_of_pair", "Yp") + (() if gather else ("Xp",)):
        a, b = getattr(one, name), getattr(steps, name)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name
    assert torch.equal(one.out.view(torch.int16), steps.out.view(torch.int16))
    if Is > 0:
        assert torch.equal(one.sg, steps.sg) and torch.equal(one.S.view(torch.int16), steps.S.view(torch.int16))
        f32 = {k: v.float().numpy() for k, v in w.items() if v is not None}
        S_ref, _ = oracle64.shared_forward(x.float().numpy(), f32["Wsg"], f32["Wsu"], f32["Wsd"], f32["wgate"])
        check_close(f64(one.S), S_ref, "S")


@pytest.mark.parametrize("T", [1, 13, 16, 17, 32, 33])
# K parts of 20 and 21 steps; three; one; four of 22; one, and more sets than can ride along
@pytest.mark.parametrize("H,E,K,I,Is", [(512, 12, 2, 384, 2624), (256, 60, 4, 576, 3904), (128, 16, 2, 64, 448), (192, 20, 2, 1408, 5632),
                                        (320, 16, 1, 64, 1024)])
def test_output_is_bitwise_independent_of_blocks_streams_and_sequence(moe, oracle64, monkeypatch, T, H, E, K, I, Is):
    print(f"[case] few tokens in every sequence T={T} H={H} E={E} K={K} I={I} Is={Is}", flush=True)
    w = workloads.layer_weights(H, E, I, Is, 21 + T, 0.05, 0.1, torch.bfloat16, device="cpu")
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T * 3 + E)).to(torch.bfloat16)
    d, xg = {k: v.cuda() for k, v in w.items()}, x.cuda()
    run = lambda **kw: moe.moe_layer_forward(xg, d["Wr"], None, d["Wg"], d["Wu"], d["Wd"], (d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"]), K,
                                             False, **kw)
    served = record_one_calls(monkeypatch)
    bufs = {"one block": run(), "gathered": run(fused_gather=True), "two blocks": run(groups=[(0, 5), (5, E)]),
            "a block per expert": run(groups=[(e, e + 1) for e in range(E)]), "two streams": run(shared_stream=torch.cuda.Stream()),
            "blocks and streams": run(groups=[(0, 1), (1, E)], shared_stream=torch.cuda.Stream())}
    torch.cuda.synchronize()
    assert served[:3] == [True, True, False]
    one = bufs["one block"]
    f32 = {k: v.float().numpy() for k, v in w.items()}
    S_ref, sg_ref = oracle64.shared_forward(x.float().numpy(), f32["Wsg"], f32["Wsu"], f32["Wsd"], f32["wgate"])
    check_close(f64(one.S), S_ref, "S")
    assert np.allclose(one.sg.cpu().numpy(), sg_ref, rtol=1e-4, atol=1e-5)
    for name, b in bufs.items():
        for what in ("S", "sg", "Yp", "out"):
            assert torch.equal(getattr(b, what).view(torch.uint8), getattr(one, what).view(torch.uint8)), f"{what} of {name}"
    # the shared expert by hand, in workspaces from the smallest that is taken (K parts where K divides evenly) to the helper's
    h_only = (T * Is * 2 + 255) // 256 * 256
    least = h_only + next((p for p in (8, 4, 2) if Is % (64 * p) == 0), 0) * T * H * 4
    for nbytes in {least, int(moe.load().moe_shared_workspace_bytes(T, H, Is))}:
        for flags in (0, 0x400):
            S, sg = torch.full_like(one.S, 768.0), torch.full_like(one.sg, 768.0)
            moe.moe_shared_forward(xg, d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"], S, sg, torch.empty(nbytes, dtype=torch.uint8, device="cuda"),
                                   flags)
            torch.cuda.synchronize()
            assert torch.equal(S.view(torch.int16), one.S.view(torch.int16)) and torch.equal(sg, one.sg), f"workspace {nbytes}"


@pytest.mark.parametrize("T", [1, 13, 16, 17, 32, 33])
@pytest.mark.parametrize("shared_memory", ["workspaces", "Xp", "out", "src_of_row", "S", "x", "out over x"])
def test_layer_in_one_call_with_memory_shared_between_its_steps(moe, oracle64, T, shared_memory):
    # One buffer as every workspace; or the shared expert's scratch in memory of a step that is over by then (the row
    # copies, the index list) or not yet begun (the output), or S or the tokens behind the hidden rows, in room that this K is
    # not cut for (17 steps); or the output one row behind the tokens: right when the steps run in turn, so right in one call too.
    H, E, K, I, Is = 192, 8, 1, 256, 1088
    print(f"[case] layer in one call, shared memory: {shared_memory}, T={T}", flush=True)
    w = workloads.layer_weights(H, E, I, Is, 70 + T, 0.05, 0.1, torch.bfloat16, device="cpu")
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16)
    d, xg = {k: v.cuda() for k, v in w.items()}, x.cuda()
    f32 = {k: v.float().numpy() for k, v in w.items()}
    buf = moe.LayerBuffers.allocate(T, H, E, K, I, Is)
    need = moe.moe_workspace_bytes(T, H, E, K, I, Is)
    if shared_memory == "workspaces":
        buf.workspace = buf.workspace_shared = buf.workspace_permute = torch.empty(need, dtype=torch.uint8, device="cuda")
    elif shared_memory == "out over x":
        both = torch.empty((T + 1, H), dtype=torch.bfloat16, device="cuda")
        both[:T] = xg
        xg, buf.out = both[:T], both[1:]
    else:
        whole = torch.empty(need, dtype=torch.uint8, device="cuda")
        buf.workspace_shared = whole
        old = xg if shared_memory == "x" else getattr(buf, shared_memory)
        at = (T * Is * 2 + 255) // 256 * 256 if shared_memory in ("S", "x") else 0
        room = whole[at:at + old.numel() * old.element_size()]
        assert room.numel() == old.numel() * old.element_size()
        new = room.view(old.dtype).view(old.shape)
        if shared_memory == "x":
            new.copy_(xg)
            xg = new
        else:
            setattr(buf, shared_memory, new)
    moe.moe_layer_forward(xg, d["Wr"], None, d["Wg"], d["Wu"], d["Wd"], (d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"]), K, False,
                          buf=buf, fused_gather=shared_memory in ("workspaces", "src_of_row"))
    torch.cuda.synchronize()
    ref = oracle64.layer(x.float().numpy(), f32["Wr"], None, f32["Wg"], f32["Wu"], f32["Wd"],
                         (f32["Wsg"], f32["Wsu"], f32["Wsd"], f32["wgate"]), K, False)
    assert np.array_equal(buf.topk_ids.cpu().numpy(), ref["ids"])
    check_close(f64(buf.out), ref["out"], f"out, {shared_memory}")


@pytest.mark.parametrize("T", [1, 16, 17])
def test_a_second_stream_keeps_its_order_whatever_runs_on_it(moe, T):
    # The shared expert's weights are uploaded on the second stream behind a long copy, and S is read there behind the
    # layer while the caller's stream is still busy: both were ordered when the shared expert ran on that stream.
    H, E, K, I, Is = 128, 8, 2, 64, 192
    print(f"[case] order of the second stream T={T}", flush=True)
    w = {k: v.cuda() for k, v in workloads.layer_weights(H, E, I, Is, 80 + T, 0.05, 0.1, torch.bfloat16, device="cpu").items()}
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16).cuda()
    run = lambda sh, b, st: moe.moe_layer_forward(x, w["Wr"], None, w["Wg"], w["Wu"], w["Wd"], sh, K, False, buf=b, shared_stream=st)
    real = (w["Wsg"], w["Wsu"], w["Wsd"], w["wgate"])
    late = tuple(torch.zeros_like(t) for t in real)
    bufs = [moe.LayerBuffers.allocate(T, H, E, K, I, Is) for _ in range(2)]
    a, b = (torch.zeros(1 << 28, dtype=torch.uint8, device="cuda") for _ in range(2))
    side, seen = torch.cuda.Stream(), torch.zeros_like(bufs[1].S)
    run(real, bufs[0], side)                  # (kernels loaded, expected result)
    torch.cuda.synchronize()
    bufs[1].S.fill_(768.0)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(40):                   # some milliseconds
            b.copy_(a)
        for t, r in zip(late, real):
            t.copy_(r)
    run(late, bufs[1], side)
    torch.cuda.synchronize()
    assert torch.equal(bufs[0].out.view(torch.int16), bufs[1].out.view(torch.int16)), "ran before the upload"
    bufs[1].S.fill_(768.0)
    torch.cuda.synchronize()
    for _ in range(40):
        b.copy_(a)
    run(real, bufs[1], side)
    with torch.cuda.stream(side):
        seen.copy_(bufs[1].S)
    torch.cuda.synchronize()
    assert torch.equal(bufs[0].S.view(torch.int16), seen.view(torch.int16)), "read before it was written"


@pytest.mark.parametrize("T", [1, 16, 17])
def test_capture_with_a_second_stream_at_few_tokens(moe, T):
    H, E, K, I, Is = 128, 8, 2, 64, 192
    print(f"[case] capture with a second stream T={T}", flush=True)
    w = {k: v.cuda() for k, v in workloads.layer_weights(H, E, I, Is, 90 + T, 0.05, 0.1, torch.bfloat16, device="cpu").items()}
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16).cuda()
    side, buf = torch.cuda.Stream(), moe.LayerBuffers.allocate(T, H, E, K, I, Is)
    run = lambda b, st: moe.moe_layer_forward(x, w["Wr"], None, w["Wg"], w["Wu"], w["Wd"], (w["Wsg"], w["Wsu"], w["Wsd"], w["wgate"]),
                                              K, False, buf=b, shared_stream=st)
    warm = torch.cuda.Stream()
    warm.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(warm):
        run(buf, side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run(buf, side)
        run(buf, side)      # the second stream is in the capture already
    for i in range(3):
        x.copy_(torch.randn((T, H), generator=torch.Generator().manual_seed(50 + i)).to(torch.bfloat16))
        buf.out.fill_(768.0)
        graph.replay()
        torch.cuda.synchronize()
        eager = run(None, side)
        torch.cuda.synchronize()
        assert torch.equal(buf.out.view(torch.int16), eager.out.view(torch.int16)), f"replay {i}"
        assert torch.equal(buf.S.view(torch.int16), eager.S.view(torch.int16)), f"replay {i}"


@pytest.mark.parametrize("T,H,E,K,I,Is", [(1, 64, 8, 2, 64, 0), (33, 2112, 8, 2, 64, 128), (520, 128, 8, 2, 64, 192), (700, 64, 4, 1, 64, 0),
                                          (5, 8192, 4, 1, 64, 0), (1, 320, 16, 2, 384, 2624), (16, 192, 12, 2, 256, 1088),
                                          (32, 128, 20, 2, 64, 448)])
def test_residual_step_from_the_aggregation_has_the_bits_of_its_own_call(moe, monkeypatch, T, H, E, K, I, Is):
    # 520 tokens and 33 form the gate logit in the aggregation or beside the sum of the K parts; up to 32 tokens the shared
    # expert rides along and the aggregation adds its parts as well; the layers run in place
    print(f"[case] stack against its steps T={T} H={H} E={E} Is={Is}", flush=True)
    layers = [{k: None if v is None else v.cuda() for k, v in
               workloads.layer_weights(H, E, I, Is, 5 + i, 0.05, 0.1, torch.bfloat16, device="cpu").items()} for i in range(3)]
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16).cuda()
    served = record_one_calls(monkeypatch)
    out = moe.moe_stack_forward(x, layers, K, False, eps=1e-5)
    assert served == [True] * 3
    cur = x
    for w in layers:
        shared = None if Is == 0 else (w["Wsg"], w["Wsu"], w["Wsd"], w["wgate"])
        buf = moe.moe_layer_forward(cur, w["Wr"], None, w["Wg"], w["Wu"], w["Wd"], shared, K, False, groups=[(0, 1), (1, E)])
        cur = moe.moe_residual_norm(cur, buf.out, eps=1e-5)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), cur.view(torch.int16))


@pytest.mark.parametrize("T", [1, 5, 33, 130])
@pytest.mark.parametrize("where", ["x", "out", "Yp", "S", "Xp"])
def test_residual_step_into_memory_of_the_layer(moe, T, where):
    # the next layer's tokens may take the place of anything that is over by then, also of rows the aggregation still reads
    H, E, K, I, Is = 192, 8, 2, 64, 128
    print(f"[case] residual step into {where} T={T}", flush=True)
    w = {k: v.cuda() for k, v in workloads.layer_weights(H, E, I, Is, 40 + T, 0.05, 0.1, torch.bfloat16, device="cpu").items()}
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16).cuda()
    expect = moe.moe_stack_forward(x, [w], K, False)
    buf = moe.LayerBuffers.allocate(T, H, E, K, I, Is)
    cur = x.clone()
    into = cur if where == "x" else getattr(buf, where)[:T]
    got = moe.moe_stack_forward(cur, [w], K, False, buf=buf, x_out=into)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int16), expect.view(torch.int16))


@pytest.mark.parametrize("T,H,Is", [(383, 64, 11264), (384, 192, 11200), (385, 64, 11264), (6000, 2048, 64)])
def test_shared_expert_in_192_row_tiles(moe, oracle64, T, H, Is):
    # sizes at which the choice falls on 192-row tiles (gate/up of a wide hidden layer; down of many rows), and one beside them
    print(f"[case] shared expert T={T} H={H} Is={Is}", flush=True)
    w = workloads.layer_weights(H, 2, 64, Is, T, 0.05, 0.1, torch.bfloat16, device="cpu")
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16)
    d = {k: v.cuda() for k, v in w.items()}
    S, sg = torch.empty((T, H), dtype=torch.bfloat16, device="cuda"), torch.empty(T, device="cuda")
    ws = torch.empty(int(moe.load().moe_shared_workspace_bytes(T, H, Is)), dtype=torch.uint8, device="cuda")
    moe.moe_shared_forward(x.cuda(), d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"], S, sg, ws)
    torch.cuda.synchronize()
    S_ref, sg_ref = oracle64.shared_forward(x.float().numpy(), *[w[k].float().numpy() for k in ("Wsg", "Wsu", "Wsd", "wgate")])
    check_close(f64(S), S_ref, "S")
    assert np.allclose(sg.cpu().numpy(), sg_ref, rtol=1e-4, atol=1e-5)


@pytest.mark.parametrize("mean,bm", [(60, 128), (140, 160), (232, 256)])     # the height of the layer's tiles
# full width in gate/up, in the down projection; one K step, four, and seven (longer than every ring and no multiple of one)
@pytest.mark.parametrize("H,I", [(256, 1152), (448, 1152), (2304, 64), (2304, 448)])
def test_calls_on_a_few_experts_take_narrower_tiles_to_the_same_bits(moe, oracle64, mean, bm, H, I):
    # 60 experts: the uncut call has two rounds of whole tiles, calls on a few of them have compute units to spare
    E = 60
    edges = [bm - 1, bm, bm + 1, 0, 1, 31, 32, 33, 64, bm - 32, 2 * bm + 1]
    counts = (edges * 6)[:E]
    rest = (mean * E - sum(counts)) // 20
    counts = [n + (rest if i % 3 == 2 else 0) for i, n in enumerate(counts)]
    counts = [max(0, n) for n in counts]
    print(f"[case] narrower tiles mean={mean} H={H} I={I}", flush=True)
    c = block_case(oracle64, counts, H, I, 300 + mean)
    Yp = run_blocks(moe, c, 0)
    check_close(f64(Yp), c["ref"], f"Yp mean {mean}")
    for cuts in ([(i, i + 1) for i in range(E)], [(0, 3), (3, 10), (10, 17), (17, 32), (32, 40), (40, 60)]):
        Yc = run_blocks(moe, c, 0, cuts)
        assert torch.equal(Yp.view(torch.int16), Yc.view(torch.int16)), cuts[:2]


# (which of these sizes are sorted there: test_launch_routes_host.py holds the library to it, as to the memory)
@pytest.mark.parametrize("T,K,E", [(T, K, E) for T, K, E, _ in SORT_BESIDE])
@pytest.mark.parametrize("gather,ids_in", [(False, "their own memory"), (True, "their own memory"), (False, "the hidden rows"),
                                           (True, "row_of_pair")])
def test_micro_batch_constructed_beside_gate_up_equals_the_sort(moe, oracle64, monkeypatch, T, K, E, gather, ids_in):
    # up to 128 pairs the sort is part of the experts' first launch; most tokens choose the same expert, so that its rows
    # take several passes over the ids; ids in memory that this launch writes keep the sort's own launch
    H, I = 64, 64
    print(f"[case] sort beside gate/up T={T} K={K} E={E} gather={gather} ids in {ids_in}", flush=True)
    w = workloads.layer_weights(H, E, I, 0, 90 + T, 0.05, 0.1, torch.bfloat16, device="cpu")
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T + E)).to(torch.bfloat16)
    bias = torch.zeros(E)
    bias[E // 2] = 3.0
    d, xg = {k: None if v is None else v.cuda() for k, v in w.items()}, x.cuda()
    run = lambda buf, groups: moe.moe_layer_forward(xg, d["Wr"], bias.cuda(), d["Wg"], d["Wu"], d["Wd"], None, K, True, groups=groups,
                                                    buf=buf, fused_gather=gather)
    one, steps = (moe.LayerBuffers.allocate(T, H, E, K, I, 0) for _ in range(2))
    if ids_in != "their own memory":
        one.topk_ids = (one.workspace if ids_in == "the hidden rows" else one.row_of_pair).view(torch.int32)[:T * K].view(T, K)
    served = record_one_calls(monkeypatch)
    run(one, None), run(steps, [(0, 1), (1, E)])
    torch.cuda.synchronize()
    assert served == [True, False]
    assert int((steps.expert_offsets[1:] - steps.expert_offsets[:-1]).max()) > 16
    for name in ("topk_w", "expert_offsets", "src_of_row", "row_of_pair", "Yp", "out") + (() if gather else ("Xp",)):
        a, b = getattr(one, name), getattr(steps, name)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name


# 60 experts take tiles of 128, 160 and 256 rows; the shared hidden layer is whole sets of I columns, or ends in a
# narrower one that covers less than the column tiles of a set, or is narrower than one; too many sets for one launch
# (which of these sizes take the one launch: the table says so, and test_launch_routes_host.py holds the library to it)
@pytest.mark.parametrize("T,Is", [(T, Is) for T, Is, _ in SHARED_BESIDE])
@pytest.mark.parametrize("gather", [False, True])
def test_shared_expert_formed_beside_the_routed_gate_up_has_the_bits_of_its_own_call(moe, oracle64, monkeypatch, T, Is, gather):
    H, E, K, I = 128, 60, 4, 1152
    print(f"[case] shared gate/up beside the routed T={T} Is={Is} gather={gather}", flush=True)
    w = workloads.layer_weights(H, E, I, Is, 120 + T, 0.05, 0.1, torch.bfloat16, device="cpu")
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T + Is)).to(torch.bfloat16)
    d, xg = {k: v.cuda() for k, v in w.items()}, x.cuda()
    sh = (d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"])
    run = lambda groups: moe.moe_layer_forward(xg, d["Wr"], None, d["Wg"], d["Wu"], d["Wd"], sh, K, True, groups=groups, fused_gather=gather)
    served = record_one_calls(monkeypatch)
    one, steps = run(None), run([(0, 25), (25, E)])
    torch.cuda.synchronize()
    assert served == [True, False]
    for name in ("Yp", "S", "sg", "out"):
        a, b = getattr(one, name), getattr(steps, name)
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name
    f32 = {k: v.float().numpy() for k, v in w.items()}
    rows = np.arange(0, T, 7)
    S_ref, _ = oracle64.shared_forward(x.float().numpy()[rows], f32["Wsg"], f32["Wsu"], f32["Wsd"], f32["wgate"])
    check_close(f64(one.S)[rows], S_ref, "S")


@pytest.mark.parametrize("memory", ["workspaces", "Xp", "src_of_row", "expert_offsets"])
def test_shared_expert_whose_rows_lie_in_memory_of_the_routed_ones_has_its_own_launch(moe, memory):
    # right when the steps run in turn: each of these is of no further use when the shared expert's own call begins
    T, H, E, K, I, Is = 640, 128, 60, 4, 1152, 2304
    print(f"[case] shared hidden rows in memory of the routed experts: {memory}", flush=True)
    w = workloads.layer_weights(H, E, I, Is, 17, 0.05, 0.1, torch.bfloat16, device="cpu")
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(T)).to(torch.bfloat16).cuda()
    d = {k: v.cuda() for k, v in w.items()}
    apart, one = (moe.LayerBuffers.allocate(T, H, E, K, I, Is) for _ in range(2))
    if memory == "workspaces":
        need = moe.moe_workspace_bytes(T, H, E, K, I, Is)
        one.workspace = one.workspace_shared = one.workspace_permute = torch.empty(need, dtype=torch.uint8, device="cuda")
    else:
        old = getattr(one, memory)
        setattr(one, memory, one.workspace_shared[:old.numel() * old.element_size()].view(old.dtype).view(old.shape))
    for buf in (apart, one):
        moe.moe_layer_forward(x, d["Wr"], None, d["Wg"], d["Wu"], d["Wd"], (d["Wsg"], d["Wsu"], d["Wsd"], d["wgate"]), K, True, buf=buf,
                              fused_gather=memory != "Xp")
    torch.cuda.synchronize()
    for name in ("Yp", "S", "sg", "out"):
        assert torch.equal(getattr(one, name).view(torch.uint8), getattr(apart, name).view(torch.uint8)), name


def test_a_layer_whose_block_is_refused_leaves_the_steps_before_it(moe):
    T, H, E, K, I = 5, 64, 8, 2, 64
    print("[case] refused block behind gating and sort", flush=True)
    w = {k: None if v is None else v.cuda() for k, v in workloads.layer_weights(H, E, I, 0, 7, 0.05, 0.1, torch.bfloat16, device="cpu").items()}
    x = torch.randn((T, H), generator=torch.Generator().manual_seed(2)).to(torch.bfloat16).cuda()
    want = moe.moe_layer_forward(x, w["Wr"], None, w["Wg"], w["Wu"], w["Wd"], None, K, True)
    b = moe.LayerBuffers.allocate(T, H, E, K, I, 0)
    b.src_of_row.fill_(-1)
    p = lambda t: t.data_ptr()
    rc = moe.load().moe_layer_forward(
        p(x), p(w["Wr"]), None, None, 0, p(w["Wg"]), p(w["Wu"]), p(w["Wd"]), None, None, None, None, T, H, E, K, I, 0, 1, 0, E, 0, 0,
        p(b.topk_ids), p(b.topk_w), p(b.expert_offsets), p(b.src_of_row), p(b.row_of_pair), p(b.Xp), None, None, None, p(b.out),
        p(b.workspace_permute), b.workspace_permute.numel(), p(b.workspace), b.workspace.numel(), None, 0, 0.0, None,
        torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == -1     # MOE_ERR_NULL: no Yp
    for name in ("topk_ids", "expert_offsets", "src_of_row", "row_of_pair", "Xp"):
        assert torch.equal(getattr(b, name).view(torch.uint8), getattr(want, name).view(torch.uint8)), name
