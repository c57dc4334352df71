"""The launches without dedicated consumers (two launches without waits; small
tiles, or full tiles with smaller ones for the rest) against the CPU oracle,
and bitwise against the persistent kernel, which an explicit consumer count
always takes."""
import numpy as np
import pytest

from oracle import combine as oc
from workloads import custom, explicit

pytestmark = pytest.mark.gpu


def _edge_counts(counts, T, H, I, seed):
    """Workload whose expert e owns exactly counts[e] rows."""
    rng = np.random.default_rng(seed)
    sel = [[] for _ in range(T)]
    for e, c in enumerate(counts):
        for t in rng.choice(T, size=c, replace=False):
            sel[t].append(e)
    gates = [rng.random(len(s)).astype(np.float32) + 0.1 for s in sel]
    return explicit(T=T, H=H, I=I, E=len(counts), sel=sel, gates=gates, L=1, seed=seed)


CASES = {
    # 64 x 64 tiles: one token; a reduction of 40 (not a multiple of 16)
    "one_token": lambda: custom(T=1, H=2048, I=704, E=32, topk=6, L=2, seed=3),
    "k_tail": lambda: custom(T=19, H=264, I=40, E=5, topk=2, L=1, seed=4),
    # 64 x 128 tiles, deep ring (256..511 tiles) and shallow (512 and more)
    "deep_ring": lambda: custom(T=64, H=1024, I=72, E=32, topk=8, L=1, seed=5),
    "many_tiles": lambda: custom(T=128, H=2056, I=104, E=64, topk=4, L=1,
                                 routing=("zipf", 1.0), seed=6),
    # 128 x 256 tiles (32-deep stages, a reduction that ends inside one), and
    # with 128 x 128 ones for a last column block that is at most half full
    "wide": lambda: custom(T=515, H=8192, I=72, E=8, topk=2, L=2, seed=7),
    "wide_edges": lambda: _edge_counts([127, 128, 129, 255, 256, 257, 70], 300, 8456, 40, 24),
    "half_block": lambda: custom(T=520, H=4168, I=64, E=8, topk=2, L=1, seed=25),
    # more experts than a wave has lanes, most of them without rows
    "experts_200": lambda: custom(T=40, H=512, I=64, E=200, topk=3, L=1, seed=8),
    # expert row counts at the edges of the 64- and 128-row tiles, empty experts
    "edges_64": lambda: _edge_counts([63, 0, 64, 65, 1, 0, 33], 130, 520, 136, 9),
    "edges_128": lambda: _edge_counts([127, 128, 0, 129, 255, 256, 257, 1], 300, 2056, 24, 10),
    # more than two 256 x 256 tiles per CU: full tiles, with 256 x 128 edges and
    # 128 x 256 bottoms if the launch's plan has them (each plan: LARGE below);
    # rows past a full tile at the plan's limits (64, 128 and 192), empty experts
    "full_and_rest": lambda: _edge_counts([300] * 14, 400, 8320, 264, 21),
    "full_edges": lambda: _edge_counts([256, 257, 0, 255, 192, 193, 320, 321, 384, 385, 448, 449,
                                        64, 63, 1], 500, 8328, 40, 22),
    "full_100_experts": lambda: _edge_counts([20 + (37 * e) % 310 for e in range(100)], 600, 1096,
                                             72, 23),
    "full_rounds": lambda: _edge_counts([2000, 2060, 1, 1990, 2048], 2100, 4104, 24, 24),
    "topk_64": lambda: custom(T=70, H=256, I=32, E=64, topk=64, L=1, seed=11),
}


# the tiles each of them is meant to run as (checked on the CPU by test_launches.py)
TILES = {
    "one_token": "64x64", "k_tail": "64x64", "deep_ring": "64x128 deep", "many_tiles": "64x128",
    "wide": "128x256", "wide_edges": "128x256", "half_block": "128x256", "experts_200": "64x128 deep",
    "edges_64": "64x64", "edges_128": "128x128", "full_and_rest": "full", "full_edges": "full",
    "full_100_experts": "full", "full_rounds": "full", "topk_64": "64x128 deep",
}


def _bits(a):
    return np.ascontiguousarray(a).view(np.uint32)


@pytest.mark.parametrize("name", list(CASES))
def test_stage_matches_oracle_and_persistent_kernel(gpu_lib, name):
    import gpu_util
    w = CASES[name]()
    print(f"{name}: T={w.T} H={w.H} I={w.I} E={w.E} k={w.topk} rows={w.Mtot}", flush=True)
    ref = oc.combine_reference(w.x_perm, w.w2, w.expert_offsets, w.token_ids, w.gate_w, w.T)
    dev = gpu_util.to_device(w)
    got, _, ws = gpu_util.run(w, C=0, dev=dev)
    assert oc.rel_l2(got, ref) <= oc.REL_L2_TOL
    assert oc.max_abs_ratio(got, ref) <= oc.MAX_ABS_TOL
    # both paths in turn on one workspace (they share its epoch and counters)
    for C in (3, 0, -1, 3, -1, 0):
        again, _, ws = gpu_util.run(w, C=C, dev=dev, workspace=ws)
        assert np.array_equal(_bits(again), _bits(got)), C
    bands, _, _ = gpu_util.run(w, C=0, dev=dev, mode=2)
    assert np.array_equal(_bits(bands), _bits(got))


def test_small_batch_unsorted_rows_and_no_rows(gpu_lib):
    """Rows in any order inside an expert, tokens without rows, and a call
    whose experts hold no rows at all."""
    import torch

    import gpu_util
    from paper_2609_07536_amd import binding as B
    w = custom(T=90, H=512, I=96, E=6, topk=3, L=1, seed=12)
    rng = np.random.default_rng(1)
    for e in range(w.E):
        a, b = w.expert_offsets[e], w.expert_offsets[e + 1]
        p = a + rng.permutation(b - a)
        w.x_perm[a:b], w.token_ids[a:b] = w.x_perm[p], w.token_ids[p]
        w.gate_w[a:b] = w.gate_w[p]
    ref = oc.combine_reference(w.x_perm, w.w2, w.expert_offsets, w.token_ids, w.gate_w, w.T)
    dev = gpu_util.to_device(w)
    got, _, ws = gpu_util.run(w, C=0, dev=dev)
    assert oc.rel_l2(got, ref) <= oc.REL_L2_TOL
    persistent, _, _ = gpu_util.run(w, C=3, dev=dev, workspace=ws)
    assert np.array_equal(_bits(persistent), _bits(got))
    x, w2, off, tid, g = dev
    out = torch.full((w.T, w.H), float("nan"), device="cuda")
    B.combine(x, w2, torch.zeros_like(off), tid, g, T=w.T, topk=w.topk, num_consumers=0, out=out,
              workspace=ws)
    torch.cuda.synchronize()
    assert (out == 0).all()


@pytest.mark.parametrize("T,H,E", [(60, 520, 6), (2500, 4104, 5)], ids=["small", "full"])
def test_scatter_adds_rows_past_topk(gpu_lib, T, H, E):
    """Mode 1 without dedicated consumers adds every in-range row, also those
    past a token's topk, and flags nothing; two such tokens, several times on
    one workspace."""
    import gpu_util
    w = custom(T=T, H=H, I=40, E=E, topk=2, L=1, seed=14)
    w.token_ids = w.token_ids.copy()
    w.token_ids[::3] = 7          # one token owns a third of all rows
    w.token_ids[1::31] = T - 1
    ref = oc.combine_reference(w.x_perm, w.w2, w.expert_offsets, w.token_ids, w.gate_w, w.T)
    dev = gpu_util.to_device(w)
    ws = None
    for C in (0, -1, 3, 0):
        got, _, ws = gpu_util.run(w, C=C, dev=dev, workspace=ws, mode=1)
        assert oc.rel_l2(got, ref) <= oc.REL_L2_TOL, C
        assert oc.max_abs_ratio(got, ref) <= oc.MAX_ABS_TOL, C


# the up-projection: E, H, I, T, topk for each tile shape, edges of its rows
# and columns (2I = 96, 160, 1344 packed columns), a gather of repeated tokens
UP = {
    "one_token": (32, 2048, 704, 1, 6),
    "odd": (11, 1352, 336, 130, 3),
    "k_tail": (5, 264, 48, 40, 2),
    "deep_ring": (32, 520, 512, 64, 8),
    "many_tiles": (64, 264, 672, 128, 4),
    "tiles_128": (8, 136, 2048, 515, 2),
    "tiles_128_tail": (8, 136, 2064, 515, 2),
    "wide": (8, 136, 4096, 515, 2),
    "half_block": (8, 128, 4160, 515, 2),
    "wide_edge": (14, 264, 2112, 1400, 3),
    "experts_200": (200, 256, 80, 60, 3),
    # full tiles (with smaller ones for the rest: LARGE below)
    "full_no_edge": (10, 136, 1984, 2100, 4),
    "full_100_experts": (100, 64, 1072, 3000, 6),
}
UP_TILES = {
    "one_token": "64x64", "odd": "64x64", "k_tail": "64x64", "deep_ring": "64x128 deep",
    "many_tiles": "64x128", "tiles_128": "128x128", "tiles_128_tail": "128x128", "wide": "128x256",
    "half_block": "128x256", "wide_edge": "128x256", "experts_200": "64x128 deep",
    "full_no_edge": "full", "full_100_experts": "full",
}


@pytest.mark.parametrize("name", list(UP))
def test_up_projection_tiles(gpu_lib, name):
    """Against fp32 torch on the device: one bf16 rounding of the activation
    (2^-9 of its value) on top of fp32 sums of H products."""
    import torch

    import gpu_util
    from paper_2609_07536_amd import binding as B
    E, H, I, T, k = UP[name]
    print(f"{name}: E={E} H={H} I={I} T={T} k={k}", flush=True)
    w = custom(T=T, H=H, I=I, E=E, topk=k, L=1, routing=("zipf", 1.0), seed=13)
    _, _, off, tid, _ = gpu_util.to_device(w)
    gen = torch.Generator(device="cuda").manual_seed(1)
    hidden = torch.randn((T, H), generator=gen, device="cuda").bfloat16()
    w1 = (torch.randn((E, H, 2 * I), generator=gen, device="cuda") / H ** 0.5).bfloat16()
    got = B.gemm1_swiglu(hidden, B.pack_w1(w1), off, tid, k, w.Mtot)
    ref = torch.empty((w.Mtot, I), device="cuda")
    for e in range(E):
        a, b = int(w.expert_offsets[e]), int(w.expert_offsets[e + 1])
        h = hidden[tid[a:b].long()].float() @ w1[e].float()
        ref[a:b] = torch.nn.functional.silu(h[:, :I]) * h[:, I:]
    # fp32 sums of up to 2048 products of unit variance: about 1e-6 each way
    assert (got.float() - ref).abs().le(2 ** -8 * ref.abs() + 2e-4).all()


# Full tiles with smaller ones for the rest: E, columns, reduction, rows of
# expert e, and what the stage's plan has: rows past a full tile that are one
# themselves (255: all), and whether a narrow last column block has its own tiles.
LARGE = {
    "bottoms_192": (24, 2048, 1040, lambda e: 1100 + 37 * e % 60, 63, 0),
    "bottoms_128": (60, 2048, 1040, lambda e: 600 + 37 * e % 60, 127, 0),
    "whole": (60, 2048, 520, lambda e: 100 + 37 * e % 120, 255, 0),
    "edge_bottoms_192": (16, 2120, 520, lambda e: 1100 + 37 * e % 60, 63, 1),
    "edge_bottoms_128": (60, 1096, 1040, lambda e: 600 + 37 * e % 256, 127, 1),
    "edge": (60, 2120, 520, lambda e: 100 + 37 * e % 60, 255, 1),
    # many more smaller tiles than CUs: a workgroup takes several
    "many_bottoms": (300, 2048, 1040, lambda e: 30 + e % 31, 63, 0),
    "many_edges": (700, 264, 512, lambda e: 1 + 5 * e % 90, 255, 1),
    "many_both": (150, 1096, 1040, lambda e: 100 + 7 * e % 400, None, 1),
    "few_full": (270, 2304, 768, lambda e: 240 + e % 40 if e % 3 else 0, None, 0),
}
# the same of the up-projection, whose plan has other prices
UP_LARGE = {
    "bottoms_192": (24, 2048, 1040, lambda e: 300 + 37 * e % 256),
    "bottoms_128": (60, 2048, 1040, lambda e: 600 + 37 * e % 60),
    "whole": (40, 2048, 1040, lambda e: 100 + 37 * e % 256),
    "edge_bottoms_192": (16, 2112, 1040, lambda e: 1100 + 37 * e % 60),
    "edge_bottoms_128": (60, 1088, 1040, lambda e: 400 + 37 * e % 256),
    "edge": (60, 2112, 1040, lambda e: 100 + 37 * e % 60),
    "many_bottoms": (300, 2080, 2048, lambda e: 30 + e % 31),
    "many_edges": (700, 320, 512, lambda e: 1 + 5 * e % 90),
}


def _routing(E, rows_of, k=4):
    """Row counts, token count, offsets, tokens: every token has k rows at most."""
    import torch
    counts = np.array([rows_of(e) for e in range(E)])
    rows = int(counts.sum())
    T = -(-rows // k)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    rng = np.random.default_rng(5)
    tid = rng.permutation(np.repeat(np.arange(T), k)[:rows]).astype(np.int32)
    return rows, T, torch.from_numpy(off).cuda(), torch.from_numpy(tid).cuda()


def _left_plan(ws):
    """What the stage's GEMM left in the workspace: pad, edge, edges, bottoms."""
    at = ws.ptr - ws.tensor.data_ptr() + 352
    w = ws.tensor[at:at + 24].cpu().numpy().view(np.uint64) & 0xffffffff
    return int(w[0]) >> 1, int(w[0]) & 1, int(w[1]), int(w[2])


@pytest.mark.parametrize("name", list(LARGE))
def test_stage_full_tiles_with_smaller_ones(gpu_lib, name):
    """Bitwise against the persistent kernel (three consumers), several calls on
    one workspace; the plan is the one the case is for."""
    import torch

    from paper_2609_07536_amd import binding as B
    E, H, I, rows_of, pad, edge = LARGE[name]
    rows, T, off, tid = _routing(E, rows_of)
    print(f"{name}: E={E} H={H} I={I} T={T} rows={rows}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn((rows, I), generator=gen, device="cuda").bfloat16()
    w2 = torch.randn((E, I, H), generator=gen, device="cuda").bfloat16()
    gate = torch.rand(rows, generator=gen, device="cuda")
    wl, _ = B.make_workload(T, H, I, E, 4, 1, rows=rows)
    ws = B.Workspace(B.workspace_size(wl))
    out = torch.empty((T, H), device="cuda")

    def stage(C):
        out.fill_(float("nan"))
        B.combine(x, w2, off, tid, gate, T=T, topk=4, num_consumers=C, out=out, workspace=ws)
        return out.clone()

    ref = stage(3)
    for i in range(3):
        assert torch.equal(stage(0), ref), i
    plan = _left_plan(ws)
    print(f"plan: pad {plan[0]}, edge {plan[1]}, {plan[2]} edges, {plan[3]} bottoms", flush=True)
    assert plan[1] == edge and pad in (None, plan[0])
    assert torch.equal(stage(3), ref) and ws.status() == 0


@pytest.mark.parametrize("name", list(UP_LARGE))
def test_up_projection_full_tiles_with_smaller_ones(gpu_lib, name):
    """Against fp32 torch (the bound of test_up_projection_tiles), three calls."""
    import torch

    from paper_2609_07536_amd import binding as B
    E, N, H, rows_of = UP_LARGE[name]
    I = N // 2
    rows, T, off, tid = _routing(E, rows_of)
    print(f"{name}: E={E} H={H} I={I} T={T} rows={rows}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    hidden = torch.randn((T, H), generator=gen, device="cuda").bfloat16()
    w1 = (torch.randn((E, H, N), generator=gen, device="cuda") * H ** -0.5).bfloat16()
    packed, ref = B.pack_w1(w1), torch.empty((rows, I), device="cuda")
    bounds = off.tolist()
    for e in range(E):
        a, b = bounds[e], bounds[e + 1]
        h = hidden[tid[a:b].long()].float() @ w1[e].float()
        ref[a:b] = torch.nn.functional.silu(h[:, :I]) * h[:, I:]
    for i in range(3):
        got = B.gemm1_swiglu(hidden, packed, off, tid, 4, rows)
        assert (got.float() - ref).abs().le(2 ** -8 * ref.abs() + 2e-4).all(), i


def test_overlapping_expert_ranges_have_no_tiles(gpu_lib):
    """Decreasing offsets that give half of the experts all rows make a large
    batch's tiles many times those of the workload: the launch flags them and
    computes none of them (the workspace's Y keeps what it held); the next call
    on the workspace is right."""
    import torch

    from paper_2609_07536_amd import binding as B
    T, H, I, E, k = 4096, 2048, 64, 32, 8
    rows, gen = T * k, torch.Generator(device="cuda").manual_seed(6)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda").bfloat16()

    x, w2, gate = normal(rows, I), normal(E, I, H), torch.rand(rows, generator=gen, device="cuda")
    tid = torch.arange(T, device="cuda", dtype=torch.int32).repeat(k)
    off = torch.arange(E + 1, device="cuda", dtype=torch.int32) * (rows // E)
    bad = torch.tensor([0, rows] * (E // 2) + [rows], device="cuda", dtype=torch.int32)
    wl, _ = B.make_workload(T, H, I, E, k, 1, rows=rows)
    ws = B.Workspace(B.workspace_size(wl))
    out = torch.empty((T, H), device="cuda")

    def stage(offsets, C):
        B.combine(x, w2, offsets, tid, gate, T=T, topk=k, num_consumers=C, out=out, workspace=ws)
        return out.clone()

    ref = stage(off, 3)
    y = ws.tensor[ws.nbytes // 2:ws.nbytes - 256]   # Y is the workspace's last and largest part
    y.fill_(0x11)
    stage(bad, 0)
    assert ws.status(clear=True) == B.MOE_ERR_BAD_ROUTING
    assert bool((y == 0x11).all())
    assert torch.equal(stage(off, 0), ref) and ws.status() == 0
