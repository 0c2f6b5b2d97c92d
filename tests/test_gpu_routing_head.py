"""The routing steps where their paths meet: rows of the router that are not whole 2048s (dot products), 64 and 128 experts
(ranking), 64 and 1024 assignments, 64 slots, and scratch memory that does or does not reach the lists' place (lists)."""
import numpy as np
import pytest

from paper_2603_09983_amd import synth

pytestmark = pytest.mark.gpu

CASES = [  # T, k, E, C, H
    (1, 1, 1, 1, 8), (13, 5, 70, 64, 256), (16, 64, 128, 64, 64), (32, 32, 128, 64, 64), (32, 8, 64, 63, 264),
    (9, 8, 128, 64, 1408), (4, 6, 64, 64, 2040), (17, 6, 65, 65, 2056), (3, 2, 9, 9, 4104), (33, 4, 64, 20, 520),
    (70, 3, 64, 40, 2040), (129, 2, 64, 33, 72), (17, 6, 64, 48, 256), (19, 16, 64, 64, 64), (31, 17, 64, 64, 64), (50, 16, 33, 10, 64),
    (18, 7, 7, 7, 128)]


@pytest.mark.parametrize("T,k,E,C,H", CASES)
def test_layer(T, k, E, C, H):
    """Two layers of one shape after one another on one workspace, every output overwritten in between: neither an output nor a list
    in the workspace that the second call fails to write can pass for its own."""
    import gpu_util as G
    print(f"[case] {T} {k} {E} {C} {H}", flush=True)
    buf = None
    for seed in (70 + T + k, 700 + T + k):
        li = synth.make_layer(synth.small_recipe("head", seed, T=T, H=H, F=64, E=E, k=k, C=C, hidden="unit"), margin=1e-5)
        if buf is not None:
            for x in (buf.topk_idx, buf.hist, buf.slot_idx, buf.miss_list, buf.miss_count):
                x.fill_(-77)
            for x in (buf.topk_w, buf.out):
                x.fill_(float("nan"))
        buf = G.run_layer(G.upload(li), buf)
        G.check_against_oracle(li, buf, tag=f"{T} {k} {E} {C} {H} seed {seed}", rms_over_nonzero_rows=True)


@pytest.mark.parametrize("T,H,E", [(1, 8, 5), (5, 264, 64), (70, 2040, 64), (129, 2056, 64), (257, 2048, 130), (513, 4104, 64), (193, 1032, 64), (192, 264, 65),
                                   (3073, 8, 5)])
def test_logits(T, H, E):
    import torch
    from paper_2603_09983_amd import binding as B
    print(f"[case] {T} {H} {E}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(T + H)
    x = torch.randn(T, H, device="cuda", generator=g).bfloat16()
    w = torch.randn(E, H, device="cuda", generator=g) * 0.02
    bias = torch.randn(E, device="cuda", generator=g)
    idx = torch.zeros(T, 2, dtype=torch.int32, device="cuda")
    gate, logits = torch.zeros(T, 2, device="cuda"), torch.zeros(T, E, device="cuda")
    ws = B.new_workspace(B.make_shape(T, H, E, 2, 64, 0))
    B.moe_route_topk(x, w, bias, T, H, E, 2, idx, gate, logits, ws)
    ref = x.double() @ w.double().T + bias.double()
    # a lane adds H / 256 + 1 terms of four products, six more additions over the wavefront, one of the bias: so many roundings
    # of at most the sum of the magnitudes
    bound = (x.double().abs() @ w.double().abs().T + bias.double().abs()) * (H / 256 + 13) * 2.0 ** -24
    assert bool(((logits.double() - ref).abs() <= bound).all())
    assert torch.equal(idx.long(), logits.topk(2, dim=1).indices)


@pytest.mark.parametrize("T", [9, 18, 50])
def test_ties_over_rows_of_lanes(T):
    """Experts with the same router row tie exactly, within a row of lanes and between rows: the lower id comes first."""
    import torch
    from paper_2603_09983_amd import binding as B
    print(f"[case] {T}", flush=True)
    E, H, k, F, C = 64, 64, 12, 64, 8
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    w = (torch.randn(8, H, device="cuda", generator=g) * 0.02)[torch.randint(0, 8, (E,), generator=g, device="cuda")].contiguous()
    x = torch.randn(T, H, device="cuda", generator=g).bfloat16()
    table = torch.full((E,), -1, dtype=torch.int32, device="cuda")
    sh = B.make_shape(T, H, E, k, F, C)
    buf = B.LayerBuffers.allocate(sh)
    pools = [torch.zeros(C, F, H, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    B.moe_verify_layer(sh, x, w, None, table, *pools, None, None, None, buf.topk_idx, buf.topk_w, buf.hist, buf.slot_idx,
                       buf.miss_list, buf.miss_count, buf.out, False, False, buf.workspace)
    s = (x.double() @ w.double().T).cpu().numpy()
    want = np.argsort(-s.round(9), axis=1, kind="stable")[:, :k]   # (equal rows give equal sums; stable: the lower id first)
    assert np.array_equal(buf.topk_idx.cpu().numpy(), want)


@pytest.mark.parametrize("T,E", [(9, 40), (9, 96), (24, 40), (24, 96), (50, 64), (50, 96)])
def test_nan_and_infinite_logits(T, E):
    """A NaN logit ranks as minus infinity, ties to the lower id: in the gate/up launch (one token to a wavefront up to 16, four or
    two beyond) and in the routing kernel."""
    import gpu_util as G
    import oracle
    import torch
    from paper_2603_09983_amd import binding as B
    print(f"[case] {T} {E}", flush=True)
    H, k, F, C = 64, 8, 64, 8
    rng = np.random.default_rng(T + E)
    order = rng.permutation(E).astype(np.float32)
    bias = np.zeros(E, dtype=np.float32)
    bad = rng.choice(E, E - 5, replace=False)   # five finite logits are left, k = 8
    bias[bad] = np.where(rng.random(bad.size) < 0.5, np.nan, -np.inf)
    router = np.zeros((E, H), dtype=np.float32)
    router[:, 0] = order
    x = torch.zeros(T, H, dtype=torch.bfloat16, device="cuda")
    x[:, 0] = 1.0
    sh = B.make_shape(T, H, E, k, F, C)
    buf = B.LayerBuffers.allocate(sh)
    table = torch.full((E,), -1, dtype=torch.int32, device="cuda")
    pools = [torch.zeros(C, F, H, dtype=torch.bfloat16, device="cuda") for _ in range(3)]
    B.moe_verify_layer(sh, x, torch.from_numpy(router).cuda(), torch.from_numpy(bias).cuda(), table, *pools, None, None, None,
                       buf.topk_idx, buf.topk_w, buf.hist, buf.slot_idx, buf.miss_list, buf.miss_count, buf.out, False, False,
                       buf.workspace)
    want, gate = oracle.topk_gate(np.tile(np.where(np.isnan(bias), -np.inf, order + bias).astype(np.float64), (T, 1)), k)
    assert np.array_equal(buf.topk_idx.cpu().numpy(), want) and list(want[0][5:]) == sorted(bad)[:3]
    w = buf.topk_w.cpu().numpy()
    assert np.max(np.abs(w - gate)) <= G.GATE_ATOL and np.all(w[:, 5:] == 0.0)
