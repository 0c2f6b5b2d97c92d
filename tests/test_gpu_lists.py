"""The per-slot lists of larger batches (one assignment per thread and block of 1024, several blocks, ids beyond the
LDS copy) against plain torch: slot lookup and miss list bit-exact, and the lists through the expert FFN that reads
them.  The FFN of a list entry that is lost, doubled or out of place is wrong by the whole entry."""
import pytest
import torch

from paper_2603_09983_amd import binding as B

pytestmark = pytest.mark.gpu


# edges: one wavefront, a block of 1024 and one more, several blocks, past the 4096 ids kept in LDS; 1 slot, 1024 slots
@pytest.mark.parametrize("T,k,E,C", [(1, 1, 1, 1), (16, 4, 9, 3), (13, 5, 40, 33), (128, 8, 128, 64), (205, 5, 64, 64),
                                     (512, 8, 512, 1024), (700, 6, 100, 65), (4097, 1, 8, 5), (1500, 5, 60, 17)])
def test_resolve(T, k, E, C):
    g = torch.Generator().manual_seed(T * 31 + C)
    idx = torch.stack([torch.randperm(E, generator=g)[:k] for _ in range(T)]).int()
    tab = torch.full((E,), -1, dtype=torch.int32)
    n = min(E, C) - (min(E, C) > 2)
    tab[torch.randperm(E, generator=g)[:n]] = torch.randperm(C, generator=g)[:n].int()
    if n > 1:
        tab[(tab < 0).nonzero()[:1]] = C   # out of range: not resident
    i32 = dict(dtype=torch.int32, device="cuda")
    slot, miss, cnt = torch.empty(T, k, **i32), torch.zeros(T * k, **i32), torch.empty(1, **i32)
    ws = B.new_workspace(B.make_shape(T, 64, E, k, 64, C))
    print(f"[case] resolve {T} {k} {E} {C}", flush=True)
    B.moe_slot_resolve(idx.cuda(), tab.cuda(), T, k, E, C, slot, miss, cnt, ws)
    ref = tab[idx.long()]
    ref = torch.where((ref < 0) | (ref >= C), -1, ref)
    m = (ref.flatten() < 0).nonzero().flatten().int()
    assert torch.equal(slot.cpu(), ref)
    assert int(cnt.cpu()) == m.numel() and torch.equal(miss.cpu()[:m.numel()], m)


@pytest.mark.parametrize("T,k,C,kind", [(9, 6, 8, "distinct"), (300, 4, 7, "distinct"), (1100, 4, 3, "repeated"),
                                        (300, 6, 40, "one_slot"), (70, 2, 600, "sparse")])
def test_lists_through_the_ffn(T, k, C, kind):
    H, F = 64, 64
    g = torch.Generator(device="cuda").manual_seed(T + C)
    n = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).bfloat16()
    x, wg, wu, wd = n(T, H), n(C, F, H, std=0.1), n(C, F, H, std=0.1), n(C, H, F, std=0.1)
    w = torch.rand(T, k, device="cuda", generator=g)
    if kind == "one_slot":
        slot = torch.full((T, k), -1, device="cuda")
        slot[:, 0] = C - 1
    elif kind == "repeated":   # a caller's own ids: a token may name a slot twice, ids outside [0,C) count as missed
        slot = torch.randint(-2, C + 2, (T, k), device="cuda", generator=g)
    else:
        slot = torch.rand(T, C, device="cuda", generator=g).argsort(1)[:, :k]
        slot = torch.where(torch.rand(T, k, device="cuda", generator=g) < 0.3, -1, slot)
    slot = slot.int().contiguous()
    out = torch.empty(T, H, device="cuda")
    ws = B.new_workspace(B.make_shape(T, H, max(C, k), k, F, C))
    print(f"[case] lists {T} {k} {C} {kind}", flush=True)
    B.moe_grouped_ffn(x, w, slot, wg, wu, wd, T, H, F, k, C, out, False, False, ws)
    B.moe_workspace_status(ws)
    ref = torch.zeros(T, H, dtype=torch.float64, device="cuda")
    for c in range(C):
        t, j = (slot == c).nonzero(as_tuple=True)
        if t.numel():
            a = x[t].double() @ wg[c].double().T
            y = (a * torch.sigmoid(a) * (x[t].double() @ wu[c].double().T)) @ wd[c].double().T
            ref.index_add_(0, t, w[t, j, None].double() * y)
    rms = ref.square().mean().sqrt()
    # (activations rounded to bf16: 2^-9 of each; a wrong list entry is off by about rms)
    assert (out.double() - ref).abs().max() <= 2e-2 * max(rms, ref.abs().max() * 0.25)
