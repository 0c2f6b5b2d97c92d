"""Calls whose workspace regions lie at the same offsets but hold another kind of entry (plain floats from the larger-batch
kernels, (call number, value) words from the streaming kernels' final sum): the second one is reported, as a call with
another layout is, and served after a new initialisation."""
import pytest
import torch

from paper_2603_09983_amd import binding as B

pytestmark = pytest.mark.gpu

H, F, E, C = 2112, 2048, 8, 3   # 78 MB of weights: 17 to 32 tokens take the larger-batch kernels


def _call(T, k, form, ws, wts, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    shape = B.make_shape(T, H, E, k, F, C)
    buf = B.LayerBuffers.allocate(shape)
    if ws is not None:
        buf.workspace = ws
    x = torch.randn(T, H, device="cuda", generator=g).bfloat16()
    router = torch.randn(E, H, device="cuda", generator=g) * 0.02
    table = torch.tensor([0, -1, 1, -1, 2, -1, -1, -1], dtype=torch.int32, device="cuda")
    B.moe_verify_layer(B.with_form(shape, form), x, router, None, table, *wts, None, None, None, buf.topk_idx, buf.topk_w, buf.hist,
                       buf.slot_idx, buf.miss_list, buf.miss_count, buf.out, False, False, buf.workspace)
    torch.cuda.synchronize()
    return buf


@pytest.mark.parametrize("first,second", [((32, 1, B.LAUNCH_AUTO), (16, 2, B.LAUNCH_AUTO)), ((16, 2, B.LAUNCH_AUTO), (32, 1, B.LAUNCH_AUTO)),
                                          ((24, 2, B.LAUNCH_AUTO), (24, 2, B.LAUNCH_THREE)), ((24, 2, B.LAUNCH_TWO), (24, 2, B.LAUNCH_AUTO))])
def test_other_entries_at_the_same_offsets(first, second):
    g = torch.Generator(device="cuda").manual_seed(3)
    n = lambda *s: (torch.randn(*s, device="cuda", generator=g) * 0.02).bfloat16()
    wts = n(C, F, H), n(C, F, H), n(C, H, F)
    print(f"[case] {first} {second}", flush=True)
    a = _call(*first, None, wts, 1)
    assert B.moe_workspace_status(a.workspace, check=False) == B.OK
    want = _call(*second, None, wts, 2)
    assert want.workspace.numel() == a.workspace.numel()
    got = _call(*second, a.workspace, wts, 2)
    assert B.moe_workspace_status(a.workspace, check=False) == B.ERR_WORKSPACE
    assert int(got.miss_count.cpu()[0]) == -1 and bool(torch.isnan(got.out).all())
    B.moe_workspace_init(a.workspace)
    got = _call(*second, a.workspace, wts, 2)
    assert B.moe_workspace_status(a.workspace, check=False) == B.OK
    assert torch.equal(got.out, want.out) and torch.equal(got.miss_count, want.miss_count)
