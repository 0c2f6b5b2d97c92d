"""The larger-batch kernels in the forms that full sizes run: items of 64 rows, several chunks of 512 columns to an item,
several items to a workgroup, lists of more than 32 tokens; and the line from 17 to 32 tokens at which wide matrices go to them
(64 MB of weights, contractions beyond 2048).  Against 64-bit sums, or the oracle where there are shared experts."""
import pytest
import torch

from paper_2603_09983_amd import binding as B
from paper_2603_09983_amd import synth

pytestmark = pytest.mark.gpu


def _ffn_case(T, H, F, k, C, on0=None):
    g = torch.Generator(device="cuda").manual_seed(T + H + F)
    n = lambda *s, std: (torch.randn(*s, device="cuda", generator=g) * std).bfloat16()
    wts = n(C, F, H, std=2.0 * H ** -0.5), n(C, F, H, std=2.0 * H ** -0.5), n(C, H, F, std=F ** -0.5)
    x, w = n(T, H, std=1.0), torch.rand(T, k, device="cuda", generator=g)
    slot = torch.rand(T, C, device="cuda", generator=g).argsort(1)[:, :k]
    if on0 is not None:   # slot 0 for the first tokens only
        slot = torch.rand(T, C - 1, device="cuda", generator=g).argsort(1)[:, :k] + 1
        slot[:on0, 0] = 0
    slot = torch.where(torch.rand(T, k, device="cuda", generator=g) < 0.1, -1, slot).int().contiguous()
    out = torch.empty(T, H, device="cuda")
    ws = B.new_workspace(B.make_shape(T, H, max(C, k), k, F, C))
    print(f"[case] {T} {H} {F} {k} {C} {on0}", flush=True)
    for _ in range(2):
        B.moe_grouped_ffn(x, w, slot, *wts, T, H, F, k, C, out, False, False, ws)
    B.moe_workspace_status(ws)
    ref = torch.zeros(T, H, dtype=torch.float64, device="cuda")
    for c in range(C):
        t, j = (slot == c).nonzero(as_tuple=True)
        if t.numel():
            a = x[t].double() @ wts[0][c].double().T
            y = (a * torch.sigmoid(a) * (x[t].double() @ wts[1][c].double().T)) @ wts[2][c].double().T
            ref.index_add_(0, t, w[t, j, None].double() * y)
    # (activations rounded to bf16: 2^-9 of each; a chunk or an item out of place is off by about rms)
    assert (out.double() - ref).abs().max() <= 2e-2 * max(ref.square().mean().sqrt(), ref.abs().max() * 0.25)


# chunks of 512 columns to an item: 3 (with a remainder of 8 and 24) | 6 and 3 | 2 and 5, from a chunk of the row's own
@pytest.mark.parametrize("T,H,F,k,C,on0", [(40, 1032, 1048, 8, 64, None), (64, 1032, 1048, 6, 64, 33), (80, 2600, 1096, 4, 24, 64),
                                           (130, 1000, 2312, 4, 40, 97), (200, 2056, 2056, 4, 16, None)])
def test_tall_items(T, H, F, k, C, on0):
    _ffn_case(T, H, F, k, C, on0)


# 6 H F C bytes of weights: 65 and 78 MB around the line, H or F beyond 2048 or neither, widths of 64s and of 8s
@pytest.mark.parametrize("T", [16, 17, 32])
@pytest.mark.parametrize("H,F,C", [(2112, 1024, 5), (2112, 1024, 6), (512, 4160, 5), (512, 4160, 6), (2056, 1048, 6), (1048, 2056, 6), (2048, 1024, 6)])
def test_either_side_of_the_line_from_17_to_32_tokens(T, H, F, C):
    _ffn_case(T, H, F, 3, C)


@pytest.mark.parametrize("T,H,F,C,n,Fs", [(17, 2112, 256, 8, 2, 2048), (32, 2112, 1024, 6, 1, 512), (24, 2056, 1000, 6, 1, 2568), (24, 256, 128, 8, 1, 45000)])
def test_shared_experts_from_17_to_32_tokens(T, H, F, C, n, Fs):
    import gpu_util as G
    assert 6 * H * (C * F + n * Fs) >= 64 << 20
    li = synth.make_layer(synth.small_recipe("line", 1500 + T + H, T=T, H=H, F=F, E=8, k=2, C=C, n_shared=n, F_shared=Fs, hidden="unit",
                                             residency="all" if C >= 8 else "uniform"))
    print(f"[case] {T} {H} {F} {C} {n} {Fs}", flush=True)
    d = G.upload(li)
    buf = G.run_layer(d)
    G.run_layer(d, buf)
    G.check_against_oracle(li, buf, tag=f"{T} {H} {F}", rms_over_nonzero_rows=True)
