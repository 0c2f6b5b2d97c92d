"""Batches of more than 32 tokens in the streaming kernels (contractions of up to 2048 columns in whole 64s): an expert's
list is one entry of the item list for each 32 tokens.  Lists on both sides of whole blocks, shared experts (all tokens) of
another width, one slot, many slots; and a caller's own lists in which a token names a slot several times."""
import numpy as np
import pytest
import torch

from paper_2603_09983_amd import binding as B
from paper_2603_09983_amd import synth

pytestmark = pytest.mark.gpu

# (T, H, F, E, k, C, n_shared, F_shared, tokens on expert 0)
CASES = [(33, 64, 64, 8, 2, 8, 1, 64, 33), (64, 128, 192, 8, 2, 8, 2, 320, 64), (65, 2048, 64, 8, 2, 8, 1, 2048, 65),
         (100, 64, 1984, 70, 2, 70, 0, 0, 96), (100, 64, 128, 70, 2, 70, 3, 64, 97), (40, 256, 64, 1, 1, 1, 0, 0, 40),
         (128, 64, 64, 300, 3, 290, 1, 64, 31), (200, 192, 128, 16, 2, 5, 0, 0, 161), (36, 64, 64, 16, 2, 0, 2, 128, 3)]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_blocks(i):
    import gpu_util as G
    T, H, F, E, k, C, n, Fs, on0 = CASES[i]
    li = synth.make_layer(synth.small_recipe(f"large{i}", 500 + i, T=T, H=H, F=F, E=E, k=k, C=C, n_shared=n, F_shared=Fs,
                                             hidden="unit", residency="all" if C >= E else "uniform"))
    # column 0 of the hidden states decides who goes to expert 0: +1 for the first `on0` tokens, -1 for the others
    li.router_w[:, 0] = 0.0
    li.router_w[0] = 0.0
    li.router_w[0, 0] = 100.0
    li.hidden[:, 0] = synth.f32_to_bf16_bits(np.where(np.arange(T) < on0, 1.0, -1.0).astype(np.float32))
    print(f"[case] {CASES[i]}", flush=True)
    ref = G.oracle.layer_from_inputs(li)
    assert E == 1 or ref.hist[0] == on0
    d = G.upload(li)
    buf = G.run_layer(d)
    G.run_layer(d, buf)   # again on the same workspace
    G.check_against_oracle(li, buf, ref, tag=str(CASES[i]), rms_over_nonzero_rows=True)


@pytest.mark.parametrize("T,k,C", [(33, 4, 3), (40, 6, 1), (64, 8, 40)])
def test_a_token_that_names_a_slot_several_times(T, k, C):
    H, F = 128, 192
    g = torch.Generator(device="cuda").manual_seed(T + C)
    n = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).bfloat16()
    x, wg, wu, wd = n(T, H), n(C, F, H, std=0.1), n(C, F, H, std=0.1), n(C, H, F, std=0.1)
    w = torch.rand(T, k, device="cuda", generator=g)
    slot = torch.randint(-1, C, (T, k), device="cuda", generator=g).int()
    slot[: T // 2] = C - 1   # half of the tokens name the last slot k times: a list of more than T entries
    out = torch.empty(T, H, device="cuda")
    ws = B.new_workspace(B.make_shape(T, H, max(C, k), k, F, C))
    print(f"[case] repeated {T} {k} {C}", flush=True)
    B.moe_grouped_ffn(x, w, slot, wg, wu, wd, T, H, F, k, C, out, False, False, ws)
    B.moe_workspace_status(ws)
    ref = torch.zeros(T, H, dtype=torch.float64, device="cuda")
    for c in range(C):
        t, j = (slot == c).nonzero(as_tuple=True)
        a = x[t].double() @ wg[c].double().T
        y = (a * torch.sigmoid(a) * (x[t].double() @ wu[c].double().T)) @ wd[c].double().T
        ref.index_add_(0, t, w[t, j, None].double() * y)
    # (activations rounded to bf16: 2^-9 of each, as many of one sign as a token names its slot; a wrong entry is off by about rms)
    assert (out.double() - ref).abs().max() <= 2e-2 * max(ref.square().mean().sqrt(), ref.abs().max() * 0.25)
