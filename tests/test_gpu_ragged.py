"""Widths that are multiples of 8 only, in batches the streaming kernels take (up to 32 tokens), against the oracle: one
and several contraction panels, the last of which begins inside the one before; a last tile of 8 rows; pieces that
end inside a half tile; routed and shared experts of different widths; widths of 64 times a prime."""
import numpy as np
import pytest
import torch

from paper_2603_09983_amd import binding as B
from paper_2603_09983_amd import synth

pytestmark = pytest.mark.gpu

# (T, H, F, E, k, C, n_shared, F_shared)
CASES = [(1, 8, 8, 4, 2, 3, 0, 0), (5, 24, 40, 8, 2, 8, 1, 16), (7, 136, 1032, 8, 2, 6, 0, 0), (9, 2056, 72, 6, 3, 6, 1, 64),
         (16, 72, 2056, 6, 2, 5, 0, 0), (3, 4104, 24, 4, 2, 4, 0, 0), (17, 200, 1000, 16, 4, 12, 2, 120),
         (32, 328, 328, 16, 8, 16, 1, 2600), (31, 2040, 88, 8, 3, 7, 0, 0), (24, 64, 4072, 8, 2, 8, 1, 64),
         (4, 2368, 64, 4, 2, 4, 1, 2368), (20, 64, 2368, 8, 2, 8, 1, 200), (32, 8, 64, 64, 8, 40, 0, 0), (6, 1024, 1016, 130, 6, 9, 1, 512)]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_ragged(i):
    import gpu_util as G
    T, H, F, E, k, C, n, Fs = CASES[i]
    li = synth.make_layer(synth.small_recipe(f"ragged{i}", 300 + i, T=T, H=H, F=F, E=E, k=k, C=C, n_shared=n, F_shared=Fs,
                                             hidden="unit", residency="all"))
    print(f"[case] {CASES[i]}", flush=True)
    d = G.upload(li)
    ref = G.oracle.layer_from_inputs(li)
    G.check_against_oracle(li, G.run_layer(d), ref, tag=str(CASES[i]), rms_over_nonzero_rows=True)
    # the routing kernel and the same FFN launches, by name; a second call on the same workspace
    buf = G.run_layer(d, form=B.LAUNCH_THREE)
    G.run_layer(d, buf, form=B.LAUNCH_THREE)
    G.check_against_oracle(li, buf, ref, tag=str(CASES[i]), rms_over_nonzero_rows=True)
    buf = B.LayerBuffers.allocate(d.shape, out_bf16=True)   # added to a previous result, in bf16
    buf.out.fill_(1.0)
    G.run_layer(d, buf, out_bf16=True, accumulate=True)
    y = buf.out.float().cpu().numpy() - 1.0
    # (1 + y rounded to bf16: half a unit in the last place of at most 1 + max|y|)
    assert np.max(np.abs(y - ref.y)) <= G.RTOL_RMS * G.rms(ref.y) + 2.0 ** -8 * (1 + np.max(np.abs(ref.y)))
    with pytest.raises(B.MoeError):   # the two-launch form by name stays for widths of whole 64s
        if H % 64 or F % 64 or Fs % 64:
            G.run_layer(d, form=B.LAUNCH_TWO)
        else:
            raise B.MoeError(B.ERR_SHAPE, "")


@pytest.mark.parametrize("F", [72, 2056])
def test_an_infinite_weight_stays_in_its_own_row(F):
    """The columns past a row's end (in the tile buffer: the next row's first ones) and those that two panels share
    must not reach the row's result."""
    import gpu_util as G
    li = synth.make_layer(synth.small_recipe("inf", 77, T=4, H=72, F=F, E=4, k=2, C=4, hidden="unit", residency="all"))
    ref = G.run_layer(G.upload(li)).out.cpu()
    li.w_down[:, 33, 0] = 0x7F80      # +inf in row 33, first column
    li.w_down[:, 50, F - 1] = 0x7F80  # ... and row 50, last column
    out = G.run_layer(G.upload(li)).out.cpu()
    rest = [h for h in range(72) if h not in (33, 50)]
    assert torch.equal(out[:, rest], ref[:, rest]) and not torch.isfinite(out[:, [33, 50]]).any()
    li.w_down[:, 50, F - 2056 if F > 2048 else 0] = 0x7F80
    out = G.run_layer(G.upload(li)).out.cpu()
    assert torch.equal(out[:, rest], ref[:, rest])


def test_static_call_where_only_the_general_layout_fits():
    """32 tokens x 64 experts each, F = 120: the streaming kernels' regions exceed the library's static array, the general
    kernel's do not.  The call was always accepted and has to stay so."""
    import gpu_util as G
    T, H, F, E, k, C = 32, 1000, 120, 64, 64, 6
    li = synth.make_layer(synth.small_recipe("static", 91, T=T, H=H, F=F, E=E, k=k, C=C, hidden="unit"), margin=0.0)
    d = G.upload(li)
    buf = B.LayerBuffers.allocate(d.shape)
    print("[case] static, general layout", flush=True)
    args = (d.hidden, d.router_w, d.router_bias, d.slot_table, d.w_gate, d.w_up, d.w_down, d.sh_gate, d.sh_up, d.sh_down,
            buf.topk_idx, buf.topk_w, buf.hist, buf.slot_idx, buf.miss_list, buf.miss_count, buf.out, False, False)
    B.moe_verify_layer_static(d.shape, *args)
    torch.cuda.synchronize()
    own, small = buf.out.clone(), torch.empty(10 << 20, dtype=torch.uint8, device="cuda")
    B.moe_workspace_init(small)   # a workspace of the general layout's size does too
    B.moe_verify_layer(d.shape, *args, small)
    assert torch.equal(own, buf.out)
    ref = G.run_layer(d).out
    assert (own - ref).abs().max() <= G.RTOL_RMS * ref.square().mean().sqrt()
