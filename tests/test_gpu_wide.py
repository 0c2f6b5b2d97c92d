"""Batches of more than 32 tokens against the oracle: experts with one token, with 16 / 17 / 32 / 33 / many (several
blocks of 32), rows and contractions at the edges of the 512-column chunks and of the larger-batch kernels' items of 32 rows,
shared experts, bf16 output and accumulation, fewer items than workgroups.  (Items of 64 rows: test_gpu_wide_tall.py.)"""
import numpy as np
import pytest

from paper_2603_09983_amd import binding as B
from paper_2603_09983_amd import synth

pytestmark = pytest.mark.gpu

# (T, H, F, E, k, C, n_shared, F_shared)
CASES = [(33, 8, 8, 2, 1, 2, 0, 0), (64, 512, 512, 4, 2, 3, 0, 0), (40, 520, 504, 8, 3, 6, 1, 24), (100, 136, 40, 3, 3, 3, 0, 0),
         (257, 64, 72, 4, 2, 4, 2, 64), (47, 1024, 1032, 16, 1, 12, 0, 0), (128, 2056, 64, 8, 2, 8, 1, 2560), (65, 72, 2600, 4, 4, 2, 0, 0),
         (48, 256, 128, 64, 6, 0, 1, 136), (36, 128, 128, 300, 8, 200, 0, 0), (33, 4096, 64, 4, 1, 4, 0, 0)]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_wide(i):
    import gpu_util as G
    T, H, F, E, k, C, n, Fs = CASES[i]
    li = synth.make_layer(synth.small_recipe(f"wide{i}", 700 + i, T=T, H=H, F=F, E=E, k=k, C=C, n_shared=n, F_shared=Fs,
                                             hidden="unit", residency="all" if C >= E else "uniform"))
    print(f"[case] {CASES[i]}", flush=True)
    d = G.upload(li)
    ref = G.oracle.layer_from_inputs(li)
    buf = G.run_layer(d)
    G.run_layer(d, buf)   # again on the same workspace
    G.check_against_oracle(li, buf, ref, tag=str(CASES[i]), rms_over_nonzero_rows=True)
    buf = B.LayerBuffers.allocate(d.shape, out_bf16=True)
    buf.out.fill_(1.0)
    G.run_layer(d, buf, out_bf16=True, accumulate=True)
    y = buf.out.float().cpu().numpy() - 1.0
    # (1 + y rounded to bf16: half a unit in the last place of at most 1 + max|y|)
    assert np.max(np.abs(y - ref.y)) <= G.RTOL_RMS * G.rms(ref.y) + 2.0 ** -8 * (1 + np.max(np.abs(ref.y)))


@pytest.mark.parametrize("T,most", [(33, 32), (34, 32), (33, 33), (128, 32), (128, 33)])
def test_either_side_of_32_tokens_an_expert(T, most):
    """Widths of whole 64s: an expert with more than 32 tokens is several entries of the streaming kernels' list.  Column 0
    of the hidden states sends exactly `most` tokens to expert 0."""
    import gpu_util as G
    import torch
    E, k, H, F = 64, 2, 64, 128
    li = synth.make_layer(synth.small_recipe("either", 40, T=T, H=H, F=F, E=E, k=k, C=E, hidden="unit", residency="all"))
    # column 0 of the hidden states decides: +1 for the chosen tokens, -1 for the others, and only expert 0 looks at it
    li.router_w[:, 0] = 0.0
    li.router_w[0] = 0.0
    li.router_w[0, 0] = 100.0
    li.hidden[:, 0] = synth.f32_to_bf16_bits(np.where(np.arange(T) < most, 1.0, -1.0).astype(np.float32))
    ref = G.oracle.layer_from_inputs(li)
    assert ref.hist[0] == most and ref.hist[1:].max() <= 32
    print(f"[case] {T} tokens, {most} on one expert", flush=True)
    buf = G.run_layer(G.upload(li))
    G.check_against_oracle(li, buf, ref, tag=f"{T} {most}")
    assert torch.equal(G.run_layer(G.upload(li)).out, buf.out)
