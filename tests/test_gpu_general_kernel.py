"""The general FFN kernel: it runs where a caller's workspace holds its partial sums but not the regions of the faster kernels.
Both token tilings, whole 32s and multiples of 8 only, its pipelined and its plain loops, slices that end early, several passes
over a list, against the oracle; and one byte less than its layout is refused."""
import pytest
import torch

from paper_2603_09983_amd import binding as B
from paper_2603_09983_amd import synth

pytestmark = pytest.mark.gpu


def _layout_bytes(T, H, F, k, C, n, Fs):
    """Control block, stamped logits and ids, the lists, then 4 bytes for each slice of 128, assignment and column."""
    a256, sl = lambda x: (x + 255) // 256 * 256, lambda f: (f + 127) // 128
    A = T * k
    return (256 + 65536 * 8 + 4096 * 8 + 2 * a256(A * 4) + 2 * a256(max(C, 1) * 4) + a256((C + 1) * 4) + a256(sl(F) * A * H * 4) +
            a256(n * sl(Fs) * T * H * 4))


# (T, H, F, E, k, C, n_shared, F_shared)
CASES = [(9, 512, 160, 8, 2, 8, 0, 0), (20, 512, 160, 8, 3, 6, 1, 96), (1, 96, 96, 4, 2, 3, 1, 32), (32, 1000, 120, 64, 8, 6, 0, 0),
         (5, 72, 1000, 8, 2, 8, 0, 0), (17, 40, 520, 8, 4, 5, 2, 264), (12, 2048, 96, 8, 2, 8, 0, 0), (60, 136, 104, 4, 2, 3, 0, 0),
         (200, 96, 96, 4, 2, 4, 1, 96), (31, 4960, 8, 4, 1, 4, 0, 0)]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_general_kernel(i):
    import gpu_util as G
    T, H, F, E, k, C, n, Fs = CASES[i]
    li = synth.make_layer(synth.small_recipe(f"general{i}", 4000 + i, T=T, H=H, F=F, E=E, k=k, C=C, n_shared=n, F_shared=Fs, hidden="unit",
                                             residency="all" if C >= E else "uniform"))
    d = G.upload(li)
    buf = B.LayerBuffers.allocate(d.shape)
    size = _layout_bytes(T, H, F, k, C, n, Fs)
    assert size < buf.workspace.numel()
    args = (d.hidden, d.router_w, d.router_bias, d.slot_table, d.w_gate, d.w_up, d.w_down, d.sh_gate, d.sh_up, d.sh_down,
            buf.topk_idx, buf.topk_w, buf.hist, buf.slot_idx, buf.miss_list, buf.miss_count, buf.out, False, False)
    few = torch.empty(size - 16, dtype=torch.uint8, device="cuda")
    B.moe_workspace_init(few)
    assert B.moe_verify_layer(d.shape, *args, few, check=False) == B.ERR_WORKSPACE
    buf.workspace = torch.empty(size, dtype=torch.uint8, device="cuda")
    B.moe_workspace_init(buf.workspace)
    print(f"[case] {CASES[i]}", flush=True)
    B.moe_profile_enable(True)
    B.moe_verify_layer(d.shape, *args, buf.workspace)
    torch.cuda.synchronize()
    B.moe_profile_enable(False)
    assert B.moe_profile_read(B.KERNEL_DOWN)[1] == 0 and B.moe_profile_read(B.KERNEL_FFN)[1] == 1   # no down launch: it was the general kernel
    B.moe_verify_layer(d.shape, *args, buf.workspace)
    B.moe_workspace_status(buf.workspace)
    G.check_against_oracle(li, buf, tag=str(CASES[i]), rms_over_nonzero_rows=True)
