"""The per-slot lists that the routing steps inside the gate/up launch build: by one wavefront up to 64 assignments and
64 slots, by the workgroup beyond; both sides of each limit against the oracle."""
import pytest

from paper_2603_09983_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,C", [(1, 1, 1), (16, 4, 64), (16, 4, 65), (13, 5, 64), (32, 2, 64), (32, 2, 65), (8, 8, 33), (1, 64, 64)])
def test_lists(T, k, C):
    import gpu_util as G
    li = synth.make_layer(synth.small_recipe("lists", 60 + T + C, T=T, H=64, F=64, E=70, k=k, C=C, n_shared=T % 2, F_shared=64,
                                             hidden="unit"), margin=1e-5)
    print(f"[case] {T} {k} {C}", flush=True)
    d = G.upload(li)
    buf = G.run_layer(d)
    G.run_layer(d, buf)   # again on the same workspace
    G.check_against_oracle(li, buf, tag=f"{T} {k} {C}", rms_over_nonzero_rows=True)
