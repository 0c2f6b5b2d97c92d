"""A token's expert outputs depend on the token, the expert and the widths, not on what else is in the batch: bits equal
between batches of 16 and larger ones (contractions of up to 2048 columns in whole 64s: the streaming kernels at any batch
size), between larger batches of any width that differ in size and in the number of slots (64 and 32 rows to an item), and
between two larger batches that route the other tokens differently."""
import pytest
import torch

from paper_2603_09983_amd import binding as B

pytestmark = pytest.mark.gpu


def _weights(g, H, F, C):
    n = lambda *s, std: (torch.randn(*s, device="cuda", generator=g) * std).bfloat16()
    return n(C, F, H, std=2.0 * H ** -0.5), n(C, F, H, std=2.0 * H ** -0.5), n(C, H, F, std=F ** -0.5)


def _ffn(x, slot, wts, bf16=False):
    (T, H), k = x.shape, slot.shape[1]
    C, F = wts[0].shape[:2]
    out = torch.empty(T, H, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32)
    ws = B.new_workspace(B.make_shape(T, H, max(C, k), k, F, C))
    B.moe_grouped_ffn(x, torch.full((T, k), 1.0 / k, device="cuda"), slot, *wts, T, H, F, k, C, out, bf16, False, ws)
    B.moe_workspace_status(ws)
    return out


def _slots(g, T, k, C, on_first):
    """k distinct slots a token; slot 0 for the first `on_first` tokens, never for the others."""
    s = torch.rand(T, C - 1, device="cuda", generator=g).argsort(1)[:, :k] + 1
    s[:on_first, 0] = 0
    return s.int().contiguous()


# (H, F, T, tokens on slot 0)
@pytest.mark.parametrize("H,F,T,first", [(1088, 576, 64, 33), (2048, 1408, 64, 64), (2048, 1408, 40, 20), (512, 2048, 130, 97),
                                         (192, 1984, 33, 33), (64, 64, 200, 150)])
def test_same_bits_as_in_batches_of_sixteen(H, F, T, first):
    g = torch.Generator(device="cuda").manual_seed(H + F + T)
    C, k = 9, 2
    wts = _weights(g, H, F, C)
    x = torch.randn(T, H, device="cuda", generator=g).bfloat16()
    slot = _slots(g, T, k, C, first)
    print(f"[case] {H} {F} {T} {first}", flush=True)
    whole = _ffn(x, slot, wts)
    parts = torch.cat([_ffn(x[i:i + 16].contiguous(), slot[i:i + 16].contiguous(), wts) for i in range(0, T, 16)])
    assert torch.equal(whole, parts), f"{(whole != parts).float().mean().item():.2g} of the values differ"


# (H, F, tokens of the smaller batch and of the larger): one chunk of 512 columns and several, with remainders
@pytest.mark.parametrize("H,F,small,large", [(1000, 1048, 33, 130), (2040, 520, 40, 64), (4096, 576, 34, 100), (520, 4104, 48, 70)])
def test_batch_size_and_item_height_do_not_matter(H, F, small, large):
    g = torch.Generator(device="cuda").manual_seed(H + F)
    C, k = 48, 2
    wts = _weights(g, H, F, C)
    x = torch.randn(large, H, device="cuda", generator=g).bfloat16()
    slot = _slots(g, large, k, 5, 70)   # slots 0 to 4
    print(f"[case] {H} {F} {small} {large}", flush=True)
    whole = _ffn(x, slot, wts)
    assert torch.equal(_ffn(x[:small].contiguous(), slot[:small].contiguous(), wts), whole[:small])
    assert torch.equal(_ffn(x, slot, tuple(w[:5].contiguous() for w in wts)), whole)


@pytest.mark.parametrize("H,F,T", [(4096, 128, 40), (256, 2560, 64), (4104, 72, 100), (2048, 1408, 128), (1088, 576, 64)])
def test_the_other_tokens_routing_does_not_matter(H, F, T):
    g = torch.Generator(device="cuda").manual_seed(H + F + T)
    C, k = 12, 2
    wts = _weights(g, H, F, C)
    x = torch.randn(T, H, device="cuda", generator=g).bfloat16()
    print(f"[case] {H} {F} {T}", flush=True)
    a = _slots(g, T, k, C, 5)
    first = _ffn(x, a, wts)
    for others in (T, T // 2, 0):   # slot 0 in the lists' front with many tokens, with some, and not at all
        b = _slots(g, T, k, C, others)
        b[-3:] = a[-3:]
        assert torch.equal(_ffn(x, b, wts)[-3:], first[-3:]), others
