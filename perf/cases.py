"""The calls whose time counts, over the range of sizes that a program using the library has them in.

Four kinds of work, each through the public binding:
  layer    one moe_verify_layer call (routing, histogram, slot lookup, expert FFN, final sum)
  steps    the same layer as the four single-step calls, for a program with a routing of its own in between
  control  one step of the control loop for all layers: utility update, threshold, cache plan
  load     the fetched experts of one layer moved into their slots

Hidden states are what a layer gets behind a normalisation (unit variance), weights N(0, 0.02), routers N(0, 0.02).
Every token's k+1 best logits are kept a small margin apart, so that no correct implementation ranks them otherwise.
"""
import math

import torch

from paper_2603_09983_amd import binding as B

W_STD = 0.02
MARGIN = 1e-3


def _layer(name, T, H, E, k, F, C, n_shared=0, F_shared=0, zipf=False, out_bf16=False, accumulate=False):
    return {"name": name, "kind": "layer", "T": T, "H": H, "E": E, "k": k, "F": F, "C": C, "n_shared": n_shared,
            "F_shared": F_shared, "zipf": zipf, "out_bf16": out_bf16, "accumulate": accumulate}


def listed():
    return [
        # the smallest call there is: a toy model's verify step, all experts resident; launches and host work
        _layer("tiny_T5", 5, 256, 8, 2, 512, 8),
        # plain decoding (no draft accepted or none made): one token through a 64-expert layer
        _layer("one_token", 1, 2048, 64, 6, 1408, 48),
        # the ordinary verify step: 8 draft tokens + 1, two shared experts, half of the experts resident
        _layer("verify_T9", 9, 2048, 64, 6, 1408, 32, n_shared=2, F_shared=1408),
        # skewed routing, one wide shared expert, bf16 output added to what the host computed for the misses
        _layer("zipf_wide_shared_T5", 5, 2048, 60, 4, 1408, 24, n_shared=1, F_shared=5632, zipf=True, out_bf16=True,
               accumulate=True),
        # two requests verified together
        _layer("batch_T17", 17, 2048, 64, 6, 1408, 48),
        # the largest batch of the verification sweep
        _layer("batch_T128", 128, 2048, 64, 6, 1408, 48),
        # large experts, one request
        _layer("large_T8", 8, 4096, 8, 2, 14336, 8),
        # large experts, a batch of requests
        _layer("large_T64", 64, 4096, 8, 2, 14336, 8),
        # widths that no tile divides
        _layer("ragged_T7", 7, 2040, 40, 4, 1000, 20, n_shared=1, F_shared=1480),
        # the single-step calls on a batch larger than the sweep's
        dict(_layer("steps_T256", 256, 2048, 64, 6, 1408, 48, out_bf16=True), kind="steps"),
        # the control loop of a 24-layer model after each verify step
        {"name": "control_24x64", "kind": "control", "T": 9, "k": 6, "L": 24, "N": 64, "C": 32, "K": 4, "budget": 4},
        # four experts of one layer prefetched from a store in device memory
        {"name": "load_4", "kind": "load", "H": 2048, "F": 1408, "C": 32, "n": 4, "store": "device"},
    ]


def _logint(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, lo, hi):
    step = rng.choice([64, 64, 64, 128, 32, 8])
    return max(step, _logint(rng, lo, hi) // step * step)


def draw(rng):
    while True:
        p = rng.random()
        if p < 0.12:
            N = rng.choice([8, 32, 60, 64, 100, 128, 256])
            return {"kind": "control", "T": rng.randint(2, 16), "k": rng.randint(1, min(8, N)), "L": rng.randint(1, 48),
                    "N": N, "C": rng.randint(1, N), "K": rng.randint(1, 8), "budget": rng.randint(1, 8)}
        if p < 0.24:
            H, F = _width(rng, 256, 4096), _width(rng, 256, 4096)
            return {"kind": "load", "H": H, "F": F, "C": rng.randint(8, 16), "n": rng.randint(1, 8),
                    "store": "host" if rng.random() < 0.25 else "device"}
        E = rng.choice([4, 8, 16, 40, 60, 64, 64, 64, 100, 128])
        case = _layer("", _logint(rng, 1, 128 if p < 0.85 else 256), _width(rng, 256, 4096), E,
                      rng.randint(1, min(8, E)), _width(rng, 256, 8192 if rng.random() < 0.3 else 2048),
                      rng.randint(max(1, E // 4), E))
        del case["name"]
        case["zipf"] = rng.random() < 0.25
        case["out_bf16"] = rng.random() < 0.5
        case["accumulate"] = rng.random() < 0.3
        if p < 0.85:
            case["n_shared"] = rng.choice([0, 0, 1, 2])
            case["F_shared"] = _width(rng, 256, 4096) if case["n_shared"] else 0
        else:
            case["kind"] = "steps"
        if work(case)["bytes"] <= 9e8 and 6 * case["C"] * case["H"] * case["F"] <= 4e9:
            return case


def _normal(g, *shape, std=1.0, dtype=torch.bfloat16):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, std, generator=g)


def _layer_inputs(case, seed):
    """Plain tensors of one layer: the same for every implementation."""
    T, H, E, k, F, C = (case[n] for n in ("T", "H", "E", "k", "F", "C"))
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    router = _normal(g, E, H, std=W_STD, dtype=torch.float32)
    bias, popular = None, torch.ones(E, device="cuda")
    if case["zipf"]:
        # logits are normal with deviation 0.02 sqrt(H): with this bias a token picks experts about as often as
        # their popularity rank^-1.1 says
        rank = torch.randperm(E, generator=g, device="cuda") + 1
        popular = rank.float() ** -1.1
        bias = (W_STD * math.sqrt(H) / 1.2825 * popular.log()).float()
    hidden = _normal(g, T, H)
    todo = torch.arange(T, device="cuda")
    for _ in range(200):   # draw rows again until the best k+1 logits are apart
        s = hidden[todo].double() @ router.double().T
        if bias is not None:
            s = s + bias.double()
        top = s.topk(min(k + 1, E), dim=1).values
        todo = todo[((top[:, :-1] - top[:, 1:]) < MARGIN).any(dim=1)]
        if todo.numel() == 0:
            break
        hidden[todo] = _normal(g, todo.numel(), H)
    n = min(C, E)
    resident = torch.multinomial(popular, n, generator=g)
    table = torch.full((E,), -1, dtype=torch.int32, device="cuda")
    table[resident] = torch.randperm(C, generator=g, device="cuda")[:n].int()
    t = {"hidden": hidden, "router": router, "bias": bias, "table": table,
         "gate": _normal(g, C, F, H, std=W_STD), "up": _normal(g, C, F, H, std=W_STD),
         "down": _normal(g, C, H, F, std=W_STD), "sh_gate": None, "sh_up": None, "sh_down": None}
    if case["n_shared"]:
        m, Fs = case["n_shared"], case["F_shared"]
        t["sh_gate"], t["sh_up"] = _normal(g, m, Fs, H, std=W_STD), _normal(g, m, Fs, H, std=W_STD)
        t["sh_down"] = _normal(g, m, H, Fs, std=W_STD)
    dt = torch.bfloat16 if case["out_bf16"] else torch.float32
    # what the host has computed for the experts that are not resident
    t["partial"] = _normal(g, T, H, std=0.2, dtype=dt) if case["accumulate"] else torch.zeros(T, H, dtype=dt, device="cuda")
    return t


def _prepare_layer(case, seed):
    t = _layer_inputs(case, seed)
    shape = B.make_shape(case["T"], case["H"], case["E"], case["k"], case["F"], case["C"], case["n_shared"],
                         case["F_shared"])
    buf = B.LayerBuffers.allocate(shape, out_bf16=case["out_bf16"])
    buf.out.copy_(t["partial"])
    buf.miss_list.zero_()
    st = {"case": case, "t": t, "shape": shape, "buf": buf}
    if case["kind"] == "steps":
        st["logits"] = torch.zeros(case["T"], case["E"], device="cuda")
        # each single step keeps scratch in a workspace of its own
        st["ws_route"], st["ws_slot"], st["ws_ffn"] = (B.new_workspace(shape) for _ in range(3))
    return st


def _prepare_control(case, seed):
    L, N, C, K, T, k = (case[n] for n in ("L", "N", "C", "K", "T", "k"))
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    # eight steps' activation frequencies: every layer's popularity drifts slowly
    p = torch.randn(L, N, device="cuda", generator=g)
    f = []
    for _ in range(8):
        p = p + 0.3 * torch.randn(L, N, device="cuda", generator=g)
        picks = torch.multinomial(p.softmax(1).repeat_interleave(T, 0), k, generator=g).view(L, T * k)
        f.append(torch.zeros(L, N, dtype=torch.int32, device="cuda").scatter_add_(
            1, picks, torch.ones(L, T * k, dtype=torch.int32, device="cuda")))
    i32 = dict(dtype=torch.int32, device="cuda")
    table = torch.full((L, N), -1, **i32)
    for l in range(L):
        n = min(C, N)
        table[l, torch.randperm(N, generator=g, device="cuda")[:n]] = torch.randperm(C, generator=g, device="cuda")[:n].int()
    st = {"case": case, "step": 0, "f": f, "in_use": [(x > 0).int() for x in f], "table": table,
          "state": [torch.zeros(L, N, **i32) for _ in range(4)], "n_tau": torch.zeros(L, K + 1, **i32),
          "r_c": torch.rand(L, K + 1, device="cuda", generator=g, dtype=torch.float64).sort(1).values,
          "r_g": torch.rand(L, K + 1, device="cuda", generator=g, dtype=torch.float64).sort(1, descending=True).values.contiguous(),
          "params": B.BalanceParams(40.0, 3.0, 6.0, 600.0, L, 17 << 20, 16 * (17 << 20)),
          "tau": torch.zeros(L, **i32), "b": torch.zeros(L, **i32), "budget": torch.full((L,), case["budget"], **i32),
          "evict": torch.zeros(L, N, **i32), "n_evict": torch.zeros(L, **i32), "fetch": torch.zeros(L, C, **i32),
          "fetch_slot": torch.zeros(L, C, **i32), "n_fetch": torch.zeros(L, **i32)}
    f_prev, s, up, dn = st["state"]
    B.moe_utility_init(f_prev, s, up, dn, L, N, T - 1)
    for x in f[:4]:   # a few steps of history
        B.moe_utility_update(x, f_prev, s, up, dn, table, st["n_tau"], L, N, K, 1, 10)
    return st


def _prepare_load(case, seed):
    H, F, C, n = case["H"], case["F"], case["C"], case["n"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    E = 2 * n
    store = [_normal(g, E, F, H, std=W_STD), _normal(g, E, F, H, std=W_STD), _normal(g, E, H, F, std=W_STD)]
    if case["store"] == "host":
        pinned = []
        for w in store:
            h = torch.empty(w.shape, dtype=w.dtype, pin_memory=True)
            h.copy_(w)
            pinned.append(h)
        store = pinned
    pool = [torch.zeros(C, F, H, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    pool.append(torch.zeros(C, H, F, dtype=torch.bfloat16, device="cuda"))
    return {"case": case, "store": store, "pool": pool,
            "fetch": torch.randperm(E, generator=g, device="cuda")[:n].int().contiguous(),
            "slot": torch.randperm(C, generator=g, device="cuda")[:n].int().contiguous(),
            "n_fetch": torch.full((1,), n, dtype=torch.int32, device="cuda")}


def prepare(case, seed):
    if case["kind"] == "control":
        return _prepare_control(case, seed)
    if case["kind"] == "load":
        return _prepare_load(case, seed)
    return _prepare_layer(case, seed)


def run(st):
    c = st["case"]
    if c["kind"] == "control":
        i = st["step"] % 8
        st["step"] += 1
        f_prev, s, up, dn = st["state"]
        B.moe_utility_update(st["f"][i], f_prev, s, up, dn, st["table"], st["n_tau"], c["L"], c["N"], c["K"], 1, 10)
        B.moe_balance_threshold(st["f"][i], st["n_tau"], st["r_c"], st["r_g"], c["L"], c["N"], c["K"], c["T"] - 1, c["k"],
                                st["params"], st["tau"], st["b"])
        B.moe_cache_plan(s, st["in_use"][i], st["table"], st["tau"], st["budget"], c["L"], c["N"], c["C"], c["K"],
                         st["evict"], st["n_evict"], st["fetch"], st["fetch_slot"], st["n_fetch"])
        return (s, up, dn, f_prev, st["n_tau"], st["tau"], st["b"], st["table"], st["evict"], st["n_evict"], st["fetch"],
                st["fetch_slot"], st["n_fetch"])
    if c["kind"] == "load":
        B.moe_pool_load(*st["store"], *st["pool"], st["fetch"], st["slot"], st["n_fetch"], c["n"], c["H"], c["F"])
        return tuple(st["pool"])
    t, b = st["t"], st["buf"]
    if c["kind"] == "steps":
        T, H, E, k, F, C = (c[n] for n in ("T", "H", "E", "k", "F", "C"))
        B.moe_route_topk(t["hidden"], t["router"], t["bias"], T, H, E, k, b.topk_idx, b.topk_w, st["logits"], st["ws_route"])
        B.moe_expert_histogram(b.topk_idx, T, k, E, b.hist)
        B.moe_slot_resolve(b.topk_idx, t["table"], T, k, E, C, b.slot_idx, b.miss_list, b.miss_count, st["ws_slot"])
        B.moe_grouped_ffn(t["hidden"], b.topk_w, b.slot_idx, t["gate"], t["up"], t["down"], T, H, F, k, C, b.out,
                          c["out_bf16"], c["accumulate"], st["ws_ffn"])
        return {"out": b.out, "topk_w": b.topk_w, "logits": st["logits"], "topk_idx": b.topk_idx, "hist": b.hist,
                "slot_idx": b.slot_idx, "miss_list": b.miss_list, "miss_count": b.miss_count}
    B.moe_verify_layer(st["shape"], t["hidden"], t["router"], t["bias"], t["table"], t["gate"], t["up"], t["down"],
                       t["sh_gate"], t["sh_up"], t["sh_down"], b.topk_idx, b.topk_w, b.hist, b.slot_idx, b.miss_list,
                       b.miss_count, b.out, c["out_bf16"], c["accumulate"], b.workspace)
    return {"out": b.out, "topk_w": b.topk_w, "topk_idx": b.topk_idx, "hist": b.hist, "slot_idx": b.slot_idx,
            "miss_list": b.miss_list, "miss_count": b.miss_count}


def work(case):
    if case["kind"] == "control":
        L, N, C, K = (case[n] for n in ("L", "N", "C", "K"))
        # f, in_use and the five words of state read, the state and the table written; tables and lists
        words = L * N * (2 + 5 + 5) + 2 * L * (K + 1) + 6 * L + L * C
        return {"bytes": 4 * words + 16 * L * (K + 1), "flops": 20 * L * N}
    if case["kind"] == "load":
        return {"bytes": 2 * 6 * case["n"] * case["H"] * case["F"], "flops": 0}
    T, H, E, k, F, C = (case[n] for n in ("T", "H", "E", "k", "F", "C"))
    n = min(C, E)
    # resident experts that at least one of the T tokens picks; each one's matrices are read once.  With skewed
    # routing this counts the experts as if they were picked alike (a little too many).
    active = n * (1.0 - (1.0 - k / E) ** T)
    weights = 6.0 * H * F * active + 6.0 * H * case["n_shared"] * case["F_shared"]
    out = T * H * (2 if case["out_bf16"] else 4) * (2 if case["accumulate"] else 1)
    flops = 6.0 * H * (F * T * k * n / E + case["n_shared"] * case["F_shared"] * T) + 2.0 * T * E * H
    return {"bytes": weights + 4.0 * E * H + 2.0 * T * H + out + 16 * T * k, "flops": flops}


def tolerance(case):
    if case["kind"] in ("control", "load"):
        return "exact"
    # The activations are rounded to bf16 between the projections (relative error 1.7e-3 of each, averaged over the
    # width), the output once more where it is bf16.  Measured against 64 bits: 1.6e-3 to 2.4e-3; stated: about four times that.
    return {"rel": 7e-3, "max": 0.1}


def exact(case, seed):
    if case["kind"] in ("control", "load"):
        return None   # whole numbers and copied bytes
    t = _layer_inputs(case, seed)
    T, k = case["T"], case["k"]
    x = t["hidden"].double()
    logits = x @ t["router"].double().T
    if t["bias"] is not None:
        logits = logits + t["bias"].double()
    top = logits.topk(k, dim=1)
    gate = torch.softmax(top.values, dim=1)
    slot = t["table"].long()[top.indices]
    y = t["partial"].double().clone() if case["accumulate"] else torch.zeros(T, case["H"], dtype=torch.float64, device="cuda")

    def expert(xe, wg, wu, wd):
        a = xe @ wg.double().T
        return (a * torch.sigmoid(a) * (xe @ wu.double().T)) @ wd.double().T

    for c in slot.unique().tolist():
        if c >= 0:
            rows, j = (slot == c).nonzero(as_tuple=True)
            y[rows] += gate[rows, j, None] * expert(x[rows], t["gate"][c], t["up"][c], t["down"][c])
    for i in range(case["n_shared"]):
        y += expert(x, t["sh_gate"][i], t["sh_up"][i], t["sh_down"][i])
    r = {"out": y, "topk_w": gate, "topk_idx": None, "hist": None, "slot_idx": None, "miss_list": None, "miss_count": None}
    if case["kind"] == "steps":
        r["logits"] = logits
    return r
