"""A step's grouping (perm, inv, offsets, gathered rows) against the oracle's
stable permutation, on both sides of the one-workgroup kernel's limits: 32
pieces of up to 64 tokens, 128 pieces x slots, 23040 LDS words; where 256-token
chunks hold more than two pieces on average, 16 pieces and 128 pieces x (slots +
experts / 96), elsewhere 149 of these.  All integers and copies: exact."""
import numpy as np
import pytest
import torch

from gpu_helpers import log
from oracle import permute as operm

pytestmark = pytest.mark.gpu


# name: (dtype, L, E, S, k, tokens of each entry[, H]); layers cycle, so one layer's
# entries are not neighbours
CASES = {
    "one_token": ("bf16", 1, 64, 2, 6, [1]),
    "one_token_wide": ("bf16", 1, 64, 1, 8, [1], 7168),      # 126 KB of rows: copied by the same launch
    "copy_full": ("bf16", 2, 8, 0, 2, [1, 0, 41], 768),      # 84 rows of 1.5 KB: 126 KB; 88 rows: 132 KB
    "copy_over": ("bf16", 2, 8, 0, 2, [1, 0, 43], 768),
    "copy_f32": ("f32", 2, 8, 1, 2, [3, 6], 1024),
    "piece_edges": ("bf16", 2, 60, 4, 4, [63, 64, 65, 0, 127, 128, 129, 1]),
    "many_entries": ("bf16", 5, 8, 0, 2, [1 + i % 7 for i in range(32)]),
    "64_entries": ("bf16", 5, 8, 0, 2, [1 + i % 7 for i in range(64)]),
    "32_pieces": ("bf16", 2, 16, 1, 3, [1024, 1, 64, 895]),
    "33_pieces": ("bf16", 2, 16, 1, 3, [1024, 1, 65, 895]),
    "32_full_pieces": ("bf16", 2, 16, 1, 3, [64] * 32),
    "16_in_chunks": ("bf16", 2, 16, 1, 3, [512, 1, 64, 320, 1]),
    "17_in_chunks": ("bf16", 2, 16, 1, 3, [512, 1, 64, 321, 1]),
    "cost_full": ("bf16", 2, 192, 0, 6, [1024]),                    # 16 x (6 + 2) = 128; 193 experts: over
    "cost_over": ("bf16", 2, 193, 0, 6, [1024]),
    "short_cost_full": ("bf16", 2, 128, 0, 8, [65] * 8),            # 16 x (8 + 4/3) = 149
    "short_cost_over": ("bf16", 2, 129, 0, 8, [65] * 8),
    "slots_full": ("bf16", 3, 256, 0, 8, [65] * 8),
    "slots_over": ("bf16", 3, 256, 1, 8, [65] * 8),
    "lds_full": ("bf16", 3, 256, 0, 1, [64] * 30),
    "lds_over": ("bf16", 3, 256, 0, 1, [64] * 31),
    "many_keys": ("f32", 15, 1000, 4, 12, [64, 3, 64, 130]),
    "all_slots": ("f32", 3, 20, 0, 16, [70, 0, 90]),
    "three_launches": ("f32", 3, 500, 2, 5, [300, 1, 512, 77, 256]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_grouping(name, device):
    from paper_2608_07964_amd import binding as B
    log(f"grouping {name}")
    dtype, L, E, S, k, lens, *rest = CASES[name]
    H, F = rest[0] if rest else 256, 128
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(11)
    g = torch.Generator(device=device).manual_seed(11)
    layers = [i % L for i in range(len(lens))]
    # skewed picks: the low experts take most tokens
    idx = [np.argsort(rng.random((T, E)) * (1.0 + np.arange(E)) ** 0.7, axis=1)[:, :k] for T in lens]
    a = [torch.randn(max(T, 1), H, generator=g, device=device).to(tdt) for T in lens]
    used = sorted(set(layers))
    gu = [torch.zeros(E + S, 2 * F, H, dtype=tdt, device=device) if l in used else None for l in range(L)]
    dn = [torch.zeros(E + S, H, F, dtype=tdt, device=device) if l in used else None for l in range(L)]
    desc = B.make_desc(L, H, F, E, k, S, 1, dtype)
    P = sum(lens) * (k + S)
    keep = [torch.from_numpy(np.ascontiguousarray(i, np.int32)).to(device) for i in idx]
    w = torch.ones(max(lens), k, device=device)
    run = B.work_array([(j, l, T, x, i, w) for j, (l, T, x, i) in enumerate(zip(layers, lens, a, keep))])
    o = torch.full((P, H), 1.0, dtype=tdt, device=device)
    inv = torch.full((P,), -1, dtype=torch.int32, device=device)
    v = dict(a_perm=torch.zeros(P, H, dtype=tdt, device=device), h=torch.empty(P, F, dtype=tdt, device=device),
             perm=torch.full((P,), -1, dtype=torch.int32, device=device),
             offsets=torch.full((L * (E + S) + 1,), -1, dtype=torch.int32, device=device))
    wsb = B.easybalance_moe_step_workspace_size(desc, lens)
    ws = torch.full((wsb + 256,), 255, dtype=torch.uint8, device=device)
    B.easybalance_moe_step(desc, run, len(lens), gu, dn, ws.data_ptr() + (-ws.data_ptr()) % 256, wsb, o, inv, v)
    torch.cuda.synchronize()
    perm, want_inv, offsets = operm.stable_permutation(operm.step_keys(list(zip(layers, idx)), E, S), L * (E + S))
    assert np.array_equal(v["offsets"].cpu().numpy(), offsets)
    assert np.array_equal(v["perm"].cpu().numpy(), perm)
    assert np.array_equal(inv.cpu().numpy(), want_inv)
    src = torch.cat([x[:T] for x, T in zip(a, lens)])
    rows = torch.from_numpy(perm // (k + S)).to(device)
    assert torch.equal(v["a_perm"], src[rows])
    assert not o.any()                               # zero experts: every row was computed


@pytest.mark.parametrize("T", [65, 200, 600])
def test_grouping_of_repeated_picks(T, device):
    """Tokens that pick an expert twice (or ids outside [0, E), clamped) alone, grouped
    by the one-workgroup kernel, and before 2100 tokens of another layer, grouped by the
    three launches: the same positions, and each pair's position holds its token's row."""
    from paper_2608_07964_amd import binding as B
    log(f"repeated picks T {T}")
    H, F, E, k, L, T2 = 256, 128, 5, 3, 2, 2100
    g = torch.Generator(device=device).manual_seed(T)
    idx = torch.randint(-1, E + 1, (T, k), generator=g, device=device, dtype=torch.int32)
    idx2 = torch.randint(0, E, (T2, k), generator=g, device=device, dtype=torch.int32)
    a = torch.randn(T, H, generator=g, device=device).bfloat16()
    a2 = torch.randn(T2, H, generator=g, device=device).bfloat16()
    w = torch.ones(T2, k, device=device)
    gu = [torch.zeros(E, 2 * F, H, dtype=torch.bfloat16, device=device) for _ in range(L)]
    dn = [torch.zeros(E, H, F, dtype=torch.bfloat16, device=device) for _ in range(L)]
    desc = B.make_desc(L, H, F, E, k, 0, 1, "bf16")
    pos = []
    for ents in ([(0, 0, T, a, idx, w)], [(0, 0, T, a, idx, w), (1, 1, T2, a2, idx2, w)]):
        P = sum(e[2] for e in ents) * k
        o = torch.empty(P, H, dtype=torch.bfloat16, device=device)
        inv = torch.full((P,), -1, dtype=torch.int32, device=device)
        v = dict(a_perm=torch.zeros(P, H, dtype=torch.bfloat16, device=device),
                 offsets=torch.full((L * E + 1,), -1, dtype=torch.int32, device=device))
        wsb = B.easybalance_moe_step_workspace_size(desc, [e[2] for e in ents])
        ws = torch.empty(wsb + 256, dtype=torch.uint8, device=device)
        B.easybalance_moe_step(desc, B.work_array(ents), len(ents), gu, dn, ws.data_ptr() + (-ws.data_ptr()) % 256,
                               wsb, o, inv, v)
        torch.cuda.synchronize()
        p = inv[:T * k].long()
        key = idx.clamp(0, E - 1).reshape(-1).long()
        assert ((p >= v["offsets"][key]) & (p < v["offsets"][key + 1])).all()
        assert torch.equal(v["a_perm"][p], a.repeat_interleave(k, 0))
        pos.append((p, v["offsets"][:E + 1]))
    assert torch.equal(pos[0][1], pos[1][1])
    assert torch.equal(pos[0][0], pos[1][0])
