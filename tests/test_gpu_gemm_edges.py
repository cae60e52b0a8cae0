"""The grouped expert GEMMs at the edges of their tiles: groups of exactly the
row counts where a tile, a row block or a kernel choice begins, against a plain
float64 computation of the same experts (through the C ABI).

Tolerance: the suite's own bar, max-abs error <= 1e-5 max|ref| (fp32) and
1e-2 max|ref| (bf16, whose h and o are each rounded once to 8 bits)."""
import numpy as np
import pytest
import torch

from gpu_helpers import assert_close, log

pytestmark = pytest.mark.gpu


def _step(device, dtype, H, F, E, S, lens, experts, seed=3, spoil=None):
    """One layer of E routed (top-1) and S shared experts; micro-batch i's tokens all pick
    experts[i].  spoil(gu, dn, rows): changes the weights or the micro-batches' rows first.
    Returns (o, h, a_perm) of the step and their float64 values."""
    from paper_2608_07964_amd import binding as B
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device=device).manual_seed(seed)
    gu = (torch.randn(E + S, 2 * F, H, generator=g, device=device) * 0.05).to(tdt)
    dn = (torch.randn(E + S, H, F, generator=g, device=device) * 0.05).to(tdt)
    acts = [torch.randn(T, H, generator=g, device=device).to(tdt) for T in lens]
    if spoil:
        spoil(gu, dn, acts)
    desc = B.make_desc(1, H, F, E, 1, S, 1, dtype)
    pgu, pdn = torch.empty_like(gu), torch.empty_like(dn)
    B.easybalance_pack_weights(desc, B.EB_WEIGHTS_GATE_UP, E + S, gu, pgu)
    B.easybalance_pack_weights(desc, B.EB_WEIGHTS_DOWN, E + S, dn, pdn)
    ents = []
    for i, (T, e, a) in enumerate(zip(lens, experts, acts)):
        ents.append((i, 0, T, a, torch.full((T, 1), e, dtype=torch.int32, device=device),
                     torch.ones(T, 1, device=device)))
    P = sum(lens) * (1 + S)
    nan = float("nan")
    o = torch.full((P, H), nan, dtype=tdt, device=device)
    views = dict(h=torch.full((P, F), nan, dtype=tdt, device=device),
                 a_perm=torch.full((P, H), nan, dtype=tdt, device=device))
    inv = torch.empty(P, dtype=torch.int32, device=device)
    wsb = B.easybalance_moe_step_workspace_size(desc, list(lens))
    ws = torch.empty(wsb + 256, dtype=torch.uint8, device=device)
    B.easybalance_moe_step(desc, B.work_array(ents), len(ents), [pgu], [pdn],
                           ws.data_ptr() + (-ws.data_ptr()) % 256, wsb, o, inv, views)
    torch.cuda.synchronize()
    # grouped order: experts ascending, then entries in order; shared slots last
    rows = [torch.cat([en[3] for en, e in zip(ents, experts) if e == x]) if x in experts else None
            for x in range(E)] + [torch.cat([en[3] for en in ents])] * S
    ref_h, ref_o = [], []
    for x, a in enumerate(rows):
        if a is None:
            continue
        z = a.double() @ gu[x].double().t()
        h = torch.nn.functional.silu(z[:, :F]) * z[:, F:]
        ref_h.append(h)
        ref_o.append(h.to(tdt).double() @ dn[x].double().t())
    return (o, views["h"], views["a_perm"]), (torch.cat(ref_o), torch.cat(ref_h),
                                              torch.cat([a for a in rows if a is not None]))


def _check(got, ref, dtype, what):
    for g, r, n in zip(got, ref, ("o", "h", "a_perm")[-len(got):]):
        assert_close(g.float().cpu().numpy(), r.float().cpu().numpy(), dtype, f"{what} {n}")


# decode launches: at most 32 tokens at a layer (row loads of 8, 16 and 32), one
# K part (F = 384) and two (F = 8192); 33 tokens take the tiled kernel
@pytest.mark.parametrize("H,F", [(256, 384), (768, 8192)])
@pytest.mark.parametrize("rows", [1, 7, 8, 9, 16, 17, 31, 32, 33])
def test_bf16_decode_rows(rows, H, F, device):
    log(f"bf16 rows {rows} H {H} F {F}")
    lens, experts = ([rows], [1]) if rows < 3 else ([rows - 2, 2], [1, 2])
    got, ref = _step(device, "bf16", H, F, 3, 1, lens, experts)
    _check(got, ref, "bf16", f"rows {rows}")


def test_bf16_decode_repeated_pick(device):
    """Two micro-batches whose tokens pick one expert in all four slots: its group
    spans 128 rows (16 of each 64 defined) while the layer has 32 tokens."""
    from paper_2608_07964_amd import binding as B
    T, k, H, F, E = 16, 4, 512, 384, 4
    log("bf16 repeated pick")
    g = torch.Generator(device=device).manual_seed(5)
    gu = (torch.randn(E, 2 * F, H, generator=g, device=device) * 0.05).bfloat16()
    dn = (torch.randn(E, H, F, generator=g, device=device) * 0.05).bfloat16()
    desc = B.make_desc(1, H, F, E, k, 0, 1, "bf16")
    pgu, pdn = torch.empty_like(gu), torch.empty_like(dn)
    B.easybalance_pack_weights(desc, B.EB_WEIGHTS_GATE_UP, E, gu, pgu)
    B.easybalance_pack_weights(desc, B.EB_WEIGHTS_DOWN, E, dn, pdn)
    a = torch.randn(2 * T, H, generator=g, device=device).bfloat16()
    idx = torch.ones(2 * T, k, dtype=torch.int32, device=device)
    w = torch.ones(2 * T, k, device=device)
    P = 2 * T * k
    o = torch.zeros(P, H, dtype=torch.bfloat16, device=device)
    a_perm = torch.zeros(P, H, dtype=torch.bfloat16, device=device)  # rows no pair fills stay zero
    h = torch.empty(P, F, dtype=torch.bfloat16, device=device)
    inv = torch.empty(P, dtype=torch.int32, device=device)
    wsb = B.easybalance_moe_step_workspace_size(desc, [T, T])
    ws = torch.empty(wsb + 256, dtype=torch.uint8, device=device)
    run = B.work_array([(i, 0, T, a[i * T:], idx, w) for i in range(2)])
    B.easybalance_moe_step(desc, run, 2, [pgu], [pdn], ws.data_ptr() + (-ws.data_ptr()) % 256, wsb, o, inv,
                           dict(a_perm=a_perm, h=h))
    torch.cuda.synchronize()
    z = a.double() @ gu[1].double().t()
    hr = (torch.nn.functional.silu(z[:, :F]) * z[:, F:]).bfloat16().double()
    ref = hr @ dn[1].double().t()
    pos = inv.reshape(2 * T, k).long()
    assert int(pos.max()) >= 64                      # past the rows a decode launch is sized for
    for r in range(k):
        assert_close(o[pos[:, r]].float().cpu().numpy(), ref.float().cpu().numpy(), "bf16", f"slot {r}")


def test_bf16_decode_rows_do_not_depend_on_the_launch(device):
    """The same tokens alone (a decode launch) and next to 300 others (tiles): the same bits."""
    H, F = 512, 8192
    log("bf16 decode launch against tiles")
    (o1, h1, _), _ = _step(device, "bf16", H, F, 2, 0, [20], [1])
    (o2, h2, _), _ = _step(device, "bf16", H, F, 2, 0, [20, 300], [1, 1])
    assert torch.equal(h1.view(torch.int16), h2[:20].view(torch.int16))
    assert torch.equal(o1.view(torch.int16), o2[:20].view(torch.int16))


# items of up to 64 (bf16) and 16 rows (fp32) on both sides of the 128 tokens at
# a layer up to which their weight loads are non-temporal
@pytest.mark.parametrize("dtype,row", [("bf16", 40), ("f32", 10)])
@pytest.mark.parametrize("tokens", [128, 129])
def test_weight_load_policy(tokens, dtype, row, device):
    log(f"{dtype} rows {row} of {tokens} tokens")
    lens, experts = [row, tokens - row], [1, 0]
    got, ref = _step(device, dtype, 512, 384, 3, 0, lens, experts)
    _check(got, ref, dtype, f"{tokens} tokens")


# Small groups set aside for the end of a launch, every row of every group
# checked.  K in one part: 64 small groups against the 35 that F = 1408 sets
# aside.  Split K (8 down items a group here, on 256 workgroups): one round
# exactly, a last round of 8 items, of half the workgroups and of 8 more, and
# two rounds exactly -- set aside in the first three only.
@pytest.mark.parametrize("H,F,groups", [(256, 1408, 64), (1024, 8192, 32), (1024, 8192, 33), (1024, 8192, 48),
                                        (1024, 8192, 49), (1024, 8192, 64)])
def test_bf16_groups_set_aside(H, F, groups, device):
    log(f"bf16 set aside H {H} F {F} groups {groups}")
    # rows of the 64- and 128-row tile shapes and a few of the 256-row shape
    lens = [(1 + 7 * i) % 64 + 1 if i % 4 else 65 + (29 * i) % 64 for i in range(groups)]
    lens[5], lens[groups - 2] = 129, 256
    got, ref = _step(device, "bf16", H, F, groups, 0, lens, [(5 * i) % groups if groups % 5 else i for i in range(groups)])
    _check(got, ref, "bf16", f"{groups} groups")


# fp32 row blocks of 16, m-tiles of 64 sharing a group's rows evenly
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 33, 48, 63, 64, 65, 127, 129, 200, 513])
def test_f32_group_rows(rows, device):
    log(f"f32 rows {rows}")
    got, ref = _step(device, "f32", 256, 384, 3, 1, [rows, 5], [1, 2])
    _check(got, ref, "f32", f"rows {rows}")


# fewest K stages (H = 256, F = 128) and column tiles; long K
@pytest.mark.parametrize("H,F", [(256, 128), (512, 128), (256, 2176), (1280, 640)])
def test_f32_shapes(H, F, device):
    log(f"f32 H {H} F {F}")
    got, ref = _step(device, "f32", H, F, 2, 0, [70, 9], [0, 1])
    _check(got, ref, "f32", f"H {H} F {F}")


# Launches of as many items as workgroups (256 of bf16, 512 of fp32: every item
# has a workgroup by number, none is drawn), fewer and more
@pytest.mark.parametrize("dtype,rows", [("bf16", 257), ("bf16", 65536), ("bf16", 65537), ("f32", 65), ("f32", 16384),
                                        ("f32", 16385)])
def test_items_by_number(dtype, rows, device):
    log(f"{dtype} {rows} rows of one expert")
    got, ref = _step(device, dtype, 256, 128, 1, 0, [rows], [0])
    _check(got, ref, dtype, f"{rows} rows")


# One row of infinities, one of NaN at the ends of neighbouring groups, and an
# expert of infinite weights: rows of every kernel and tile shape (decode
# launches with one and two K parts, 64-, 128- and 256-row tiles, fp32 row
# blocks) do not see their neighbours'.
@pytest.mark.parametrize("dtype,F,rows", [("bf16", 384, 7), ("bf16", 8192, 13), ("bf16", 384, 30), ("bf16", 384, 90),
                                          ("bf16", 8192, 90), ("bf16", 384, 200), ("f32", 384, 10), ("f32", 384, 90)])
def test_nonfinite_rows_stay_alone(dtype, F, rows, device):
    log(f"{dtype} F {F} rows {rows} infinities and NaN")
    lens, experts = [rows, rows + 1, 2], [0, 1, 2]

    def spoil(gu, dn, acts):
        acts[0][-1] = float("inf")
        acts[1][0] = float("nan")
        gu[2], dn[2] = float("inf"), float("-inf")

    (o, h, _), _ = _step(device, dtype, 256, F, 3, 0, lens, experts)
    (o2, h2, _), _ = _step(device, dtype, 256, F, 3, 0, lens, experts, spoil=spoil)
    bad = torch.zeros(sum(lens), dtype=torch.bool, device=device)
    bad[rows - 1:rows + 1] = True
    bad[-2:] = True
    for got, ref in ((o2, o), (h2, h)):
        assert torch.equal(got[~bad], ref[~bad])
        assert not torch.isfinite(got[bad]).any()


def test_f32_subnormal_operands(device):
    """fp32 products with a subnormal operand, and subnormal sums: rows that see only
    column 0 (gate) and a subnormal column 1 (up), down weights near the smallest normal."""
    log("f32 subnormals")
    H, F = 256, 128

    def spoil(gu, dn, acts):
        for a in acts:
            a[:, 1] = 1e-41 * (1 + torch.arange(a.shape[0], device=device))
            a[:, 2:] = 0
        gu.zero_()
        gu[:, :F, 0] = 0.5
        gu[:, F:, 1] = 1e38
        dn.mul_(1e-37)

    got, ref = _step(device, "f32", H, F, 2, 0, [70, 9], [0, 1], spoil=spoil)
    assert 0 < ref[0].abs().max() < 1e-38
    # each of the sums' F terms and the sums themselves are rounded to multiples of 2^-149
    assert (got[0].double() - ref[0]).abs().max() <= (F + 2) * 2.0 ** -149 + 1e-5 * ref[0].abs().max()
    _check(got[1:], ref[1:], "f32", "subnormals")
