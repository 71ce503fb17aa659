"""Parity at the edges of the sizes that choose a kernel: the smallest and the ragged ends of each range, against the oracle."""
import pytest

from tests.test_gpu_parity import _full_parity

pytestmark = pytest.mark.gpu


def _bf16(name, N, L=1, heads=3, d=64, B=16, K=8, kind="gaussian", **kw):
    return dict(name=name, batch=1, heads=heads, d=d, N=N, B=B, K=K, L=L, dtype="bf16", kind=kind, **kw)


@pytest.mark.parametrize("cfg", [
    # lengths that are multiples of the block and of nothing larger (fp32 P and dS): one query tile in all, one tile into the
    # third workgroup, one short of it
    _bf16("one_tile", 16, K=4),
    _bf16("tiles_9", 144),
    _bf16("tiles_15_d128", 240, d=128, K=4),
    _bf16("tiles_169", 2704, kind="smooth"),
    _bf16("tiles_33_Le0", 528, Le=0),
    _bf16("blocks32_3", 96, B=32, K=2),
    _bf16("blocks64_5", 320, B=64, K=3),
    # more than 64 level-0 tiles per list at such a length: one wave per query tile
    _bf16("blocks32_K33", 1120, B=32, K=33),
], ids=lambda c: c["name"])
def test_lengths_that_fill_no_workgroup(cfg):
    _full_parity(cfg, 0xD15A + cfg["N"])


@pytest.mark.parametrize("cfg", [
    _bf16("tiles_9", 144),
    _bf16("tiles_169_d128", 2704, d=128, kind="smooth"),
    _bf16("blocks32_33", 1056, B=32, K=5),
], ids=lambda c: c["name"])
def test_lengths_that_are_no_multiple_of_64_have_fp32_probabilities(cfg):
    """Their attention and gradients are those of the fp32-arithmetic kernels, bit for bit: nothing of P or dS is rounded to bf16."""
    import torch
    from tests import harness as H
    x = H.make_inputs(cfg, 0xD162)
    got, want = (H.gpu_forward_backward(cfg, x, plan=H.make_plan(cfg, kernel_path=path)) for path in (0, 1))
    for name in ("indices", "O", "LSE", "dQ", "dK", "dV"):
        assert torch.equal(got[name], want[name]), name


def test_lists_of_six_levels():
    """Levels beyond the fourth coarse one (1048576 tokens in blocks of 16, the coarsest level a single token): the bf16 MFMA kernels
    against the fp32-arithmetic ones, both within the bf16 bound of the same result."""
    import torch
    from paper_2512_16615_amd import llsa
    from tests import harness as H
    N, d = 16 ** 5, 64
    gen = torch.Generator(device="cuda").manual_seed(11)
    Q, K, V, dO = (torch.randn(1, 1, N, d, generator=gen, device="cuda").bfloat16() for _ in range(4))
    got = []
    for path in (0, 1):
        plan = llsa.Plan(1, 1, N, d, 16, 2, 5, kernel_path=path)
        O, LSE, idx, ws = llsa.forward(plan, Q, K, V, workspace=plan.alloc_workspace(True))
        got.append((O, LSE, idx) + tuple(llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)))
    assert torch.equal(got[0][2], got[1][2])
    tol = H.TOL["bf16"]["out"]
    for name, i in (("O", 0), ("dQ", 3), ("dK", 4), ("dV", 5)):
        assert float((got[0][i].float() - got[1][i].float()).abs().max()) <= 2 * tol, name
    assert float((got[0][1] - got[1][1]).abs().max()) <= 1e-3


@pytest.mark.parametrize("d,B", [(64, 16), (128, 16), (128, 32), (32, 8), (16, 16)])
def test_bf16_tiles_round_outputs_only(d, B):
    """bf16 shapes in fp32 arithmetic, every block listed (a dense softmax): all but a few outputs are the correctly rounded result.  fp32
    sums of 144 to 160 terms are off by some 1e-6 of it, which crosses a rounding border (2^-8 apart) in 1 of 2000 elements, more
    where terms cancel; P or dS rounded to bf16 would change a quarter."""
    import torch
    from paper_2512_16615_amd import llsa
    N = 160 if B == 32 else 144
    gen = torch.Generator().manual_seed(d + B)
    Q, K, V, dO = (torch.randn(1, 2, N, d, generator=gen).bfloat16().cuda() for _ in range(4))
    plan = llsa.Plan(1, 2, N, d, B, N // B, 1, Le=0)
    O, LSE, idx, ws = llsa.forward(plan, Q, K, V, workspace=plan.alloc_workspace(True))
    dQ, dK, dV = llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)
    q, k, v, g = (x.double() for x in (Q, K, V, dO))
    mm = lambda a, b: torch.matmul(a, b.contiguous())
    P = torch.softmax(mm(q, k.transpose(2, 3)) * d ** -0.5, -1)
    dS = P * (mm(g, v.transpose(2, 3)) - (g * O.double()).sum(-1, keepdim=True)) * d ** -0.5
    for name, got, want in (("O", O, mm(P, v)), ("dV", dV, mm(P.transpose(2, 3), g)), ("dQ", dQ, mm(dS, k)),
                            ("dK", dK, mm(dS.transpose(2, 3), q))):
        assert float((got != want.bfloat16()).float().mean()) < 0.01, name


@pytest.mark.parametrize("d,B", [(64, 16), (128, 16), (64, 32), (128, 64)])
def test_largest_probability_takes_no_rounding(d, B):
    """Lengths that are no multiple of 256: P relative to the exact running maximum.  One key, behind the first tiles, holds 78 to 94 %
    of every query's weight; its P is 1, and rounding the others' moves O by less than 2^-9 x 0.22 x |mean V| ~ 3e-5, a
    thirtieth of half a unit of O's last place, so that O is the correctly rounded result but for some 3 % of the elements."""
    import torch
    from paper_2512_16615_amd import llsa
    N, top = 192, 100
    gen = torch.Generator().manual_seed(3)
    Q, K = torch.zeros(1, 2, N, d), torch.zeros(1, 2, N, d)
    Q[..., 0] = 6.5 + 1.5 * torch.rand(1, 2, N, generator=gen)
    K[..., top, 0] = 1.0
    V = torch.randn(1, 2, N, d, generator=gen)
    Q, K, V = (t.bfloat16().cuda() for t in (Q, K, V))
    plan = llsa.Plan(1, 2, N, d, B, N // B, 1, Le=0, sm_scale=1.0)
    O = llsa.forward(plan, Q, K, V)[0]
    P = torch.softmax(torch.matmul(Q.double(), K.double().transpose(2, 3).contiguous()), -1)
    want = torch.matmul(P, V.double()).bfloat16()
    assert float((O != want).float().mean()) < 0.1


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_fp32_arithmetic_takes_exponentials_to_the_last_place(dtype):
    """Logits of 16 to 64, equal for all 64 keys of a query: a factor of log2(e) rounded at that size costs the logsumexp more than a
    unit of its last place and P up to 3e-6.  LSE: logf and the sum, below one unit.  dV holds single P's: a unit of expf (2 x 2^-24)
    and two roundings.  dQ holds the sum of 64 equal ones: partial sum k is rounded at k / 64 of the result, 32.5 x 2^-24 in all, on
    top of expf and three factors."""
    import torch
    from paper_2512_16615_amd import llsa
    N = d = 64
    gen = torch.Generator().manual_seed(7)
    sign = torch.tensor([1.0, -1.0]).repeat(N // 2)
    Q, K = torch.zeros(2, 1, 3, N, d)
    Q[..., 0] = 16 + 48 * torch.rand(1, 3, N, generator=gen)
    K[..., 0], K[..., 1] = 1.0, sign
    V = sign[:, None].expand(1, 3, N, d)
    dO = torch.eye(N).expand(1, 3, N, d)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dO = (x.to(t).contiguous().cuda() for x in (Q, K, V, dO))
    plan = llsa.Plan(1, 3, N, d, 16, N // 16, 1, Le=0, sm_scale=1.0, dtype=llsa.F32 if dtype == "f32" else llsa.BF16, kernel_path=1)
    O, LSE, idx, ws = llsa.forward(plan, Q, K, V, workspace=plan.alloc_workspace(True))
    dQ, dK, dV = llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)
    z = Q[..., 0].double()
    want = z + torch.log(torch.tensor(64.0, dtype=torch.float64, device="cuda"))
    assert float(((LSE.double() - want).abs() / torch.exp2(torch.floor(torch.log2(want)) - 23)).max()) < 1.0
    P = torch.exp(z - LSE.double())
    out = 0 if dtype == "f32" else 2.0 ** -8                # bf16: the output's own rounding
    assert float((dV.double() / P[..., None, :] - 1).abs().max()) < 4 * 2.0 ** -24 + out
    assert float((dQ[..., 1].double() / (64 * P) - 1).abs().max()) < 38 * 2.0 ** -24 + out


def _tile(name, N, B, K, L, d=64, dtype="f32", heads=2, **kw):
    return dict(name=name, batch=1, heads=heads, d=d, N=N, B=B, K=K, L=L, dtype=dtype, kind="gaussian", **kw)


@pytest.mark.parametrize("cfg", [
    # fp32 tiles: blocks of one and a quarter tile, of two, of less than one; every channel count; lists of 64 and of 65 tokens;
    # a dense level with a ragged last tile; coarse lists split over many workgroups; no coarse level in the list
    _tile("B20_d128", 800, 20, 3, 2, d=128),
    _tile("B32_d16", 2048, 32, 2, 2, d=16),
    _tile("B5_d32", 625, 5, 7, 3, d=32),
    _tile("list_64", 256, 16, 3, 1),
    _tile("list_65", 17 * 16, 16, 3, 1, heads=3),
    _tile("split_lists", 8192, 16, 8, 2, heads=1),
    _tile("B64_Le0", 4096, 64, 2, 2, Le=0),
    _tile("bf16_B8_d64", 512, 8, 4, 3, dtype="bf16"),
    _tile("bf16_B16_d32_Le0", 1024, 16, 4, 2, d=32, dtype="bf16", Le=0),
    # the walk of the list: more than 64 and 128 blocks of it, a dense level cut into blocks with a short last one; bf16 tiles of
    # odd blocks at every channel count; lists split over workgroups
    _tile("blocks_144", 512, 2, 40, 2, d=32),
    _tile("bf16_blocks_144", 512, 2, 40, 2, d=32, dtype="bf16"),
    _tile("bf16_B5_d16", 625, 5, 7, 3, d=16, dtype="bf16"),
    _tile("bf16_B20_d128", 800, 20, 3, 2, d=128, dtype="bf16"),
    _tile("bf16_B3_dense_67", 201, 3, 5, 1, dtype="bf16"),
    _tile("bf16_B48_split", 48 * 48 * 2, 48, 5, 2, dtype="bf16", heads=1),
    _tile("B3_dense_1", 27, 3, 2, 3),
], ids=lambda c: c["name"])
def test_fp32_tiles(cfg):
    _full_parity(cfg, 0xD15B + cfg["N"])


@pytest.mark.parametrize("cfg", [
    # candidates per query at the edges of a wave's 64 and of four waves': 64, 65, 128, 256, 257 and 1024; picks at the edges of
    # the 8- and 16-entry lists; tiles of fewer queries than 16
    _bf16("dense_64", 1024, K=8, heads=2),
    _bf16("dense_65", 1040, K=9, heads=2),
    _bf16("dense_128_K16", 2048, K=16, heads=1),
    _bf16("dense_257_K1", 4112, K=1, heads=1),
    _bf16("sparse_256_K16", 4096, K=16, L=2, heads=1, d=128),
    _bf16("sparse_1024_B64", 65536, K=16, L=2, heads=1, B=64),
    _tile("f32_B4_dense_4", 1024, 4, 3, 4, d=16),
    _tile("f32_B20_dense_340", 6800, 20, 16, 1, d=32, heads=1),
    _tile("f32_B48_d128", 48 * 48, 48, 5, 2, d=128, heads=1),
    _tile("f32_K17", 1024, 4, 17, 2, heads=1),
], ids=lambda c: c["name"])
def test_selection_of_tied_scores(cfg):
    """Inputs of a few integers: many equal scores, so the tie rule (lower key id) decides most rows; lists must be exact."""
    import numpy as np
    from tests import harness as H
    x = {n: np.clip(np.round(v), -1, 1) for n, v in H.make_inputs(cfg, 0xD15C).items()}
    gpu = H.gpu_forward_backward(cfg, x, backward=False)
    for (b, h), r in H.oracle_all_heads(cfg, x, backward=False).items():
        for l in range(cfg["L"]):
            assert np.array_equal(gpu["plan"].level_indices(gpu["indices"], l)[b, h].cpu().numpy(), r["I"][l]), f"level {l}"


_MANY_PICKS = [
    # one pass: 18 and 256 candidates, blocks of 32; two passes with one candidate in the second
    _bf16("K17_of_18", 288, K=17),
    _bf16("K64_of_256", 4096, K=64),
    _bf16("K48_of_128_B32_d128", 4096, B=32, K=48, d=128),
    _bf16("K64_of_257", 4112, K=64),
    # the coarsest level in the same launch: 16 tokens above 256 candidates, 4 above 64
    _bf16("K20_top16_d128", 4096, L=2, K=20, d=128),
    _bf16("K64_top4", 16384, L=3, K=64, heads=1),
]


@pytest.mark.parametrize("heads,N,K,L,Le", [
    (1, 256, 8, 2, 2),                                     # one level-2 token: one pick of it, 16 candidates
    (3, 1024, 8, 2, 2),                                    # four picks: 64 candidates, one a lane
    (2, 1280, 5, 2, 2), (16, 4096, 8, 2, 2), (5, 2304, 1, 2, 1),
    (2, 16384, 8, 2, 2), (7, 16384, 7, 2, 2),              # 64 level-2 tokens, the most that a wave takes; the most workgroups (896)
    (4, 1024, 4, 2, 0),                                    # no coarse level in the lists
    (2, 4096, 8, 3, 3), (1, 12288, 3, 3, 1), (1, 65536, 8, 4, 4),   # level 1's lists come from a launch of their own
])
@pytest.mark.parametrize("kind", ["gaussian", "ties", "constant", "special", "nan"])
def test_lists_selected_by_the_attention(heads, N, K, L, Le, kind):
    """A forward call whose attention selects its own lists against the same call one step at a time: every output bit for bit, whatever the scores are."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    shape = (1, heads, N, 64)
    if kind == "ties":                                     # pooled values and scores take few different values; zeros of both signs
        Q, K_, V = (torch.randint(-1, 2, shape, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
        Q = torch.where(torch.rand(shape, generator=gen, device="cuda") < 0.5, -0.0, Q.float()).bfloat16()
    elif kind == "constant":
        Q, K_, V = (torch.full(shape, 0.5, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    else:
        Q, K_, V = (torch.randn(shape, generator=gen, device="cuda").bfloat16() for _ in range(3))
    if kind == "special":                                  # infinite and NaN scores among the others, scores that underflow
        K_[:, :, 5] = float("inf")
        K_[:, :, N // 2, 3] = float("nan")
        K_[:, 0, N // 4: N // 4 + 64] = 1e-39
        Q[:, :, 40:60] *= 1e-38
    if kind == "nan":                                      # of both signs, several payloads, quiet and not, in single channels of either
        bits = torch.tensor([0x7fc0, -64, 0x7f81, -127, 0x7fff, -1], dtype=torch.int16, device="cuda").view(torch.bfloat16)
        for x, every in ((K_, 7 * 16), (Q, 11 * 16)):
            at = torch.arange(3, N, every, device="cuda")
            x[:, :, at, (5 * at) % 64] = bits[torch.arange(len(at), device="cuda") % 6]
    plan = llsa.Plan(1, heads, N, 64, 16, K, L, Le=Le)
    O, LSE, idx, ws = llsa.forward(plan, Q, K_, V)
    ws1, idx1 = plan.alloc_workspace(False), plan.alloc_indices()
    llsa.pool(plan, Q, K_, V, ws1)
    parent = None
    for l in range(L, 0, -1):
        out = plan.level_indices(idx1, l - 1)
        llsa.select_level(plan, l, ws1, parent, out)
        parent = out
    for l in range(L):
        assert torch.equal(plan.level_indices(idx, l), plan.level_indices(idx1, l)), f"level {l}"
    O1, LSE1 = llsa.attention(plan, Q, K_, V, idx1, ws1)
    assert torch.equal(O.view(torch.int16), O1.view(torch.int16)) and torch.equal(LSE.view(torch.int32), LSE1.view(torch.int32))


@pytest.mark.parametrize("dtype,heads,N,d,B,K,L", [
    ("fp32", 1, 256, 32, 4, 2, 3), ("fp32", 3, 1024, 16, 4, 3, 4),   # one workgroup a head; three levels above
    ("fp32", 2, 16384, 64, 8, 8, 4), ("fp32", 5, 16384, 64, 8, 8, 4),   # 64 candidates: all levels; more workgroups at level 1 (1280) than are few
    ("bf16", 2, 4096, 64, 4, 5, 5),                          # four levels above: a launch more
    ("bf16", 1, 8192, 32, 16, 4, 3), ("bf16", 2, 4096, 128, 2, 9, 7), ("bf16", 1, 16384, 64, 4, 16, 6),
    ("fp32", 1, 13824, 64, 24, 2, 2), ("bf16", 1, 2 * 24 ** 3, 64, 24, 2, 3),   # rows of more than 16 tokens: two tiles a token
])
@pytest.mark.parametrize("kind", ["gaussian", "ties", "constant", "special"])
def test_levels_selected_in_one_launch(dtype, heads, N, d, B, K, L, kind):
    """A forward call, which selects several levels in a launch where they are small, against the same selection level by level."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    shape, t = (1, heads, N, d), torch.float32 if dtype == "fp32" else torch.bfloat16
    if kind == "ties":
        Q, K_, V = (torch.randint(-1, 2, shape, generator=gen, device="cuda").to(t) for _ in range(3))
    elif kind == "constant":
        Q, K_, V = (torch.full(shape, 0.5, device="cuda", dtype=t) for _ in range(3))
    else:
        Q, K_, V = (torch.randn(shape, generator=gen, device="cuda").to(t) for _ in range(3))
    if kind == "special":                                  # infinite and NaN scores among the others, NaN of both signs
        K_[:, :, 5], K_[:, :, N // 4] = float("inf"), float("-inf")
        K_[:, :, N // 2, 3], K_[:, :, N // 3, 1] = float("nan"), -float("nan")
        Q[:, :, N // 5, 2], Q[:, :, 2 * N // 3, 7] = float("nan"), float("inf")
    plan = llsa.Plan(1, heads, N, d, B, K, L, Le=1, dtype=llsa.F32 if dtype == "fp32" else llsa.BF16)
    O, LSE, idx, ws = llsa.forward(plan, Q, K_, V)
    ws1, idx1 = plan.alloc_workspace(False), plan.alloc_indices()
    llsa.pool(plan, Q, K_, V, ws1)
    parent = None
    for l in range(L, 0, -1):
        out = plan.level_indices(idx1, l - 1)
        llsa.select_level(plan, l, ws1, parent, out)
        parent = out
    for l in range(L):
        assert torch.equal(plan.level_indices(idx, l), plan.level_indices(idx1, l)), f"level {l}"


@pytest.mark.parametrize("heads,N,K,L,Le", [
    (1, 256, 8, 1, 1), (3, 256, 4, 1, 1), (16, 512, 8, 2, 1),    # 1, 3 and 32 query blocks of 256 rows: fewer than XCDs, not a multiple of them
    (5, 2816, 16, 2, 2), (2, 4096, 8, 2, 2), (16, 4096, 8, 2, 2), (31, 4096, 8, 2, 2), (1, 8192, 32, 2, 2),
    (2, 4352, 8, 2, 2),                                          # 17 rows: the dense level is not taken along
    (2, 8192, 8, 3, 3), (1, 8192, 60, 2, 2),                     # levels above in kernels of their own; 32 listed blocks, four to a wave
])
def test_dq_takes_the_grouped_kernel_along(heads, N, K, L, Le):
    """A backward pass whose dQ launch does the grouped dK / dV kernel's work too against the pass with a launch for each: every gradient bit for bit."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator(device="cuda").manual_seed(N + K + heads)
    Q, K_, V, dO = (torch.randn((1, heads, N, 64), generator=gen, device="cuda").bfloat16() for _ in range(4))
    plan = llsa.Plan(1, heads, N, 64, 16, K, L, Le=Le)
    ws = plan.alloc_workspace(True)
    O, LSE, idx, ws = llsa.forward(plan, Q, K_, V, workspace=ws)
    grads = llsa.backward(plan, Q, K_, V, O, LSE, idx, dO, ws)
    llsa.stage_timing_begin(-1, 1)                               # (a pass that is timed by its stages runs them one by one)
    apart = llsa.backward(plan, Q, K_, V, O, LSE, idx, dO, ws)
    llsa.stage_timing_end()
    for name, x, y in zip(("dQ", "dK", "dV"), grads, apart):
        assert torch.equal(x.view(torch.int16), y.view(torch.int16)), name


@pytest.mark.parametrize("heads,N,d,B,K,L,dtype", [
    (1, 256, 64, 16, 8, 1, "bf16"), (16, 4096, 64, 16, 8, 2, "bf16"), (31, 4096, 64, 16, 8, 2, "bf16"), (2, 8192, 64, 16, 8, 3, "bf16"),   # few rows at d = 64
    (2, 4096, 128, 16, 8, 2, "bf16"), (2, 16384, 64, 64, 4, 2, "bf16"), (2, 16640, 64, 16, 8, 2, "bf16"), (16, 16384, 64, 16, 8, 2, "bf16"), (3, 1088, 64, 16, 8, 1, "bf16"),
    (2, 1152, 64, 64, 18, 1, "bf16"), (2, 2704, 64, 16, 8, 1, "bf16"), (2, 1024, 32, 4, 3, 3, "f32")])
def test_dq_written_over_o(heads, N, d, B, K, L, dtype):
    """A backward pass that writes dQ over O, by every kernel that makes dQ, against one with a buffer for it: every gradient bit for bit."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator(device="cuda").manual_seed(N + K + heads)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K_, V, dO = (torch.randn((1, heads, N, d), generator=gen, device="cuda").to(t) for _ in range(4))
    plan = llsa.Plan(1, heads, N, d, B, K, L, dtype=llsa.F32 if dtype == "f32" else llsa.BF16)
    O, LSE, idx, ws = llsa.forward(plan, Q, K_, V, workspace=plan.alloc_workspace(True))
    apart = llsa.backward(plan, Q, K_, V, O, LSE, idx, dO, ws)
    over = llsa.backward(plan, Q, K_, V, O, LSE, idx, dO, ws, dQ=O)
    assert over[0].data_ptr() == O.data_ptr()
    for name, x, y in zip(("dQ", "dK", "dV"), apart, over):
        assert torch.equal(x, y), name


@pytest.mark.parametrize("cfg", _MANY_PICKS, ids=lambda c: c["name"])
def test_selection_of_more_than_16(cfg):
    _full_parity(cfg, 0xD165)


@pytest.mark.parametrize("cfg", _MANY_PICKS + [_bf16("K8", 4096, L=2), _tile("f32_K8", 1024, 4, 8, 2), _tile("f32_K17", 1024, 4, 17, 2),
                                               dict(_bf16("K8_path1", 4096, L=2), kernel_path=1)], ids=lambda c: c["name"])
def test_lists_hold_different_blocks_whatever_the_scores_are(cfg):
    """NaN and infinite scores: every list is still K_l different blocks of its range, in ascending order (the attention reads
    what they name)."""
    import torch
    from paper_2512_16615_amd import llsa
    from tests import harness as H
    plan = H.make_plan(cfg, kernel_path=cfg.get("kernel_path", 0))
    x = H.make_inputs(cfg, 0xD166)
    Q, K, V = (H.to_dev(x[n], cfg) for n in ("Q", "K", "V"))
    N, B = cfg["N"], cfg["B"]
    K[:, :, :B, 0], K[:, :, 2 * B:3 * B, 1], K[:, :, 5 * B:6 * B, 2] = float("nan"), float("-inf"), float("inf")
    Q[:, :, B:2 * B], Q[:, :, N // 2:] = float("nan"), float("inf")
    idx = llsa.forward(plan, Q, K, V)[2]
    for l in range(cfg["L"]):
        lists = plan.level_indices(idx, l).cpu()
        assert int(lists.min()) >= 0 and int(lists.max()) < N // B ** (l + 1)
        assert bool((lists.diff(dim=-1) > 0).all())


@pytest.mark.parametrize("T,K,heads", [(1, 1, 2), (33, 3, 3), (64, 8, 2), (65, 5, 2), (512, 8, 2), (513, 3, 2), (1025, 8, 2),
                                         (2048, 64, 1), (4099, 7, 2), (16384, 8, 1), (16385, 2, 1)])
def test_index_transpose_by_size(T, K, heads):
    """Alg. 2 on forced lists at the edges of its paths: few rows, rows that fill no 64-row word, segment, group or key range, the
    largest level of each path and the smallest beyond it; one key listed by every row, the last keys listed by none."""
    import numpy as np
    import torch
    from oracle import llsa_oracle as orc
    from tests import harness as H
    from paper_2512_16615_amd import llsa
    cfg = dict(batch=1, heads=heads, d=64, N=16 * T, B=16, K=K, L=1, dtype="bf16")
    plan = H.make_plan(cfg)
    ws, idx = plan.alloc_workspace(True), plan.alloc_indices()
    rng = np.random.default_rng(T)
    top = max(K, T - T // 8)
    I = np.stack([np.stack([np.sort(rng.choice(min(top, 4 * K) if r % 3 else top, K, replace=False)) for r in range(T)])
                  for _ in range(heads)]).astype(np.int32)
    I[0, :, 0] = 0
    for r in range(T):                                       # keep the rows ascending and distinct with key 0 in each
        if K > 1 and I[0, r, 1] == 0:
            I[0, r] = np.arange(K)
    plan.level_indices(idx, 0).copy_(torch.from_numpy(I).cuda().view(1, heads, T, K))
    ws.fill_(0x7F)
    llsa.index_transpose(plan, idx, ws)
    torch.cuda.synchronize()
    C, Iq = plan.csc_level(ws, 0)
    for h in range(heads):
        iq_ref, c_ref = orc.transpose(I[h], T)
        assert np.array_equal(C[h].cpu().numpy(), c_ref)
        assert np.array_equal(Iq[h].cpu().numpy(), iq_ref)


@pytest.mark.parametrize("heads,N,L,d,Le", [
    # every query lists the first K blocks: lists of all T = N / 16 query blocks beside T - K empty ones.  Pieces of 8 tiles: 4 tiles, 10 and
    # 12 (the first that are cut), 32 and 34 (one window of places and its end), no parent, of 14 tiles a wave at d = 128; of 16 at either width; and,
    # in waves of eight places, of 32 at either width (229376 places in all) and of 64 (d = 128, 573440)
    (1, 64, 1, 64, 1), (2, 320, 1, 64, 1), (3, 384, 1, 64, 0), (1, 1024, 1, 64, 1), (2, 1088, 1, 64, 1), (1, 1088, 1, 128, 1),
    (16, 16384, 2, 64, 2), (8, 65536, 3, 64, 3), (8, 16384, 2, 128, 2), (16, 16384, 2, 128, 2), (16, 65536, 3, 64, 3), (8, 131072, 3, 128, 3),
    (10, 262144, 3, 128, 3),
    (5, 16640, 2, 64, 2), (7, 69632, 3, 64, 3)])             # waves of three places and of six, which the places are no multiple of
def test_level0_lists_of_every_query(heads, N, L, d, Le):
    """dK and dV where lists are cut into pieces that several waves add up: within the bf16 kernels' rounding of the fp32-arithmetic kernels,
    and the same bits every time, whichever wave comes last."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, V, dO = (torch.randn(1, heads, N, d, generator=gen, device="cuda").bfloat16() for _ in range(3))
    K = torch.ones_like(Q)
    got = []
    for path in (0, 1):
        plan = llsa.Plan(1, heads, N, d, 16, 6, L, Le=Le, kernel_path=path)
        O, LSE, idx, ws = llsa.forward(plan, Q, K, V, workspace=plan.alloc_workspace(True))
        got.append(llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws))
        for _ in range(3 if path == 0 else 0):
            for a, b in zip(got[0], llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)):
                assert torch.equal(a, b)
    for name, a, b in zip(("dQ", "dK", "dV"), *got):
        if name == "dQ":
            continue                                        # K is constant: dQ is a sum that cancels
        rel = float((a.double() - b.double()).norm() / b.double().norm())
        assert rel < 1e-2, (name, rel)


@pytest.mark.parametrize("heads,N,d,K", [
    # few picks of heads of more than 16 MB of Q and dO: XCDs take 64 waves at a time, the last few hundred waves one each; and just below
    (1, 66560, 64, 3), (3, 66560, 64, 4), (1, 33792, 128, 4), (2, 65536, 64, 4), (1, 66560, 64, 5)])
def test_level0_waves_dealt_in_stretches(heads, N, d, K, L=2):
    """Every row of dK and dV is written, within the bf16 kernels' rounding of P and dS of the fp32-arithmetic kernels."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    Q, Kt, V, dO = (torch.randn(1, heads, N, d, generator=gen, device="cuda").bfloat16() for _ in range(4))
    got = []
    for path in (0, 1):
        plan = llsa.Plan(1, heads, N, d, 16, K, L, kernel_path=path)
        O, LSE, idx, ws = llsa.forward(plan, Q, Kt, V, workspace=plan.alloc_workspace(True))
        out = [torch.full_like(Q, float("nan")) for _ in range(3)]
        got.append(llsa.backward(plan, Q, Kt, V, O, LSE, idx, dO, ws, *out))
    for name, a, b in list(zip(("dQ", "dK", "dV"), *got))[1:]:
        rel = float((a.double() - b.double()).norm() / b.double().norm())
        assert rel < 1e-2, (name, rel)


@pytest.mark.parametrize("heads,N,d,K", [
    # no multiple of eight heads: all heads' waves for tiles, then their waves for key blocks that nothing lists (K = 1: a third of them).  Fewer
    # waves than XCDs, a last wave with a few blocks, as many waves of one kind as of the other, lists of 12; and eight heads, one after the other
    (1, 64, 64, 1), (3, 320, 64, 1), (7, 1088, 64, 1), (9, 1088, 128, 1), (12, 8256, 64, 1), (5, 16640, 128, 8), (2, 33024, 64, 12), (8, 1088, 64, 1)])
def test_level0_waves_of_several_heads(heads, N, d, K):
    """Every row of dK and dV is written, within the bf16 kernels' rounding of P and dS of the fp32-arithmetic kernels."""
    test_level0_waves_dealt_in_stretches(heads, N, d, K, L=1 if N % 256 else 2)


@pytest.mark.parametrize("heads,N,K", [(1, 256, 8), (3, 2816, 4), (16, 4096, 8), (73, 3840, 8)])
def test_gather_adds_up_a_dense_parent(heads, N, K):
    """Level 1's gather with 1, 11, 16 and 15 partials of a parent token, the last in more workgroups (1095) than are few, against the general path."""
    test_level0_waves_dealt_in_stretches(heads, N, 64, K, L=2)


@pytest.mark.parametrize("heads,N,d,K,L", [
    # the tiles of level 0's lists, written along with the lists from 513 to 16384 rows (516: 5 segments share 1024 keys; one range of keys and
    # the first keys of the next; two groups of segments; all 128 segments) and by a launch of their own beyond
    (3, 8256, 64, 1, 1), (1, 16384, 64, 8, 2), (2, 16640, 128, 3, 2), (1, 33024, 64, 8, 2), (1, 262144, 64, 2, 3), (1, 262400, 64, 2, 2)])
def test_level0_tiles_by_number_of_rows(heads, N, d, K, L):
    """Every row of dK and dV is written, within the bf16 kernels' rounding of P and dS of the fp32-arithmetic kernels."""
    test_level0_waves_dealt_in_stretches(heads, N, d, K, L)


@pytest.mark.parametrize("heads,N,L,d", [
    # partials of levels >= 1 added eight at a time: lists of 1, 7, 8, 9 and 17 query blocks beside empty ones, of more than the threads of a
    # workgroup (272 of 256; 528 of 512 at d = 128), of an upper level; one launch of more than 1024 workgroups, which add them one by one
    (2, 256, 2, 64), (2, 7 * 256, 2, 64), (2, 8 * 256, 2, 64), (2, 9 * 256, 2, 128), (1, 17 * 256, 2, 64), (3, 272 * 256, 2, 64),
    (1, 528 * 256, 2, 128), (2, 16384, 3, 64), (2, 16384, 3, 128), (5, 207 * 256, 2, 64)])
def test_gather_of_lists_of_every_query(heads, N, L, d):
    test_level0_lists_of_every_query(heads, N, L, d, L)


@pytest.mark.parametrize("cfg", [
    # the dense level 2 in the group kernel: one token (one query block a head), a ragged tile, all 16; two passes of listed blocks behind it;
    # the widest launch that the chain kernel does not take yet, and the first one that it does
    _bf16("top_1", 256, L=2, heads=3, K=1),
    _bf16("top_5_K3", 5 * 256, L=2, heads=2, K=3),
    _bf16("top_16_K12", 4096, L=2, heads=2, K=12),
    _bf16("top_15_K16", 15 * 256, L=2, heads=1, K=16),
    _bf16("top_16_heads_63", 4096, L=2, heads=63, K=2),
    _bf16("top_16_heads_64", 4096, L=2, heads=64, K=2),
], ids=lambda c: c["name"])
def test_dense_level_in_the_group_kernel(cfg):
    _full_parity(cfg, 0xD16C)


@pytest.mark.parametrize("cfg", [
    # at most 512 level-0 rows: one row, a ragged range of 32 keys, the most; workgroups of eight and of four waves; blocks of 64; fp32
    # arithmetic in both types
    _bf16("rows_4_L1", 64, K=2, heads=1),
    _bf16("rows_80", 1280, L=2, heads=3, K=5),
    _bf16("rows_512", 8192, L=2, heads=2),
    _bf16("rows_256_of_64_heads", 4096, L=2, heads=64),
    _bf16("rows_256_B64", 16384, B=64, K=4, L=2, heads=2),
    _bf16("rows_48_d128_Le0", 768, d=128, K=3, heads=2, Le=0),
    _bf16("rows_169_tiles", 2704, heads=2),
    dict(name="rows_500_f32", batch=1, heads=3, d=32, N=2000, B=4, K=3, L=2, dtype="f32", kind="gaussian"),
], ids=lambda c: c["name"])
def test_lists_made_along_with_dq(cfg):
    """The key-major lists that the dQ launch makes are those of the index transpose by itself, whole numbers for whole numbers."""
    import torch
    from paper_2512_16615_amd import llsa
    from tests import harness as H
    x = H.make_inputs(cfg, 0xD16B)
    Q, K, V, dO = (H.to_dev(x[n], cfg) for n in ("Q", "K", "V", "dO"))
    plan = H.make_plan(cfg)
    ws = plan.alloc_workspace(True)
    O, LSE, idx, _ = llsa.forward(plan, Q, K, V, workspace=ws)
    llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)
    levels = range(min(plan.Le + 1, plan.L))
    got = [[t.clone() for t in plan.csc_level(ws, l)] for l in levels]
    other = plan.alloc_workspace(True)
    other.zero_()
    llsa.index_transpose(plan, idx, other)
    for l in levels:
        for a, b in zip(got[l], plan.csc_level(other, l)):
            assert torch.equal(a, b), f"level {l}"


@pytest.mark.parametrize("cfg", [
    # levels >= 2 of the grouped dK/dV kernels: a dense level of two blocks (17 tokens), of 16 blocks behind no sparse level, of
    # two blocks behind 8 listed ones; its single block owned by a wave (3 and 12 listed blocks) and shared by all (8)
    _bf16("dense_17", 17 * 256, L=2, heads=2),
    _bf16("dense_256", 65536, L=2, heads=1, K=4),
    _bf16("dense_18_K8", 18 * 4096, L=3, heads=1),
    _bf16("dense_13_K3", 13 * 4096, L=3, heads=1, K=3),
    _bf16("dense_12_K12", 12 * 4096, L=3, heads=1, K=12),
    _bf16("dense_8_K8", 8 * 4096, L=3, heads=1),
    # d = 128, query groups of one or two query blocks: the dense level in the split kernel
    _bf16("dense_7_K7_d128", 7 * 4096, L=3, heads=1, K=7, d=128),
    _bf16("dense_17_K4_d128", 17 * 4096, L=3, heads=1, K=4, d=128),
    _bf16("dense_12_K12_d128", 12 * 4096, L=3, heads=1, K=12, d=128),
    _bf16("dense_8_K8_d128", 8 * 4096, L=3, heads=1, d=128),
    _bf16("dense_2_heads16_d128", 2 * 4096, L=3, heads=16, d=128),
    # d = 128, of four: owned by waves in a share that has one to spare (a ragged tile; two blocks behind 4 listed ones: a share of their own), in
    # a share of its own behind 8
    _bf16("dense_7_K7_heads10_d128", 7 * 4096, L=3, heads=10, K=7, d=128),
    _bf16("dense_17_K4_heads4_d128", 17 * 4096, L=3, heads=4, K=4, d=128),
    _bf16("dense_8_K8_heads8_d128", 8 * 4096, L=3, heads=8, d=128),
], ids=lambda c: c["name"])
def test_grouped_upper_levels(cfg):
    _full_parity(cfg, 0xD15E)


@pytest.mark.parametrize("cfg", [
    # dK/dV of key blocks of several tiles: blocks of 32 (two waves a tile) and 64, at d = 64 and 128; lists split over
    # workgroups; dense levels of 33, 65 and 129 tokens (a ragged tile, a spare wave, a spare block) under an odd number of query
    # tiles; no coarse level in the list
    _bf16("B32_L2", 32 * 1024, L=2, heads=1, B=32, K=4),
    _bf16("B32_d128", 32 * 33, heads=2, B=32, K=4, d=128),
    _bf16("B64_d128", 64 * 65, heads=1, B=64, K=2, d=128),
    _bf16("B64_L2_split", 64 * 64 * 33, L=2, heads=1, B=64, K=3),
    _bf16("B64_Le0", 64 * 20, heads=2, B=64, K=4, Le=0),
    _bf16("dense_129", 16 * 129, heads=2),
    _bf16("dense_33_d128", 16 * 33, heads=2, d=128),
    _bf16("dense_65_L2_d128", 256 * 65, L=2, heads=1, d=128, K=4),
], ids=lambda c: c["name"])
def test_key_blocks_of_several_tiles(cfg):
    _full_parity(cfg, 0xD15F)


@pytest.mark.parametrize("heads,N,B,d,L", [
    # every query lists the same key blocks: tiles in a ring of two or three places, taken in turn by one group of waves (blocks of 64) or two.
    # 1 tile a group, 2, 3, 4, 5 and 7; lists of more than 64 entries, the next 64 looked up while tiles are on their way; a level 1 whose lists
    # are shared out; d = 128
    (2, 64, 32, 64, 1), (1, 128, 32, 64, 1), (3, 192, 32, 64, 1), (1, 448, 32, 128, 1), (1, 2112, 32, 64, 1), (2, 32768, 32, 64, 2),
    (2, 64, 64, 64, 1), (3, 192, 64, 64, 1), (1, 320, 64, 128, 1), (1, 4160, 64, 64, 1), (1, 4160, 64, 128, 1), (2, 36864, 64, 64, 2),
    (1, 36864, 64, 128, 2)])
def test_key_blocks_of_several_tiles_listed_by_every_query(heads, N, B, d, L):
    """dK and dV within the bf16 kernels' rounding of P and dS of the fp32-arithmetic kernels, and the same bits every time."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator(device="cuda").manual_seed(N + B)
    Q, V, dO = (torch.randn(1, heads, N, d, generator=gen, device="cuda").bfloat16() for _ in range(3))
    K = torch.ones_like(Q)
    got = []
    for path in (0, 1):
        plan = llsa.Plan(1, heads, N, d, B, 6, L, kernel_path=path)
        O, LSE, idx, ws = llsa.forward(plan, Q, K, V, workspace=plan.alloc_workspace(True))
        got.append([x.clone() for x in llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)])
        for _ in range(2 if path == 0 else 0):
            for a, b in zip(got[0], llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)):
                assert torch.equal(a, b)
    for name, a, b in list(zip(("dQ", "dK", "dV"), *got))[1:]:   # K is constant: dQ is a sum that cancels
        rel = float((a.double() - b.double()).norm() / b.double().norm())
        assert rel < 1e-2, (name, rel)


@pytest.mark.parametrize("cfg", [
    # the fp32-arithmetic kernels (no multiple of 64) on a chip full of query tiles, on lists of 33 blocks, on blocks of two tiles
    _bf16("B16_400_heads256", 400, heads=256),
    _bf16("B32_416_heads256", 416, heads=256, B=32, K=3),
    _bf16("K33", 16 * 43, heads=2, K=33),
    _bf16("K33_d128", 16 * 43, heads=2, K=33, d=128),
    _bf16("B32_odd_d128", 32 * 21, heads=2, B=32, K=5, d=128),
], ids=lambda c: c["name"])
def test_bf16_tiles_by_size(cfg):
    _full_parity(cfg, 0xD160)


@pytest.mark.parametrize("cfg", [
    # query tiles per wave of the shared forward (multiples of 256) and dQ (of 64): from 1024 workgroups on two at d = 64, the
    # last workgroup of a head ragged, blocks of 16, 32 and 64; lists longer than a pair of tiles may have (33 and 64 blocks)
    # at d = 64 and, with 128 KB of rows in LDS, at d = 128, spare waves among them (1088 tokens); blocks of 32 at d = 128
    _bf16("B16_1024_wgs", 448, heads=256),
    _bf16("B32_1024_wgs", 448, heads=256, B=32, K=3),
    _bf16("B64_1026_wgs", 320, heads=342, B=64, K=2),
    _bf16("B16_256_1024_wgs", 256, heads=512),
    _bf16("K33", 1024, heads=2, K=33),
    _bf16("K33_d128", 1024, heads=2, K=33, d=128),
    _bf16("K64_d128", 1280, heads=2, K=64, d=128),
    _bf16("K33_d128_17", 1088, heads=2, K=33, d=128),
    _bf16("K64_d128_17", 1088, heads=2, K=64, d=128),
    _bf16("B32_d128_11", 32 * 22, heads=2, B=32, K=5, d=128),
    _bf16("B32_d128", 1280, heads=2, B=32, K=32, d=128),
], ids=lambda c: c["name"])
def test_query_tiles_per_wave(cfg):
    _full_parity(cfg, 0xD160)


@pytest.mark.parametrize("cfg", [
    # level-1 dK/dV carried along 2 or 4 query blocks (heads x level-1 query blocks >= 1024): rows shorter than the register
    # slots, rows of all slots, rows that two workgroups share, at d = 64 and 128
    _bf16("chain_K3", 8192, L=2, heads=32, K=3),
    _bf16("chain_K4", 8192, L=2, heads=64, K=4),
    _bf16("chain_K6", 8192, L=2, heads=32, K=6),
    _bf16("chain_K9", 8192, L=2, heads=32, K=9),
    _bf16("chain_K16", 8192, L=2, heads=32, K=16),
    _bf16("chain_K9_d128", 8192, L=2, heads=32, K=9, d=128),
    _bf16("chain_K6_d128", 8192, L=2, heads=32, K=6, d=128),
    _bf16("chain_K8_d128", 8192, L=2, heads=32, K=8, d=128),
], ids=lambda c: c["name"])
def test_level1_sums_carried_along_query_blocks(cfg):
    _full_parity(cfg, 0xD161)


@pytest.mark.parametrize("cfg", [
    # d = 128, workgroups of four waves: level 1 of one, three and four listed blocks; levels >= 2 of 1, 5 and 9 listed blocks (one share, two and
    # three, the last with one block)
    _bf16("chain_K1", 8192, L=2, heads=32, K=1, d=128),
    _bf16("chain_K3", 8192, L=2, heads=32, K=3, d=128),
    _bf16("chain_K4", 8192, L=2, heads=32, K=4, d=128),
    _bf16("upper_K1", 2 * 4096, L=3, heads=2, K=1, d=128),
    _bf16("upper_K5", 9 * 4096, L=3, heads=1, K=5, d=128),
    _bf16("upper_K9", 10 * 4096, L=3, heads=1, K=9, d=128),
], ids=lambda c: c["name"])
def test_coarse_levels_of_wide_heads(cfg):
    _full_parity(cfg, 0xD162)


@pytest.mark.parametrize("heads,K,d", [(64, 3, 64), (64, 6, 64), (32, 8, 64), (64, 6, 128), (64, 8, 128), (64, 12, 64), (32, 16, 128)])
def test_level1_sums_carried_through_several_query_blocks(heads, K, d):
    """Chains of 8 (heads x level-1 query blocks >= 4096) or 4 query blocks on smooth inputs, whose blocks stay listed: slots are kept,
    released and taken again several times.  Two heads' inputs, repeated, so that the oracle has two to do."""
    import torch
    from paper_2512_16615_amd import llsa
    from tests import harness as H
    two = _bf16(f"chain_K{K}_d{d}", 16384, L=2, heads=2, K=K, d=d, kind="smooth")
    x = H.make_inputs(two, 0xD168)
    Q, Kt, V, dO = (H.to_dev(x[n], two).repeat(1, heads // 2, 1, 1) for n in ("Q", "K", "V", "dO"))
    plan = H.make_plan(dict(two, heads=heads))
    O, LSE, idx, ws = llsa.forward(plan, Q, Kt, V, workspace=plan.alloc_workspace(True))
    got = dict(zip(("dQ", "dK", "dV"), llsa.backward(plan, Q, Kt, V, O, LSE, idx, dO, ws)))
    tol = H.TOL["bf16"]
    for (b, h), r in H.oracle_all_heads(two, x).items():
        for l in range(2):
            assert (plan.level_indices(idx, l)[b, h].cpu().numpy() == r["I"][l]).all(), f"level {l}"
        for n, t in got.items():
            H.check_close(f"{n}{(b, h)}", H.f32(t[b, h]), r[n], tol["out"], tol["ulp"])
            assert torch.equal(t[:, h::2], t[:, h:h + 1].expand_as(t[:, h::2])), n


def _key_gradients_64(plan, ws, idx, Q, K, V, O, LSE, dO):
    """dK and dV of head 0 in 64 bits from the forward's lists, pooled levels, O and logsumexp, and the root of the sum of the squares of
    the terms that each of their elements adds up."""
    import math
    import torch
    B, N, d, scale = plan.B, plan.N, plan.d, plan.d ** -0.5
    q, g, lse = Q[0, 0].double(), dO[0, 0].double(), LSE[0, 0].double()
    D = (g * O[0, 0].double()).sum(-1)
    levels = []
    for l in range(plan.Le + 1):
        k, v = ((t if l == 0 else plan.pyramid_level(ws, x, l))[0, 0].double() for t, x in ((K, 1), (V, 2)))
        toks = torch.arange(len(k), device="cuda")[None]
        if l < plan.L:
            toks = (plan.level_indices(idx, l)[0, 0].long()[:, :, None] * B + torch.arange(B, device="cuda")).flatten(1)
        rows, n, T = len(toks), N // len(toks), toks.shape[1]
        dk, dv, k2, v2 = (torch.zeros_like(k) for _ in range(4))
        c = min(n, 4096)
        step = max(1, (1 << 24) // (T * max(c, d)))
        for r in range(0, rows, step):
            tk = toks[r:r + step]
            kt, vt = k[tk].transpose(1, 2).contiguous(), v[tk].transpose(1, 2).contiguous()
            for x in range(0, n, c):
                qq, gg, ll, dd = (t.view(rows, n, -1)[r:r + step, x:x + c] for t in (q, g, lse, D))
                P = torch.exp(torch.matmul(qq, kt) * scale + l * math.log(B) - ll)
                dS = P * (torch.matmul(gg, vt) - dd) * scale
                for out, w, t in ((dk, dS, qq), (dv, P, gg), (k2, dS * dS, qq * qq), (v2, P * P, gg * gg)):
                    out.index_add_(0, tk.flatten(), torch.matmul(w.transpose(1, 2), t.contiguous()).flatten(0, 1))
        levels.append([dk, dv, k2, v2])
    for l in range(plan.Le, 0, -1):
        for x in range(4):
            levels[l - 1][x] += levels[l][x].repeat_interleave(B, 0) / (B if x < 2 else B * B)
    return {"dK": (levels[0][0], levels[0][2].sqrt()), "dV": (levels[0][1], levels[0][3].sqrt())}


def _check_key_gradients(N, d, K, L, heads, side):
    """Heads alike, so that one is enough for 64 bits.  dS and P enter their products rounded to bf16 (each term off by up to 2^-9 of
    itself, independently: 2^-9 / sqrt(3) of the root of the sum of their squares, of which 8 are allowed for the largest of some
    10^7 elements), the result is rounded once, and fp32 sums and exponentials are off by some 1e-6 of values of up to 10."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K)
    rand = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")
    y, x = torch.meshgrid(torch.arange(N // side, device="cuda"), torch.arange(side, device="cuda"), indexing="ij")
    wave = torch.stack([torch.sin(2 * torch.pi * (a * x + b * y) / side + c) for a, b, c in [(1, 0, 0), (0, 1, 1), (2, 1, 2), (1, 2, 3)]], -1)
    Q, Kt = (wave.reshape(N, 4) @ rand(4, d) + 0.1 * rand(N, d) for _ in range(2))
    Q, Kt, V, dO = (t.bfloat16().expand(1, heads, N, d).contiguous() for t in (Q, Kt, rand(N, d), rand(N, d)))
    plan = llsa.Plan(1, heads, N, d, 16, K, L)
    O, LSE, idx, ws = llsa.forward(plan, Q, Kt, V, workspace=plan.alloc_workspace(True))
    got = dict(zip(("dK", "dV"), llsa.backward(plan, Q, Kt, V, O, LSE, idx, dO, ws)[1:]))
    for n, (want, rms) in _key_gradients_64(plan, ws, idx, Q, Kt, V, O, LSE, dO).items():
        assert torch.equal(got[n], got[n][:, :1].expand_as(got[n])), n
        over = (got[n][0, 0].double() - want).abs() - (8 / 3 ** 0.5 * 2.0 ** -9 * rms + 2.0 ** -8 * want.abs())
        assert float(over.max()) < 5e-6, n


@pytest.mark.parametrize("K,d,side", [(8, 64, 512), (12, 64, 512), (16, 128, 512), (5, 64, 1024), (12, 64, 1024), (8, 128, 1024)])
def test_level1_sums_carried_to_the_query_block_below(K, d, side):
    """Chains of query blocks 2 (262144 tokens) and 4 (1048576) apart, whose partials the gather finds."""
    _check_key_gradients(side * side, d, K, 2, heads=4 if side == 512 else 2, side=side)


@pytest.mark.parametrize("N,d,K,L", [(260 * 256, 64, 4, 2), (262144, 64, 20, 4), (262144, 128, 20, 4), (36864, 64, 12, 3), (139264, 64, 16, 3)])
def test_listed_blocks_of_the_upper_levels_shared_by_workgroups(N, d, K, L):
    """Blocks of levels >= 2 of a query group: 17 (three workgroups of eight, the last with a ragged block of four tokens), 24 and a
    dense block that all waves share (three of eight, the first takes it), 24 and a dense one at d = 128 (seven of four), 13 (one of 16),
    18 (three of eight)."""
    _check_key_gradients(N, d, K, L, heads=2, side=256)


def _all_listed_64(plan, ws, Q, K, V, O, dO):
    """Attention and gradients in 64 bits where every block is listed: softmax over all tokens and, with Le = 1, the pooled ones.  D from
    the O given, as in the backward."""
    import math
    import torch
    q, k, v, o, g = (x.double().cpu() for x in (Q, K, V, O, dO))
    bias = torch.zeros(plan.N, dtype=torch.float64)
    if plan.Le:
        k, v = (torch.cat([x, plan.pyramid_level(ws, i, 1).double().cpu()], 2) for x, i in ((k, 1), (v, 2)))
        bias = torch.cat([bias, torch.full((plan.N // plan.B,), math.log(plan.B), dtype=torch.float64)])
    scale = plan.d ** -0.5
    P = torch.softmax(torch.matmul(q, k.transpose(2, 3)) * scale + bias, -1)
    dS = P * (torch.matmul(g, v.transpose(2, 3)) - (g * o).sum(-1, keepdim=True)) * scale
    out = {"O": torch.matmul(P, v), "dQ": torch.matmul(dS, k), "dK": torch.matmul(dS.transpose(2, 3), q), "dV": torch.matmul(P.transpose(2, 3), g)}
    if plan.Le:
        for n in ("dK", "dV"):
            out[n] = out[n][:, :, :plan.N] + out[n][:, :, plan.N:].repeat_interleave(plan.B, 2) / plan.B
    return out


def _check_infinities(got, want, tol=2e-2):
    """An infinity where 64 bits give one, a value where they give one (where they give a NaN, anything)."""
    import torch
    for n, t in got.items():
        x, w = t.double().cpu(), want[n]
        inf, fin = torch.isinf(w), torch.isfinite(w)
        assert torch.equal(x[inf], w[inf]), f"{n}: {int((x[inf] != w[inf]).sum())} of {int(inf.sum())} infinities are something else"
        assert bool(((x[fin] - w[fin]).abs() <= tol).all()), n


@pytest.mark.parametrize("d,B,N,Le,path", [
    # lists of an odd multiple of 16 tokens (half a tile of 32 past the end), with and without a dense level, every channel count, lists
    # that end inside 16 tokens, a length that the bf16 MFMA kernels take
    (64, 16, 144, 0, 0), (64, 16, 144, 1, 0), (128, 16, 144, 0, 0), (32, 8, 104, 0, 0), (16, 16, 80, 1, 0), (64, 5, 105, 1, 0),
    (128, 20, 180, 1, 0), (64, 16, 512, 1, 1), (16, 4, 208, 0, 0), (64, 32, 96, 0, 0),
])
def test_infinite_values_in_bf16_tiles(d, B, N, Le, path):
    """bf16 shapes in fp32 arithmetic, whose P and dS enter their products in three parts: an infinite row times a part that is 0, or
    an infinite dS, must not become a NaN.  Heads: an infinite V at the last key; at another; an infinite dO at the last query; at
    another; neither.  A query of zeros has P = 1 before the sum: two of its parts are 0."""
    import torch
    from paper_2512_16615_amd import llsa
    gen = torch.Generator().manual_seed(N + d)
    Q, K, V, dO = torch.randn(4, 1, 5, N, d, generator=gen)
    c = d // 2 + 1
    Q[..., 0], dO[..., c] = Q[..., 0].abs() + 0.1, dO[..., c].abs() + 0.1     # so that infinite dS add up with one sign
    Q[:, :, 3] = 0
    V[:, 0, N - 1, c] = V[:, 1, 7, c] = dO[:, 2, N - 1, c] = float("inf")
    dO[:, 3, 5, c] = float("-inf")
    Q, K, V, dO = (x.bfloat16().cuda() for x in (Q, K, V, dO))
    plan = llsa.Plan(1, 5, N, d, B, N // B, 1, Le=Le, kernel_path=path)
    O, LSE, idx, ws = llsa.forward(plan, Q, K, V, workspace=plan.alloc_workspace(True))
    got = dict(zip(("dQ", "dK", "dV"), llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)), O=O)
    want = _all_listed_64(plan, ws, Q, K, V, O, dO)
    assert int(torch.isinf(want["O"]).sum()) and int(torch.isinf(want["dV"]).sum()) and int(torch.isinf(want["dK"]).sum())
    _check_infinities(got, want)
