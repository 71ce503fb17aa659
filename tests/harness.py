"""Shared helpers of the GPU parity tests: seeded inputs -> GPU library and CPU oracle -> comparisons.

Tolerances (written here once, used by every parity test):
  * pooled levels: bit-exact (the pooling order and rounding are a contract, selection depends on them);
  * selection indices: bit-exact, level by level with teacher forcing (the oracle's level-l selection is fed the
    GPU's own parent lists); a row may differ only where the gap between the K-th and (K+1)-th fp64 score is
    below 1e-5 relative;
  * O, dQ, dK, dV: plain max-abs error <= 2e-2 (bf16 I/O) or 1e-4 (fp32 I/O), as stated for this build; no
    scaling with the magnitude of the value.  (check_close can add a term `ulp * |ref|`; every parity test passes
    ulp = 0.)  Every comparison records the max-abs error, the largest |ref| and the number of elements above the
    bound (`STATS`, written to parity_stats.json at the end of a GPU test session);
  * LSE (always fp32): plain 1e-4 (fp32 I/O) or 1e-3 (bf16 I/O).
"""
from __future__ import annotations

import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

from oracle import llsa_oracle as orc
from paper_2512_16615_amd import inputs, llsa

BF16_ULP = 0.0          # no magnitude-scaled term: the plain bound holds on every shape tested (largest error seen 1.9e-2, on an edge case with a large softmax scale)
TOL = {"f32": dict(out=1e-4, lse=1e-4, ulp=0.0), "bf16": dict(out=2e-2, lse=1e-3, ulp=BF16_ULP)}
STATS: dict = {}        # output kind -> observed figures over every comparison of the session


def make_inputs(cfg: dict, seed: int):
    """fp32 numpy tensors [batch, heads, N, d] already rounded to the I/O type."""
    out = {}
    for name in ("Q", "K", "V", "dO"):
        x = inputs.make_tensor(cfg["kind"], seed, name, cfg["batch"], cfg["heads"], cfg["N"], cfg["d"])
        out[name] = orc.to_bf16(x) if cfg["dtype"] == "bf16" else x
    return out


def to_dev(x: np.ndarray, cfg: dict) -> torch.Tensor:
    t = torch.from_numpy(x).cuda()
    return t.to(torch.bfloat16) if cfg["dtype"] == "bf16" else t   # exact: values are bf16-representable


def make_plan(cfg: dict, **kw) -> llsa.Plan:
    args = dict(batch=cfg["batch"], heads=cfg["heads"], N=cfg["N"], d=cfg["d"], B=cfg["B"], K=cfg["K"], L=cfg["L"],
                Le=cfg.get("Le"), dtype=llsa.BF16 if cfg["dtype"] == "bf16" else llsa.F32,
                reweight=cfg.get("reweight", 1), sm_scale=cfg.get("sm_scale", 0.0))
    args.update(kw)
    return llsa.Plan(**args)


def gpu_forward_backward(cfg: dict, x: dict, plan: llsa.Plan | None = None, backward: bool = True):
    plan = plan or make_plan(cfg)
    Q, K, V, dO = (to_dev(x[n], cfg) for n in ("Q", "K", "V", "dO"))
    ws = plan.alloc_workspace(True)
    O, LSE, idx, _ = llsa.forward(plan, Q, K, V, workspace=ws)
    res = {"plan": plan, "O": O, "LSE": LSE, "indices": idx, "ws": ws, "Q": Q, "K": K, "V": V, "dO": dO}
    if backward:
        res["dQ"], res["dK"], res["dV"] = llsa.backward(plan, Q, K, V, O, LSE, idx, dO, ws)
    torch.cuda.synchronize()
    return res


def geometry(cfg: dict) -> orc.Geometry:
    return orc.Geometry(cfg["N"], cfg["d"], cfg["B"], cfg["K"], cfg["L"])


def oracle_head(cfg: dict, x: dict, b: int, h: int, backward: bool = True, rows=None):
    g = geometry(cfg)
    Le = cfg.get("Le")
    Le = g.L if Le is None else Le
    sc = cfg.get("sm_scale", 0.0)
    sc = None if sc <= 0 else sc
    f = orc.forward(x["Q"][b, h], x["K"][b, h], x["V"][b, h], g, Le=Le, bf16=cfg["dtype"] == "bf16",
                    reweight=cfg.get("reweight", 1), scale=sc, rows=rows, want_margin=True)
    if backward:
        f.update(orc.backward(x["Q"][b, h], f["Kp"], f["Vp"], f["idx_cat"], x["dO"][b, h], g, Le=Le,
                              reweight=cfg.get("reweight", 1), scale=sc))
    return f


def oracle_all_heads(cfg: dict, x: dict, heads=None, backward: bool = True, threads: int = 8):
    heads = heads or [(b, h) for b in range(cfg["batch"]) for h in range(cfg["heads"])]
    with ThreadPoolExecutor(max_workers=threads) as ex:
        res = list(ex.map(lambda bh: oracle_head(cfg, x, bh[0], bh[1], backward), heads))
    return dict(zip(heads, res))


def f32(t: torch.Tensor) -> np.ndarray:
    return t.detach().float().cpu().numpy()


def check_pyramid(cfg, gpu, ref, b, h):
    plan = gpu["plan"]
    for x, name in enumerate(("Qp", "Kp", "Vp")):
        for l in range(1, cfg["L"] + 1):
            got = f32(plan.pyramid_level(gpu["ws"], x, l)[b, h])
            assert np.array_equal(got, ref[name][l]), f"pooled {name} level {l} head {(b, h)} not bit-exact"


def check_indices(cfg, gpu, ref, b, h, x):
    """Teacher-forced, level-by-level comparison; returns (#rows differing from the free-running oracle,
    #rows excused as near-ties)."""
    plan, g = gpu["plan"], geometry(cfg)
    excused = free_diff = 0
    for l in range(g.L, 0, -1):
        got = plan.level_indices(gpu["indices"], l - 1)[b, h].cpu().numpy()
        assert got.shape == (g.n(l), g.K_l(l - 1))
        assert np.all(np.diff(got, axis=1) > 0), "rows must be ascending and distinct"
        parent = None if l == g.L else plan.level_indices(gpu["indices"], l)[b, h].cpu().numpy()
        want, margin = orc.select_level(ref["Qp"][l], ref["Kp"][l], g.B, parent, g.K_l(l - 1), want_margin=True)
        bad = np.nonzero((got != want).any(axis=1))[0]
        for i in bad:
            assert margin[i] < 1e-5, f"level {l} row {i} head {(b, h)}: indices differ, margin {margin[i]:.3e}"
        excused += len(bad)
        free_diff += int((got != ref["I"][l - 1]).any(axis=1).sum())
    return free_diff, excused


def check_close(name, got, ref, tol, ulp=0.0):
    """Asserts |got - ref| <= tol + ulp * |ref| element-wise; returns the plain max-abs error."""
    err = np.abs(got.astype(np.float64) - ref)
    aref = np.abs(ref)
    over = err - ulp * aref                      # what is left for the plain tolerance
    kind = (name.split("(")[0].strip(), "ulp" if ulp > 0 else "plain", tol)
    st = STATS.setdefault(kind, dict(max_abs_err=0.0, max_ref=0.0, max_err_minus_ulp_term=-1.0, elements=0,
                                     above_plain_tol=0, worst=""))
    e = float(err.max())
    if e > st["max_abs_err"]:
        st["max_abs_err"], st["worst"] = e, name
    st["max_ref"] = max(st["max_ref"], float(aref.max()))
    st["max_err_minus_ulp_term"] = max(st["max_err_minus_ulp_term"], float(over.max()))
    st["elements"] += int(err.size)
    st["above_plain_tol"] += int((err > tol).sum())
    assert float(over.max()) <= tol, (f"{name}: max-abs err {e:.3e}, {int((over > tol).sum())} elements beyond "
                                      f"{tol} + {ulp:.2e}*|ref| (max |ref| {float(aref.max()):.3e})")
    return e


def dump_stats(path):
    import json
    rows = [dict(output=k[0], rule=k[1], tol=k[2], **v) for k, v in sorted(STATS.items())]
    if rows:
        with open(path, "w") as f:
            json.dump(rows, f, indent=1)


def oracle_backward_threads(Q, Kp, Vp, idx_cat, dO, g, Le, threads=16, reweight=1, scale=None):
    """The oracle's backward of one head with the query rows split into `threads` ranges run on host threads
    (the C call releases the interpreter lock): each range's fp64 share of dQ / dK / dV over the whole pyramid,
    summed here, then the pooling adjoint.  Same arithmetic as orc.backward up to fp64 summation order."""
    Kc, Vc = orc.cat_pyramid(Kp), orc.cat_pyramid(Vp)
    cuts = [g.N * i // threads for i in range(threads + 1)]
    ranges = [(a, b) for a, b in zip(cuts[:-1], cuts[1:]) if b > a]
    tot = None
    with ThreadPoolExecutor(max_workers=threads) as ex:
        for part in ex.map(lambda r: orc.attn_bwd(Q, Kc, Vc, idx_cat, dO, g, Le, reweight, scale, rows=r), ranges):
            if tot is None:
                tot = list(part)
            else:
                for t_, p_ in zip(tot, part):
                    t_ += p_
    return {"dQ": tot[0], "dK": orc.unpool(tot[1], g), "dV": orc.unpool(tot[2], g)}


# ---- large shapes: the oracle checks sampled rows, properties cover every head ----
def make_inputs_parallel(cfg, seed, threads=8):
    out = {n: np.empty((cfg["batch"], cfg["heads"], cfg["N"], cfg["d"]), np.float32) for n in ("Q", "K", "V", "dO")}
    jobs = [(n, b, h) for n in out for b in range(cfg["batch"]) for h in range(cfg["heads"])]

    def one(job):
        n, b, h = job
        x = inputs.make_head(cfg["kind"], seed, n, b, h, cfg["N"], cfg["d"])
        out[n][b, h] = orc.to_bf16(x) if cfg["dtype"] == "bf16" else x

    with ThreadPoolExecutor(max_workers=threads) as ex:
        list(ex.map(one, jobs))
    return out


def properties_all_heads(cfg, gpu, x):
    """Checks that need no oracle: valid index lists, gradient sum identities."""
    plan, g = gpu["plan"], geometry(cfg)
    for l in range(g.L):
        I = plan.level_indices(gpu["indices"], l)
        assert bool((I[..., 1:] > I[..., :-1]).all()) if I.shape[-1] > 1 else True
        assert int(I.min()) >= 0 and int(I.max()) < g.n(l + 1)
        if l + 1 < g.L:        # every pick is a child of a pick of the parent row
            par = plan.level_indices(gpu["indices"], l + 1)                       # [b, h, rows/B, K]
            parent_of_pick = (I // cfg["B"]).unsqueeze(-1)                         # [b, h, rows, K, 1]
            rows = I.shape[2]
            par_rows = par[:, :, torch.arange(rows, device=I.device) // cfg["B"]]  # [b, h, rows, Kp]
            assert bool((parent_of_pick == par_rows.unsqueeze(-2)).any(-1).all())
    assert bool(torch.isfinite(gpu["LSE"]).all()) and bool(torch.isfinite(gpu["O"].float()).all())
    dO, dV = gpu["dO"].float(), gpu["dV"].float()
    s_ref, s_got = dO.sum(dim=2), dV.sum(dim=2)                                    # [b, h, d]
    scale = dO.abs().sum(dim=2)
    assert float(((s_ref - s_got).abs() / scale).max()) < 2e-3, "sum_t dV[t] != sum_q dO[q]"
    lhs = (gpu["dQ"].float() * gpu["Q"].float()).sum(dim=(2, 3))
    rhs = (gpu["dK"].float() * gpu["K"].float()).sum(dim=(2, 3))
    norm = (gpu["dQ"].float().abs() * gpu["Q"].float().abs()).sum(dim=(2, 3))
    assert float(((lhs - rhs).abs() / norm).max()) < 5e-3, "<dQ,Q> != <dK,K>"


def sampled_parity(cfg, gpu, x, heads, n_row_chunks=6, chunk=32, full_backward_head=None):
    """Pooled levels and indices bit-exact on `heads`; O, LSE, dQ element-wise on sampled runs of query rows;
    dK, dV element-wise on one whole head if asked (the oracle's full backward must fit the test's time)."""
    g = geometry(cfg)
    Le = g.L if cfg.get("Le") is None else cfg["Le"]
    tol = TOL[cfg["dtype"]]
    rng = np.random.default_rng(1234)
    for (b, h) in heads:
        Qp, Kp, Vp = (orc.pyramid(x[n][b, h], g, cfg["dtype"] == "bf16") for n in ("Q", "K", "V"))
        ref = {"Qp": Qp, "Kp": Kp, "Vp": Vp, "I": orc.select_all(Qp, Kp, g)}
        check_pyramid(cfg, gpu, ref, b, h)
        free_diff, excused = check_indices(cfg, gpu, ref, b, h, x)
        assert excused == 0 and free_diff == 0
        idx = orc.cat_indices(ref["I"])
        Kc, Vc = orc.cat_pyramid(Kp), orc.cat_pyramid(Vp)
        starts = sorted(set([0, g.N - chunk] + [int(s) for s in rng.integers(0, g.N - chunk, n_row_chunks)]))
        for s0 in starts:
            o, lse = orc.attn_fwd(x["Q"][b, h], Kc, Vc, idx, g, Le, rows=(s0, s0 + chunk))
            dq, _, _ = orc.attn_bwd(x["Q"][b, h], Kc, Vc, idx, x["dO"][b, h], g, Le, rows=(s0, s0 + chunk))
            sl = slice(s0, s0 + chunk)
            check_close(f"O{(b, h, s0)}", f32(gpu["O"][b, h, sl]), o[sl], tol["out"], tol["ulp"])
            check_close(f"LSE{(b, h, s0)}", f32(gpu["LSE"][b, h, sl]), lse[sl], tol["lse"])
            check_close(f"dQ{(b, h, s0)}", f32(gpu["dQ"][b, h, sl]), dq[sl], tol["out"], tol["ulp"])
        if full_backward_head == (b, h):
            bw = oracle_backward_threads(x["Q"][b, h], Kp, Vp, idx, x["dO"][b, h], g, Le)
            for name in ("dQ", "dK", "dV"):
                err = check_close(f"{name}{(b, h)}", f32(gpu[name][b, h]), bw[name], tol["out"], tol["ulp"])
                print(f"{cfg['name']} full-head {name} max-abs err {err:.3e}")
