"""The work that a trainer has this library do, as cases that can be timed and checked.

Every case is one policy update, or the part of one that a trainer calls by itself, through the
package's public entry points:

  update      policy_update: token statistics, step selection, loss and dlogits of given logits
  loss        dart_policy_loss under torch.autograd: the same path as a training loop's loss
  variants    the update with the objective's options: several task groups, GRPO advantages,
              an inverse temperature, step ratios, a KL term, zero rows skipped
  objective   the same without the logits (their statistics come from the LM head, or from a
              gather over ranks): advantages, selection per group, loss and coefficients
  head_stats  dart_lmhead_tok_stats_ex: log-probs and entropies straight from the LM head's
              inputs (the recompute of the old policy's log-probs; forward only)
  head_loss   dart_lmhead_policy_loss under torch.autograd: forward and backward to the hidden
              states and the LM-head weight

The inputs are made on the GPU from the seed alone, by torch and numpy.
"""

import math

import numpy as np
import torch

import paper_2509_23866_amd as dart
from paper_2509_23866_amd.autograd import dart_lmhead_policy_loss, dart_policy_loss

EPS_LOW, EPS_HIGH, CAP, BETA = 0.2, 0.28, 2.0, 0.1
CHUNK = 1 << 27  # elements of logits that the preparation and the 64-bit path hold at a time


def listed():
    return [
        # the smallest update: a toy policy's fp32 logits, where latency and launches count
        dict(name="update_tiny", kind="update", T=512, S=16, V=4096, ld=4096, dtype="f32", rho=0.5),
        # two steps of one episode under the 7B policy's vocabulary: few rows, each of them long
        dict(name="update_steps", kind="update", T=96, S=2, V=152064, ld=152064, dtype="bf16", rho=0.8),
        # the 7B policy's step group, the headline workload of the benchmark
        dict(name="update_group", kind="update", T=4096, S=64, V=152064, ld=152064, dtype="bf16", rho=0.8),
        # a large step group of which a quarter of the steps is kept
        dict(name="update_large", kind="update", T=16384, S=256, V=151936, ld=151936, dtype="bf16", rho=0.25),
        # logits of a padded head, cut back to the tokenizer's own (odd) vocabulary
        dict(name="update_sliced", kind="update", T=2000, S=40, V=50257, ld=50304, dtype="bf16", rho=0.8),
        # a training loop that upcasts its logits to fp32 and samples at a temperature
        dict(name="loss_f32", kind="loss", T=2048, S=32, V=32000, ld=32000, dtype="f32", rho=0.8,
             inv_temp=1.25),
        # several tasks in one batch with the objective's options on, an odd vocabulary
        dict(name="variants_groups", kind="variants", T=6000, S=100, V=32003, ld=32003, dtype="bf16",
             rho=0.5, inv_temp=1.25, traj_steps=10, group_trajs=4, kl="k3", aggregation="step_mean",
             ratio="step_geomean"),
        # the long-horizon batch without its logits: 32 episodes of 50 steps
        dict(name="objective_long", kind="objective", T=152569, S=1600, rho=0.5, traj_steps=50,
             group_trajs=8, kl="k3", aggregation="step_mean", ratio="step_geomean"),
        # log-probs of one step's tokens under the 7B policy's head
        dict(name="head_stats_step", kind="head_stats", T=64, S=1, V=152064, d=3584, inv_temp=1.0),
        # log-probs of a whole step group under it
        dict(name="head_stats_group", kind="head_stats", T=4096, S=64, V=152064, d=3584, inv_temp=1.0),
        # forward and backward of the head for one episode's tokens
        dict(name="head_loss_episode", kind="head_loss", T=1000, S=16, V=152064, d=3584, rho=0.8,
             skip=False, inv_temp=1.0),
        # forward and backward of the head for a step group, dropped rows left out
        dict(name="head_loss_group", kind="head_loss", T=4096, S=64, V=152064, d=3584, rho=0.8,
             skip=True, inv_temp=1.0),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, evenly spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges above: T from one short step to a large group, vocabularies
    from 2048 to 152064 (odd ones among them), rows padded or not, every option."""
    kind = rng.choice(["update", "update", "loss", "variants", "objective", "head_stats",
                       "head_stats", "head_loss", "head_loss"])
    c = dict(kind=kind)
    if kind == "objective":
        c["T"] = _spread(rng, 1000, 160000)
    else:
        c["T"] = _spread(rng, 16, 4096 if kind.startswith("head") else 16384)
    c["S"] = max(1, min(c["T"], int(c["T"] / rng.uniform(16, 128))))
    if kind != "objective":
        V = _spread(rng, 2048, 152064)
        c["V"] = V if rng.random() < 0.5 else V // 64 * 64
    if kind.startswith("head"):
        c["d"] = _spread(rng, 512, 3584) // 8 * 8
    elif kind != "objective":
        c["dtype"] = rng.choice(["bf16", "bf16", "f32"])
        if c["dtype"] == "f32":
            c["T"] = max(16, min(c["T"], 4 * 10 ** 8 // c["V"]))
            c["S"] = min(c["S"], c["T"])
        c["ld"] = c["V"] if rng.random() < 0.6 else (c["V"] + 127) // 64 * 64
    if kind != "head_stats":
        c["rho"] = rng.choice([0.25, 0.5, 0.8, 1.0])
    if kind not in ("update", "objective"):
        c["inv_temp"] = rng.choice([1.0, 1.0, 0.8, 1.25])
    if kind in ("variants", "objective"):
        c["traj_steps"] = rng.randint(5, 50)
        c["group_trajs"] = rng.choice([4, 8])
        c["kl"] = rng.choice(["none", "k1", "k2", "k3"])
        c["aggregation"] = rng.choice(["token_mean", "token_mean_all", "step_mean"])
        c["ratio"] = rng.choice(["token", "step_geomean", "step_geomean"])
    if kind == "head_loss":
        c["skip"] = rng.random() < 0.5
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------


def _offsets(rs, n, parts):
    """Offsets that cut n things into that many parts of at least one, the lengths of the parts
    within a factor of a few of each other."""
    w = rs.uniform(0.4, 1.6, parts)
    lens = 1 + np.floor((n - parts) * w / w.sum()).astype(np.int64)
    lens[: n - int(lens.sum())] += 1
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


def _even(n, size):
    """Offsets of runs of `size` out of n things, the last run shorter."""
    return np.array(list(range(0, n, size)) + [n], np.int32)


def _rows(T, width):
    step = max(1, CHUNK // width)
    return [(r, min(T, r + step)) for r in range(0, T, step)]


def _target_logp(z, y):
    """log softmax(z)[y] of rows of logits, in float32."""
    z = z.float()
    return z.gather(1, y.long()[:, None])[:, 0] - torch.logsumexp(z, 1)


def _noise(g, dev, n, sigma):
    return torch.randn(n, generator=g, device=dev) * sigma


def prepare(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(seed)
    rs = np.random.RandomState(seed % (1 << 31))
    kind, T, S = case["kind"], case["T"], case["S"]
    off = _offsets(rs, T, S)
    lens = np.diff(off)
    cuda = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    per_token = lambda a: cuda(np.repeat(a, lens).astype(np.float32))  # noqa: E731
    st = dict(case=case, T=T, off=cuda(off))
    it = case.get("inv_temp", 1.0)
    # steps differ in how sure the policy is: the selection works on that
    sharp = per_token(rs.uniform(1.5, 3.5, S))
    if kind == "objective":
        st["entropy"] = torch.rand(T, generator=g, device=dev) * 2 + sharp
        logp = -torch.rand(T, generator=g, device=dev) * 6
    elif kind.startswith("head"):
        V, d = case["V"], case["d"]
        h = torch.randn(T, d, generator=g, device=dev) * (sharp[:, None] / 3)
        h = st["hidden"] = h.to(torch.bfloat16)
        w = st["weight"] = torch.randn(V, d, generator=g, device=dev, dtype=torch.bfloat16)
        w *= 3 / math.sqrt(d)
        # generated tokens are likely ones: the best of a few candidates
        cand = torch.randint(V, (T, 16), generator=g, device=dev)
        zc = torch.cat([(w[cand[a:b]].float() * h[a:b, None].float()).sum(2)
                        for a, b in _rows(T, 16 * d)])
        st["target"] = cand.gather(1, zc.argmax(1, True))[:, 0].to(torch.int32)
        if kind == "head_stats":
            return st
        logp = torch.cat([_target_logp((h[a:b] @ w.t()).float() * it, st["target"][a:b])
                          for a, b in _rows(T, V)])
    else:
        V, ld = case["V"], case["ld"]
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        buf = torch.empty(T, ld, dtype=dt, device=dev)
        y = torch.randint(V, (T, 1), generator=g, device=dev)
        spike = torch.rand(T, 1, generator=g, device=dev) * 6 + 2
        lp = []
        for a, b in _rows(T, ld):
            z = torch.randn(b - a, ld, generator=g, device=dev).mul_(sharp[a:b, None])
            z.scatter_add_(1, y[a:b], spike[a:b])
            buf[a:b] = z
            lp.append(_target_logp(buf[a:b, :V].float() * it, y[a:b, 0]))
        st["logits"] = buf[:, :V]
        st["target"] = y[:, 0].to(torch.int32)
        logp = torch.cat(lp)
    st["old"] = logp + _noise(g, dev, T, 0.08)
    st["roll"] = st["old"] + _noise(g, dev, T, 0.3)
    st["adv"] = per_token(0.3 + rs.standard_normal(S))
    if "traj_steps" in case:
        st["logp"] = logp
        st["ref"] = logp + _noise(g, dev, T, 0.08)
        traj = _even(S, case["traj_steps"])
        group = _even(len(traj) - 1, case["group_trajs"])
        st["reward"] = cuda(rs.uniform(0, 1, len(traj) - 1).astype(np.float32))
        st["traj_off"], st["group_off"] = cuda(traj), cuda(group)
        st["group_step_off"] = cuda(traj[group])
    return st


# ---------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------


def _objective(st, logp, entropy):
    c = st["case"]
    adv, mean, std = dart.dart_grpo_advantage(st["reward"], st["traj_off"], st["group_off"],
                                              st["off"], T=st["T"])
    step_ent, mask, kept = dart.dart_step_select_groups(entropy, st["off"], st["group_step_off"],
                                                        c["rho"])
    loss, coef, stats = dart.dart_tis_loss_fwd_ex(
        logp, st["old"], st["roll"], adv, st["off"], mask, EPS_LOW, EPS_HIGH, CAP,
        logp_ref=st["ref"], kl=c["kl"], beta=BETA, aggregation=c["aggregation"], ratio=c["ratio"])
    return dict(adv=adv, group_mean=mean, group_std=std, step_entropy=step_ent, step_mask=mask,
                n_kept_steps=kept, loss=loss, tok_coef=coef, stats=stats)


def run(st):
    c = st["case"]
    kind, it = c["kind"], c.get("inv_temp", 1.0)
    if kind == "update":
        return dart.policy_update(st["logits"], st["target"], st["old"], st["roll"], st["adv"],
                                  st["off"], c["rho"], EPS_LOW, EPS_HIGH, CAP)
    if kind == "loss":
        z = st["logits"].detach().requires_grad_()
        loss = dart_policy_loss(z, st["target"], st["old"], st["roll"], st["adv"], st["off"],
                                c["rho"], EPS_LOW, EPS_HIGH, CAP, inv_temp=it)
        return dict(loss=loss.detach(), dlogits=torch.autograd.grad(loss, z)[0])
    if kind == "variants":
        logp, ent, lse = dart.dart_tok_stats(st["logits"], st["target"], inv_temp=it)
        out = _objective(st, logp, ent)
        out["dlogits"] = dart.dart_tis_grad(st["logits"], st["target"], logp, lse, out["tok_coef"],
                                            inv_temp=it, skip_zero_rows=True)
        return dict(out, logp=logp, entropy=ent, lse=lse)
    if kind == "objective":
        return _objective(st, st["logp"], st["entropy"])
    if kind == "head_stats":
        logp, ent, lse = dart.dart_lmhead_tok_stats_ex(st["hidden"], st["weight"], st["target"], it)
        return dict(logp=logp, entropy=ent, lse=lse)
    h, w = st["hidden"].detach().requires_grad_(), st["weight"].detach().requires_grad_()
    loss = dart_lmhead_policy_loss(h, w, st["target"], st["old"], st["roll"], st["adv"], st["off"],
                                   c["rho"], EPS_LOW, EPS_HIGH, CAP, inv_temp=it,
                                   flags=dart.DART_LMHEAD_SKIP_ZERO_ROWS if c["skip"] else 0)
    dh, dw = torch.autograd.grad(loss, (h, w))
    return dict(loss=loss.detach(), dhidden=dh, dweight=dw)


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how far a correct result may be off
# ---------------------------------------------------------------------------


def work(case):
    kind, T, S = case["kind"], case["T"], case["S"]
    if kind == "objective":
        # entropy, three or four log-probs in; advantage and coefficient out; the steps' arrays
        return {"bytes": T * 4 * (6 if case["kl"] == "none" else 7) + S * 13, "flops": 0}
    if kind.startswith("head"):
        V, d = case["V"], case["d"]
        gemm = 2.0 * T * V * d
        if kind == "head_stats":
            return {"bytes": (T + V) * d * 2 + T * 16, "flops": gemm}
        # the logits once, dh and dW for the rows that count
        rows = case["rho"] if case["skip"] else 1.0
        return {"bytes": 2 * (T + V) * d * 2 + T * 20, "flops": gemm * (1 + 2 * rows)}
    b = 4 if case["dtype"] == "f32" else 2
    return {"bytes": 2 * T * case["V"] * b + T * 36 + S * 9, "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind in ("objective", "head_stats") or case.get("dtype") == "f32":
        return {"rel": 1e-5}
    # dlogits, dh and dW in bf16: half a unit of 2^-8 each
    return {"rel": 8e-3}


# ---------------------------------------------------------------------------
# the same results in 64 bits, by torch and numpy alone
# ---------------------------------------------------------------------------


def _stats64(z, y):
    """logp, entropy, lse and softmax of rows of 64-bit logits."""
    lse = torch.logsumexp(z, 1)
    x = z - lse[:, None]
    p = x.exp()
    return x.gather(1, y.long()[:, None])[:, 0], -(p * x).sum(1), lse, p


def _select64(ent, off, groups, rho):
    """Step means (rounded to float32, as the selection reads them) and the mask of each group's
    ceil(rho S) highest, equal ones by the lower index."""
    e = ent.cpu().numpy()
    mean = np.array([e[a:b].mean() for a, b in zip(off[:-1], off[1:])])
    mask = np.zeros(len(mean), bool)
    for a, b in zip(groups[:-1], groups[1:]):
        k = max(0, min(b - a, math.ceil(rho * (b - a) - 1e-6)))
        mask[a + np.argsort(-mean[a:b].astype(np.float32), kind="stable")[:k]] = True
    return mean, mask


def _loss64(case, st, logp, adv, off, mask):
    """Loss, coefficients and the sums behind the stats."""
    np64 = lambda t: t.double().cpu().numpy()  # noqa: E731
    lp, lo, lr, adv = np64(logp), np64(st["old"]), np64(st["roll"]), np64(adv)
    lens = np.diff(off)
    step = np.repeat(np.arange(len(lens)), lens)
    M = mask[step].astype(np.float64)
    N, K, L = M.sum(), mask.sum(), lens[step].astype(np.float64)
    agg = case.get("aggregation", "token_mean")
    om = {"token_mean": 1 / N, "token_mean_all": 1 / len(lp), "step_mean": 1 / (K * L)}[agg]
    u, d, share = lp - lo, lo - lr, np.ones_like(lp)
    if case.get("ratio", "token") != "token":
        mean = lambda x: (np.add.reduceat(x, off[:-1]) / lens)[step]  # noqa: E731
        # every token of a step gets the step's whole derivative, |s| weights times 1 / |s|
        u, d, adv = mean(u), mean(d), mean(adv)
    r, w = np.exp(u), np.minimum(np.exp(d), CAP)
    a, b = r * adv, np.clip(r, 1 - EPS_LOW, 1 + EPS_HIGH) * adv
    flow = a <= b
    kl = dkl = np.zeros_like(lp)
    if case.get("kl", "none") != "none":
        x = np64(st["ref"]) - lp
        kl = {"k1": -x, "k2": x * x / 2, "k3": np.expm1(x) - x}[case["kl"]]
        dkl = {"k1": share, "k2": -x, "k3": -np.expm1(x)}[case["kl"]]
    loss = -(M * om * (w * np.minimum(a, b) - BETA * kl)).sum()
    coef = -M * om * (w * flow * a - BETA * dkl)
    stats = np.array([(M * ~flow).sum(), (M * w).sum(), (M * (d >= math.log(CAP))).sum(), N * N,
                      (M * kl).sum(), K * N]) / N
    return np.array([loss]), coef, stats


def exact(case, seed):
    st = prepare(case, seed)
    kind, it = case["kind"], case.get("inv_temp", 1.0)
    off = st["off"].cpu().numpy()
    head = kind.startswith("head")
    out = {}
    T = case["T"]
    if kind == "objective":
        logp, ent = st["logp"].double(), st["entropy"].double()
    else:
        if head:
            h, w = st["hidden"].double(), st["weight"].double()
            z_rows = lambda a, b: (h[a:b] @ w.t()) * it  # noqa: E731
        else:
            z_rows = lambda a, b: st["logits"][a:b].double() * it  # noqa: E731
        parts = [_stats64(z_rows(a, b), st["target"][a:b])[:3] for a, b in _rows(T, case["V"])]
        logp, ent, lse = (torch.cat(p) for p in zip(*parts))
        out = dict(logp=logp, entropy=ent, lse=lse)
        if kind == "head_stats":
            return out
    groups, adv = [0, case["S"]], st["adv"]
    if "traj_steps" in case:
        groups, traj = st["group_step_off"].cpu().numpy(), st["traj_off"].cpu().numpy()
        gt, R = st["group_off"].cpu().numpy(), st["reward"].double().cpu().numpy()
        n = np.diff(traj).astype(np.float64)
        cut = list(zip(gt[:-1], gt[1:]))
        mean = np.array([np.average(R[a:b], weights=n[a:b]) for a, b in cut])
        std = np.array([math.sqrt(np.average((R[a:b] - m) ** 2, weights=n[a:b]))
                        for (a, b), m in zip(cut, mean)])
        size = np.diff(gt)
        m, s = np.repeat(mean, size), np.repeat(std, size)
        a_traj = np.where(s > 0, (R - m) / np.where(s > 0, s, 1), 0)
        adv = torch.from_numpy(np.repeat(np.repeat(a_traj, np.diff(traj)), np.diff(off)))
        out.update(adv=adv, group_mean=mean, group_std=std)
    step_ent, mask = _select64(ent, off, groups, case["rho"])
    loss, coef, stats = _loss64(case, st, logp, adv, off, mask)
    out.update(step_entropy=step_ent, step_mask=None, n_kept_steps=None, loss=loss, tok_coef=coef,
               stats=stats if "traj_steps" in case else stats[:4])
    if kind == "objective":
        return out
    gcoef = torch.from_numpy(coef).to(logp.device) * it
    wide = head and torch.zeros_like(w)
    rows = []
    for a, b in _rows(T, case["V"]):
        z = z_rows(a, b)
        dz = -gcoef[a:b, None] * (z - lse[a:b, None]).exp()
        dz.scatter_(1, st["target"][a:b].long()[:, None],
                    (gcoef[a:b] * -torch.expm1(logp[a:b]))[:, None])
        if head:
            rows.append(dz @ w)
            wide += dz.t() @ h[a:b]
        else:
            rows.append(dz)
    if head:
        return dict(loss=loss[0], dhidden=torch.cat(rows), dweight=wide)
    out["dlogits"] = torch.cat(rows)
    return dict(loss=loss[0], dlogits=out["dlogits"]) if kind == "loss" else out
