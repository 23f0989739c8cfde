"""What is timed when the library is made faster: the calls a user of this framework makes, over their real range.

A case is one pass through the public entry points of paper_2604_18348_amd.binding:
  kind "attn"   adacluster_attn on one layer's Q, K, V.  warm False: the first denoising step (Algorithm 1 from
                scratch); warm True: any later step, which starts from the centres of the step before and hands
                its own on (the buffers are updated in place, as in a sampling loop).
  kind "dense"  adacluster_dense_attn: layers or heads that keep full attention.
  kind "steps"  the entry points one by one (query clustering, key clustering, selection, attention) and the
                compactness score, as a study of a layer calls them.
  kind "scores" adacluster_quest_scores: token rows against key pages.

Inputs follow the recipe of the package's workloads (tokens of a T x Y x X video grid plus text tokens, a token
is its component's mean plus noise, a share of outliers, heads without structure at the end), drawn on the GPU:
the components are the boxes of an uneven per-head grid, the query mean of a component leans towards its key
mean, so that attention is concentrated as it is in a trained model, and V has component means too.
"""
import dataclasses
import math

import torch

from paper_2604_18348_amd import binding as B


def _attn(name, H, grid, text, d, dtype, M, warm, q_clusters, m0, m_min, n_max, frac, topk, select="topk", score="tq",
          sigma=0.3, outlier=0.0, lognorm=False, diffuse=0, neariso=0, kind="attn"):
    return dict(name=name, kind=kind, H=H, T=grid[0], Y=grid[1], X=grid[2], text=text, d=d, dtype=dtype, M=M, warm=warm,
                q_clusters=q_clusters, m0=m0, m_min=m_min, n_max=n_max, frac=frac, topk=topk, select=select, score=score,
                sigma=sigma, outlier=outlier, lognorm=lognorm, diffuse=diffuse, neariso=neariso)


def listed():
    return [
        # the smallest call: a short clip in few heads (the package's smoke test); launches and host time
        _attn("attn_1.5k", 2, (10, 10, 15), 0, 64, "bf16", 12, False, 9, 16, 4, 64, 0.03, 5),
        # the fp32 accuracy path at its usual size
        _attn("attn_f32_4k", 1, (16, 16, 16), 0, 64, "f32", 32, False, 32, 16, 4, 128, 0.0, 8),
        # fp32, the wide head, a ragged token count, a later denoising step
        _attn("attn_f32_5k_warm", 3, (9, 23, 24), 39, 128, "f32", 32, True, 65, 32, 8, 256, 0.03, 16),
        # 720x480, 49 frames, first step and later steps (text tokens, outliers, some heads without structure)
        _attn("attn_17k", 30, (13, 30, 45), 226, 64, "bf16", 256, False, 65, 128, 16, 512, 0.03, 64, outlier=0.02, diffuse=6),
        _attn("attn_17k_warm", 30, (13, 30, 45), 226, 64, "bf16", 256, True, 65, 128, 16, 512, 0.03, 64, outlier=0.02, diffuse=6),
        # 832x480, 81 frames, wide head, the top-p budget (skewed key lists)
        _attn("attn_32k_topp", 12, (21, 30, 52), 0, 128, "bf16", 512, False, 65, 256, 16, 1024, 0.03, 64, select="topp", lognorm=True),
        # 1280x720, 81 frames: the main model, first step and later steps
        _attn("attn_75k", 30, (21, 45, 80), 0, 64, "bf16", 1024, False, 65, 512, 16, 2048, 0.03, 64, sigma=0.4, outlier=0.02),
        _attn("attn_75k_warm", 30, (21, 45, 80), 0, 64, "bf16", 1024, True, 65, 512, 16, 2048, 0.03, 64, sigma=0.4, outlier=0.02),
        # the longest sequence, wide head
        _attn("attn_180k", 24, (50, 45, 80), 0, 128, "bf16", 2048, False, 65, 1024, 16, 4096, 0.03, 64, lognorm=True, neariso=8),
        # full attention of a layer that stays dense
        _attn("dense_32k", 12, (21, 30, 52), 0, 128, "bf16", 512, False, 65, 256, 16, 1024, 0.03, 64, kind="dense"),
        # a study of one layer through the single entry points: box scores, a ragged token count
        _attn("steps_9k_box", 5, (11, 28, 30), 7, 128, "bf16", 64, False, 65, 64, 8, 256, 0.03, 32, score="box", kind="steps"),
        # token rows against the key clusters of the main model, matrix-core form
        dict(name="scores_75k", kind="scores", H=2, Lq=75600, Lk=450, d=64, dtype="bf16", form="mfma", clamp=False),
    ]


def draw(rng):
    """One more case of the same ranges: token counts over their logarithm, any head count, both widths."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choices(["attn", "dense", "steps", "scores"], [10, 2, 2, 2])[0]
    d = rng.choice([64, 128])
    if kind == "scores":
        bf16 = rng.random() < 0.75
        H = rng.randint(1, 24)
        Lq, Lk = logint(65, 180000), logint(48, 1200)
        while H * Lq * Lk > 24 * 10 ** 7:
            H, Lq = max(1, H // 2), (Lq * 3 + 3) // 4
        return dict(kind=kind, H=H, Lq=Lq, Lk=Lk, d=d, dtype="bf16" if bf16 else "f32",
                    form="mfma" if bf16 and rng.random() < 0.75 else "alu", clamp=rng.random() < 0.3)
    f32 = rng.random() < 0.2
    H = rng.randint(1, 30)
    N = logint(1200, 12000 if f32 else 180000)
    if kind == "steps":
        N = min(N, logint(1200, 48000))
    if kind == "dense":
        N = min(N, logint(1200, 33000))
        while 4.0 * d * H * N * N > (3e10 if f32 else 6e12):
            H, N = max(1, H // 2), N - N // 5
    while H * N * d > 24 * 180000 * 128:
        H -= 1
    if f32:
        H = (H - 1) % 4 + 1
    T = rng.randint(5, 24)
    Y = max(2, int(math.sqrt(N / T / rng.uniform(1.0, 2.0))))
    X = max(2, N // (T * Y))
    text = rng.choice([0, 0, rng.randint(1, 256)])
    N = T * Y * X + text
    m0 = max(16, int(N / rng.uniform(110, 260)))
    lognorm = rng.random() < 0.4
    topp = rng.random() < (0.3 if lognorm or N < 10000 else 0.0) and N < 60000     # (even norms: a top-p budget takes most keys)
    q = rng.choice([65, 65, 65, rng.randint(9, 100)])
    loose = N < 40000                      # heads without structure may end in full attention: not at the largest sizes
    return _attn("", H, (T, Y, X), text, d, "f32" if f32 else "bf16", max(12, int(N / rng.uniform(60, 130))),
                 kind == "attn" and rng.random() < 0.4, q, m0, min(16, m0 // 2), 4 * m0, rng.choice([0.0, 0.03, 0.03]),
                 max(4, min(64, m0 // 2)), select="topp" if topp else "topk",
                 score="box" if kind == "steps" and rng.random() < 0.5 else rng.choice(["tq", "tq", "tq", "dot"]),
                 sigma=rng.uniform(0.2, 0.6), outlier=rng.choice([0.0, 0.02]), lognorm=lognorm,
                 diffuse=rng.choice([0, 0, H // 5]) if loose else 0, neariso=rng.choice([0, 0, H // 3]) if loose else 0, kind=kind) | {"name": ""}


def _n(case):
    return case["T"] * case["Y"] * case["X"] + case["text"]


def _tdtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _params(case):
    return B.Params(
        H=case["H"], N=_n(case), d=case["d"], dtype=B.BF16 if case["dtype"] == "bf16" else B.F32,
        q_clusters=case["q_clusters"], q_iters=3, k_iters=3, k_m0=case["m0"], k_m_min=case["m_min"],
        k_max_clusters=case["n_max"], k_max_stages=10, tau_factor=1.5, min_unassigned_frac=case["frac"],
        score_mode={"tq": B.SCORE_TQ, "box": B.SCORE_BOX, "dot": B.SCORE_DOT}[case["score"]],
        select_mode=B.SELECT_TOPP if case["select"] == "topp" else B.SELECT_TOPK, topk=case["topk"], top_p=0.9)


def _components(case, gen):
    """Component of every token, [H, N]: the cells of an uneven grid over the video box, text tokens in 8 of their own."""
    H, dims = case["H"], (case["T"], case["Y"], case["X"])
    side = (dims[0] * dims[1] * dims[2] / case["M"]) ** (1.0 / 3.0)
    cells = [min(L, max(1, round(L / side))) for L in dims]
    axis = []
    for L, n in zip(dims, cells):
        jitter = 0.8 * (torch.rand((H, n - 1), generator=gen, device="cuda") - 0.5)
        cuts = (torch.arange(1, n, device="cuda") + jitter) * (L / n)
        at = torch.arange(L, device="cuda", dtype=torch.float32) + 0.5
        axis.append((at[None, :, None] > cuts[:, None, :]).sum(-1))
    comp = (axis[0][:, :, None, None] * cells[1] + axis[1][:, None, :, None]) * cells[2] + axis[2][:, None, None, :]
    comp = comp.reshape(H, -1)
    n = cells[0] * cells[1] * cells[2]
    if case["text"]:
        text = n + torch.arange(case["text"], device="cuda") % 8
        comp = torch.cat([comp, text[None].expand(H, -1)], 1)
        n += 8
    return comp, n


def _qkv(case, gen):
    H, N, d = case["H"], _n(case), case["d"]
    comp, n = _components(case, gen)
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda")  # noqa: E731

    def means():
        m = rand(H, n, d)
        if case["lognorm"]:
            m = m / m.norm(dim=2, keepdim=True) * (0.5 * rand(H, n, 1)).exp() * math.sqrt(d)
        return m

    muk = means()
    muq = 0.5 * muk + math.sqrt(0.75) * means()
    scale, sigma = torch.ones(H, device="cuda"), torch.full((H,), case["sigma"], device="cuda")
    if case["neariso"]:                    # means pulled in, noise as wide as they are apart
        scale[-case["neariso"]:], sigma[-case["neariso"]:] = 0.25, 1.0
    if case["diffuse"]:                    # no structure at all
        scale[-case["diffuse"]:], sigma[-case["diffuse"]:] = 0.0, 1.0
    out = []
    for mu, noise in ((muq, sigma), (muk, sigma), (rand(H, n, d), 0.5 * torch.ones_like(sigma))):
        x = torch.empty((H, N, d), dtype=_tdtype(case), device="cuda")
        for h in range(H):
            t = rand(N, d) * noise[h] + (mu[h] * scale[h])[comp[h]]
            if case["outlier"] and len(out) < 2:
                t = torch.where(torch.rand((N, 1), generator=gen, device="cuda") < case["outlier"], rand(N, d), t)
            x[h] = t
        out.append(x)
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    if case["kind"] == "scores":
        H, Lq, Lk, d = case["H"], case["Lq"], case["Lk"], case["d"]
        q = torch.randn((H, Lq, d), generator=gen, device="cuda").to(_tdtype(case))
        c = torch.randn((H, Lk, d), generator=gen, device="cuda")
        w = torch.randn((H, Lk, d), generator=gen, device="cuda").abs()
        return dict(case=case, Q=q, hi=(c + w).to(_tdtype(case)), lo=(c - w).to(_tdtype(case)),
                    S=torch.empty((H, Lq, Lk), device="cuda"), form=B.QUEST_MFMA if case["form"] == "mfma" else B.QUEST_ALU)
    p = _params(case)
    Q, K, V = _qkv(case, gen)
    s = dict(case=case, p=p, Q=Q, K=K, V=V, O=torch.empty_like(Q), ws=B.workspace(p))
    if case["kind"] == "attn":
        s["outs"] = B.alloc_outputs(p, "cuda", want_box=case["score"] == "box", want_stage=False)
        if case["warm"]:
            # the step before: a cold call, then every tensor drifts a little; from here on two passes per clustering
            B.adacluster_attn(p, Q, K, V, outs=s["outs"], out=s["O"], ws=s["ws"])
            for x in (Q, K, V):
                for h in range(case["H"]):
                    x[h] += (0.05 * torch.randn(x[h].shape, generator=gen, device="cuda")).to(x.dtype)
            s["p"] = dataclasses.replace(p, q_init_mode=1, k_init_mode=1, q_iters=2, k_iters=2)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "scores":
        return B.adacluster_quest_scores(s["Q"], s["hi"], s["lo"], s["form"], clamp=s["case"]["clamp"], out=s["S"])
    p, Q, K, V = s["p"], s["Q"], s["K"], s["V"]
    if kind == "dense":
        return B.adacluster_dense_attn(p, Q, K, V, out=s["O"], ws=s["ws"])
    if kind == "attn":
        o = s["outs"]
        O = B.adacluster_attn(p, Q, K, V, outs=o, out=s["O"], ws=s["ws"])
        # the output, the assignments, and the centres that the next step starts from
        return dict(O=O, **{n: o[n] for n in ("q_labels", "k_labels", "q_centroids", "k_centroids", "k_count", "full_flag")})
    q = B.adacluster_qcluster(p, Q, ws=s["ws"])
    k = B.adacluster_kcluster(p, K, want_box=s["case"]["score"] == "box", ws=s["ws"])
    mse = B.adacluster_compactness(p, K, k["k_labels"], k["k_centroids"], ws=s["ws"])
    idx, cnt = B.adacluster_select(p, q["q_centroids"], q["q_mean_norm"], k["k_centroids"], k["k_box_min"], k["k_box_max"],
                                   k["k_sizes"], k["k_count"], k["full_flag"], ws=s["ws"])
    O = B.adacluster_sparse_attn(p, Q, K, V, q["q_labels"], k["k_labels"], k["k_count"], idx, cnt, out=s["O"], ws=s["ws"])
    return dict(O=O, q_labels=q["q_labels"], q_centroids=q["q_centroids"], k_labels=k["k_labels"], k_centroids=k["k_centroids"],
                k_count=k["k_count"], k_stage_of=k["k_stage_of"], sel_cnt=cnt, mse=mse)


def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "scores":
        H, Lq, Lk, d = case["H"], case["Lq"], case["Lk"], case["d"]
        return {"bytes": H * ((Lq + 2 * Lk) * d * es + 4 * Lq * Lk), "flops": 4.0 * H * Lq * Lk * d}
    H, N, d = case["H"], _n(case), case["d"]
    io = 4 * H * N * d * es                # Q, K, V read once, O written once
    if case["kind"] == "dense":
        return {"bytes": io, "flops": 4.0 * H * N * N * d}
    # the assignment products of every pass (Algorithm 1: those of its first stage, over all keys) and the
    # attention over the share of the keys that a selection of this size holds
    passes = 2 if case["warm"] else 3
    assign = 2.0 * H * N * d * passes * (case["q_clusters"] + case["m0"])
    share = 0.006 if case["select"] == "topp" else min(1.0, (0.33 if case["lognorm"] else 0.55) * case["topk"] / case["m0"])
    return {"bytes": io + 8 * H * N, "flops": assign + 4.0 * H * N * (share * N) * d}


def tolerance(case):
    """About four times what another order of the same sums gives (measured: the parts, walks and partial sums of the
    centre updates and the row sums of the soft-max in another order, the soft-max reference moved at another limit).
    Where bf16 centres are updated, a sum that rounds the other way moves a centre by one bf16 step and with it, now
    and then, a token between two clusters as near as each other; in a cluster of one or two tokens that shows."""
    if case["kind"] == "scores":           # fp32 sums of up to 256 products
        return {"rel": 2e-6, "max": 5e-5}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-4}
    if case["kind"] == "dense":            # one rounding to bf16
        return {"rel": 1.5e-3, "max": 0.032}
    return {"rel": 0.02, "max": 0.99, "differ": 3e-4}
