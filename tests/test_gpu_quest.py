"""GPU Quest scores (Eq. 1 with vector arithmetic, Eq. 2 / Algorithm 2 on the matrix cores) against the
fp64 oracle.  The inputs are bf16 (or fp32) values both sides read exactly; every product of two bf16
values is exact in fp32, so the only error is the fp32 accumulation over d terms: 1e-5 relative to the
sum of the absolute terms."""
import numpy as np
import pytest
import torch

from oracle import adacluster_oracle as orc
from paper_2604_18348_amd import binding as B
from paper_2604_18348_amd import workloads as wl

pytestmark = pytest.mark.gpu


def inputs(seed, H, Lq, Lk, d, bf16):
    rng = np.random.default_rng(seed)
    Q = rng.standard_normal((H, Lq, d)).astype(np.float32)
    C = rng.standard_normal((H, Lk, d)).astype(np.float32)
    spread = np.abs(rng.standard_normal((H, Lk, d))).astype(np.float32)
    lo, hi = C - spread, C + spread
    if bf16:
        Q, C, lo, hi = (wl.round_bf16_f32(a) for a in (Q, C, lo, hi))
    return Q, C, lo, hi


def dev(a, bf16):
    t = torch.from_numpy(a).cuda()
    return t.to(torch.bfloat16) if bf16 else t


@pytest.mark.parametrize("form,bf16", [(B.QUEST_ALU, True), (B.QUEST_MFMA, True), (B.QUEST_ALU, False)])
@pytest.mark.parametrize("Lq,Lk,d", [(65, 173, 64), (300, 70, 128), (1, 1, 64), (129, 257, 128)])
def test_box_scores_match_eq1(form, bf16, Lq, Lk, d):
    H = 2
    Q, _, lo, hi = inputs(3, H, Lq, Lk, d, bf16)
    S = B.adacluster_quest_scores(dev(Q, bf16), dev(hi, bf16), dev(lo, bf16), form).cpu().numpy()
    for h in range(H):
        ref = orc.score_box(Q[h].astype(np.float64), lo[h].astype(np.float64), hi[h].astype(np.float64))
        mag = np.abs(Q[h].astype(np.float64)) @ np.maximum(np.abs(lo[h]), np.abs(hi[h])).astype(np.float64).T
        assert np.all(np.abs(S[h] - ref) <= 1e-5 * mag + 1e-6), float(np.abs(S[h] - ref).max())


@pytest.mark.parametrize("Lq,Lk,d", [(257, 64, 64), (300, 65, 128), (70, 128, 64), (33, 129, 128), (65, 256, 64),
                                     (31, 512, 128), (40, 513, 64), (64, 993, 128), (97, 1201, 64)])
def test_matrix_core_form_at_the_edges_of_its_spans(Lq, Lk, d):
    """Page counts around the spans a workgroup collects (64, 128, 256, 512 slots) and past the largest, where rows leave
    in line-aligned pieces; same bound as above.  Scores are written once: S starts as NaN."""
    H = 2
    Q, _, lo, hi = inputs(11, H, Lq, Lk, d, True)
    S = torch.full((H, Lq, Lk), float("nan"), device="cuda")
    B.adacluster_quest_scores(dev(Q, True), dev(hi, True), dev(lo, True), B.QUEST_MFMA, out=S)
    S = S.cpu().numpy()
    for h in range(H):
        ref = orc.score_box(Q[h].astype(np.float64), lo[h].astype(np.float64), hi[h].astype(np.float64))
        mag = np.abs(Q[h].astype(np.float64)) @ np.maximum(np.abs(lo[h]), np.abs(hi[h])).astype(np.float64).T
        assert np.all(np.abs(S[h] - ref) <= 1e-5 * mag + 1e-6)


@pytest.mark.parametrize("Lq,Lk,d,shift", [(1, 1, 64, 1), (33, 3, 64, 2), (67, 31, 128, 3), (97, 127, 64, 1), (65, 255, 128, 2),
                                           (2085, 450, 64, 3), (96, 511, 64, 0), (35, 512, 128, 1),
                                           (67, 515, 64, 2), (34, 1001, 128, 3)])
def test_matrix_core_form_writes_rows_at_any_alignment(Lq, Lk, d, shift):
    """Scores leave in aligned 16-byte pieces, whatever float of such a piece a head or a row starts at; nothing else is
    written.  Same bound as above."""
    H = 3
    Q, _, lo, hi = inputs(13, H, Lq, Lk, d, True)
    buf = torch.full((H * Lq * Lk + 8,), float("nan"), device="cuda")
    S = buf[4 + shift:][:H * Lq * Lk].view(H, Lq, Lk)
    B.adacluster_quest_scores(dev(Q, True), dev(hi, True), dev(lo, True), B.QUEST_MFMA, out=S)
    assert torch.isnan(buf[:4 + shift]).all() and torch.isnan(buf[4 + shift + H * Lq * Lk:]).all()
    S = S.cpu().numpy()
    for h in range(H):
        ref = orc.score_box(Q[h].astype(np.float64), lo[h].astype(np.float64), hi[h].astype(np.float64))
        mag = np.abs(Q[h].astype(np.float64)) @ np.maximum(np.abs(lo[h]), np.abs(hi[h])).astype(np.float64).T
        assert np.all(np.abs(S[h] - ref) <= 1e-5 * mag + 1e-6)


@pytest.mark.parametrize("form", [B.QUEST_ALU, B.QUEST_MFMA])
def test_clamped_centroids_are_algorithm_2(form):
    """One vector per page: R+ = max(c, 0), R- = min(c, 0), taken on the fly from the centroid tensor."""
    H, Lq, Lk, d = 3, 97, 200, 64
    Q, C, _, _ = inputs(5, H, Lq, Lk, d, True)
    Cd = dev(C, True)
    S = B.adacluster_quest_scores(dev(Q, True), Cd, Cd, form, clamp=True).cpu().numpy()
    for h in range(H):
        ref = orc.score_tensorquest(Q[h].astype(np.float64), C[h].astype(np.float64))
        mag = np.abs(Q[h].astype(np.float64)) @ np.abs(C[h]).astype(np.float64).T
        assert np.all(np.abs(S[h] - ref) <= 1e-5 * mag + 1e-6)


def test_the_two_forms_agree_and_bound_every_member():
    """Eq. 1 and Eq. 2 are the same number, and that number bounds q.k for every key inside the box."""
    H, Lq, Lk, d = 1, 64, 40, 128
    Q, C, lo, hi = inputs(7, H, Lq, Lk, d, True)
    a = B.adacluster_quest_scores(dev(Q, True), dev(hi, True), dev(lo, True), B.QUEST_ALU).cpu().numpy()
    b = B.adacluster_quest_scores(dev(Q, True), dev(hi, True), dev(lo, True), B.QUEST_MFMA).cpu().numpy()
    assert np.allclose(a, b, rtol=0, atol=2e-4)
    inner = (Q[0].astype(np.float64) @ C[0].astype(np.float64).T)       # the centre lies inside its box
    assert np.all(b[0] >= inner - 1e-4)


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("H,Lq,Lk,d,shift", [(8, 32801, 65, 64, 0), (2, 131073, 64, 128, 0),      # eight rows a thread
                                             (4, 8201, 66, 128, 1), (3, 12000, 68, 64, 0),        # four
                                             (1, 33, 3, 64, 2), (2, 31, 64, 128, 0), (1, 1, 129, 64, 3)])      # two
def test_vector_form_at_the_edges_of_its_tiles(H, Lq, Lk, d, shift, bf16):
    """Rows and pages around the tiles, any alignment of S; minima above maxima, infinities and NaN are what Eq. 1 makes of them term by
    term (a NaN beside a number is ignored).  Same bound as above for finite scores; nothing else is written."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(Lq)
    Q, hi, lo = (torch.randn(s, generator=gen, device="cuda") for s in ((H, Lq, d), (H, Lk, d), (H, Lk, d)))     # (boxes that are none, too)
    hi[0, Lk // 2, d - 1], lo[0, 0, d // 2], Q[0, Lq // 3, 5] = float("inf"), float("nan"), 0.0
    hi[0, 0, 3], Q[H - 1, Lq - 1, 1] = float("-inf"), float("inf")
    Q[0, 0, d - 1] = 0.0
    if bf16:
        Q, hi, lo = (t.to(torch.bfloat16) for t in (Q, hi, lo))
    if shift:                                                    # inputs that start anywhere
        Q, hi, lo = (torch.cat([t.new_zeros(shift), t.flatten()])[shift:].view(t.shape) for t in (Q, hi, lo))
    buf = torch.full((H * Lq * Lk + 8,), 7.5, device="cuda")
    S = buf[4 + shift:][:H * Lq * Lk].view(H, Lq, Lk)
    B.adacluster_quest_scores(Q, hi, lo, B.QUEST_ALU, out=S)
    assert (buf[:4 + shift] == 7.5).all() and (buf[4 + shift + H * Lq * Lk:] == 7.5).all()
    rows = torch.unique(torch.cat([torch.arange(min(Lq, 130)), torch.arange(max(0, Lq - 130), Lq), torch.tensor([Lq // 3])])).cuda()
    for h in range(H):
        q, p, n = Q[h, rows].double()[:, None], hi[h].double()[None], lo[h].double()[None]
        ref = torch.fmax(q * p, q * n).sum(2)
        mag = torch.fmax((q * p).abs(), (q * n).abs()).sum(2)
        got = S[h, rows].double()
        fin = torch.isfinite(ref)
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and torch.equal(got[~fin & ~torch.isnan(ref)], ref[~fin & ~torch.isnan(ref)])
        assert ((got - ref).abs()[fin] <= 1e-5 * mag[fin] + 1e-6).all()


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("H,Lq,Lk", [(8, 32801, 65), (4, 8201, 66), (1, 33, 3)])      # eight, four and two rows a thread
def test_vector_form_where_products_overflow(H, Lq, Lk, bf16):
    """Finite values whose products are infinite: Eq. 1 term by term in fp32, so one term of each sign makes NaN, one alone infinity."""
    d = 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(Lq)
    Q, hi, lo = (torch.randn(s, generator=gen, device="cuda") for s in ((H, Lq, d), (H, Lk, d), (H, Lk, d)))
    Q[:, :, 2], Q[:, :, 40] = 2.0 ** 70, 2.0 ** 80
    hi[:, 0, 2], lo[:, 0, 2], hi[:, 0, 40], lo[:, 0, 40] = 2.0 ** 60, -1.0, -2.0 ** 60, -2.0 ** 61      # +inf and -inf
    hi[:, 1, 2], lo[:, 1, 2], hi[:, 1, 40], lo[:, 1, 40] = 2.0 ** 60, -1.0, 0.0, -1.0                     # +inf
    hi[:, 2, 2], lo[:, 2, 2], hi[:, 2, 40], lo[:, 2, 40] = 1.0, -1.0, 0.0, -2.0 ** 60                     # none: the larger product
    if bf16:
        Q, hi, lo = (t.to(torch.bfloat16) for t in (Q, hi, lo))
    S = B.adacluster_quest_scores(Q, hi, lo, B.QUEST_ALU)
    assert S[:, :, 0].isnan().all() and (S[:, :, 1] == float("inf")).all() and S[:, :, 2].isfinite().all()
