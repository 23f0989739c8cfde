"""The label sort behind the attention step, through adacluster_sparse_attn with labels given by the caller: lengths
around the change from one workgroup to the counting sort and around its segments, label counts from one to thousands,
labels past the caller's own cluster count (they belong to no cluster).  Reference: fp32 soft-max over the keys whose
cluster is selected.  Inputs are bf16 values both sides read; the library rounds probabilities and outputs to bf16 (2^-9
each), so 1e-2 relative L2 has a factor of two in hand."""
import numpy as np
import pytest
import torch

from paper_2604_18348_amd import binding as B
from paper_2604_18348_amd import workloads as wl
from tests.helpers import to_dev
from tests.test_gpu_cluster import check_kcluster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,kc,cap,past", [(4096, 40, 64, 0), (4097, 129, 300, 7), (4097, 1, 16, 2), (6143, 700, 1300, 50),
                                           (6144, 2500, 2600, 1), (8193, 4000, 7000, 400)])
def test_rows_follow_their_labels(N, kc, cap, past):
    H, d, Cq = 2, 64, 5
    rng = np.random.default_rng(N + kc)
    m0 = min(cap // 2, 16)
    p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=Cq, k_m0=m0, k_m_min=1, k_max_clusters=cap - m0)
    Q, K, V = (torch.from_numpy(rng.standard_normal((H, N, d)).astype(np.float32)).cuda().to(torch.bfloat16) for _ in range(3))
    # skewed label sizes, and some labels at or past the count
    kl = np.minimum((kc * rng.random((H, N)) ** 2).astype(np.int32), kc - 1)
    if past:
        kl[:, rng.integers(0, N, past)] = kc + rng.integers(0, 3, past)
    ql = rng.integers(0, Cq, (H, N)).astype(np.int32)
    sel = np.zeros((H, Cq, cap), dtype=np.int32)
    cnt = np.zeros((H, Cq), dtype=np.int32)
    pick = rng.random((H, Cq, kc)) < 0.3
    pick[:, :, 0] = True
    for h in range(H):
        for i in range(Cq):
            j = np.nonzero(pick[h, i])[0]
            sel[h, i, :len(j)], cnt[h, i] = j, len(j)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    O = B.adacluster_sparse_attn(p, Q, K, V, dev(ql), dev(kl), torch.full((H,), kc, dtype=torch.int32, device="cuda"),
                                 dev(sel), dev(cnt)).float()
    for h in range(H):
        allowed = np.zeros((Cq, int(kl.max()) + 1), dtype=bool)
        allowed[:, :kc] = pick[h]
        S = (Q[h].float() @ K[h].float().T) / d ** 0.5
        S.masked_fill_(~dev(allowed)[dev(ql[h]).long()][:, dev(kl[h]).long()], float("-inf"))
        ref = torch.softmax(S, 1) @ V[h].float()
        rel = float((O[h] - ref).norm() / ref.norm())
        assert rel < 1e-2, rel


@pytest.mark.parametrize("kc_extra", [0, 5])
@pytest.mark.parametrize("N,kc,cap", [(700, 40, 64), (1500, 127, 128), (1500, 128, 128), (4096, 300, 384), (4097, 128, 128),
                                      (4097, 300, 384)])
def test_labels_and_counts_outside_their_range(N, kc, cap, kc_extra):
    """Either form of the sort: labels below zero, at the count, at and past the capacity, and with the low digits of a valid
    label belong to no cluster and leave the others in place; a count above the capacity (kc_extra) is taken as the capacity,
    and a selected cluster past it is left out.  Query labels outside [0, Cq): those rows are not written."""
    H, d, Cq = 2, 64, 5
    rng = np.random.default_rng(N + kc)
    m0 = min(cap // 2, 16)
    p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=Cq, k_m0=m0, k_m_min=1, k_max_clusters=cap - m0)
    Q, K, V = (torch.from_numpy(rng.standard_normal((H, N, d)).astype(np.float32)).cuda().to(torch.bfloat16) for _ in range(3))
    good = rng.integers(0, kc, (H, N)).astype(np.int64)
    kl, ql = good.copy(), rng.integers(0, Cq, (H, N)).astype(np.int64)
    strange = [-1, -127, -2 ** 31, cap, cap + 3, 2 ** 31 - 1, 128 * 7 + 1, 16384 * 3 + 2, 2 ** 24]
    for h in range(H):
        at = rng.permutation(N)[:N // 8]
        kl[h, at] = rng.choice([s for s in strange if not 0 <= s < cap], at.size)
        at = rng.permutation(N)[:N // 16]
        ql[h, at] = rng.choice([-1, -128, Cq, 128 + 1, 2 ** 31 - 1], at.size)
    sel = np.zeros((H, Cq, cap), dtype=np.int32)
    cnt = np.zeros((H, Cq), dtype=np.int32)
    pick = rng.random((H, Cq, kc)) < 0.3
    pick[:, :, 0] = True
    for h in range(H):
        for i in range(Cq):
            j = np.append(np.nonzero(pick[h, i])[0], cap + 2)[:cap]
            sel[h, i, :len(j)], cnt[h, i] = j, len(j)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    count = cap + kc_extra if kc_extra else kc
    O = torch.full((H, N, d), -7.0, dtype=torch.bfloat16, device="cuda")
    B.adacluster_sparse_attn(p, Q, K, V, dev(ql.astype(np.int32)), dev(kl.astype(np.int32)),
                             torch.full((H,), count, dtype=torch.int32, device="cuda"), dev(sel), dev(cnt), out=O)
    for h in range(H):
        rows = (ql[h] >= 0) & (ql[h] < Cq)
        keys = (kl[h] >= 0) & (kl[h] < kc)
        S = (Q[h].float() @ K[h].float().T) / d ** 0.5
        allowed = np.zeros((N, N), dtype=bool)
        allowed[np.ix_(rows, keys)] = pick[h][ql[h][rows]][:, kl[h][keys]]
        S.masked_fill_(~dev(allowed), float("-inf"))
        r = dev(np.flatnonzero(rows))
        ref = torch.softmax(S[r], 1) @ V[h].float()
        got = O[h].float()
        rel = float((got[r] - ref).norm() / ref.norm())
        assert rel < 1e-2, rel
        assert bool((got[dev(np.flatnonzero(~rows))] == -7.0).all())


@pytest.mark.parametrize("dtype,d,N,m0", [(B.BF16, 64, 4096, 140), (B.BF16, 64, 4097, 140), (B.BF16, 128, 6145, 129),
                                          (B.F32, 64, 4096, 20), (B.F32, 64, 4097, 200)])
def test_key_clustering_around_the_change_of_the_sort(dtype, d, N, m0):
    """More than 128 first-stage centres are updated from sorted labels (fp32: by members up to a size), and the final sort has
    more than 128 clusters, or fewer, on either side of one workgroup's 4 096 items: labels, member means, sizes and boxes
    against the oracle (check_kcluster)."""
    H = 2
    _, K, _ = wl.make_small(61, N, d, 30, dtype="bf16" if dtype == B.BF16 else "f32", H=H)
    p = B.Params(H=H, N=N, d=d, dtype=dtype, q_clusters=4, k_iters=3, k_m0=m0, k_m_min=4, k_max_clusters=3 * m0, tau_factor=1.1)
    out = B.adacluster_kcluster(p, to_dev(K, dtype), want_box=True)
    torch.cuda.synchronize()
    check_kcluster(K, p, out, dtype)


@pytest.mark.parametrize("H,N,cap", [(2, 9000, 100), (60, 9000, 63), (2, 24000, 1791), (2, 24000, 1792), (2, 4097, 1983), (2, 4097, 1984),
                                     (2, 4097, 2047), (2, 4097, 2048),
                                     (2, 10240, 4031), (2, 10240, 4032), (2, 10240, 4095), (2, 10240, 4096), (2, 81920, 64), (2, 81921, 64)])
def test_sort_with_the_prefix_in_the_scatter_and_in_a_launch(H, N, cap):
    """Sixteen, eight and four waves a segment, the prefix over the segments in the scatter or in a launch before it, on either
    side of every line between them; sampled rows of the first and the last head."""
    d, Cq = 64, 3
    rng = np.random.default_rng(N + cap)
    m0 = min(cap // 2, 16)
    p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=Cq, k_m0=m0, k_m_min=1, k_max_clusters=cap - m0)
    Q, K, V = (torch.from_numpy(rng.standard_normal((H, N, d), dtype=np.float32)).cuda().to(torch.bfloat16) for _ in range(3))
    kl = np.minimum((cap * rng.random((H, N)) ** 2).astype(np.int32), cap - 1)
    kl[:, rng.integers(0, N, 9)] = cap + 1
    ql = rng.integers(0, Cq, (H, N)).astype(np.int32)
    pick = rng.random((H, Cq, cap)) < 0.2
    pick[:, :, 0] = True
    cnt = pick.sum(2).astype(np.int32)
    sel = np.argsort(~pick, axis=2, kind="stable").astype(np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    O = B.adacluster_sparse_attn(p, Q, K, V, dev(ql), dev(kl), torch.full((H,), cap, dtype=torch.int32, device="cuda"),
                                 dev(sel), dev(cnt)).float()
    for h in (0, H - 1):
        r = np.append(rng.integers(0, N, 62), [0, N - 1])
        allowed = np.concatenate([pick[h], np.zeros((Cq, 2), dtype=bool)], axis=1)[ql[h][r]][:, kl[h]]
        S = (Q[h][dev(r)].float() @ K[h].float().T) / d ** 0.5
        ref = torch.softmax(S.masked_fill(~dev(allowed), float("-inf")), 1) @ V[h].float()
        rel = float((O[h][dev(r)] - ref).norm() / ref.norm())
        assert rel < 1e-2, rel
