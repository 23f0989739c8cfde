"""The label sort behind the attention step, through adacluster_sparse_attn with labels given by the caller: lengths
around the change from one workgroup to the counting sort and around its segments, label counts from one to thousands,
labels past the caller's own cluster count (they belong to no cluster).  Reference: fp32 soft-max over the keys whose
cluster is selected.  Inputs are bf16 values both sides read; the library rounds probabilities and outputs to bf16 (2^-9
each), so 1e-2 relative L2 has a factor of two in hand."""
import numpy as np
import pytest
import torch

from paper_2604_18348_amd import binding as B

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
