"""GPU parity of the attention kernels against the fp64 oracle (Alg. 3 lines 9-10, dense branch).

Tolerances (from the benchmark spec): fp32 I/O 1e-4 max-abs; bf16 I/O 1e-2 relative L2 and 2e-2
max-abs against the fp64 oracle fed the same bf16-rounded inputs."""
import numpy as np
import pytest
import torch

from oracle import adacluster_oracle as orc
from paper_2604_18348_amd import binding as B
from paper_2604_18348_amd import workloads as wl
from tests.helpers import attn_errors, sel_to_dev, to_dev, to_np

pytestmark = pytest.mark.gpu


def check(got, ref, dtype):
    rel, mx = attn_errors(got, ref)
    if dtype == B.F32:
        assert mx < 1e-4, (rel, mx)
    else:
        assert rel < 1e-2 and mx < 2e-2, (rel, mx)
    return rel, mx


def make_case(seed, N, d, dtype, H=2, Cq=5, Ck=23, M=12):
    Q, K, V = wl.make_small(seed, N, d, M, dtype="bf16" if dtype == B.BF16 else "f32", H=H)
    rng = np.random.default_rng(seed + 100)
    ql = rng.integers(0, Cq, (H, N)).astype(np.int32)
    kl = rng.integers(0, Ck, (H, N)).astype(np.int32)
    # ragged clusters: squeeze most keys into a few clusters, leave one empty
    kl[kl == 3] = 4
    sel = []
    for h in range(H):
        rows = []
        for i in range(Cq):
            k = int(rng.integers(1, Ck))
            rows.append(np.sort(rng.choice(Ck, size=k, replace=False)).astype(np.int64))
        sel.append(rows)
    return Q, K, V, ql, kl, sel


def run_sparse(Q, K, V, ql, kl, sel, dtype, Cq, Ck):
    H, N, d = Q.shape
    p = B.Params(H=H, N=N, d=d, dtype=dtype, q_clusters=Cq, k_m0=min(4, N), k_m_min=1,
                 k_max_clusters=max(Ck, 4))
    assert p.cap >= Ck
    si, sc = sel_to_dev(sel, Cq, p.cap)
    O = B.adacluster_sparse_attn(p, to_dev(Q, dtype), to_dev(K, dtype), to_dev(V, dtype),
                                 torch.from_numpy(ql).cuda(), torch.from_numpy(kl).cuda(),
                                 torch.full((H,), Ck, dtype=torch.int32, device="cuda"), si, sc)
    torch.cuda.synchronize()
    return to_np(O)


@pytest.mark.parametrize("dtype,d,N", [(B.BF16, 64, 1000), (B.BF16, 128, 1537), (B.BF16, 64, 37),
                                       (B.F32, 64, 700), (B.F32, 128, 333)])
def test_sparse_attention_matches_oracle(dtype, d, N):
    Cq, Ck = 5, 23
    Q, K, V, ql, kl, sel = make_case(1, N, d, dtype)
    got = run_sparse(Q, K, V, ql, kl, sel, dtype, Cq, Ck)
    for h in range(Q.shape[0]):
        ref = orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h])
        print("sparse", dtype, d, N, h, check(got[h], ref, dtype))


@pytest.mark.parametrize("dtype,d,N", [(B.BF16, 64, 1000), (B.BF16, 128, 777), (B.F32, 64, 515), (B.BF16, 128, 1),
                                       (B.BF16, 64, 64), (B.BF16, 64, 2048 + 63)])
def test_dense_attention_matches_oracle(dtype, d, N):
    H = 2
    Q, K, V = wl.make_small(2, N, d, max(1, min(12, N)), dtype="bf16" if dtype == B.BF16 else "f32", H=H)
    p = B.Params(H=H, N=N, d=d, dtype=dtype, q_clusters=1, k_m0=1, k_m_min=1, k_max_clusters=1)
    O = to_np(B.adacluster_dense_attn(p, to_dev(Q, dtype), to_dev(K, dtype), to_dev(V, dtype)))
    for h in range(H):
        print("dense", dtype, d, N, h, check(O[h], orc.dense_attention(Q[h], K[h], V[h]), dtype))


@pytest.mark.parametrize("d,H,N", [(64, 1, 129), (64, 2, 2500), (128, 1, 1300), (128, 2, 2049), (64, 9, 1025), (128, 1, 4100), (64, 1, 16385)])
def test_dense_attention_of_small_launches(d, H, N):
    """128 queries a workgroup, whole key lists or pieces of them (the last one short), and heads left over by the eight XCDs."""
    rng = np.random.default_rng(N)
    Q, K, V = (wl.round_bf16_f32(rng.standard_normal((H, N, d)).astype(np.float32)) for _ in range(3))
    Q[0, 0] *= 40.0                             # one query's scores far above the others'
    Q = wl.round_bf16_f32(Q)
    p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=1, k_m0=4, k_m_min=1, k_max_clusters=8)
    O = to_np(B.adacluster_dense_attn(p, to_dev(Q, B.BF16), to_dev(K, B.BF16), to_dev(V, B.BF16)))
    rows = np.unique(np.concatenate([[0, N - 1], np.arange(0, N, max(1, N // 200))]))
    for h in {0, H - 1}:
        S = Q[h, rows].astype(np.float64) @ K[h].astype(np.float64).T / np.sqrt(d)
        P = np.exp(S - S.max(1, keepdims=True))
        check(O[h, rows], (P / P.sum(1, keepdims=True)) @ V[h].astype(np.float64), B.BF16)


def reference_with_dead_keys(Q, K, V, dead, scale):
    """Softmax in fp64 over the keys that are not dead (scores of -inf weigh nothing)."""
    live = np.setdiff1d(np.arange(K.shape[0]), dead)
    S = Q.astype(np.float64) @ K[live].astype(np.float64).T * scale
    P = np.exp(S - S.max(1, keepdims=True))
    return (P / P.sum(1, keepdims=True)) @ V[live].astype(np.float64)


@pytest.mark.parametrize("d,H,N", [(64, 1, 2500), (128, 1, 1300), (128, 2, 2049),          # in pieces of the key list
                                   (64, 30, 545), (128, 9, 1025), (64, 1, 37)])             # whole lists
def test_bf16_scores_of_minus_infinity_weigh_nothing(d, H, N):
    """Queries are positive and dead keys -inf, so whole key tiles have no other score, the first ones or the last ones of a
    list or of its pieces: they add nothing, and a query all of whose scores are -inf gets NaN, as exp(-inf) / sum exp(-inf)
    is.  At scale 2 the lowest finite score would leave the range of a float when scaled."""
    rng = np.random.default_rng(31)
    Q = wl.round_bf16_f32(rng.random((H, N, d)).astype(np.float32) + 0.1)
    K, V = (wl.round_bf16_f32(rng.standard_normal((H, N, d)).astype(np.float32)) for _ in range(2))
    tile = np.arange(N) // 64
    for dead, scale in ((np.arange(N * 3 // 4, N), d ** -0.5), (np.arange(min(N - 1, 161)), d ** -0.5), (np.arange(N - 1), 2.0),
                        (np.arange(1, N), 2.0), (np.flatnonzero(tile % 2 == 0)[:N - 1], d ** -0.5), (np.arange(0, N, 3), d ** -0.5)):
        K2 = K.copy()
        K2[:, dead] = -np.inf
        p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=1, k_m0=1, k_m_min=1, k_max_clusters=1, softmax_scale=scale)
        O = to_np(B.adacluster_dense_attn(p, to_dev(Q, B.BF16), to_dev(K2, B.BF16), to_dev(V, B.BF16)))
        for h in (0, H - 1):
            check(O[h], reference_with_dead_keys(Q[h], K[h], V[h], dead, scale), B.BF16)
    K2[:] = -np.inf
    assert np.all(np.isnan(to_np(B.adacluster_dense_attn(p, to_dev(Q, B.BF16), to_dev(K2, B.BF16), to_dev(V, B.BF16)))))


@pytest.mark.parametrize("d", [64, 128])
def test_bf16_cut_lists_with_dead_keys(d):
    """A list of every cluster, four times the mean list and so cut into chunks: the first clusters hold -inf keys alone, more
    of them than a chunk.  The others have a cluster of live keys each, one a cluster of dead ones, one none."""
    H, N, Cq, Ck = 1, 6000, 8, 23
    rng = np.random.default_rng(37)
    Q = wl.round_bf16_f32(rng.random((H, N, d)).astype(np.float32) + 0.1)
    K, V = (wl.round_bf16_f32(rng.standard_normal((H, N, d)).astype(np.float32)) for _ in range(2))
    ql, kl = (rng.integers(0, c, (H, N)).astype(np.int32) for c in (Cq, Ck))
    dead = np.flatnonzero(kl[0] < 10)
    K2 = K.copy()
    K2[:, dead] = -np.inf
    sel = [[np.arange(Ck), np.array([3]), np.zeros(0)] + [np.array([i + 9]) for i in range(3, Cq)]]
    sel = [[s.astype(np.int64) for s in rows] for rows in sel]
    got = run_sparse(Q, K2, V, ql, kl, sel, B.BF16, Cq, Ck)[0]
    for i in range(Cq):
        rows = ql[0] == i
        keys = np.isin(kl[0], sel[0][i])
        if i == 1:
            assert np.all(np.isnan(got[rows]))
        elif i == 2:
            assert np.all(got[rows] == 0)
        else:
            check(got[rows], reference_with_dead_keys(Q[0][rows], K[0], V[0], np.union1d(dead, np.flatnonzero(~keys)), d ** -0.5), B.BF16)


@pytest.mark.parametrize("dtype", [B.BF16, B.F32])
def test_selecting_every_cluster_reproduces_dense(dtype):
    Cq, Ck = 5, 23
    Q, K, V, ql, kl, _ = make_case(3, 900, 64, dtype)
    sel = [[np.arange(Ck, dtype=np.int64) for _ in range(Cq)] for _ in range(Q.shape[0])]
    got = run_sparse(Q, K, V, ql, kl, sel, dtype, Cq, Ck)
    for h in range(Q.shape[0]):
        check(got[h], orc.dense_attention(Q[h], K[h], V[h]), dtype)


def test_more_ranges_than_the_lds_table_holds():
    """A query cluster whose selection is > 256 separate row ranges walks its range table from HBM
    instead of the LDS copy; every other of 700 tiny key clusters gives 350 ranges."""
    H, N, d, Cq, Ck = 2, 2800, 64, 3, 700
    Q, K, V = wl.make_small(7, N, d, 10, dtype="bf16", H=H)
    rng = np.random.default_rng(8)
    ql = rng.integers(0, Cq, (H, N)).astype(np.int32)
    kl = (np.arange(N) % Ck).astype(np.int32)[None].repeat(H, 0)
    kl = np.ascontiguousarray(rng.permuted(kl, axis=1))
    sel = [[np.arange(i % 2, Ck, 2, dtype=np.int64) if i < 2 else np.arange(0, Ck, 7, dtype=np.int64)
            for i in range(Cq)] for _ in range(H)]
    got = run_sparse(Q, K, V, ql, kl, sel, B.BF16, Cq, Ck)
    for h in range(H):
        ref = orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h])
        print("many ranges", h, check(got[h], ref, B.BF16))


@pytest.mark.parametrize("dtype,d", [(B.BF16, 64), (B.BF16, 128), (B.F32, 64)])
def test_key_lists_of_many_one_key_ranges(dtype, d):
    """The planner writes four entries of a key list at a time, from its ranges in LDS (up to 512 of them) or in memory.
    Every other cluster of one key gives lists of r ranges that end one key further each; the last list joins two-key ranges
    to the large cluster at the end."""
    counts = [1, 2, 3, 4, 5, 63, 65, 511, 512, 513, 0]
    H, N, Cq, Ck = 1, 1400, len(counts), 1031
    Q, K, V = wl.make_small(17, N, d, 10, dtype="bf16" if dtype == B.BF16 else "f32", H=H)
    rng = np.random.default_rng(18)
    ql = rng.integers(0, Cq, (H, N)).astype(np.int32)
    kl = np.minimum(rng.permutation(N), Ck - 1).astype(np.int32)[None, :]
    sel = [[np.arange(1, 2 * r, 2, dtype=np.int64) for r in counts[:-1]] + [np.flatnonzero(np.arange(Ck) % 3)]]
    sel[0][-1] = np.append(sel[0][-1], Ck - 1) if sel[0][-1][-1] != Ck - 1 else sel[0][-1]
    got = run_sparse(Q, K, V, ql, kl, sel, dtype, Cq, Ck)
    check(got[0], orc.sparse_attention_gather(Q[0], K[0], V[0], ql[0], kl[0], sel[0]), dtype)


@pytest.mark.parametrize("H", [8, 11])
def test_heads_dealt_to_xcds_whole_and_leftover_heads(H):
    """Small heads take the mapping that gives every XCD whole heads, eight at a time, and splits the
    H mod 8 leftover heads by tile: H = 8 has no leftover, H = 11 has both kinds."""
    N, d, Cq, Ck = 300, 64, 5, 23
    Q, K, V, ql, kl, sel = make_case(9, N, d, B.BF16, H=H)
    got = run_sparse(Q, K, V, ql, kl, sel, B.BF16, Cq, Ck)
    for h in range(H):
        ref = orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h])
        check(got[h], ref, B.BF16)
    p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=1, k_m0=1, k_m_min=1, k_max_clusters=1)
    O = to_np(B.adacluster_dense_attn(p, to_dev(Q, B.BF16), to_dev(K, B.BF16), to_dev(V, B.BF16)))
    for h in range(H):
        check(O[h], orc.dense_attention(Q[h], K[h], V[h]), B.BF16)


@pytest.mark.parametrize("d", [64, 128])
def test_skewed_selection_cuts_the_long_key_list(d):
    """One query cluster selects every key cluster (a list of 94 key tiles) while the others select one
    small cluster each: the long list is cut into chunks handled by separate workgroups and merged."""
    H, N, Cq, Ck = 2, 6000, 6, 40
    Q, K, V = wl.make_small(12, N, d, 10, dtype="bf16", H=H)
    rng = np.random.default_rng(13)
    ql = rng.integers(0, Cq, (H, N)).astype(np.int32)
    kl = rng.integers(0, Ck, (H, N)).astype(np.int32)
    sel = [[np.arange(Ck, dtype=np.int64) if i == 2 else np.array([i], dtype=np.int64) for i in range(Cq)]
           for _ in range(H)]
    got = run_sparse(Q, K, V, ql, kl, sel, B.BF16, Cq, Ck)
    for h in range(H):
        ref = orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h])
        print("skewed", d, h, check(got[h], ref, B.BF16))


def test_more_cut_lists_than_partial_slots():
    """Ten query clusters of three query tiles select every key; the rest select one small cluster.  The
    chunks wanted (10 x 3 x 5) exceed the partial slots of a head, so the last lists are cut into fewer
    chunks or stay whole; every row must still match."""
    H, N, d, Cq, Ck = 1, 36000, 64, 60, 300
    Q, K, V = wl.make_small(14, N, d, 16, dtype="bf16", H=H)
    rng = np.random.default_rng(15)
    sizes = np.array([380] * 10 + [644] * 50)
    assert sizes.sum() == N
    ql = np.repeat(np.arange(Cq), sizes).astype(np.int32)
    ql = ql[rng.permutation(N)][None, :]
    kl = rng.integers(0, Ck, (H, N)).astype(np.int32)
    sel = [[np.arange(Ck, dtype=np.int64) if i < 10 else np.array([i], dtype=np.int64) for i in range(Cq)]]
    got = run_sparse(Q, K, V, ql, kl, sel, B.BF16, Cq, Ck)
    ref = orc.sparse_attention_gather(Q[0], K[0], V[0], ql[0], kl[0], sel[0])
    print("slot shortage", check(got[0], ref, B.BF16))


def test_empty_selection_gives_zero_rows_and_custom_scale():
    Cq, Ck = 5, 23
    Q, K, V, ql, kl, sel = make_case(4, 600, 64, B.BF16)
    for h in range(Q.shape[0]):
        sel[h][2] = np.zeros(0, dtype=np.int64)
        sel[h][3] = np.array([3], dtype=np.int64)        # cluster 3 is empty by construction
    got = run_sparse(Q, K, V, ql, kl, sel, B.BF16, Cq, Ck)
    for h in range(Q.shape[0]):
        assert np.all(got[h][ql[h] == 2] == 0) and np.all(got[h][ql[h] == 3] == 0)
        ref = orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h])
        check(got[h], ref, B.BF16)
    # explicit softmax scale
    H, N, d = Q.shape
    p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=1, k_m0=1, k_m_min=1, k_max_clusters=1, softmax_scale=0.05)
    O = to_np(B.adacluster_dense_attn(p, to_dev(Q, B.BF16), to_dev(K, B.BF16), to_dev(V, B.BF16)))
    check(O[0], orc.dense_attention(Q[0], K[0], V[0], 0.05), B.BF16)


def test_large_logits_do_not_overflow():
    H, N, d = 1, 300, 64
    rng = np.random.default_rng(5)
    Q = wl.round_bf16_f32((6 * rng.standard_normal((H, N, d))).astype(np.float32))
    K = wl.round_bf16_f32((6 * rng.standard_normal((H, N, d))).astype(np.float32))
    V = wl.round_bf16_f32(rng.standard_normal((H, N, d)).astype(np.float32))
    p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=1, k_m0=1, k_m_min=1, k_max_clusters=1)
    O = to_np(B.adacluster_dense_attn(p, to_dev(Q, B.BF16), to_dev(K, B.BF16), to_dev(V, B.BF16)))
    assert np.all(np.isfinite(O))
    check(O[0], orc.dense_attention(Q[0], K[0], V[0]), B.BF16)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [1, 31, 33, 256, 257, 545])
def test_fp32_key_lists_split_over_the_waves(d, N):
    """The fp32 kernel deals 32-key tiles to the waves of up to four workgroups: fewer tiles than waves, exactly as many,
    one more, a ragged last tile, and query tiles of one row and of 32; the dense form and a selection with an
    empty list."""
    Q, K, V, ql, kl, sel = make_case(17, N, d, B.F32, H=2, Cq=1 if N == 1 else 3, Ck=6, M=max(1, min(12, N)))
    Cq = len(sel[0])
    sel[1][Cq - 1] = np.zeros(0, dtype=np.int64)
    got = run_sparse(Q, K, V, ql, kl, sel, B.F32, Cq, 6)
    for h in range(2):
        check(got[h], orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h]), B.F32)
    p = B.Params(H=2, N=N, d=d, dtype=B.F32, q_clusters=1, k_m0=1, k_m_min=1, k_max_clusters=1)
    O = to_np(B.adacluster_dense_attn(p, to_dev(Q, B.F32), to_dev(K, B.F32), to_dev(V, B.F32)))
    for h in range(2):
        check(O[h], orc.dense_attention(Q[h], K[h], V[h]), B.F32)


@pytest.mark.parametrize("dtype", [B.BF16, B.F32])
def test_a_list_that_names_clusters_twice_stays_inside_its_row(dtype):
    """A selection whose clusters hold more than N keys in all (the interface asks for distinct ones) is cut at N keys: the
    lists of the other query clusters, whose rows of the key-row table lie before and behind it, are not touched."""
    Cq, Ck, N = 5, 23, 900
    Q, K, V, ql, kl, sel = make_case(21, N, 64, dtype)
    for h in range(Q.shape[0]):
        sel[h][2] = np.tile(np.arange(Ck // 2, dtype=np.int64), 2)       # fits the capacity, nearly all keys of it twice
    kl[kl >= Ck // 2] = 4
    got = run_sparse(Q, K, V, ql, kl, sel, dtype, Cq, Ck)
    for h in range(Q.shape[0]):
        rows = ql[h] != 2
        ref = orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], [np.unique(s) for s in sel[h]])
        check(got[h][rows], ref[rows], dtype)
        assert np.all(np.isfinite(got[h]))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,H", [(33, 1), (600, 2), (545, 70)])
def test_fp32_scores_of_minus_infinity_weigh_nothing(d, N, H):
    """Whole key tiles whose every score is -inf (queries are positive, those keys -inf): the waves and workgroups that see
    nothing else add nothing, and a query all of whose scores are -inf gets NaN, as exp(-inf) / sum exp(-inf) is.  With 70
    heads the lists are not split over workgroups."""
    rng = np.random.default_rng(31)
    Q = rng.random((H, N, d)).astype(np.float32) + 0.1
    K, V = (rng.standard_normal((H, N, d)).astype(np.float32) for _ in range(2))
    for dead, scale in ((np.arange(32), d ** -0.5), (np.arange(32, min(N, 161)), d ** -0.5), (np.arange(N - 1), 2.0),
                        (np.arange(0, N, 3), d ** -0.5)):
        K2 = K.copy()
        K2[:, dead] = -np.inf
        p = B.Params(H=H, N=N, d=d, dtype=B.F32, q_clusters=1, k_m0=1, k_m_min=1, k_max_clusters=1, softmax_scale=scale)
        O = to_np(B.adacluster_dense_attn(p, to_dev(Q, B.F32), to_dev(K2, B.F32), to_dev(V, B.F32)))
        live = np.setdiff1d(np.arange(N), dead)
        for h in (0, H - 1):
            S = Q[h].astype(np.float64) @ K[h][live].astype(np.float64).T * scale
            P = np.exp(S - S.max(1, keepdims=True))
            check(O[h], (P / P.sum(1, keepdims=True)) @ V[h][live].astype(np.float64), B.F32)
    K2[:] = -np.inf
    assert np.all(np.isnan(to_np(B.adacluster_dense_attn(p, to_dev(Q, B.F32), to_dev(K2, B.F32), to_dev(V, B.F32)))))


def test_fp32_more_workgroups_than_one_grid_dimension_takes():
    """65 535 heads of 130 one-query clusters: 17.8 million workgroups of 256 threads, more than 2^32 threads.  (Past 256 heads
    each has a grid row of its own.)"""
    H, N, d = 65535, 130, 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    Q, K, V = (torch.randn((H, N, d), generator=gen, device="cuda") for _ in range(3))
    p = B.Params(H=H, N=N, d=d, dtype=B.F32, q_clusters=N, k_m0=1, k_m_min=1, k_max_clusters=1)
    labels = torch.arange(N, dtype=torch.int32, device="cuda").repeat(H, 1)
    sel = torch.zeros((H, N, p.cap), dtype=torch.int32, device="cuda")
    one = torch.ones((H, N), dtype=torch.int32, device="cuda")
    O = B.adacluster_sparse_attn(p, Q, K, V, labels, (labels > 99).int(), 2 * one[:, 0].contiguous(), sel, one)
    for h in range(0, H, 8192):                    # every query takes the keys of cluster 0, the first 100
        S = torch.bmm(Q[h:h + 8192], K[h:h + 8192, :100].transpose(1, 2).contiguous()) / d ** 0.5
        ref = torch.bmm(torch.softmax(S, 2), V[h:h + 8192, :100].contiguous())
        assert float((O[h:h + 8192] - ref).abs().max()) < 1e-4


def pieces_of_the_last_round(tiles, N, d):
    """(whole rounds, tiles left over, pieces of their lists) of an XCD, by the rule of the fp32 kernel; `tiles` per head."""
    full = 3 if d == 64 else 2
    whole, rest = divmod(sum(-(-int(t) // 8) for t in tiles), 32 * full)
    cost = {}
    for sp in (1, 2, 3, 4):
        f, r = divmod(rest * sp, 32 * full)
        k = -(-r // 32)
        turns = 32 * full * f + (0 if r == 0 else 24 * k + 8 * full if f else 32 * k if k > 1 else 33)
        cost[sp] = turns * (2 * -(-(-(-N // 32)) // (4 * sp)) + 1)
    return whole, rest, min(cost, key=lambda sp: (cost[sp], sp))


@pytest.mark.parametrize("H,N,d,whole,rest,pieces",
                         [(64, 545, 64, 0, 0, 1), (65, 545, 128, 0, 0, 1), (256, 330, 64, 0, 0, 1), (257, 330, 128, 0, 0, 1),      # left whole
                          (6, 545, 64, 0, 18, 3), (5, 545, 64, 0, 15, 2), (31, 545, 64, 0, 93, 1), (12, 1321, 64, 0, 72, 4),      # one round
                          (32, 545, 64, 1, 0, 1), (45, 545, 64, 1, 39, 2), (35, 545, 64, 1, 9, 3), (48, 545, 64, 1, 48, 2), (56, 545, 64, 1, 72, 1),        # and past it
                          (13, 545, 128, 0, 39, 3), (5, 545, 128, 0, 15, 2), (21, 545, 128, 0, 63, 1), (8, 1321, 128, 0, 48, 4),
                          (43, 545, 128, 2, 1, 3), (64, 300, 128, 2, 0, 1), (25, 545, 128, 1, 11, 2), (31, 545, 128, 1, 29, 1), (11, 1321, 128, 1, 2, 4)])
def test_fp32_lists_whole_and_split_over_up_to_four_workgroups(H, N, d, whole, rest, pieces):
    """A launch of many tiles leaves key lists whole (the kernel writes the output itself); in smaller ones the tiles past the
    last whole round of an XCD go in up to four pieces, none left over and one among them; up to 256 heads are dealt from the
    tile counts, 64 at a time, more have a grid row each.  Sparse, with an empty list and an empty cluster (the counts are those
    of the dense call); every output element is written."""
    Cq = 5
    cut = H <= 256 and H * (N // 32 + 1) < 1024
    if cut:
        assert pieces_of_the_last_round([-(-N // 32)] * H, N, d) == (whole, rest, pieces)
    Q, K, V, ql, kl, sel = make_case(41, N, d, B.F32, H=H)
    for h in range(0, H, 3):
        sel[h][2] = np.zeros(0, dtype=np.int64)
    ql[1][ql[1] == 4] = 0
    p = B.Params(H=H, N=N, d=d, dtype=B.F32, q_clusters=Cq, k_m0=4, k_m_min=1, k_max_clusters=23)
    si, sc = sel_to_dev(sel, Cq, p.cap)
    Qd, Kd, Vd = to_dev(Q, B.F32), to_dev(K, B.F32), to_dev(V, B.F32)
    O = torch.full_like(Qd, float("nan"))
    B.adacluster_sparse_attn(p, Qd, Kd, Vd, torch.from_numpy(ql).cuda(), torch.from_numpy(kl).cuda(),
                             torch.full((H,), 23, dtype=torch.int32, device="cuda"), si, sc, out=O)
    D = B.adacluster_dense_attn(p, Qd, Kd, Vd, out=torch.full_like(Qd, float("nan")))
    for h in sorted({0, 1, H // 2, H - 2, H - 1}):
        check(to_np(O[h]), orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h]), B.F32)
        check(to_np(D[h]), orc.dense_attention(Q[h], K[h], V[h]), B.F32)
    assert bool(torch.isfinite(O).all()) and bool(torch.isfinite(D).all())


@pytest.mark.parametrize("H,N,d,Cq", [(18, 3700, 64, 3600), (33, 3001, 128, 2700)])
def test_fp32_key_rows_searched_in_the_ranges(H, N, d, Cq):
    """So many query clusters that the table of key rows would take more than 1 GiB: the kernel finds its rows from the ranges
    of a list.  Lists of a range per key cluster (every other one, up to 700 ranges), of one long range, of all keys, of
    single keys, and an empty one; the dense call of the same params."""
    Ck = 1400
    assert Cq > 2 * d and 4 * H * Cq * ((N + 63) // 64 * 64 + 512) > 2 ** 30
    Q, K, V, _, _, _ = make_case(51, N, d, B.F32, H=H)
    rng = np.random.default_rng(52)
    ql = np.sort(rng.integers(0, Cq, (H, N)), axis=1).astype(np.int32)
    ql[:, N // 2:] %= 9                                             # some clusters of whole query tiles
    kl = rng.permuted(np.minimum(np.arange(N) % Ck + (np.arange(N) % 7 == 0) * 3, Ck - 1).astype(np.int32)[None].repeat(H, 0), axis=1)
    kinds = [np.arange(0, Ck, 2), np.arange(100, 900), np.arange(Ck), np.array([5]), np.zeros(0), np.arange(1, Ck, 3),
             np.array([0, 1, 700, Ck - 1]), np.concatenate([np.arange(0, 600), np.arange(601, Ck, 2)])]
    sel = [[kinds[(i + h) % len(kinds)].astype(np.int64) for i in range(Cq)] for h in range(H)]
    p = B.Params(H=H, N=N, d=d, dtype=B.F32, q_clusters=Cq, k_m0=4, k_m_min=1, k_max_clusters=Ck)
    si, sc = sel_to_dev(sel, Cq, p.cap)
    Qd, Kd, Vd = to_dev(Q, B.F32), to_dev(K, B.F32), to_dev(V, B.F32)
    O = torch.full_like(Qd, float("nan"))
    ws = B.workspace(p)
    B.adacluster_sparse_attn(p, Qd, Kd, Vd, torch.from_numpy(ql).cuda(), torch.from_numpy(kl).cuda(),
                             torch.full((H,), Ck, dtype=torch.int32, device="cuda"), si, sc, out=O, ws=ws)
    D = B.adacluster_dense_attn(p, Qd, Kd, Vd, out=torch.full_like(Qd, float("nan")), ws=ws)
    for h in (0, H - 1):
        check(to_np(O[h]), orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h]), B.F32)
    check(to_np(D[H - 1]), orc.dense_attention(Q[H - 1], K[H - 1], V[H - 1]), B.F32)
    assert bool(torch.isfinite(O).all()) and bool(torch.isfinite(D).all())


def test_fp32_head_of_more_than_4_gib():
    """Byte offsets inside a head pass 2^32: 100 keys of 8.4 million, the last rows among them."""
    H, N, d = 1, 2 ** 23 + 4001, 128
    assert N * d * 4 > 2 ** 32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(4)
    Q, K, V = (torch.randn((H, N, d), generator=gen, device="cuda") for _ in range(3))
    at = torch.cat([torch.randint(0, N, (60,), generator=gen, device="cuda"), torch.arange(N - 40, N, device="cuda")]).unique()
    kl = torch.zeros((H, N), dtype=torch.int32, device="cuda")
    kl[0, at] = 1
    p = B.Params(H=H, N=N, d=d, dtype=B.F32, q_clusters=1, k_m0=1, k_m_min=1, k_max_clusters=3)
    sel = torch.ones((H, 1, p.cap), dtype=torch.int32, device="cuda")
    one = torch.ones((H, 1), dtype=torch.int32, device="cuda")
    O = torch.full_like(Q, float("nan"))
    B.adacluster_sparse_attn(p, Q, K, V, torch.zeros_like(kl), kl, 2 * one[0], sel, one, out=O)
    for n in range(0, N, 2 ** 20):
        P = torch.softmax(Q[0, n:n + 2 ** 20] @ K[0, at].T.contiguous() / d ** 0.5, 1)
        assert float((O[0, n:n + 2 ** 20] - P @ V[0, at]).abs().max()) < 1e-4


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_lists_shorter_than_their_split(d):
    """Two heads have their lists split over up to four workgroups of four waves: lists of 1 to 17 key tiles of 32 keys, so that
    one workgroup writes the row, or two, three or four leave parts (and the first stands in for the others), beside an empty
    list, with the workspace full of NaN before the call."""
    H, tiles = 2, [0, 1, 4, 5, 8, 9, 12, 13, 16, 17]
    Cq, Ck, N = len(tiles), len(tiles), 32 * sum(tiles) - 40
    rng = np.random.default_rng(71)
    Q, K, V = (rng.standard_normal((H, N, d)).astype(np.float32) for _ in range(3))
    sizes = [max(0, 32 * t - (5 if t < 9 else 0)) for t in tiles]
    kl = np.repeat(np.arange(Ck), sizes)[:N]
    kl = np.concatenate([kl, np.full(N - kl.size, 1)])
    kl = np.stack([rng.permutation(kl) for _ in range(H)]).astype(np.int32)
    ql = rng.integers(0, Cq, (H, N)).astype(np.int32)
    sel = [[np.array([i], dtype=np.int64) for i in range(Cq)] for _ in range(H)]
    p = B.Params(H=H, N=N, d=d, dtype=B.F32, q_clusters=Cq, k_m0=4, k_m_min=1, k_max_clusters=Ck)
    si, sc = sel_to_dev(sel, Cq, p.cap)
    ws = B.workspace(p)
    ws.fill_(0xFF)
    O = to_np(B.adacluster_sparse_attn(p, to_dev(Q, B.F32), to_dev(K, B.F32), to_dev(V, B.F32), torch.from_numpy(ql).cuda(),
                                       torch.from_numpy(kl).cuda(), torch.full((H,), Ck, dtype=torch.int32, device="cuda"), si, sc, ws=ws))
    for h in range(H):
        check(O[h], orc.sparse_attention_gather(Q[h], K[h], V[h], ql[h], kl[h], sel[h]), B.F32)


@pytest.mark.parametrize("H,N,d,Cq", [(64, 2600, 64, 24),       # as many heads as are dealt by work
                                      (5, 9247, 128, 65),       # a tile more than places on an XCD
                                      (2, 34000, 128, 3),       # 256 queries a workgroup, a list of all keys
                                      (16, 5000, 64, 256),      # as many query clusters as are dealt by work, many of a row or none
                                      (7, 6001, 128, 33)])
def test_tiles_dealt_by_work(H, N, d, Cq):
    """Heads and clusters of very different lists (none, one cluster, all), so that parts, order and pieces of the tiles differ from XCD
    to XCD; every row against float64 on the device, and a second call bit for bit."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * N)
    Ck = 40
    Q, K, V = (torch.randn((H, N, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    rng = np.random.default_rng(N)
    ql = np.minimum((Cq * rng.random((H, N)) ** 2).astype(np.int32), Cq - 1)
    kl = rng.integers(0, Ck, (H, N)).astype(np.int32)
    sel = [[np.sort(rng.choice(Ck, size=Ck if i == Cq // 2 else int(rng.integers(0, max(2, Ck * (h + 1) // H))), replace=False)) for i in range(Cq)]
           for h in range(H)]
    p = B.Params(H=H, N=N, d=d, dtype=B.BF16, q_clusters=Cq, k_m0=4, k_m_min=1, k_max_clusters=Ck)
    si, sc = sel_to_dev(sel, Cq, p.cap)
    qt, kt = torch.from_numpy(ql).cuda(), torch.from_numpy(kl).cuda()
    kc = torch.full((H,), Ck, dtype=torch.int32, device="cuda")
    ws = B.workspace(p)
    O = B.adacluster_sparse_attn(p, Q, K, V, qt, kt, kc, si, sc, ws=ws)
    again = B.adacluster_sparse_attn(p, Q, K, V, qt, kt, kc, si, sc, ws=ws)
    assert torch.equal(O, again)
    worst = 0.0
    for h in range(H):
        ref = torch.zeros((N, d), dtype=torch.float64, device="cuda")
        for i in range(Cq):
            rows = torch.nonzero(qt[h] == i)[:, 0]
            keys = torch.nonzero(torch.isin(kt[h], torch.from_numpy(sel[h][i].astype(np.int32)).cuda()))[:, 0]
            for r in rows.split(4096) if len(keys) else ():
                P = torch.softmax(Q[h, r].double() @ K[h, keys].double().T.contiguous() / d ** 0.5, 1)
                ref[r] = P @ V[h, keys].double()
        got = O[h].double()
        rel, mx = float((got - ref).norm() / ref.norm().clamp_min(1e-30)), float((got - ref).abs().max())
        assert rel < 1e-2 and mx < 2e-2, (h, rel, mx)
        worst = max(worst, rel)
    print("dealt", H, N, d, Cq, worst)


@pytest.mark.parametrize("H,N,d,Cq", [(2, 6400, 128, 65),       # one round of workgroups: every list in pieces
                                      (3, 9001, 64, 41),        # more: the last tiles
                                      (4, 9100, 128, 200),      # 1 024 tiles and more: whole lists
                                      (64, 1200, 64, 100)])
def test_fp32_tiles_dealt_by_work(H, N, d, Cq):
    """As test_tiles_dealt_by_work, for fp32: heads and clusters of very different lists, every row against float64 on the device."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(H * N)
    Ck = 40
    Q, K, V = (torch.randn((H, N, d), generator=gen, device="cuda") for _ in range(3))
    rng = np.random.default_rng(N)
    ql = np.minimum((Cq * rng.random((H, N)) ** 2).astype(np.int32), Cq - 1)
    kl = rng.integers(0, Ck, (H, N)).astype(np.int32)
    sel = [[np.sort(rng.choice(Ck, size=Ck if i == Cq // 2 else int(rng.integers(0, max(2, Ck * (h + 1) // H))), replace=False)) for i in range(Cq)]
           for h in range(H)]
    p = B.Params(H=H, N=N, d=d, dtype=B.F32, q_clusters=Cq, k_m0=4, k_m_min=1, k_max_clusters=Ck, select_mode=B.SELECT_TOPP)
    si, sc = sel_to_dev(sel, Cq, p.cap)
    qt, kt = torch.from_numpy(ql).cuda(), torch.from_numpy(kl).cuda()
    kc = torch.full((H,), Ck, dtype=torch.int32, device="cuda")
    ws = B.workspace(p)
    O = B.adacluster_sparse_attn(p, Q, K, V, qt, kt, kc, si, sc, out=torch.full_like(Q, float("nan")), ws=ws)
    assert torch.equal(O, B.adacluster_sparse_attn(p, Q, K, V, qt, kt, kc, si, sc, ws=ws))
    for h in range(0, H, max(1, H // 8)):
        ref = torch.zeros((N, d), dtype=torch.float64, device="cuda")
        for i in range(Cq):
            rows = torch.nonzero(qt[h] == i)[:, 0]
            keys = torch.nonzero(torch.isin(kt[h], torch.from_numpy(sel[h][i].astype(np.int32)).cuda()))[:, 0]
            if len(keys):
                P = torch.softmax(Q[h, rows].double() @ K[h, keys].double().T.contiguous() / d ** 0.5, 1)
                ref[rows] = P @ V[h, keys].double()
        assert float((O[h].double() - ref).abs().max()) < 1e-4, h


@pytest.mark.parametrize("H,N,d,Cq", [(4, 13200, 128, 65),      # a few tiles more than places on an XCD
                                      (9, 9001, 64, 33),        # less than a round
                                      (3, 31000, 128, 30)])     # 256 queries a workgroup
def test_a_head_has_the_same_bits_alone_and_among_others(H, N, d, Cq):
    """bf16 sparse attention: which workgroups run a head's tiles depends on the other heads' lists, how their sums are formed does not."""
    Ck = 40
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    Q, K, V = (torch.randn((H, N, d), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(3))
    rng = np.random.default_rng(N)
    ql = torch.from_numpy(np.minimum((Cq * rng.random((H, N)) ** 2).astype(np.int32), Cq - 1)).cuda()
    kl = torch.from_numpy(rng.integers(0, Ck, (H, N)).astype(np.int32)).cuda()
    sel = [[np.sort(rng.choice(Ck, size=int(rng.integers(0, max(2, Ck * (h + 1) // H))), replace=False)) for _ in range(Cq)] for h in range(H)]

    def attend(heads):
        p = B.Params(H=len(heads), N=N, d=d, dtype=B.BF16, q_clusters=Cq, k_m0=4, k_m_min=1, k_max_clusters=Ck)
        si, sc = sel_to_dev([sel[h] for h in heads], Cq, p.cap)
        x = [t[heads].contiguous() for t in (Q, K, V, ql, kl)]
        return B.adacluster_sparse_attn(p, *x, torch.full((len(heads),), Ck, dtype=torch.int32, device="cuda"), si, sc, ws=B.workspace(p))

    O = attend(list(range(H)))
    for h in range(H):
        assert torch.equal(O[h], attend([h])[0]), h


def dealt_reference(Q, K, V, ql, kl, si, sc, scale):
    """Softmax over each query's selected keys in float64 on the device; scores of -inf weigh nothing, a list of such keys gives NaN, an
    empty one 0."""
    ref = torch.zeros(Q.shape, dtype=torch.float64, device="cuda")
    for i in range(si.shape[0]):
        rows = torch.nonzero(ql == i)[:, 0]
        keys = torch.nonzero(torch.isin(kl, si[i, :int(sc[i])]))[:, 0]
        for r in rows.split(4096) if len(keys) else ():
            S = Q[r].double() @ K[keys].double().T.contiguous() * scale
            ref[r] = torch.softmax(S, 1) @ V[keys].double()
    return ref


FUSED_DEALT = [(0, 12, 5000, 128, 65, "topk"),       # between one and two rounds of workgroups
               (0, 24, 4600, 64, 65, "topp"),        # less than one
               (0, 2, 40000, 128, 30, "topk"),       # 256 queries a workgroup
               (1, 4, 8208, 64, 65, "topk"),         # fp32, whole lists
               (1, 2, 9000, 64, 65, "topp"),         # fp32, one round of workgroups: every list in pieces
               (1, 2, 6437, 128, 65, "topp"),
               (1, 3, 8300, 64, 65, "topk")]         # fp32, the tiles past the first round in pieces


@pytest.mark.parametrize("f32,H,N,d,Cq,select", FUSED_DEALT)
def test_fused_call_with_tiles_dealt_by_work(f32, H, N, d, Cq, select):
    """The fused call plans its tiles beside the key lists, the single entry point behind them: the same output to the bit, also from a second
    call on the same workspace; every row of two heads, the last one without structure, against float64."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    M = N // 90
    comp = torch.randint(0, M, (H, N), generator=gen, device="cuda")
    means = torch.randn((H, M, d), generator=gen, device="cuda") * (0.5 * torch.randn((H, M, 1), generator=gen, device="cuda")).exp()
    means[-1] = 0
    pick = lambda m: torch.gather(m, 1, comp[..., None].expand(-1, -1, d))  # noqa: E731
    noise = torch.full((H, 1, 1), 0.3, device="cuda")
    noise[-1] = 1
    Q, K = (pick(means) + noise * torch.randn((H, N, d), generator=gen, device="cuda") for _ in range(2))
    V = torch.randn((H, N, d), generator=gen, device="cuda")
    if not f32:
        Q, K, V = (t.to(torch.bfloat16) for t in (Q, K, V))
    p = B.Params(H=H, N=N, d=d, dtype=B.F32 if f32 else B.BF16, q_clusters=Cq, k_m0=N // 180, k_m_min=8, k_max_clusters=N // 45, topk=12, top_p=0.9,
                 min_unassigned_frac=0.03, select_mode=B.SELECT_TOPP if select == "topp" else B.SELECT_TOPK)
    ws, outs = B.workspace(p), B.alloc_outputs(p, "cuda")
    first = B.adacluster_attn(p, Q, K, V, outs=outs, out=torch.full_like(Q, float("nan")), ws=ws)
    again = B.adacluster_attn(p, Q, K, V, outs=outs, out=torch.full_like(Q, float("nan")), ws=ws)
    alone = B.adacluster_sparse_attn(p, Q, K, V, outs["q_labels"], outs["k_labels"], outs["k_count"], outs["sel_idx"], outs["sel_cnt"],
                                     out=torch.full_like(Q, float("nan")), ws=ws)
    assert torch.equal(first, again) and torch.equal(first, alone)
    for h in (0, H - 1):
        ref = dealt_reference(Q[h], K[h], V[h], outs["q_labels"][h], outs["k_labels"][h], outs["sel_idx"][h], outs["sel_cnt"][h], d ** -0.5)
        err = first[h].double() - ref
        if f32:
            assert float(err.abs().max()) < 1e-4
        else:
            assert float(err.norm() / ref.norm()) < 1e-2 and float(err.abs().max()) < 2e-2


DEAD_DEALT = [(0, 12, 5000, 128, 65), (1, 2, 6437, 128, 65), (1, 3, 8300, 64, 65)]


@pytest.mark.parametrize("f32,H,N,d,Cq", DEAD_DEALT)
def test_dealt_tiles_with_dead_keys(f32, H, N, d, Cq):
    """Queries are positive, the keys of the first clusters -inf: first pieces of long lists have no other score, some lists have only such keys."""
    Ck = 40
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + 1)
    rng = np.random.default_rng(N)
    Q = torch.rand((H, N, d), generator=gen, device="cuda") + 0.1
    K, V = (torch.randn((H, N, d), generator=gen, device="cuda") for _ in range(2))
    ql = torch.from_numpy(np.minimum((Cq * rng.random((H, N)) ** 2).astype(np.int32), Cq - 1)).cuda()
    kl = torch.from_numpy(rng.integers(0, Ck, (H, N)).astype(np.int32)).cuda()
    K[kl < 25] = float("-inf")
    if not f32:
        Q, K, V = (t.to(torch.bfloat16) for t in (Q, K, V))
    sel = [[np.arange(Ck) if i % 7 == 0 else np.arange(20) if i % 7 == 1 else np.arange(24, 26) if i % 7 == 2 else
            np.sort(rng.choice(Ck, size=int(rng.integers(0, Ck // 2)), replace=False)) for i in range(Cq)] for _ in range(H)]
    p = B.Params(H=H, N=N, d=d, dtype=B.F32 if f32 else B.BF16, q_clusters=Cq, k_m0=4, k_m_min=1, k_max_clusters=Ck, select_mode=B.SELECT_TOPP)
    si, sc = sel_to_dev(sel, Cq, p.cap)
    O = B.adacluster_sparse_attn(p, Q, K, V, ql, kl, torch.full((H,), Ck, dtype=torch.int32, device="cuda"), si, sc, ws=B.workspace(p))
    for h in range(H):
        ref = dealt_reference(Q[h], K[h], V[h], ql[h], kl[h], si[h], sc[h], d ** -0.5)
        got, nan = O[h].double(), ref.isnan()
        assert torch.equal(got.isnan(), nan) and bool(nan.any())
        err = (got - ref)[~nan]
        if f32:
            assert float(err.abs().max()) < 1e-4
        else:
            assert float(err.norm() / ref[~nan].norm()) < 1e-2 and float(err.abs().max()) < 2e-2
