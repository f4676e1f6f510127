"""Routing statistics at the sizes where their kernels change, against oracle/routing_stats.py (same bars as there)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import routing_stats as rs                      # noqa: E402
from paper_2603_06626_amd import binding as b               # noqa: E402
from tests.test_gpu_routing_stats import DEV, check_all     # noqa: E402


@pytest.mark.parametrize("S,L,k,E,n_nodes,dtype", [
    (3, 255, 8, 128, 16, np.uint8),     # short samples: general kernel; one token short of a workgroup
    (3, 256, 8, 128, 16, np.int32),     # the last size of the general kernel
    (3, 257, 8, 129, 4, np.uint8),      # the first of the packed one
    (256, 257, 1, 128, 4, np.int32),    # with one id per token
    (2, 300, 8, 247, 16, np.int32),
    (2, 300, 8, 248, 4, np.uint8),
    (2, 100, 9, 64, 4, np.uint8),       # more than 8 ids: the wide form
    (2, 130, 64, 256, 4, np.uint8),     # most slots a token can have
    (3, 90, 13, 6, 2, np.int32),        # more slots than experts: every token repeats some
    (1, 257, 10, 250, 5, np.int32),     # k and E beyond the packed form
    (2, 100, 8, 64, 17, np.int32),
    (1, 65280, 2, 5, 3, np.uint8),      # longest sample whose votes fit a byte per lane
    (1, 65281, 2, 5, 3, np.uint8),
    (4, 1, 1, 1, 1, np.int32),
    (3, 511, 8, 128, 16, np.uint8),     # one token short of two rounds
    (3, 512, 8, 128, 16, np.uint8),     # a column per lane, widest table, most nodes
    (3, 513, 8, 129, 5, np.uint8),      # narrower table; one token more than two rounds
    (2, 767, 8, 247, 16, np.int32),     # last E of the packed form
    (2, 768, 1, 247, 1, np.uint8),      # one id per token
    (3, 769, 5, 33, 7, np.uint8),       # ids of a token not in one word
    (2, 600, 8, 248, 4, np.uint8),      # general kernel by E
    (2, 600, 8, 64, 17, np.int32),      # by the number of nodes
    (1, 65281, 4, 9, 3, np.int32),      # by the length
    (257, 256, 8, 128, 4, np.int32),    # more samples than CUs: general kernel
    (257, 257, 4, 128, 4, np.uint8),    # packed for placement alone
    (300, 768, 3, 60, 4, np.uint8),     # both statistics in one call: the last size of the general kernel
    (300, 769, 3, 60, 4, np.int32),     # packed
    (257, 1023, 1, 8, 4, np.uint8),     # one id per token: both statistics general, either alone packed
    (257, 1023, 2, 8, 4, np.uint8),
    (257, 1024, 2, 8, 4, np.uint8),
    (257, 511, 2, 8, 4, np.uint8),      # general for the affinity alone
    (257, 512, 2, 8, 4, np.uint8),      # packed
    (257, 768, 1, 8, 4, np.uint8),      # general with one id
    (1025, 1023, 8, 64, 3, np.uint8),   # more samples than fit at once: general
    (1025, 1024, 8, 64, 3, np.uint8),   # packed
    (1025, 1281, 7, 64, 3, np.int32),   # the same with fewer ids per token
    (1025, 2047, 2, 200, 4, np.uint8),  # general
    (1025, 2048, 2, 200, 4, np.uint8),  # packed
    (512, 3, 2, 64, 4, np.uint8),       # loads in one workgroup
    (513, 3, 2, 64, 4, np.uint8),       # and in two launches
])
def test_statistics_at_the_edges_of_their_kernels(S, L, k, E, n_nodes, dtype):
    rng = np.random.default_rng(E + k)
    idx = rng.integers(0, E, size=(S, L, k)).astype(dtype)      # repeated ids inside tokens occur
    idx[:, L // 2:] = np.sort(idx[:, L // 2:], axis=2)[:, :, ::-1]
    perm = rng.permutation(E)
    check_all(idx, E, [perm[n::n_nodes] for n in range(n_nodes)], E_T_list=(max(1, E // 5),), label=f"{S}x{L}x{k} E={E}")


@pytest.mark.parametrize("L", [65280, 65281])
@pytest.mark.parametrize("n_nodes", [1, 4])
def test_votes_of_the_longest_samples(L, n_nodes):
    """Every token reaches node 0, so that a lane of the packed kernel counts 255 votes for it at 65280 tokens, which is what a
    byte holds; 65281 tokens make 256."""
    rng = np.random.default_rng(L)
    E, k = 8, 2
    idx = np.zeros((2, L, k), dtype=np.uint8)
    idx[:, :, 1] = rng.integers(1, E, size=(2, L))
    nodes = [np.array([0])] + [np.arange(1, E)[n::n_nodes - 1] for n in range(n_nodes - 1)]
    check_all(idx, E, nodes, label=f"{L} tokens, all on node 0 of {n_nodes}")


@pytest.mark.parametrize("dtype", [np.uint8, np.int32])
@pytest.mark.parametrize("T,k,E", [
    (1, 1, 1), (1, 8, 9), (3, 2, 33),               # fewer ids than one fetch takes
    (513, 2, 64), (1537, 1, 32), (2049, 3, 128), (1025, 7, 256),    # a last run of one token, whose fetch begins before it
    (511, 4, 65), (1024, 5, 97), (4097, 8, 129),    # one block, several, an odd number; 4 and 8 slots kept
    (5000, 8, 200), (30000, 6, 63), (700, 9, 60), (900, 64, 250),
    (1025, 2, 200), (1025, 9, 40),                  # runs of 512 tokens; of 256 up to 1024 on many experts or with many ids
    (98305, 2, 100), (49153, 4, 130), (98305, 2, 129), (131073, 1, 200), (262145, 1, 90),   # one token more than the shortest runs take
])
def test_coactivation_at_the_edges_of_its_kernels(T, k, E, dtype):
    """Exact counts.  Ids repeat inside tokens, and some lie outside [0, E)."""
    rng = np.random.default_rng(T + k + E)
    idx = (rng.integers(0, 1 << 30, size=(T, k)) % rng.integers(1, E + 1, size=(T, 1))).astype(dtype)
    stray = rng.random((T, k)) < 0.1
    idx[stray] = rng.choice([min(E, 255), 255] if dtype is np.uint8 else [-1, E, E + 70, 2**31 - 1, -2**31], size=stray.sum())
    P = torch.full((E, E), -1, dtype=torch.int64, device=DEV)
    b.grouter_coactivation(torch.from_numpy(idx).to(DEV), E, P)
    wide = idx.astype(np.int64)
    wide[(wide < 0) | (wide >= E)] = E      # an expert more, left out again, for the ids that do not count
    assert (P.cpu().numpy() == rs.coactivation(wide, E + 1)[:E, :E]).all()


@pytest.mark.parametrize("T,E,pair", [
    (256 * 1023 * 512, 40, (38, 39)), (256 * 1024 * 512 - 8, 40, (6, 33)),      # 65472 tokens in every wave; 65536, and a shorter last run with as many
    (256 * 1023 * 512, 64, (32, 33)), (256 * 1024 * 512 - 511, 64, (0, 63)),
    (256 * 510 * 256, 200, (198, 199)), (256 * 1024 * 128 - 100, 200, (10, 163)),   # the same with 128 of 256 tokens in a wave
    (256 * 1024 * 128 - 127, 256, (254, 255)),
    ((1 << 32) - 1, 200, (198, 199)), ((1 << 32) - 1, 200, (96, 97)),           # the most that two counts to a word hold, in both halves
])
def test_coactivation_of_one_pair_only(T, E, pair):
    """Every token picks the same two experts: the largest counts at the limits of 16 bits a wave and 32 bits a word."""
    idx = torch.tensor(pair, dtype=torch.uint8, device=DEV).repeat(T, 1)
    P = torch.full((E, E), -1, dtype=torch.int64, device=DEV)
    b.grouter_coactivation(idx, E, P)
    del idx
    ref = torch.zeros((E, E), dtype=torch.int64)
    for i in pair:
        for j in pair:
            ref[i, j] = T
    assert torch.equal(P.cpu(), ref)


def test_coactivation_of_more_tokens_than_half_a_word_counts():
    """2^32 tokens of one expert and three of another: counts that two to a word could not hold, and up to 2^21 in a wave's fp32."""
    E, T = 200, (1 << 32) + 3
    idx = torch.zeros((T, 1), dtype=torch.uint8, device=DEV)
    idx[T // 2] = idx[5] = idx[T - 1] = 199
    P = torch.full((E, E), -1, dtype=torch.int64, device=DEV)
    b.grouter_coactivation(idx, E, P)
    ref = torch.zeros((E, E), dtype=torch.int64)
    ref[0, 0], ref[199, 199] = T - 3, 3
    assert torch.equal(P.cpu(), ref)


@pytest.mark.parametrize("E_S,E_T,scale", [(1, 1, 1), (63, 5, 1), (64, 64, 1), (65, 7, 1), (128, 1, 1), (129, 40, 1), (256, 100, 1),
                                           (257, 60, 1), (128, 31, 1 << 44), (200, 9, 1 << 44), (201, 30, 1),
                                           # groups of 8 with entries up to 6 * scale + 2: the last whose sums fit a key, and one more
                                           (64, 8, 349524), (64, 8, 349525), (128, 16, 349524), (128, 16, 349525),
                                           (200, 25, 349524), (200, 25, 349525)])
def test_fold_groups_sizes_ties_and_large_entries(E_S, E_T, scale):
    """Few distinct values make many ties; sums of 2^24 and more are grouped by 64-bit keys, entries of 2^46 and more, up to 6 *
    2^44 here, by the loop that compares scores."""
    rng = np.random.default_rng(E_S)
    P = rng.integers(0, 4, size=(E_S, E_S)).astype(np.int64) * scale + (rng.integers(0, 2, size=(E_S, E_S)) if scale > 1 else 0)
    P = P + P.T
    grp = torch.full((E_S,), -1, dtype=torch.int32, device=DEV)
    b.grouter_fold_groups(torch.from_numpy(P).to(DEV), E_T, grp)
    assert (grp.cpu().numpy() == rs.fold_groups(P, E_T)).all()


@pytest.mark.parametrize("E_S,E_T", [(5, 2), (60, 1), (64, 9), (128, 1), (128, 30), (180, 50), (200, 7), (201, 30), (256, 1), (256, 60)])
@pytest.mark.parametrize("lowest,highest", [(-3, 3), (-1, 0), (-(1 << 46), (1 << 46) - 1), (-(1 << 46) - 1, 0), (0, 1 << 46), ((1 << 32) - 2, (1 << 32) + 1)])
@pytest.mark.parametrize("where", ["all", "last"])
def test_fold_groups_at_the_limits_of_64_bit_keys(E_S, E_T, lowest, highest, where):
    """Entries of either sign up to the sizes that 64-bit keys take, and one more; in every place, or only in the last ones looked at."""
    rng = np.random.default_rng(E_S + E_T)
    extreme = rng.choice([lowest, highest, lowest + 1, highest - 1], size=(E_S, E_S))
    P = extreme if where == "all" else rng.integers(0, 4, size=(E_S, E_S))
    P[-1] = extreme[-1]
    P = np.triu(P) + np.triu(P, 1).T
    P[:, -1] = P[-1] = extreme[-1]
    P[np.arange(E_S), np.arange(E_S)] = rng.choice([1 << 62, 0, -(1 << 62)], size=E_S)     # the diagonal decides nothing
    P = P.astype(np.int64)
    grp = torch.full((E_S,), -1, dtype=torch.int32, device=DEV)
    b.grouter_fold_groups(torch.from_numpy(P).to(DEV), E_T, grp)
    zero = P.copy()
    zero[np.arange(E_S), np.arange(E_S)] = 0
    assert (grp.cpu().numpy() == rs.fold_groups(zero, E_T)).all()


def _groups_in_doubles(P, E_T):
    """The same greedy grouping with scores in float64."""
    P, E_S = P.astype(np.float64), len(P)
    group_of = np.full(E_S, -1, dtype=np.int32)
    for g in range(E_T):
        score = np.zeros(E_S)
        for _ in range(E_S // E_T + (g < E_S % E_T)):
            pick = int(np.argmax(np.where(group_of < 0, score, -np.inf)))
            group_of[pick] = g
            score = score + P[pick]
    return group_of


@pytest.mark.parametrize("E_S,E_T", [(30, 6), (64, 20), (128, 31), (200, 50)])
def test_fold_groups_beyond_the_exact_range_of_doubles(E_S, E_T):
    """Entries of 2^54 and more, where doubles are four apart, that differ in the two bits below."""
    P = (1 << 54) + np.random.default_rng(E_S).integers(0, 4, size=(E_S, E_S)).astype(np.int64)
    P = np.triu(P) + np.triu(P, 1).T
    ref = rs.fold_groups(P, E_T)
    assert (rs.fold_groups(P >> 44, E_T) == _groups_in_doubles(P >> 44, E_T)).all()      # the same rule where doubles are exact
    assert (_groups_in_doubles(P, E_T) != ref).any()
    grp = torch.full((E_S,), -1, dtype=torch.int32, device=DEV)
    b.grouter_fold_groups(torch.from_numpy(P).to(DEV), E_T, grp)
    assert (grp.cpu().numpy() == ref).all()


def test_fold_weights_with_groups_that_have_no_members():
    rng = np.random.default_rng(0)
    d, E_S, E_T = 13, 40, 12
    grp = rng.choice([0, 3, 11, 7], size=E_S).astype(np.int32)
    W = rng.standard_normal((d, E_S), dtype=np.float32)
    out = torch.full((d, E_T), float("nan"), dtype=torch.float32, device=DEV)
    b.grouter_fold_weights(torch.from_numpy(W).to(DEV), torch.from_numpy(grp).to(DEV), E_T, out)
    ref = np.zeros((d, E_T))
    for e in range(E_S):
        ref[:, grp[e]] += W[:, e]
    # at most 40 fp32 additions of relative error 2^-24 each
    assert np.abs(out.cpu().numpy() - ref).max() <= 40 * 2.0 ** -24 * np.abs(W).sum(axis=1).max()


@pytest.mark.parametrize("d,E_S,E_T", [
    (1, 1, 1), (9, 64, 1), (9, 65, 1), (8, 63, 63), (3, 65, 64), (4, 66, 66), (17, 1024, 1), (5, 1024, 1024), (5, 1000, 7), (2, 513, 300),
])
@pytest.mark.parametrize("stray", [False, True])
def test_folded_weights_add_members_in_ascending_order(d, E_S, E_T, stray):
    """Bit-exact: the same fp32 additions in the same order.  stray: some experts belong to no group."""
    rng = np.random.default_rng(E_S + E_T)
    grp = (rng.integers(0, E_T, size=E_S) ** 2 // max(1, E_T)).astype(np.int32)     # groups of very different size
    if stray:
        grp[rng.integers(0, E_S, size=max(1, E_S // 5))] = rng.choice([-1, -2**31, E_T, 2**31 - 1])
    W = rng.standard_normal((d, E_S), dtype=np.float32)
    out = torch.full((d, E_T), float("nan"), dtype=torch.float32, device=DEV)
    b.grouter_fold_weights(torch.from_numpy(W).to(DEV), torch.from_numpy(grp).to(DEV), E_T, out)
    ref = np.zeros((d, E_T), dtype=np.float32)
    for e in range(E_S):
        if 0 <= grp[e] < E_T:
            ref[:, grp[e]] += W[:, e]
    assert np.array_equal(out.cpu().numpy(), ref)
