"""The plan rule as the workspace shows it (the partitioned path holds both sides' tuples, the
unpartitioned one a few hundred bytes a unit); no GPU needed."""
import pytest

n = pytest.importorskip("paper_1904_11201_amd._native",
                        reason="libjoin.so not built (python -m paper_1904_11201_amd.build)")
M = 1 << 20
CAP = 9216


def _partitioned(nR, nS, kind=n.JOIN_KIND_HASH):
    return n.lib.join_workspace_bytes(kind, nR, nS, None) >= 8 * (nR + nS)


@pytest.mark.parametrize("nS", [M, 6 * M, 6 * M + 1, 8 * M, 64 * M, (1 << 31) - 1])
def test_a_build_of_two_tables_is_never_partitioned(nS):
    assert not _partitioned(CAP, nS)
    assert not _partitioned(CAP + 1, nS)
    assert not _partitioned(2 * CAP, nS)


def test_more_tables_are_partitioned_past_the_repeats():
    for chunks in (3, 4, 16):
        line = 6 * M // (chunks - 1)
        assert not _partitioned(chunks * CAP, line)
        assert _partitioned(chunks * CAP, line + 1)
    assert _partitioned(16 * CAP + 1, 1000)


def test_the_semi_join_follows_the_same_rule():
    for nS in (6 * M, 6 * M + 1, 64 * M):
        assert not _partitioned(2 * CAP, nS, n.JOIN_KIND_HASH_PREFILTER)
    assert not _partitioned(3 * CAP, 3 * M, n.JOIN_KIND_HASH_PREFILTER)
    assert _partitioned(3 * CAP, 3 * M + 1, n.JOIN_KIND_HASH_PREFILTER)
