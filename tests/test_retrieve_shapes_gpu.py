"""Exactness of the retrieval over the shapes at which its kernels change:
few queries (one 32-query tile, features split over four waves, up to 1024
features) against the 256-query screen, and the decision by one wave or by
four (k > 1, or an index of more than 512 blocks), with the register cache of
block maxima and the rounds of block tests exceeded, many candidates, ties,
keys past the screen's range and non-finite values.  The reference is the
definition itself: fp64 sums in feature order (every product of two fp32
values is exact in fp64), larger score first, then the lower row."""
import pytest
import torch

from paper_2608_02560_amd import precog as P

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _ref(q, K, k):
    s = torch.zeros((q.shape[0], K.shape[0]), dtype=torch.float64, device=DEV)
    qd, Kd = q.double(), K.double()
    for e in range(q.shape[1]):
        s += qd[:, e, None] * Kd[None, :, e]
    v, i = torch.sort(s, dim=1, descending=True, stable=True)
    return i[:, :k].int(), v[:, :k]


def _check(q, K, k):
    i, v = _ref(q, K, k)
    prep = P.prepare_index(K)
    for got in (P.topk(q, K, k), P.topk_prepared(q, K, prep, k)):
        assert torch.equal(got[0], i) and torch.equal(got[1], v)
    if k == 1:
        assert torch.equal(P.top1(q, K), i[:, 0])
        assert torch.equal(P.topk_prepared(q, K, prep, 1, want_score=False)[0], i)


def _unit(shape, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    v = torch.randn(shape, generator=g, device=DEV)
    return v / v.norm(dim=-1, keepdim=True)


@pytest.mark.parametrize("Q,M,E,k", [
    (1, 1, 4, 1), (1, 31, 16, 3), (32, 33, 128, 10), (33, 65, 128, 10), (31, 500, 132, 64), (2, 1000, 388, 3),
    (32, 4096, 512, 5), (3, 4129, 516, 1), (5, 2050, 1024, 3), (5, 2050, 1028, 3), (40, 8200, 384, 10),
    (7, 16390, 64, 1), (3, 140001, 16, 10), (2, 1100000, 4, 3)])
def test_exact_over_shapes(Q, M, E, k):
    _check(_unit((Q, E), 1), _unit((M, E), 2), k)


@pytest.mark.parametrize("k", [1, 3, 64])
@pytest.mark.parametrize("M", [300, 3000, 20000])
def test_many_candidates(M, k):
    """Near-duplicate keys in every block, so that whole blocks are rescored
    and the candidate list overflows; the first rows repeat further on."""
    base = _unit((1, 64), 3)
    K = base + 1e-4 * _unit((M, 64), 4)
    K[M // 2:M // 2 + 40] = K[:40]
    _check(torch.cat([base, _unit((3, 64), 5)]), K.contiguous(), k)


@pytest.mark.parametrize("k", [1, 5])
def test_beyond_the_screens_range(k):
    """Keys (or a query) whose norm could overflow the screen's fp16: every
    key is scored; and all keys equal: the lowest rows."""
    q, K = _unit((3, 32), 6), _unit((17000, 32), 7)
    K[123] *= 300.0
    _check(q, K, k)
    _check(300.0 * q, _unit((700, 32), 8), k)
    _check(q, _unit((1, 32), 9).expand(900, 32).contiguous(), k)


@pytest.mark.parametrize("Q", [3, 40])
@pytest.mark.parametrize("M", [600, 17000])
def test_a_nan_key_is_never_ranked(Q, M):
    q, K = _unit((Q, 32), 10), _unit((M, 32), 11)
    i, v = _ref(q, K, 4)
    K[int(i[0, 0])] = float("nan")
    s = torch.zeros((Q, M), dtype=torch.float64, device=DEV)
    for e in range(32):
        s += q.double()[:, e, None] * K.double()[None, :, e]
    s = torch.where(s.isnan(), -torch.inf, s)
    v, i = torch.sort(s, dim=1, descending=True, stable=True)
    for got in (P.topk(q, K, 4), P.topk_prepared(q, K, P.prepare_index(K), 4)):
        assert torch.equal(got[0], i[:, :4].int()) and torch.equal(got[1], v[:, :4])
