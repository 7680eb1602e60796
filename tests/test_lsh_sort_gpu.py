"""GPU grouping step of the LSH-bucketed join (sj_lsh_sort, Section 4: the
points of every table grouped by bucket) checked by the properties that
define it, on seeded keys: per table the output is a permutation of the rows,
rows of equal keys are contiguous and in increasing row order, the groups
come in ascending key order when the keys have at most 32 bits, and in an
order fixed by the key values otherwise (two key sets sorted by separate calls
list their common keys in the same relative order: the join merges P's order
with Q's).  Sizes are ragged against the sort's 2048-entry blocks.

Keys wider than 32 bits are sorted by the top half of a bijective mix of the
key first; runs whose top halves collide while the keys differ are put in
order afterwards.  Such collisions have probability 2^-32 per pair of keys, so
one case builds them on purpose from the library's mix (multiplication by
0x9E3779B97F4A7C15 modulo 2^64, then the high half xored into the low half),
with colliding runs of thousands of rows across several blocks.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MIX_C = 0x9E3779B97F4A7C15
MASK64 = (1 << 64) - 1


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_12608_amd  # noqa: F401  (fails loudly when libsj.so is missing)
    yield
    torch.cuda.synchronize()


def gpu_sort(keys: np.ndarray, bits: int) -> np.ndarray:
    import torch
    import paper_2006_12608_amd as sj
    kd = torch.from_numpy(np.ascontiguousarray(keys, dtype=np.uint64).view(np.int64)).cuda()
    perm = sj.lsh_sort(kd, bits)
    torch.cuda.synchronize()
    return perm.cpu().numpy().view(np.uint32)


def group_order(keys: np.ndarray, perm: np.ndarray) -> list:
    """Checks one table's grouping and returns its keys in group order."""
    n = keys.size
    assert perm.shape == (n,)
    assert np.array_equal(np.sort(perm), np.arange(n, dtype=np.uint32)), "not a permutation"
    k = keys[perm.astype(np.int64)]
    if n == 0:
        return []
    change = k[1:] != k[:-1]
    assert np.all(change | (perm[1:] > perm[:-1])), "rows of a group not in increasing order"
    starts = np.concatenate([[0], np.flatnonzero(change) + 1])
    order = k[starts]
    assert np.unique(order).size == order.size, "a key is split over several groups"
    return order.tolist()


def same_relative_order(o1: list, o2: list):
    common = set(o1) & set(o2)
    a = [x for x in o1 if x in common]
    b = [x for x in o2 if x in common]
    assert a == b, "common keys listed in different orders by two calls"


def draw_keys(rng, L, n, bits, pool_frac=0.25):
    """L tables of n keys below 2^bits drawn from a pool (so keys repeat)."""
    if bits == 0:
        return np.zeros((L, n), np.uint64)
    pool = max(1, int(n * pool_frac))
    out = np.empty((L, n), np.uint64)
    for t in range(L):
        vals = rng.integers(0, 1 << min(bits, 63), size=pool, dtype=np.uint64)
        if bits == 64:
            vals |= rng.integers(0, 2, size=pool, dtype=np.uint64) << np.uint64(63)
        out[t] = vals[rng.integers(0, pool, size=n)]
    return out


@pytest.mark.parametrize("n,L,bits", [
    (1, 1, 8), (2047, 1, 20), (2048, 2, 32), (2049, 3, 33), (5000, 2, 60),
    (70001, 2, 64), (10000, 1, 0), (4097, 4, 12), (3000, 2, 1),
])
def test_sort_groups_rows(n, L, bits):
    say("lsh_sort", n, L, bits)
    rng = np.random.default_rng(1000 + n + 7 * L + bits)
    keys = draw_keys(rng, L, n, bits)
    perm = gpu_sort(keys, bits)
    for t in range(L):
        order = group_order(keys[t], perm[t])
        if bits <= 32:
            assert order == sorted(order), "groups not in ascending key order"
    if bits > 32:
        # a second key set: part of the first table's keys plus new ones,
        # shuffled, sorted by a separate call
        m = max(1, n // 2)
        sub = keys[0][rng.integers(0, n, size=m)]
        new = draw_keys(rng, 1, m, bits)[0]
        k2 = np.concatenate([sub, new])
        rng.shuffle(k2)
        perm2 = gpu_sort(k2[None, :], bits)
        same_relative_order(group_order(keys[0], perm[0]), group_order(k2, perm2[0]))


@pytest.mark.parametrize("n,L,bits", [
    (128 * 2048, 2, 20), (128 * 2048 + 1, 1, 32), (300 * 2048 - 5, 3, 9), (3, (1 << 20) + 3, 12),
])
def test_sort_block_counts(n, L, bits):
    """Tables of about 128 and 300 blocks of 2048 (128 threads share a digit's
    blocks), and more tables than one launch of the counts' sums takes: the
    stable sort's rows."""
    say("lsh_sort blocks", n, L, bits)
    rng = np.random.default_rng(n + bits)
    keys = rng.integers(0, 1 << bits, size=(L, n), dtype=np.uint64)
    assert np.array_equal(gpu_sort(keys, bits), np.argsort(keys, axis=1, kind="stable"))


def colliding_keys(rng, count: int) -> np.ndarray:
    """`count` distinct 64-bit keys whose mixes share their top 32 bits."""
    inv = pow(MIX_C, -1, 1 << 64)
    top = int(rng.integers(0, 1 << 32))
    lows = rng.choice(1 << 32, size=count, replace=False)
    out = []
    for lo in lows.tolist():
        m = (top << 32) | lo
        k1 = m ^ (m >> 32)          # undoes the xor of the high half into the low
        out.append((k1 * inv) & MASK64)
    return np.array(out, dtype=np.uint64)


def mix(k: int) -> int:
    k = (k * MIX_C) & MASK64
    return k ^ (k >> 32)


def test_colliding_top_halves_are_ordered():
    say("lsh_sort colliding top halves")
    rng = np.random.default_rng(77)
    coll = colliding_keys(rng, 40)
    assert len({mix(int(k)) >> 32 for k in coll}) == 1
    L, n = 2, 9000
    keys = draw_keys(rng, L, n, 64)
    for t in range(L):
        # 4000 rows of the table take one of the colliding keys, spread over
        # the whole table (so the colliding run spans several blocks)
        at = rng.choice(n, size=4000, replace=False)
        keys[t, at] = coll[rng.integers(0, coll.size, size=at.size)]
    perm = gpu_sort(keys, 64)
    orders = [group_order(keys[t], perm[t]) for t in range(L)]
    same_relative_order(orders[0], orders[1])
    # a separate call on a shuffled subset lists the colliding keys alike
    k2 = keys[1][rng.permutation(n)[: n // 3]]
    same_relative_order(orders[1], group_order(k2, gpu_sort(k2[None, :], 64)[0]))
    # groups follow the mixed key's order, colliding ones included
    for o in orders:
        mixed = [mix(int(k)) for k in o]
        assert mixed == sorted(mixed)


def test_sort_empty_and_errors():
    import torch
    import paper_2006_12608_amd as sj
    say("lsh_sort empty and errors")
    for shape in [(3, 0), (0, 5)]:
        perm = sj.lsh_sort(torch.zeros(shape, dtype=torch.int64, device="cuda"), 64)
        assert tuple(perm.shape) == shape
    kd = torch.zeros((1, 16), dtype=torch.int64, device="cuda")
    with pytest.raises(sj.SjError) as e:
        sj.lsh_sort(kd, 65)
    assert e.value.status == sj.SJ_E_INVAL
    with pytest.raises(ValueError):
        sj.lsh_sort(torch.zeros((1, 16), dtype=torch.int32, device="cuda"), 8)


@pytest.mark.parametrize("L,n", [
    (5, 2048), (5, 2049),                        # one block per table, two
    (1, 17 * 2048), (1, 17 * 2048 + 1),          # 17 and 18 blocks: one run, columns
    (60, 64 * 2048), (60, 64 * 2048 + 1),        # 64 and 65 blocks
    (1, 4095 * 2048), (2, 4095 * 2048 + 1),      # 4095 and 4096 blocks: columns, runs
    (70000, 33), (3000, 2100)])
def test_sort_tables_of_any_number_of_blocks(L, n):
    """The sums over a table's blocks take another kernel for one block, a run of
    at most 64, many blocks and very many; each must give the stable order."""
    import torch
    import paper_2006_12608_amd as sj
    say("sort", L, n)
    g = torch.Generator(device="cuda")
    g.manual_seed(7000 + n)
    for bits in (9, 20):
        k = torch.randint(0, 1 << bits, (L, n), generator=g, device="cuda", dtype=torch.int64)
        perm = sj.lsh_sort(k, bits).long()
        s = k.gather(1, perm)
        up = s[:, 1:] > s[:, :-1]
        assert bool((up | ((s[:, 1:] == s[:, :-1]) & (perm[:, 1:] > perm[:, :-1]))).all())
        assert bool((torch.zeros_like(k).scatter_(1, perm, 1) == 1).all())
        del k, perm, s, up


def test_many_colliding_runs():
    """Hundreds of runs of colliding top halves, of two to five keys each, several
    in one 256-position block and across blocks and tables."""
    say("lsh_sort many colliding runs")
    rng = np.random.default_rng(78)
    coll = np.concatenate([colliding_keys(rng, int(rng.integers(2, 6))) for _ in range(400)])
    L, n = 3, 7001
    keys = coll[rng.integers(0, coll.size, size=(L, n))]
    keys[:, ::7] = rng.integers(0, 1 << 62, size=keys[:, ::7].shape).astype(np.uint64)
    perm = gpu_sort(keys, 64)
    orders = [group_order(keys[t], perm[t]) for t in range(L)]
    for o in orders:
        mixed = [mix(int(k)) for k in o]
        assert mixed == sorted(mixed)
    same_relative_order(orders[0], orders[1])
    same_relative_order(orders[1], orders[2])
