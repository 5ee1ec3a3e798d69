"""HIP path vs CPU oracle, element by element (run with -m gpu on an MI355X)."""
import ctypes
import time

import numpy as np
import pytest
import torch

import sfc_inputs as si
from oracle import Oracle
from gpu_common import Pair, assert_close, same_stats

pytestmark = pytest.mark.gpu

HASHED, DENSE = 1, 2        # sfc_config.index_kind (0 = automatic: dense for every table of these tests)


def _zipf_steps(p, V, n, s, seed, steps, **kw):
    for t in range(steps):
        ids = si.zipf_ids(n, s, V, seed, t).numpy()
        p.step(ids, si.grads(n, p.D, seed, t).numpy(), **kw)


def test_paper_examples_on_gpu():
    # VSI example + MixCache example (12 slots; 7 replaces 1, 8 takes the free slot)
    p = Pair(V=32, D=4, C=12, max_ids=64)
    z = lambda n: np.zeros((n, 4), np.float32)
    pr = p.step([1, 3, 2, 5, 4, 6, 12, 13, 14, 15, 9], z(11))
    pr = p.step([3, 2, 5, 4], z(4))
    pr = p.step([6, 7, 8], z(3))
    assert p.cache.state()[0].tolist() == [7, 3, 2, 5, 4, 6, 12, 13, 14, 15, 9, 8]
    p.finish(); p.close()
    p = Pair(V=8, D=4, C=8, max_ids=16)
    pr = p.step([1, 3, 2, 2, 3, 1], np.ones((6, 4), np.float32))
    assert p.cache.unique_ids[:3].tolist() == [1, 3, 2]
    assert p.cache.inverse[:6].tolist() == [0, 1, 2, 2, 1, 0]
    p.finish(); p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
def test_tiny_config_bypass_every_step(index_kind):
    w = si.WORKLOADS["tiny"]                  # U ~ 10.7k > C = 10k: bypass rows on every step
    p = Pair(w.vocab, w.dim, w.cache_rows, w.max_ids, seed=w.seed, index_kind=index_kind)
    saw_bypass = saw_evict = False
    for t in range(6):
        ids, _ = w.batch_ids(t)
        pr = p.step(ids.numpy(), w.batch_grads(t).numpy())
        saw_bypass |= pr.stats["n_bypass"] > 0
        saw_evict |= pr.stats["n_evict"] > 0
    assert saw_bypass and saw_evict
    p.finish(); p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
@pytest.mark.parametrize("lookahead", [0, 1])
def test_eviction_heavy_small_cache(lookahead, index_kind):
    V, D, n = 5000, 8, 3000                    # several scan tiles, ragged tails (3000 % 256, % 2048)
    p = Pair(V, D, C=1500, max_ids=4096, lookahead=lookahead, index_kind=index_kind)
    _zipf_steps(p, V, n, 1.05, 21, 10)
    p.finish(); p.close()


def test_ties_in_stamp_break_by_slot():
    # fill 100 slots in one step (all stamp 1), then need 7 victims among equal stamps
    p = Pair(V=1000, D=4, C=100, max_ids=256)
    p.step(np.arange(100), np.zeros((100, 4), np.float32))
    pr = p.step(np.arange(500, 507), np.ones((7, 4), np.float32))
    assert pr.evict_slots.tolist() == list(range(7))
    pr = p.step(np.array([99, 98, 600, 601, 602]), np.ones((5, 4), np.float32))
    assert pr.evict_slots.tolist() == [7, 8, 9]
    p.finish(); p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
def test_multihot_bags(index_kind):
    V, D, nb = 20000, 16, 1500
    p = Pair(V, D, C=4000, max_ids=nb * 20, max_bags=nb, index_kind=index_kind)
    for t in range(6):
        off = si.bag_offsets(nb, 1, 20, 31, t).numpy()
        ids = si.zipf_ids(int(off[-1]), 1.1, V, 31, t).numpy()
        p.step(ids, si.grads(nb, D, 31, t).numpy(), offsets=off)
    p.finish(); p.close()


def test_multihot_with_empty_bags_and_repeats_inside_a_bag():
    p = Pair(V=50, D=4, C=8, max_ids=64, max_bags=8)
    off = np.array([0, 0, 3, 3, 7, 8])
    ids = np.array([4, 4, 9, 1, 4, 30, 30, 2])
    p.step(ids, si.grads(5, 4, 1, 0).numpy(), offsets=off)
    p.finish(); p.close()


def test_capacity_zero_is_the_host_strategy():
    V, D, n = 3000, 8, 1000
    p = Pair(V, D, C=0, max_ids=1024)
    _zipf_steps(p, V, n, 1.1, 41, 4)
    p.finish(); p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
def test_degenerate_batches(index_kind):
    p = Pair(V=100, D=4, C=16, max_ids=512, index_kind=index_kind)
    g = lambda n, t: si.grads(n, 4, 77, t).numpy()
    p.step(np.zeros(0, np.int64), np.zeros((0, 4), np.float32))     # empty batch
    p.step(np.full(300, 42), g(300, 1))                              # one id, many times
    p.step(np.array([-5, 100, 10 ** 12, -1]), g(4, 2))               # only out-of-range ids
    p.step(np.array([3, -1, 3, 200, 7]), g(5, 3))                    # mixed
    p.step(np.arange(100)[::-1].copy(), g(100, 4))                   # all distinct, > C
    p.step(np.arange(512) % 100, g(512, 5))                          # n_ids == max_ids
    p.finish(); p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
def test_medium_zipf_many_tiles(index_kind):
    # 16384 x 39 positions like the second configuration, vocabulary shrunk so that the oracle
    # and its table stay small; cache small enough to evict from the third step on
    V, D, n = 10 ** 6, 16, 16384 * 39
    p = Pair(V, D, C=200_000, max_ids=n, index_kind=index_kind)
    for t in range(5):
        ids = si.zipf_ids(n, 1.1, V, 1001, t).numpy()
        p.step(ids, si.grads(n, D, 1001, t).numpy(), check_state=(t in (0, 4)))
    p.finish(); p.close()


@pytest.mark.parametrize("D,n,optimizer", [(4, 16384, "adagrad"), (4, 16385, "adam"), (16, 10240, "adam"),
                                           (16, 10241, "adagrad"), (32, 5120, "adagrad"), (80, 2048, "adam"),
                                           (128, 1280, "adagrad"), (256, 640, "adam"), (256, 641, "adagrad")])
def test_updates_of_small_batches_up_to_their_limits(D, n, optimizer):
    # the update of a small batch in one kernel and, one position more, in two: groups of 16 and 17 positions
    # (one lane group, the whole block), one id alone, ids that are as frequent as each other, bags, bypass rows
    V = 30_000
    p = Pair(V, D, C=n // 2, max_ids=n, max_bags=n, optimizer=optimizer)
    g = lambda m, t: si.grads(m, D, 83, t).numpy()
    rng = np.random.default_rng(D)
    p.step(np.resize(np.repeat(np.arange(n // 16), rng.integers(16, 18, n // 16)), n), g(n, 0))
    p.step(np.full(n, 11), g(n, 1))
    p.step(rng.integers(0, 100, n) * 7, g(n, 2))
    p.step(rng.permutation(V)[:n], g(n, 3))                      # more distinct ids than slots
    off = np.concatenate([[0], np.sort(rng.integers(0, n + 1, n // 5)), [n]])
    p.step(si.zipf_ids(n, 1.1, V, 83, 4).numpy(), g(off.size - 1, 4), off)
    p.step(np.where(rng.random(n) < 0.3, -1, rng.integers(0, V, n)), g(n, 5))
    p.finish(); p.close()


@pytest.mark.parametrize("C", [0, 400])
@pytest.mark.parametrize("D,n,optimizer", [(8, 16384, "adam"), (20, 8192, "adagrad"), (32, 5000, "adagrad"),
                                           (128, 1280, "adam"), (256, 640, "adagrad")])
def test_frequent_ids_of_small_batches_are_summed_in_shares(D, n, optimizer, C):
    # an id with more positions than two shares of the grouping (16384 / D positions each) is summed by several blocks:
    # groups of two shares and one position more or less, that begin at, before and behind a share's edge, two of
    # them that meet inside a share, the null entry, several batches one after the other, rows that bypass the cache
    V, share = 3000, 4096 // (D // 4)
    p = Pair(V, D, C=C, max_ids=n, optimizer=optimizer)
    rng = np.random.default_rng(D)
    for t, runs in enumerate([[2 * share], [2 * share + 1], [1, 2 * share + 1, 2 * share + 2], [share, 3 * share, 2 * share],
                              [share - 1, 2 * share + 1, 3 * share], [n], [1, n - 1], [2 * share + 1, -3 * share, 2 * share + 1]]):
        ids = np.concatenate([np.full(abs(r), -1 if r < 0 else 100 * t + k) for k, r in enumerate(runs)])[:n]
        ids = np.concatenate([ids, rng.integers(2000, V, n - ids.size)])
        ids[100:] = rng.permutation(ids[100:])           # groups lie in order of first appearance
        p.step(ids, si.grads(n, D, 85, t).numpy())
    p.finish(); p.close()


@pytest.mark.parametrize("D", [4, 8, 16, 64, 80, 128, 256])
def test_row_widths(D):
    # every lane-group geometry of the row kernels (D/4 lanes per row, also a D that does not
    # divide the wavefront), with a hot id, mid-frequency ids and singletons in one batch
    V, n = 6000, 5000
    p = Pair(V, D, C=1200, max_ids=n + 37)
    for t in range(3):
        ids = si.zipf_ids(n + 37 * (t % 2), 1.3, V, 60 + D, t).numpy()
        p.step(ids, si.grads(ids.size, D, 60 + D, t).numpy())
    p.finish(); p.close()


def test_long_groups_cross_many_spans():
    # three ids own almost all of 300k positions: their groups span hundreds of wavefronts
    V, D, n = 500, 32, 300_000
    p = Pair(V, D, C=500, max_ids=n)
    rng = np.random.default_rng(11)
    r = rng.random(n)
    ids = np.where(r < 0.5, 3, np.where(r < 0.8, 5, np.where(r < 0.97, 8, rng.integers(0, V, n))))
    p.step(ids, si.grads(n, D, 12, 0).numpy())
    p.step(ids[::-1].copy(), si.grads(n, D, 12, 1).numpy())
    p.finish(); p.close()


@pytest.mark.parametrize("D,C,optimizer", [(4, 400, "adagrad"), (16, 0, "adagrad"), (80, 400, "adagrad"),
                                           (256, 7, "adagrad"), (16, 400, "adam"), (32, 0, "adam")])
def test_groups_cut_by_block_edges_are_updated_once(D, C, optimizer):
    # Adagrad and Adam path: the optimizer kernel itself adds up the partial sums of groups that the gradient
    # stream's blocks cut (a lane group per short run, the whole block for a run of many slots) and
    # updates those rows; here one id has a run of hundreds of slots, a dozen ids have runs of a few
    # slots, the rest close inside a block.  Row widths of one lane and of a whole wavefront, a width
    # that does not divide the wavefront, rows that bypass the cache (C = 0: every one; C = 7: most).
    V, n = 400, 150_000
    rng = np.random.default_rng(100 + D)
    r = rng.random(n)
    mid = 20 + (rng.integers(0, 12, n))
    ids = np.where(r < 0.45, 3, np.where(r < 0.85, mid, rng.integers(0, V, n)))
    p = Pair(V, D, C=C, max_ids=n, optimizer=optimizer, init_acc=0.0 if optimizer == "adam" else 0.1)
    p.step(ids, si.grads(n, D, 70 + D, 0).numpy())
    p.step(ids[::-1].copy(), si.grads(n, D, 70 + D, 1).numpy())
    p.finish(); p.close()


@pytest.mark.parametrize("D,C", [(4, 400), (64, 0), (128, 400), (256, 7), (20, 400)])
def test_rowwise_rows_with_cold_groups_and_cut_groups(D, C):
    # row-wise Adagrad: groups of one and two positions, groups cut by the stream's block edges and the
    # common matrix side by side, rows of one lane to a whole wavefront (20: the path for other widths), one-hot and
    # in bags, rows that bypass the cache
    V, n = 9000, 60_000
    rng = np.random.default_rng(300 + D)
    p = Pair(V, D, C=C, max_ids=n, optimizer="rowwise_adagrad")
    for t in range(2):
        r = rng.random(n)
        ids = np.where(r < 0.4, 3, np.where(r < 0.8, 20 + rng.integers(0, 12, n), -1))
        cold = rng.permutation(V)[:6000]
        ids[-8000:] = np.concatenate([cold, cold[:2000]])         # behind 8192 positions: virtual ids beyond the LDS bins too
        ids[:9000] = rng.permutation(V)
        off = None if t == 0 else np.concatenate([[0], np.sort(rng.integers(0, n + 1, n // 4)), [n]])
        p.step(ids, si.grads(n if off is None else off.size - 1, D, 84, t).numpy(), off)
    p.finish(); p.close()


@pytest.mark.parametrize("D,n,optimizer", [(4, 200_000, "adagrad"), (4, 9000, "rowwise_adagrad"), (16, 40_000, "adam"),
                                           (32, 7000, "adagrad"), (128, 9000, "rowwise_adagrad"), (252, 12_000, "adagrad")])
def test_several_long_runs_of_partial_sums_side_by_side(D, n, optimizer):
    # ten, then forty ids own the batch: each leaves a run of a few to some dozens of block-edge partials,
    # around the length from which a whole block sums them, and the runs begin close together
    p = Pair(V=100, D=D, C=100, max_ids=n, optimizer=optimizer)
    for t, k in enumerate((10, 40, 11)):
        ids = np.random.default_rng(t).integers(0, k, n - 13 * t)
        p.step(ids, si.grads(n - 13 * t, D, 25, t).numpy())
    p.finish(); p.close()


def test_frequent_ids_that_first_appear_late():
    # the grouping passes treat the lowest virtual ids (the early, usually frequent ones) in LDS and
    # rank the others with atomics: here the batch opens with 9000 distinct ids, so the frequent ids
    # that follow get virtual ids beyond that range and their long groups take the other path;
    # multi-hot as well, where the payload of a grouped entry is the bag, not the position
    V, D, n = 40_000, 16, 120_000
    rng = np.random.default_rng(21)
    head = rng.permutation(V)[:9000]
    r = rng.random(n - 9000)
    tail = np.where(r < 0.4, 39_000, np.where(r < 0.7, 39_001, np.where(r < 0.8, head[17],
                                                                        rng.integers(0, V, n - 9000))))
    ids = np.concatenate([head, tail])
    p = Pair(V, D, C=30_000, max_ids=n)
    p.step(ids, si.grads(n, D, 22, 0).numpy())
    p.step(np.concatenate([head[::-1], tail[::-1]]), si.grads(n, D, 22, 1).numpy())
    p.finish(); p.close()
    lens = rng.integers(0, 7, 30_000)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    m = int(offsets[-1])
    ids = np.concatenate([head, tail])[:m] if m <= n else None
    assert ids is not None
    p = Pair(V, D, C=30_000, max_ids=n, max_bags=lens.size)
    p.step(ids, si.grads(lens.size, D, 23, 0).numpy(), offsets)
    p.finish(); p.close()


@pytest.mark.parametrize("n,head", [(6200, 2100), (40_000, 3000), (200_000, 8191), (200_000, 8200)])
def test_frequent_ids_behind_a_head_of_distinct_ones(n, head):
    # batches of every shape of the counting pass below 2^18 that open with distinct ids: the frequent ids
    # get virtual ids in the middle, at the end and just outside the range that is counted in LDS
    V, D = 30_000, 4
    rng = np.random.default_rng(n + head)
    p = Pair(V, D, C=20_000, max_ids=n)
    for t in range(2):
        first = rng.permutation(V - 10)[:head]
        ids = np.concatenate([first, np.where(rng.random(n - head) < 0.9, V - 1 - rng.integers(0, 3, n - head),
                                              rng.integers(0, V, n - head))])
        p.step(ids, si.grads(n, D, 24, t).numpy())
    p.finish(); p.close()


@pytest.mark.parametrize("n", [1, 255, 257, 1023, 1025, 5121, (1 << 18) - 1, 1 << 18, (1 << 18) + 1,
                               (1 << 22) - 1, (1 << 22) + 1])
def test_batch_sizes_where_the_counting_passes_change_shape(n):
    # the passes that count, rank and group the positions take other block sizes and another number of
    # LDS bins by batch size, and a ragged last block; ids beyond the bins, ids outside the table
    V, D = max(8, n // 2), 4
    p = Pair(V, D, C=max(4, V // 3), max_ids=n)
    for t in range(2 if n > 1 << 20 else 3):
        ids = si.zipf_ids(n, 1.1, max(2, V - V % 10), 300 + n % 97, t).numpy()
        ids[::1001] = V + 5
        p.step(ids, si.grads(n, D, 300 + n % 97, t).numpy(), check_state=n < 1 << 20)
    p.finish(); p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
@pytest.mark.parametrize("C", [40_000, 70_000, 150_000])
@pytest.mark.parametrize("lookahead", [0, 2])
def test_one_block_batches_beside_large_ones(lookahead, C, index_kind):
    # up to 6144 ids a batch is prepared by one block, which also chooses the victims when the index is
    # dense and the cache small (40 000 slots) or as large as the table; with 70 000 slots or a hashed
    # index the general passes take over behind its resolve.  Steps of both kinds follow each other
    # through the same counters, histogram, index and step contexts; victims in most of them
    V, D = 150_000, 4
    sizes = [80_000, 6144, 500, 1, 6145, 3000, 80_000, 6000, 6144, 200, 80_000, 5000]
    p = Pair(V, D, C=C, max_ids=80_000, lookahead=lookahead, index_kind=index_kind)
    bs = []
    for t, n in enumerate(sizes):
        # (uniform ids where the batch is large, so that 70 000 slots fill)
        ids = (si.uniform_ids(n, V, 410, t) if n == 80_000 else si.zipf_ids(n, 1.02, V, 410, t)).numpy()
        ids[::611] = -3                     # some outside the table
        bs.append((ids, si.grads(n, D, 410, t).numpy(), None))
    if lookahead:
        expect = [pr for pr, _ in p.run_pipelined(bs, False)]
    else:
        expect = [p.step(ids, g) for ids, g, _ in bs]
        p.finish()
    small_victims = [pr.stats["n_evict"] for pr, n in zip(expect, sizes) if n <= 6144]
    assert (max(small_victims) > 0) == (C < V)
    p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
@pytest.mark.parametrize("n", [1, 63, 1023, 1025, 2048, 2049, 4096, 4097, 6143, 6144])
def test_one_block_batches_at_the_edges_of_their_forms(n, index_kind):
    # sizes where the positions per thread change; ids that meet in the block's table of distinct ids, whose
    # place there is the top bits of a multiplicative hash: all from a few of its 8192 or 16384 places, so that most
    # walk on, and the same batch in bags
    V, D = 200_000, 4
    h = (np.arange(V, dtype=np.uint64) * 0x9e3779b1) & 0xffffffff
    h ^= h >> 15
    near = np.nonzero((h >> (19 if n <= 2048 else 18)) % 97 < 3)[0]
    rng = np.random.default_rng(n)
    p = Pair(V, D, C=9000, max_ids=6144, max_bags=6144, index_kind=index_kind)
    for t in range(4):
        ids = rng.choice(near[t * 500:t * 500 + 5000], n)
        ids[rng.random(n) < 0.2] = near[7]
        ids[rng.random(n) < 0.01] = -1
        if t % 2:
            off = np.concatenate([[0], np.sort(rng.integers(0, n + 1, max(n // 3, 1) - 1)), [n]])
            p.step(ids, si.grads(off.size - 1, D, 93, t).numpy(), off)
        else:
            p.step(ids, si.grads(n, D, 93, t).numpy())
    p.finish(); p.close()


@pytest.mark.parametrize("n_bags", [20_000, 30_000])
def test_few_ids_in_many_mostly_empty_bags(n_bags):
    V, D = 500, 8
    rng = np.random.default_rng(n_bags)
    p = Pair(V, D, C=60, max_ids=400, max_bags=n_bags)
    for t in range(4):
        lens = np.bincount(rng.integers(0, n_bags, 300 + t), minlength=n_bags)
        off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        p.step(rng.integers(0, V, int(off[-1])), si.grads(n_bags, D, 5, t).numpy(), offsets=off)
    p.finish(); p.close()


def test_ages_beyond_the_tallied_range_in_a_one_block_batch():
    # a slot last used more than 1024 steps ago leaves the recency histogram one by one
    V, D = 60, 4
    p = Pair(V, D, C=20, max_ids=32)
    p.step(np.arange(10), si.grads(10, D, 6, 0).numpy())
    for t in range(1030):
        ids = torch.tensor([20 + t % 3], dtype=torch.int64, device=p.dev)
        p.cache.prepare(ids); p.cache.fetch_misses(); p.cache.lookup(); p.cache.discard()
        p.orc.prepare(np.array([20 + t % 3]), None); p.orc.fetch_misses(); p.orc.lookup()
        p.orc.backward_update(np.zeros((1, D), np.float32))
    p.step(np.arange(5), si.grads(5, D, 6, 1).numpy())
    p.step(np.arange(30, 50), si.grads(20, D, 6, 2).numpy())
    p.finish(); p.close()


def test_batch_table_whose_entries_take_two_words():
    # an id and a position share one 64-bit word of the batch table unless the id range is too large for
    # that: a cache told of 2^61 Host rows (all ids used lie in the rows that exist) gives what one
    # with the true row count gives
    import paper_2104_08542_amd as sfc
    V, D, n = 30_000, 8, 20_011
    caches = []
    for rows in (V, 1 << 61):
        tab = sfc.HostTable(V, D)
        tab.w_t[:] = si.table_rows(5, 0, V, D)
        tab.acc[:] = 0.1
        tab.rows = rows
        caches.append(sfc.Cache(tab, 9000, n, index_kind=HASHED))
    for t in range(4):
        ids = si.zipf_ids(n, 1.1, V, 53, t)
        ids[::97] = -1
        d_ids, g = ids.to("cuda:0"), si.grads(n, D, 53, t).to("cuda:0")
        got = []
        for c in caches:
            c.prepare(d_ids); c.fetch_misses()
            st = c.stats()
            U = st["n_unique"]
            got.append((st, c.unique_ids[:U].cpu(), c.inverse[:n].cpu(), c.slot[:U].cpu(), c.lookup().cpu()))
            c.backward_update(g)
        assert got[0][0] == got[1][0]
        for a, b in zip(got[0][1:4], got[1][1:4]):
            assert torch.equal(a, b)
        # rows a step later may differ in the last place: the order of a frequent id's fp64 sum is free
        assert torch.allclose(got[0][4], got[1][4], rtol=1e-6, atol=1e-7)
    for c in caches:
        assert c.verify() == [0, 0, 0, 0]
        c.close(); c.table.free()


@pytest.mark.parametrize("C,n,optimizer", [(60_000, 50_000, "adagrad"), (20_000, 50_000, "adagrad"),
                                           (30_000, 50_000, "adam"),
                                           (60_000, 50_000, "rowwise_adagrad"), (90_000, 300_000, "adagrad")])
def test_host_copies_in_separate_blocks(C, n, optimizer):
    # lookahead 0 and 2^14 to 2^18 misses: the victims' rows are staged beside the step's bypass rows and
    # one part of the blocks writes them to the Host while the other reads the missed rows; with bypass
    # rows in front of the staged ones
    V, D = 200_000, 12
    p = Pair(V, D, C=C, max_ids=n, optimizer=optimizer, init_acc=0.0 if optimizer == "adam" else 0.1)
    seen = []
    for t in range(5):
        m = n if t % 2 == 0 else n - n // 7
        pr = p.step(si.uniform_ids(m, V, 71, t).numpy(), si.grads(m, D, 71, t).numpy(), check_common=False)
        seen.append(pr.stats)
    assert any(st["n_miss"] >= 1 << 14 and st["n_evict"] > 0 for st in seen)
    p.finish(); p.close()


@pytest.mark.parametrize("D,optimizer,C,sizes", [
    (12, "rowwise_adagrad", 40_000, [(1 << 14) - 1, 1 << 14, (1 << 14) + 1]),     # fewest rows
    (4, "adagrad", 300_000, [1 << 18, (1 << 18) + 1]),                             # most rows
    (128, "adam", 50_000, [43_690, 43_691])])                                      # most bytes: 64 MiB of 1536-byte rows
def test_host_copies_at_the_limits_of_the_separate_blocks(D, optimizer, C, sizes):
    # batches of ids that were never seen, all distinct, behind a full cache: as many misses and victims as
    # ids, on both sides of each limit, and the victims' rows have been updated
    V = 2 * C + sum(sizes)
    p = Pair(V, D, C=C, max_ids=max([C] + sizes), optimizer=optimizer, init_acc=0.0 if optimizer == "adam" else 0.1)
    order = np.random.default_rng(D).permutation(V)
    at = 0
    for t, n in enumerate([C] + sizes):
        pr = p.step(order[at:at + n], si.grads(n, D, 73, t).numpy(), check_common=False, check_state=t == len(sizes))
        at += n
        assert pr.stats["n_miss"] == n and pr.stats["n_evict"] == (n if t else 0)
    p.finish(); p.close()


@pytest.mark.parametrize("lookahead", [1, 3])
def test_pipelined_batches_either_side_of_where_the_passes_change(lookahead):
    # at 2^18 ids the counting and grouping passes change shape, at 2^20 the sums of the positions go to another launch:
    # batches on either side follow each other on the one prepare stream, a one-block batch among them
    V, D = 300_000, 4
    sizes = [270_000, 250_000, 300_000, 1_100_000, 280_000, 4000, 265_000, 1_100_000, 262_144, 262_143]
    p = Pair(V, D, C=250_000, max_ids=1_100_000, lookahead=lookahead)
    p.run_pipelined([(si.zipf_ids(n, 1.05, V, 510, t).numpy(), si.grads(n, D, 510, t).numpy(), None)
                     for t, n in enumerate(sizes)], False)
    p.close()


def test_large_pipelined_batches_with_bags_and_without():
    # from 2^20 ids on a pipelined prepare counts positions and finds bags beside the victims' count: one-hot and in
    # bags, hits, misses and victims in every step, an index of either kind
    V, D, C = 1_300_000, 4, 800_000
    for index_kind in (DENSE, HASHED):
        p = Pair(V, D, C=C, max_ids=(1 << 20) + 77, lookahead=1, index_kind=index_kind)
        bs = []
        for t, n in enumerate([(1 << 20) + 77, 1 << 20, (1 << 20) + 5, (1 << 20) - 1, (1 << 20) + 77]):
            ids, rng = si.zipf_ids(n, 1.02, V, 512, t).numpy(), np.random.default_rng(t)
            ids[:200_000] = rng.permutation(V)[:200_000]
            off = None if t % 2 else np.concatenate([[0], np.sort(rng.integers(0, n + 1, n // 7)), [n]])
            bs.append((ids, si.grads(n if off is None else off.size - 1, D, 512, t).numpy(), off))
        expect = p.run_pipelined(bs, index_kind == DENSE)
        assert min(pr.stats["n_evict"] for pr, _ in expect[-2:]) > 0
        p.close()


class _DeletedEntries:
    """The manager's rule for rebuilding a hashed index, replayed: the deleted entries of a table of `size` entries with
    linear probing, an insert taking the first free or deleted entry on its way."""

    def __init__(self, size):
        self.size, self.live, self.deleted, self.reused, self.due = size, {}, 0, 0, False
        self.entry = bytearray(size)                  # 0 free, 1 live, 2 deleted

    def _put(self, ids):
        h = ids.astype(np.uint64)
        for mul in (0xff51afd7ed558ccd, 0xc4ceb9fe1a85ec53, 1):
            h ^= h >> np.uint64(33)
            h *= np.uint64(mul)
        reused = 0
        for i, e in zip(ids.tolist(), (((h >> np.uint64(32)) * np.uint64(self.size)) >> np.uint64(32)).tolist()):
            while self.entry[e] == 1:
                e = e + 1 if e + 1 < self.size else 0
            reused += self.entry[e] == 2
            self.entry[e] = 1
            self.live[i] = e
        return reused

    def step(self, victims, inserted):
        """Returns what the plan compares with an eighth of the table; afterwards `due` says whether the next prepare
        starts with a rebuild."""
        self.deleted -= self.reused
        if self.due:
            self.entry, ids = bytearray(self.size), np.array(list(self.live), np.int64)
            self._put(ids)
            self.deleted = 0
        level = self.deleted + len(victims)
        self.due = level > self.size // 8
        for i in victims.tolist():
            self.entry[self.live.pop(i)] = 2
        self.deleted = level
        self.reused = self._put(inserted)
        return level


def test_hashed_index_rebuilt_between_prepares_of_every_form():
    # the rebuild of a hashed index runs inside the unique passes (below and from 2^18 ids on) and as kernels of its own
    # where the batch is prepared by one block (or empty): whenever one is due, by the rule replayed here, the next batch
    # is of a form that has not had one yet
    V, D, C, max_ids, U = 1_000_000, 4, 150_000, 270_000, 45_000
    table = _DeletedEntries(4 * (C + max_ids))
    orc = Oracle(C, D, np.zeros((V, D), np.float32), np.ones((V, D), np.float32), lookahead=1)
    rng = np.random.default_rng(512)
    forms = {"below 2^18": 60_000, "from 2^18": 265_000, "one block": 5000, "empty": 0}
    to_do, had, bs = ["from 2^18", "below 2^18", "one block", "empty", "from 2^18"], [], []
    while to_do or table.due:
        form = to_do.pop(0) if table.due else ["below 2^18", "from 2^18"][len(bs) % 2]
        if table.due:
            had.append(form)
        n = forms[form]
        ids = rng.permutation(V)[:min(n, U)]
        ids = np.concatenate([ids, rng.choice(ids, n - ids.size)]) if n else np.zeros(0, np.int64)
        bs.append((ids, si.grads(n, D, 512, len(bs)).numpy(), None))
        pr, _ = orc.step(ids, bs[-1][1])
        level = table.step(pr.evict_ids, pr.unique_ids[pr.miss_vids[pr.slot[pr.miss_vids] < C]])
        # (inserts side by side may share out the deleted entries differently)
        assert abs(level - table.size // 8) > table.size // 8 // 50, (len(bs), level, table.size // 8)
    assert had == ["from 2^18", "below 2^18", "one block", "empty", "from 2^18"]
    p = Pair(V, D, C=C, max_ids=max_ids, lookahead=1, index_kind=HASHED)
    p.run_pipelined(bs, False)
    p.close()


def test_same_stream_and_separate_host_arrays():
    # copies on the main stream; Host weights and accumulators as two separate arrays
    V, D, n = 4000, 32, 2000
    p = Pair(V, D, C=1000, max_ids=2048, side_stream=False, interleaved=False)
    _zipf_steps(p, V, n, 1.2, 5, 4)
    p.finish(); p.close()


def test_hot_id_accumulation_stays_in_tolerance():
    # one id owns ~half of 400k positions: the segment sum has ~2e5 N(0,1) terms per element
    V, D, n = 1000, 32, 400_000
    p = Pair(V, D, C=1000, max_ids=n)
    rng = np.random.default_rng(3)
    ids = np.where(rng.random(n) < 0.5, 7, rng.integers(0, V, n))
    p.step(ids, si.grads(n, D, 9, 0).numpy())
    p.finish(); p.close()


def test_index_rebuild_after_many_evictions():
    # tiny cache, every step evicts almost everything: deleted index entries pile up and the
    # rebuild path runs many times; state must stay identical to the oracle throughout
    V, D = 100_000, 4
    p = Pair(V, D, C=64, max_ids=64, index_kind=HASHED)
    for t in range(60):
        ids = si.uniform_ids(64, V, 3, t).numpy()
        p.step(ids, si.grads(64, D, 3, t).numpy(), check_common=False)
    p.finish(); p.close()


def test_call_order_and_argument_errors():
    import paper_2104_08542_amd as sfc
    p = Pair(V=100, D=4, C=16, max_ids=32)
    c = p.cache
    ids = torch.arange(8, dtype=torch.int64, device="cuda:0")
    out = torch.empty(8, 4, device="cuda:0")
    for fn in (lambda: c.lookup(out), lambda: c.backward_update(out), c.fetch_misses):
        with pytest.raises(sfc.SfcError) as e:
            fn()
        assert e.value.code == sfc.SFC_ESTATE
    with pytest.raises(sfc.SfcError) as e:
        c.prepare(torch.zeros(33, dtype=torch.int64, device="cuda:0"))
    assert e.value.code == sfc.SFC_EINVAL
    c.prepare(ids)
    with pytest.raises(sfc.SfcError) as e:
        c.prepare(ids)
    assert e.value.code == sfc.SFC_ESTATE
    c.fetch_misses(); c.lookup(out); c.backward_update(out)
    p.close()


def test_step_limit():
    import paper_2104_08542_amd as sfc
    p = Pair(V=100, D=4, C=16, max_ids=32, max_steps=3)
    for t in range(3):
        p.step(np.arange(5) + t, np.zeros((5, 4), np.float32))
    with pytest.raises(sfc.SfcError) as e:
        p.cache.prepare(torch.arange(5, dtype=torch.int64, device="cuda:0"))
    assert e.value.code == sfc.SFC_ELIMIT
    p.close()


def _batches(V, D, n, s, seed, steps):
    return [(si.zipf_ids(n, s, V, seed, t).numpy(), si.grads(n, D, seed, t).numpy(), None)
            for t in range(steps)]


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
@pytest.mark.parametrize("lookahead", [1, 2, 3])
@pytest.mark.parametrize("sync_every_call", [True, False])
def test_pipelined_steps_match_sequential_oracle(sync_every_call, lookahead, index_kind):
    # prepare / fetch of later steps overlap lookup / update of the current one; the cache is
    # small enough to evict on every step and large enough never to bypass
    V, D, n = 20000, 32, 6000
    p = Pair(V, D, C=12000, max_ids=8192, lookahead=lookahead, index_kind=index_kind)
    p.run_pipelined(_batches(V, D, n, 1.05, 77, 12), sync_every_call)
    p.close()


@pytest.mark.parametrize("lookahead", [1, 2, 3])
@pytest.mark.parametrize("sync_every_call", [True, False])
def test_pipelined_steps_with_bypass_rows(sync_every_call, lookahead):
    # the working set of two consecutive batches exceeds the cache: rows bypass it, and a row that
    # bypassed in step t is missed again in step t+1 and must arrive with the update of step t
    V, D, n = 3000, 16, 2500
    p = Pair(V, D, C=500, max_ids=4096, lookahead=lookahead)
    expect = p.run_pipelined(_batches(V, D, n, 1.05, 78, 10), sync_every_call)
    assert min(pr.stats["n_bypass"] for pr, _ in expect[1:]) > 0
    p.close()


@pytest.mark.parametrize("lookahead", [2, 3])
def test_pipelined_mixed_bypass_and_none(lookahead):
    # steps with and without bypass rows alternate, so the Host copies switch between the two
    # streams from step to step
    V, D = 6000, 8
    p = Pair(V, D, C=1000, max_ids=4096, lookahead=lookahead)
    bs = []
    for t in range(16):
        n = 3500 if t % 5 == 0 else 300
        bs.append((si.zipf_ids(n, 1.02, V, 80, t).numpy(), si.grads(n, D, 80, t).numpy(), None))
    expect = p.run_pipelined(bs, False)
    nb = [pr.stats["n_bypass"] for pr, _ in expect]
    assert max(nb) > 0 and min(nb) == 0
    p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
@pytest.mark.parametrize("scale", [1, 24])
@pytest.mark.parametrize("lookahead", [1, 2, 3])
@pytest.mark.parametrize("sync_every_call", [True, False])
def test_pipelined_first_bypass_behind_steps_that_only_evict(sync_every_call, lookahead, scale, index_kind):
    # the Host copies of a step are launched twice and exactly one launch may do them, also where the older steps that
    # were in flight have been updated and their contexts prepared anew, now with bypass rows, before the second
    # launch runs: steps that write victims back and have no bypass rows, then bypass rows for the first time
    V, D, C = 20_000 * scale, 8, 1300 * scale
    p = Pair(V, D, C=C, max_ids=1250 * scale, lookahead=lookahead, index_kind=index_kind)
    bs = []
    for t in range(15):
        n = (1250 if t in (9, 10) else 300) * scale
        bs.append((np.random.default_rng(9000 + t).permutation(V)[:n], si.grads(n, D, 82, t).numpy(), None))
    st = [pr.stats for pr, _ in p.run_pipelined(bs, sync_every_call)]
    assert [s["n_bypass"] > 0 for s in st[:11]] == [False] * 9 + [True] * 2
    assert min(s["n_evict"] for s in st[5:]) > 0
    p.close()


@pytest.mark.parametrize("lookahead", [1, 2, 3])
def test_pipelined_degenerate_batches(lookahead):
    # empty batches, a single id, only out-of-range ids and full-size batches in flight together
    V, D = 300, 4
    p = Pair(V, D, C=64, max_ids=512, lookahead=lookahead)
    g = lambda n, t: si.grads(n, D, 81, t).numpy()
    ids = [np.zeros(0, np.int64), np.full(300, 42), np.zeros(0, np.int64), np.array([-5, V, 10 ** 12, -1]),
           np.arange(512) % V, np.array([3, -1, 3, 200, 7]), np.zeros(0, np.int64), np.zeros(0, np.int64),
           np.arange(200)[::-1].copy(), np.arange(512) % 100]
    p.run_pipelined([(a, g(a.size, t), None) for t, a in enumerate(ids)], False)
    p.close()
    p = Pair(V, D, C=64, max_ids=512, lookahead=lookahead)
    p.run_pipelined([(a, g(a.size, t), None) for t, a in enumerate(ids)], True)
    p.close()


@pytest.mark.parametrize("lookahead", [1, 2, 3])
def test_pipelined_multihot(lookahead):
    V, D, nb = 8000, 8, 700
    p = Pair(V, D, C=5000, max_ids=nb * 20, max_bags=nb, lookahead=lookahead)
    bs = []
    for t in range(6):
        off = si.bag_offsets(nb, 1, 20, 79, t).numpy()
        bs.append((si.zipf_ids(int(off[-1]), 1.1, V, 79, t).numpy(), si.grads(nb, D, 79, t).numpy(), off))
    p.run_pipelined(bs, False)
    p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
@pytest.mark.parametrize("lookahead", [0, 2, 3])
def test_many_rebuilds_with_many_victims(lookahead, index_kind):
    # a cache much smaller than the id range with thousands of victims per step: the hashed index
    # fills with deleted entries and is rebuilt every few steps, also while other steps are in
    # flight; the dense one just follows
    V, D, n, C = 400_000, 4, 30_000, 40_000
    p = Pair(V, D, C=C, max_ids=n, lookahead=lookahead, index_kind=index_kind)
    bs = [(si.zipf_ids(n, 1.05, V, 77, t).numpy(), si.grads(n, D, 77, t).numpy(), None) for t in range(60)]
    if lookahead:
        expect = p.run_pipelined(bs, False)
        assert sum(pr.stats["n_evict"] for pr, _ in expect) > 5 * C
    else:
        ev = 0
        for ids, g, _ in bs:
            ev += p.step(ids, g, check_common=False, check_rows=False).stats["n_evict"]
        assert ev > 5 * C
        p.finish()
    p.close()


@pytest.mark.parametrize("max_ids", [1, 5, 16, 31])
def test_tiny_max_ids_with_id_zero(max_ids):
    # batch tables smaller than the 64 entries the unique pass always probes; id 0 is the value
    # that zero-filled memory would pass for
    V, D = 50, 4
    p = Pair(V, D, C=8, max_ids=max_ids)
    rng = np.random.default_rng(max_ids)
    for t in range(6):
        n = max_ids if t % 2 == 0 else max(1, max_ids // 2)
        ids = rng.integers(0, V, n)
        ids[rng.integers(0, n)] = 0
        if n > 2:
            ids[-1] = 0                      # id 0 again, later: its first appearance must win
        p.step(ids, si.grads(n, D, 90 + max_ids, t).numpy())
    p.finish(); p.close()


def test_malformed_offsets_are_reported_not_followed():
    # the oracle refuses such a batch; the device cannot be refused on the host (the offsets live
    # in device memory), so the kernels count the violations, stay inside their buffers and the
    # step is reported by sfc_check and in the stats
    import paper_2104_08542_amd as sfc
    from oracle import Oracle
    V, D = 200, 8
    ids = np.arange(40) % 23
    good = np.array([0, 5, 5, 17, 30, 40])
    cases = [np.array([1, 5, 5, 17, 30, 40]),          # does not start at 0
             np.array([0, 5, 5, 17, 30, 39]),          # does not end at n_ids
             np.array([0, 5, 5, 17, 30, 4000]),        # ends far outside
             np.array([0, 17, 5, 30, 30, 40]),         # decreasing
             np.array([0, -7, 5, 30, 30, 40])]         # negative
    for k, off in enumerate(cases):
        p = Pair(V, D, C=64, max_ids=64, max_bags=8)
        p.step(ids, si.grads(5, D, 3, 0).numpy(), offsets=good)       # a good step first
        tab = np.zeros((V, D), np.float32)
        with pytest.raises(ValueError):                 # the oracle's -1
            Oracle(64, D, tab.copy(), tab.copy()).prepare(ids.astype(np.int64), off.astype(np.int64))
        c = p.cache
        c.prepare(torch.from_numpy(ids).to(p.dev), torch.from_numpy(off.astype(np.int64)).to(p.dev))
        st = c.stats()
        assert st["n_bad_offsets"] >= 1, (k, st)
        c.fetch_misses()
        out = c.lookup()
        c.backward_update(torch.zeros(5, D, device=p.dev))
        torch.cuda.synchronize()
        assert out.shape == (5, D)
        with pytest.raises(sfc.SfcError) as e:
            c.check()
        assert e.value.code == sfc.SFC_EINVAL and "step 2" in str(e.value)
        c.check()                                       # reported once
        assert c.verify() == [0, 0, 0, 0]               # the manager state depends on the ids alone
        pk, step = c.peek_stats()
        assert step == 2 and pk["n_bad_offsets"] == st["n_bad_offsets"]
        p.close()


@pytest.mark.parametrize("n_ids,n_bags,index_kind", [(9000, 700, DENSE), (9000, 700, HASHED), (900, 700, HASHED),
                                                     (900, 25_000, DENSE), (900, 700, DENSE)])
@pytest.mark.parametrize("where", ["first", "inner", "last"])
def test_malformed_offsets_at_every_size_and_place(where, n_ids, n_bags, index_kind):
    # the bags of a batch too large for the one-block prepare, of one that a hashed index or the number of
    # bags keeps from it, and of one that takes it; the offsets of a whole wavefront's bags and more hold
    # values far outside, so that some wavefronts see a violation and others, inside the run, none
    import paper_2104_08542_amd as sfc
    V, D = 5000, 8
    rng = np.random.default_rng(n_ids + n_bags)
    ids = rng.integers(0, V, n_ids)
    good = np.sort(np.concatenate([[0, n_ids], rng.integers(0, n_ids + 1, n_bags - 1)])).astype(np.int64)
    a = {"first": 0, "inner": n_bags // 2 - 100, "last": n_bags - 199}[where]
    for x in [-7, -2 ** 31 - 1, -2 ** 32 + 100, -0x180000001, -2 ** 63, n_ids + 1, 2 ** 32 + 5, 2 ** 63 - 4, 2 ** 63 - 1]:
        off = good.copy()
        off[a:a + 200] = x
        bad = int(np.sum(off[1:] < off[:-1])) + int(off[0] != 0 and off[1] >= off[0])
        bad += int(off[-1] != n_ids and off[-1] >= off[-2])
        p = Pair(V, D, C=4000 if n_ids < 4000 else V, max_ids=n_ids, max_bags=n_bags, index_kind=index_kind)
        c = p.cache
        c.prepare(torch.from_numpy(ids).to(p.dev), torch.from_numpy(off).to(p.dev))
        st = c.stats()
        assert st["n_bad_offsets"] == bad > 0, (x, st, bad)
        c.fetch_misses()
        out = c.lookup().cpu().numpy()
        rows = p.table.w[ids].astype(np.float64)
        lo, hi = np.clip(off[:-1], 0, n_ids), np.clip(off[1:], 0, n_ids)
        want = np.stack([rows[i:j].sum(0) for i, j in zip(lo, hi)])
        size = np.stack([np.abs(rows[i:j]).sum(0) for i, j in zip(lo, hi)])
        # fp32 additions in a row: each rounds by at most 2^-24 of what has been added up
        assert np.all(np.abs(out - want) <= 2.0 ** -24 * np.maximum(hi - lo, 1)[:, None] * size + 1e-30), x
        c.backward_update(torch.zeros(n_bags, D, device=p.dev))
        torch.cuda.synchronize()
        with pytest.raises(sfc.SfcError) as e:
            c.check()
        assert e.value.code == sfc.SFC_EINVAL and "step 1" in str(e.value)
        assert c.verify() == [0, 0, 0, 0]
        c.flush()
        assert np.array_equal(p.table.w, p.ow)         # a zero gradient changes no weight
        p.close()


@pytest.mark.parametrize("n", [40, 9000])
def test_counters_can_be_read_while_the_device_writes_them(n):
    # polled without a pause from the call on, so that many reads fall into the microseconds in which the
    # kernel writes the block
    p = Pair(V=200, D=4, C=200, max_ids=n)
    c = p.cache
    ids = torch.arange(n, device=p.dev) % 200
    for t in range(1, 301):
        c.prepare(ids)
        end = time.time() + 20
        st, step = c.peek_stats()
        while step != t and time.time() < end:
            assert step == t - 1
            st, step = c.peek_stats()
        assert step == t and st["n_unique"] == min(n, 200) and st["n_miss"] == (min(n, 200) if t == 1 else 0)
        c.fetch_misses(); c.discard()
    p.close()


@pytest.mark.parametrize("n,index_kind", [(40, DENSE), (6000, DENSE), (40, HASHED), (9000, DENSE)])
def test_malformed_offsets_are_reported_no_later_than_the_counters(n, index_kind):
    # without waiting for the device: a caller that sees a step's counters has its report as well, for
    # batches prepared by one block and by the general passes
    import paper_2104_08542_amd as sfc
    p = Pair(V=200, D=4, C=200, max_ids=n, max_bags=4, index_kind=index_kind)
    c = p.cache
    ids = torch.arange(n, device=p.dev) % 200
    off = torch.tensor([0, n, 0, n, n - 1], dtype=torch.int64, device=p.dev)
    torch.cuda.synchronize()
    for t in range(1, 201):
        c.prepare(ids, off)
        end = time.time() + 20
        st, step = c.peek_stats()
        while step != t and time.time() < end:
            st, step = c.peek_stats()
        assert step == t
        assert st["n_bad_offsets"] == 2
        with pytest.raises(sfc.SfcError) as e:
            c.check()
        assert e.value.code == sfc.SFC_EINVAL and "step %d " % t in str(e.value)
        c.fetch_misses(); c.discard()
    p.close()


@pytest.mark.parametrize("index_kind", [HASHED, DENSE])
@pytest.mark.parametrize("C", [0, 7000, 20_000])
def test_degenerate_batches_in_the_general_passes(C, index_kind):
    # the degenerate batches of the one-block prepare again at sizes that it does not take: one id many
    # times, only ids outside the table, all distinct and more than the cache holds, n_ids == max_ids
    V, D, m = 12_000, 4, 9000
    p = Pair(V, D, C=C, max_ids=m, index_kind=index_kind)
    g = lambda n, t: si.grads(n, D, 78, t).numpy()
    p.step(np.zeros(0, np.int64), np.zeros((0, D), np.float32))
    p.step(np.full(7000, 42), g(7000, 1))
    p.step(np.resize([-5, V, 10 ** 12, -1], 6145), g(6145, 2))
    p.step(np.where(np.arange(8000) % 3, np.arange(8000), -1), g(8000, 3))
    p.step(np.arange(V)[::-1][:m].copy(), g(m, 4))
    p.step(np.arange(m) % 100, g(m, 5))
    p.finish(); p.close()


def test_ties_in_stamp_break_by_slot_in_the_general_passes():
    p = Pair(V=40_000, D=4, C=10_000, max_ids=10_000)
    z = lambda n: np.ones((n, 4), np.float32)
    p.step(np.arange(10_000), z(10_000))                        # all stamp 1
    pr = p.step(np.concatenate([np.arange(3000, 10_000), np.arange(20_000, 20_300)]), z(7300))
    assert pr.evict_slots.tolist() == list(range(300))
    pr = p.step(np.concatenate([np.arange(4000, 10_000), np.arange(2999, 2499, -1), np.arange(30_000, 32_300)]), z(8800))
    # slots 300 .. 2499 still carry stamp 1, the other hundred come from stamp 2, lowest slots first; the
    # list is in slot order
    assert pr.evict_slots.tolist() == list(range(100)) + list(range(300, 2500))
    p.finish(); p.close()


def test_status_block_needs_no_waiting():
    # counters and health of the latest planned step, read from pinned memory
    V, D, n = 5000, 8, 3000
    p = Pair(V, D, C=1500, max_ids=4096, lookahead=2)
    c = p.cache
    assert c.peek_stats()[1] == 0
    want = []
    for t in range(5):
        ids = si.zipf_ids(n, 1.05, V, 21, t).numpy()
        pr = p.orc.prepare(ids, None); p.orc.fetch_misses(); p.orc.lookup()
        p.orc.backward_update(si.grads(n, D, 21, t).numpy())
        want.append(pr.stats)
        c.prepare(torch.from_numpy(ids).to(p.dev)); c.fetch_misses()
        if t >= 2:
            c.lookup(); c.backward_update(si.grads(n, D, 21, t - 2).to(p.dev))
        c.check()
        torch.cuda.synchronize()
        pk, step = c.peek_stats()
        assert step == t + 1 and {k: pk[k] for k in want[t]} == want[t]
    p.close()


def test_discard_frees_a_step_that_was_only_read():
    import paper_2104_08542_amd as sfc
    V, D, n = 3000, 8, 800
    p = Pair(V, D, C=1000, max_ids=1024, lookahead=1)
    c = p.cache
    ids = [torch.from_numpy(si.zipf_ids(n, 1.1, V, 44, t).numpy()).to(p.dev) for t in range(4)]
    c.prepare(ids[0]); c.fetch_misses()
    c.prepare(ids[1]); c.fetch_misses()
    with pytest.raises(sfc.SfcError) as e:              # both contexts hold steps that were not updated
        c.prepare(ids[2])
    assert e.value.code == sfc.SFC_ESTATE
    a = c.lookup().clone()
    c.discard()                                          # step 1 given up, rows stay as they are
    c.prepare(ids[2]); c.fetch_misses()
    b = c.lookup().clone()                               # step 2
    c.discard()
    c.prepare(ids[0]); c.fetch_misses()                  # the ids of step 1 again: all hits now
    c.lookup(); c.discard()
    again = c.lookup()                                   # step 4 = ids[0]: same rows as the first lookup
    assert torch.equal(again, a)
    assert c.stats()["n_miss"] == 0
    c.discard()
    with pytest.raises(sfc.SfcError) as e:
        c.discard()
    assert e.value.code == sfc.SFC_ESTATE
    assert c.verify() == [0, 0, 0, 0]
    p.close()


def test_steps_given_up_without_a_lookup_still_bring_their_rows():
    # lookahead 0, copies on a stream of their own: nothing on the main stream waits for the copies of
    # a step that is discarded before its lookup, and the next prepare rewrites the lists they read
    V, D, n = 400_000, 64, 60_000
    p = Pair(V, D, C=150_000, max_ids=n)
    c = p.cache
    ids = [torch.from_numpy(np.random.default_rng(t).permutation(V)[:n]).to(p.dev) for t in range(8)]
    for t in range(24):
        c.prepare(ids[t % 8]); c.fetch_misses()
        if t < 23:
            c.discard()
    out = c.lookup()
    want = p.table.w_t[ids[7].cpu()]
    assert torch.equal(out.cpu(), want)
    c.discard()
    assert c.verify() == [0, 0, 0, 0]
    c.flush()
    assert np.array_equal(p.table.w, p.ow) and np.array_equal(p.table.acc, p.oa)
    p.close()


@pytest.mark.parametrize("lookahead,n", [(0, 400), (0, 7000), (0, 40_000), (1, 400), (1, 7000)])
def test_victims_are_written_back_once_a_row_may_have_changed(lookahead, n):
    # a cache that has only been looked up evicts without writing to the Host table (here the Host rows are
    # replaced behind its back, which a write would undo); from the first update on victims are written
    V, D = 6 * n, 8
    p = Pair(V, D, C=2 * n, max_ids=n, lookahead=lookahead)
    c = p.cache
    ids = [torch.arange(k * n, (k + 1) * n, device=p.dev) for k in range(6)]
    for k in range(2):                                    # fills the cache
        c.prepare(ids[k]); c.fetch_misses(); c.lookup(); c.discard()
    torch.cuda.synchronize()
    p.table.w[:2 * n] = 7.0
    for k in range(2, 6):                                 # every row of the first two batches leaves
        c.prepare(ids[k]); c.fetch_misses(); c.lookup(); c.discard()
    st = c.stats()
    assert st["n_evict"] == n and st["d2h_bytes"] == n * 2 * D * 4
    torch.cuda.synchronize()
    assert np.all(p.table.w[:2 * n] == 7.0)
    c.prepare(ids[0]); c.fetch_misses()                   # batches 4 and 5 are resident; 4 leaves, unwritten
    out = c.lookup()
    assert torch.all(out == 7.0)
    c.backward_update(torch.ones(n, D, device=p.dev))
    for k in (2, 3):                                      # batches 5 and 0 leave: the latter was updated
        c.prepare(ids[k]); c.fetch_misses(); c.lookup(); c.discard()
    torch.cuda.synchronize()
    assert np.all(p.table.w[:n] < 7.0) and np.all(p.table.w[n:2 * n] == 7.0)
    assert np.array_equal(p.table.w[2 * n:], p.ow[2 * n:])
    assert c.verify() == [0, 0, 0, 0]
    p.close()


def _copy_on(stream, dst, src, nbytes):
    """Asynchronous copy between device and pinned Host memory on a stream."""
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipMemcpyAsync.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_void_p]
    assert hip.hipMemcpyAsync(dst, src, nbytes, 4, stream.cuda_stream) == 0       # 4: direction by the pointers


@pytest.mark.parametrize("lookahead", [0, 1])
def test_work_between_prepare_and_fetch_comes_before_the_copies(lookahead):
    # the caller fills the Host rows of a batch's ids on the main stream once the prepare has gone out
    # (rows that are set up when their id is first seen): the Host copies come behind that work, for steps
    # of every size, whichever stream their copies take
    D, sizes = 32, [60_000, 300, 300, 5000, 60_000, 7000, 200]
    V = sum(sizes)
    p = Pair(V, D, C=V, max_ids=60_000, lookahead=lookahead, interleaved=False)
    c, at = p.cache, 0
    for t, n in enumerate(sizes):
        ids = at + torch.randperm(n, generator=torch.Generator().manual_seed(t))
        new = torch.randn(n, D, generator=torch.Generator().manual_seed(100 + t)).to(p.dev)
        d_ids = ids.to(p.dev)
        torch.cuda.synchronize()
        c.prepare(d_ids)
        torch.cuda._sleep(20_000_000)
        _copy_on(c.stream, p.table._pw + 4 * D * at, new.data_ptr(), 4 * D * n)
        filled = torch.cuda.Event()
        filled.record()
        c.fetch_misses()
        assert not filled.query(), "the copies had nothing to wait for"
        out = c.lookup()
        assert torch.equal(out, new[d_ids - at]), (t, n)
        c.backward_update(torch.zeros(n, D, device=p.dev))
        at += n
    torch.cuda.synchronize()
    assert c.verify() == [0, 0, 0, 0]
    p.close()


def test_work_on_the_side_stream_comes_before_the_copies():
    # lookahead 0: what the caller has given the side stream before sfc_fetch_misses comes before the
    # copies of the step, also of a step so small that its copies would take the main stream
    D, sizes = 32, [2000, 300, 300, 5000, 200, 40_000, 300, 7000, 100]
    V = sum(sizes)
    p = Pair(V, D, C=V, max_ids=40_000, interleaved=False)
    c, at = p.cache, 0
    for t, n in enumerate(sizes):
        ids = at + torch.randperm(n, generator=torch.Generator().manual_seed(t))
        new = torch.randn(n, D, generator=torch.Generator().manual_seed(200 + t)).to(p.dev)
        d_ids = ids.to(p.dev)
        torch.cuda.synchronize()
        c.prepare(d_ids)
        if t % 2:                            # (every other step has nothing to wait for)
            with torch.cuda.stream(c.side):
                torch.cuda._sleep(20_000_000)
                _copy_on(c.side, p.table._pw + 4 * D * at, new.data_ptr(), 4 * D * n)
                filled = torch.cuda.Event()
                filled.record()
        c.fetch_misses()
        out = c.lookup()
        if t % 2:
            assert not filled.query(), "the copies had nothing to wait for"
            assert torch.equal(out, new[d_ids - at]), (t, n)
        else:
            assert torch.equal(out.cpu(), p.table.w_t[ids]), (t, n)
        c.backward_update(torch.zeros(n, D, device=p.dev))
        at += n
    torch.cuda.synchronize()
    assert c.verify() == [0, 0, 0, 0]
    p.close()


@pytest.mark.parametrize("n", [300, 20_000])
def test_main_stream_behind_the_lookup_tells_that_the_copies_are_done(n):
    # evicted rows are in the Host table once the main stream has run the step's lookup, whether the
    # step's copies were few (main stream) or many (side stream)
    V, D = 10 * n, 32
    p = Pair(V, D, C=n, max_ids=n)
    c, ids = p.cache, [torch.arange(t * n, (t + 1) * n, device=p.dev) for t in range(6)]
    for t in range(6):
        c.prepare(ids[t]); c.fetch_misses()
        c.lookup()
        c.stream.synchronize()
        if t:                                # the batch before was updated in the cache and then evicted
            now = p.table.w[(t - 1) * n:t * n]
            assert not np.any(now == p.ow[(t - 1) * n:t * n])
        c.backward_update(torch.ones(n, D, device=p.dev))
    p.close()


@pytest.mark.parametrize("n", [300, 7000])
def test_the_calls_of_a_step_can_be_captured(n):
    # lookahead 0: recorded into a graph (launched once: the step's number is part of it) the copies fork to
    # the side stream and join again, for a batch prepared by one block and by the general passes
    hip = ctypes.CDLL("libamdhip64.so")
    vp = ctypes.c_void_p
    V, D = 9000, 8
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        p = Pair(V, D, C=8000, max_ids=n)
        for t in range(3):
            p.step(si.zipf_ids(n, 1.05, V, 61, t).numpy(), si.grads(n, D, 61, t).numpy())
        c, st = p.cache, vp(s.cuda_stream)
        ids, grad = si.zipf_ids(n, 1.05, V, 61, 3).numpy(), si.grads(n, D, 61, 3).numpy()
        d_ids, d_grad, out = torch.from_numpy(ids).to(p.dev), torch.from_numpy(grad).to(p.dev), torch.empty(n, D, device=p.dev)
        torch.cuda.synchronize()
        graph, run = vp(), vp()
        assert hip.hipStreamBeginCapture(st, 2) == 0                   # relaxed
        try:
            c.prepare(d_ids); c.fetch_misses(); c.lookup(out); c.backward_update(d_grad)
        finally:
            rc = hip.hipStreamEndCapture(st, ctypes.byref(graph))
        assert rc == 0
        assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
        assert hip.hipGraphLaunch(run, st) == 0
        torch.cuda.synchronize()
        pr = p.orc.prepare(ids, None); p.orc.fetch_misses()
        assert_close(out.cpu().numpy(), p.orc.lookup(), "lookup")
        p.orc.backward_update(grad)
        assert same_stats(c.stats(), pr.stats, p.table)
        hip.hipGraphExecDestroy(run); hip.hipGraphDestroy(graph)
        p.step(si.zipf_ids(n, 1.05, V, 61, 4).numpy(), si.grads(n, D, 61, 4).numpy())
        p.finish(); p.close()


@pytest.mark.parametrize("n", [400, 40_000])
def test_what_is_recorded_writes_victims_back(n):
    # a graph may be launched when rows have been updated, so it writes victims also where the cache had never been
    # updated when it was recorded (the Host rows are replaced behind the cache's back to see it)
    hip = ctypes.CDLL("libamdhip64.so")
    vp = ctypes.c_void_p
    V, D = 3 * n, 8
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        p = Pair(V, D, C=2 * n, max_ids=n)
        c, st = p.cache, vp(s.cuda_stream)
        ids = [torch.arange(k * n, (k + 1) * n, device=p.dev) for k in range(3)]
        out = torch.empty(n, D, device=p.dev)
        for k in range(2):
            c.prepare(ids[k]); c.fetch_misses(); c.lookup(out); c.discard()
        torch.cuda.synchronize()
        p.table.w[:2 * n] = 7.0
        graph, run = vp(), vp()
        assert hip.hipStreamBeginCapture(st, 2) == 0                   # relaxed
        try:
            c.prepare(ids[2]); c.fetch_misses(); c.lookup(out)
        finally:
            rc = hip.hipStreamEndCapture(st, ctypes.byref(graph))
        assert rc == 0
        assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
        assert hip.hipGraphLaunch(run, st) == 0
        torch.cuda.synchronize()
        c.discard()
        assert c.stats()["n_evict"] == n and np.array_equal(out.cpu().numpy(), p.ow[2 * n:])
        assert np.array_equal(p.table.w[:n], p.ow[:n]) and np.all(p.table.w[n:2 * n] == 7.0)
        assert c.verify() == [0, 0, 0, 0]
        hip.hipGraphExecDestroy(run); hip.hipGraphDestroy(graph)
        p.close()


@pytest.mark.parametrize("n,bags,C,index_kind", [(6145, 0, 20_000, 0), (7000, 1500, 20_000, 2), (9001, 0, 9000, 1),
                                                 (30_000, 4000, 12_000, 1), (270_000, 40_000, 20_000, 0),
                                                 ((1 << 17) - 1, 30_000, 9000, 0), (1 << 17, 30_000, 9000, 0)])
def test_batches_of_a_cache_that_serves_lookups(n, bags, C, index_kind):
    # 64 steps given up in a row: later batches are prepared without their grouping (ids through the virtual id to the
    # slot in the gather, with and without evictions and bypass rows); a gradient has the step grouped after all
    V, D = 20_000, 20
    p = Pair(V, D, C=C, max_ids=n, max_bags=max(n, bags), index_kind=index_kind)
    for t in range(64):
        p.step(si.zipf_ids(40, 1.05, V, 77, t).numpy(), np.zeros((40, D), np.float32), update=False, check_state=False)

    def batch(t):
        ids = si.zipf_ids(n, 1.05, V, 78, t).numpy().copy()
        ids[::997] = V + 5
        off = None
        if bags:
            ends = np.sort(np.random.default_rng(t).integers(0, n + 1, bags - 1))
            off = np.concatenate([[0], ends, [n]])
        return ids, si.grads(bags or n, D, 78, t).numpy(), off

    for t in range(2):
        ids, grad, off = batch(t)
        p.step(ids, grad, off, update=False)
    if bags:
        ids, grad, off = batch(2)
        off[1] = -3
        p.cache.prepare(torch.from_numpy(ids).cuda(), torch.from_numpy(off).cuda())
        assert p.cache.stats()["n_bad_offsets"] == 1
        with pytest.raises(p.sfc.SfcError):
            p.cache.check()
        p.cache.fetch_misses(); p.cache.discard()
        p.orc.prepare(ids, np.maximum(off, 0)); p.orc.fetch_misses()
    for t in range(3, 6):                     # (the first of them is grouped when its gradient comes)
        ids, grad, off = batch(t)
        p.step(ids, grad, off)
    # once more, with the sum that takes its scratch from the library
    for t in range(64):
        p.step(si.zipf_ids(40, 1.05, V, 79, t).numpy(), np.zeros((40, D), np.float32), update=False, check_state=False)
    ids, grad, off = batch(6)
    c = p.cache
    c.prepare(torch.from_numpy(ids).cuda(), None if off is None else torch.from_numpy(off).cuda())
    p.orc.prepare(ids, off)
    c.fetch_misses(); p.orc.fetch_misses()
    out = torch.zeros(n, D, device="cuda")
    d_grad = torch.from_numpy(grad).cuda()
    p.sfc.sfc_segment_sum_static(c.h, d_grad, out)
    assert_close(c.lookup().cpu().numpy(), p.orc.lookup(), "lookup behind the sum")
    expect = p.orc.backward_update(grad, want_common_grad=True)
    assert_close(out[:expect.shape[0]].cpu().numpy(), expect, "common gradient")
    c.backward_update(d_grad)
    p.finish(); p.close()


@pytest.mark.parametrize("n,bags,D", [(270_000, 0, 32), ((1 << 22) + 3, 0, 4), ((1 << 22) + 3, 300_000, 4)])
def test_large_batches_of_a_cache_that_serves_lookups(n, bags, D):
    # the late grouping in the shapes of 2^18 and 2^22 ids on, one-hot and in bags, and lookups of 32 MB and more; device
    # timing tells that the grouping was left out: what makes up for it is added to the prepare's time
    V, C, nb = 60_000, 30_000, bags or n
    p = Pair(V, D, C=C, max_ids=n, max_bags=nb)
    c, o = p.cache, p.orc
    for k in range(64):
        p.step(si.zipf_ids(40, 1.05, V, 92, k).numpy(), np.zeros((40, D), np.float32), update=False, check_state=False)
    grad = si.grads(nb, D, 92, 0)
    d_grad = grad.to(p.dev)
    p.sfc.sfc_profile_enable(c.h, 1)
    for t in range(3):
        ids, off = si.zipf_ids(n, 1.05, V, 93, t).numpy().copy(), _bag_ends(n, bags, t) if bags else None
        ids[::997] = V + 5
        c.prepare(torch.from_numpy(ids).to(p.dev), None if off is None else off.to(p.dev)); c.fetch_misses()
        pr = o.prepare(ids, None if off is None else off.numpy()); o.fetch_misses()
        assert np.array_equal(c.inverse[:n].cpu().numpy(), pr.inverse)
        assert_close(c.lookup().cpu().numpy(), o.lookup(), "lookup of step %d" % t)
        if t == 0:
            c.discard()
            continue
        p.sfc.sfc_profile_read(c.h)
        common = c.segment_sum(d_grad)
        ms, calls = p.sfc.sfc_profile_read(c.h)["prepare"]
        assert calls == 0 and (ms > 0) == (t == 1), ms
        expect = o.backward_update(grad.numpy(), want_common_grad=True)
        assert_close(common[:expect.shape[0]].cpu().numpy(), expect, "common gradient of step %d" % t)
        c.backward_update(d_grad)
    p.finish(); p.close()


class Recorded:
    """The library calls of `calls`, recorded from stream s into a graph."""

    def __init__(self, s, calls):
        self.hip, vp = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p
        self.st, self.graph, self.run = vp(s.cuda_stream), vp(), vp()
        torch.cuda.synchronize()
        assert self.hip.hipStreamBeginCapture(self.st, 2) == 0                   # relaxed
        try:
            calls()
        finally:
            rc = self.hip.hipStreamEndCapture(self.st, ctypes.byref(self.graph))
        assert rc == 0
        assert self.hip.hipGraphInstantiate(ctypes.byref(self.run), self.graph, None, None, ctypes.c_size_t(0)) == 0

    def launch(self):
        assert self.hip.hipGraphLaunch(self.run, self.st) == 0

    def destroy(self):
        torch.cuda.synchronize()
        self.hip.hipGraphExecDestroy(self.run); self.hip.hipGraphDestroy(self.graph)


def _bag_ends(n, bags, t):
    ends = np.sort(np.random.default_rng(t).integers(0, n + 1, bags - 1))
    return torch.from_numpy(np.concatenate([[0], ends, [n]]).astype(np.int64))


@pytest.mark.parametrize("call", ["lookup", "sum", "static", "update"])
@pytest.mark.parametrize("n,bags", [(6145, 0), (9000, 2000), (40_000, 0)])
def test_recorded_calls_of_a_cache_that_serves_lookups(n, bags, call):
    # the host does not see what a graph launches: a call that was recorded once, launched behind the prepare and the
    # fetch of later steps, each of which is given up, finds what it reads there beyond the 64th of them
    V, D, nb = 12_000, 8, bags or n
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        p = Pair(V, D, C=V, max_ids=n, max_bags=nb, side_stream=False)
        c, o = p.cache, p.orc
        d_off = torch.empty(bags + 1, dtype=torch.int64, device=p.dev) if bags else None
        grad = si.grads(nb, D, 83, 0)
        d_grad, out = grad.to(p.dev), torch.zeros(n, D, device=p.dev)
        rec = None
        for t in range(70):
            ids, off = si.zipf_ids(n, 1.05, V, 83, t), _bag_ends(n, bags, t) if bags else None
            if bags:
                d_off.copy_(off)
            c.prepare(ids.to(p.dev), d_off); c.fetch_misses()
            o.prepare(ids.numpy(), None if off is None else off.numpy()); o.fetch_misses()
            if rec is None:
                rec = Recorded(s, {"lookup": lambda: c.lookup(out[:nb]), "sum": lambda: c.segment_sum(d_grad, out),
                                   "static": lambda: p.sfc.sfc_segment_sum_static(c.h, d_grad, out),
                                   "update": lambda: c.backward_update(d_grad)}[call])
            out.fill_(-1.0)
            rec.launch()
            if call != "update" or t:         # (the recording of the update has ended its step)
                c.discard()
            torch.cuda.synchronize()
            if call == "lookup":
                assert_close(out[:nb].cpu().numpy(), o.lookup(), "lookup of step %d" % t)
            else:
                expect = o.backward_update(grad.numpy(), want_common_grad=True)
                if call != "update":
                    assert_close(out[:expect.shape[0]].cpu().numpy(), expect, "common gradient of step %d" % t)
        rec.destroy()
        if call == "update":
            p.finish()
        p.close()


@pytest.mark.parametrize("call", ["lookup", "sum", "static", "update", "fetch"])
@pytest.mark.parametrize("n,bags", [(6145, 0), (9000, 2000), (140_000, 9000), (270_000, 0)])
def test_calls_recorded_on_a_step_that_is_not_grouped(n, bags, call):
    # a call recorded on a step whose prepare left the grouping out has not run: eager calls before the launch do not
    # count on it, the launch gives the same, and so do launches behind later steps, whose buffers may be others
    V, D, nb = 12_000, 8, bags or n
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        p = Pair(V, D, C=V, max_ids=n, max_bags=nb, side_stream=False)
        c, o = p.cache, p.orc
        d_off = torch.empty(bags + 1, dtype=torch.int64, device=p.dev) if bags else None
        grad = si.grads(nb, D, 87, 0)
        d_grad, out, rows = grad.to(p.dev), torch.zeros(n, D, device=p.dev), torch.zeros(nb, D, device=p.dev)

        def load(t, fetch=True):
            ids, off = si.zipf_ids(n, 1.05, V, 87, t), _bag_ends(n, bags, t) if bags else None
            if bags:
                d_off.copy_(off)
            c.prepare(ids.to(p.dev), d_off)
            if fetch:
                c.fetch_misses()
            return ids.numpy(), None if off is None else off.numpy()

        for t in range(64):
            o.prepare(*load(t % 3)); o.fetch_misses()
            c.discard()
        o.prepare(*load(64, call != "fetch")); o.fetch_misses()
        want = o.lookup()

        def everything():
            c.fetch_misses(); c.lookup(rows); c.segment_sum(d_grad, out)

        rec = Recorded(s, {"lookup": lambda: c.lookup(rows), "sum": lambda: c.segment_sum(d_grad, out),
                           "static": lambda: p.sfc.sfc_segment_sum_static(c.h, d_grad, out), "fetch": everything,
                           "update": lambda: c.backward_update(d_grad)}[call])
        if call == "fetch":                   # (the rows come with the launch)
            rec.launch()
        if call != "update":
            assert_close(c.lookup().cpu().numpy(), want, "lookup before the launch")
            common = c.segment_sum(d_grad)
        rec.launch()
        expect = o.backward_update(grad.numpy(), want_common_grad=True)
        if call != "update":
            assert_close(common[:expect.shape[0]].cpu().numpy(), expect, "common gradient before the launch")
            assert_close(c.lookup().cpu().numpy(), want, "lookup behind the launch")
            assert_close(c.segment_sum(d_grad)[:expect.shape[0]].cpu().numpy(), expect, "common gradient behind the launch")
        if call in ("lookup", "fetch"):
            assert_close(rows.cpu().numpy(), want, "recorded lookup")
        if call in ("sum", "static", "fetch"):
            assert_close(out[:expect.shape[0]].cpu().numpy(), expect, "recorded common gradient")
        if call != "update":
            c.backward_update(d_grad)
        was = {}                              # (the earlier steps' buffers stay alive)
        for t in (65, 66) if call != "fetch" else ():
            if call != "update":              # (the update reads the caller's buffers)
                c.bufs, was[t] = [p.sfc.StepBuffers(n, p.dev)], c.bufs
                c._next = 0
            o.prepare(*load(t)); o.fetch_misses()
            want = o.lookup()
            assert_close(c.lookup().cpu().numpy(), want, "lookup of step %d" % t)
            out.fill_(-1.0); rows.fill_(-1.0)
            rec.launch()
            if call != "update":
                assert_close(c.lookup().cpu().numpy(), want, "lookup of step %d, behind the launch" % t)
            expect = o.backward_update(grad.numpy(), want_common_grad=True)
            if call == "lookup":
                assert_close(rows.cpu().numpy(), want, "recorded lookup of step %d" % t)
            elif call != "update":
                assert_close(out[:expect.shape[0]].cpu().numpy(), expect, "recorded common gradient of step %d" % t)
            c.discard() if call == "update" else c.backward_update(d_grad)
        rec.destroy()
        p.finish(); p.close()


@pytest.mark.parametrize("side_stream", [True, False])
@pytest.mark.parametrize("n,bags", [(6145, 0), (9000, 2000), (140_000, 9000), (270_000, 0)])
def test_buffers_of_a_step_that_are_used_again(n, bags, side_stream):
    # behind the fetch the lookup needs the offsets alone, and behind the lookup a gradient the ids and slots: a program
    # may use the other buffers for something else, also with a cache that serves lookups (64 steps given up in a row)
    V, D, nb = 12_000, 8, bags or n
    p = Pair(V, D, C=9000, max_ids=n, max_bags=nb, side_stream=side_stream)
    c, o = p.cache, p.orc
    grad = si.grads(nb, D, 89, 0)
    d_grad = grad.to(p.dev)

    def load(t):
        ids, off = si.zipf_ids(n, 1.05, V, 89, t), _bag_ends(n, bags, t) if bags else None
        d_off = None if off is None else off.to(p.dev)
        b = c.prepare(ids.to(p.dev), d_off); c.fetch_misses()
        o.prepare(ids.numpy(), None if off is None else off.numpy()); o.fetch_misses()
        b.inverse.zero_(); b.miss_vids.zero_()
        return b, d_off

    for t in range(2):
        for k in range(64 if t else 0):
            p.step(si.zipf_ids(40, 1.05, V, 90, k).numpy(), np.zeros((40, D), np.float32), update=False, check_state=False)
        b, _ = load(3 * t)
        b.slot.zero_(); b.unique_ids.zero_()
        assert_close(c.lookup().cpu().numpy(), o.lookup(), "lookup")
        c.discard()
        for call in ("sum", "update"):
            b, d_off = load(3 * t + 1 + (call == "update"))
            want = o.lookup()
            assert_close(c.lookup().cpu().numpy(), want, "lookup of a step with a gradient")
            if bags:
                d_off.zero_()
            expect = o.backward_update(grad.numpy(), want_common_grad=True)
            assert_close(c.segment_sum(d_grad)[:expect.shape[0]].cpu().numpy(), expect, "common gradient")
            c.backward_update(d_grad)
            for k in range(64 if t else 0):
                p.step(si.zipf_ids(40, 1.05, V, 90, k).numpy(), np.zeros((40, D), np.float32), update=False, check_state=False)
    p.finish(); p.close()


@pytest.mark.parametrize("call", ["sum", "static", "update"])
@pytest.mark.parametrize("n,bags", [(7000, 0), (9000, 2000), (1 << 17, 30_000)])
def test_time_of_what_a_serving_cache_launches_later(n, bags, call):
    # device timing: the rows of the positions and a grouping that is made up for are added to the prepare's time and are
    # no calls of their own; the sum that creates no events is timed nowhere.  A batch after the gradient is grouped by its
    # prepare: nothing to make up for.
    V, D, nb = 12_000, 8, bags or n
    p = Pair(V, D, C=V, max_ids=n, max_bags=nb, side_stream=False)
    c = p.cache
    off = _bag_ends(n, bags, 0).to(p.dev) if bags else None
    ids, grad = si.zipf_ids(n, 1.05, V, 88, 0).to(p.dev), si.grads(nb, D, 88, 0).to(p.dev)
    for t in range(64):
        c.prepare(ids, off); c.fetch_misses(); c.discard()
    p.sfc.sfc_profile_enable(c.h, 1)
    prepare = lambda: p.sfc.sfc_profile_read(c.h)["prepare"]

    def gradient():
        if call == "update":
            c.backward_update(grad)
        else:
            (c.segment_sum if call == "sum" else lambda g: p.sfc.sfc_segment_sum_static(c.h, g, out))(grad)
            c.discard()

    out = torch.zeros(n, D, device=p.dev)
    for late in (True, False):
        c.prepare(ids, off)
        ms, calls = prepare()
        assert ms > 0 and calls == 1
        c.fetch_misses()
        ms, calls = prepare()
        assert calls == 0 and ms > 0
        gradient()
        ms, calls = prepare()
        assert calls == 0 and (ms > 0) == (late and call != "static"), ms
    p.close()


@pytest.mark.parametrize("side", ["idle", "busy", "recorded"])
def test_creation_leaves_a_side_stream_with_work_alone(side):
    # the prepare stream is chosen by trying streams beside the caller's two: what the caller has the side stream do or record
    # goes on as if the cache were not being created, and the cache works
    import paper_2104_08542_amd as sfc
    hip, vp = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p
    V, D, n = 3000, 8, 500
    p = Pair(V, D, C=1000, max_ids=n, lookahead=1)
    p.cache.close()
    s, x = torch.cuda.Stream(), torch.zeros(64, device="cuda:0")
    torch.cuda.synchronize()
    real = torch.cuda.Stream
    graph, run = vp(), vp()
    if side == "recorded":
        assert hip.hipStreamBeginCapture(vp(s.cuda_stream), 2) == 0           # relaxed
    if side != "idle":
        with torch.cuda.stream(s):
            if side == "busy":
                torch.cuda._sleep(20_000_000)
            x.add_(1.0)
    try:
        torch.cuda.Stream = lambda *a, **k: real(*a, **k) if k else s      # (the cache's own side stream)
        p.cache = sfc.Cache(p.table, 1000, n, lookahead=1)
    finally:
        torch.cuda.Stream = real
        if side == "recorded":
            rc = hip.hipStreamEndCapture(vp(s.cuda_stream), ctypes.byref(graph))
    assert p.cache.side is s
    if side == "recorded":
        assert rc == 0
        assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
        for k in range(3):
            assert hip.hipGraphLaunch(run, vp(s.cuda_stream)) == 0
    torch.cuda.synchronize()
    assert x.unique().tolist() == [{"idle": 0.0, "busy": 1.0, "recorded": 3.0}[side]]
    batches = [(si.zipf_ids(m, 1.05, V, 91, t), si.grads(m, D, 91, t), None) for t, m in enumerate((n, 40, n, n, 3, n))]
    p.run_pipelined(batches, False)
    if side == "recorded":
        hip.hipGraphExecDestroy(run); hip.hipGraphDestroy(graph)
    p.close()


@pytest.mark.parametrize("lookahead", [1, 2])
def test_pipelined_caches_of_one_stream_in_turn(lookahead):
    # one of them is closed on the way and another one created
    V, D, n = 40_000, 8, 20_000
    sizes = [n, 3000, 12_000, n, 7000, 16_000, n, 2000]

    class Run:
        def __init__(self, k):
            self.p = Pair(V, D, C=9000, max_ids=n, lookahead=lookahead, seed=5 + k)
            self.batches = [(si.zipf_ids(m, 1.05, V, 90 + k, t), si.grads(m, D, 90 + k, t)) for t, m in enumerate(sizes)]
            self.dev = [(i.to("cuda:0"), g.to("cuda:0")) for i, g in self.batches]
            self.expect, self.outs, self.t = [], [], 0
            for ids, grad in self.batches:
                o = self.p.orc
                o.prepare(ids.numpy()); o.fetch_misses()
                self.expect.append(o.lookup()); o.backward_update(grad.numpy())
            for t in range(lookahead):
                self.load(t)

        def load(self, t):
            if t < len(sizes):
                self.p.cache.prepare(self.dev[t][0]); self.p.cache.fetch_misses()

        def step(self):
            self.outs.append(self.p.cache.lookup())
            self.load(self.t + lookahead)
            self.p.cache.backward_update(self.dev[self.t][1])
            self.t += 1

        def end(self):
            while self.t < len(sizes):
                self.step()
            torch.cuda.synchronize()
            for t, out in enumerate(self.outs):
                assert_close(out.cpu().numpy(), self.expect[t], "lookup of step %d" % t)
            self.p.finish(); self.p.close()

    torch.cuda.synchronize()
    runs = [Run(k) for k in range(3)]
    torch.cuda.synchronize()
    for t in range(4):
        for r in runs:
            r.step()
    runs.pop(1).end()
    runs.append(Run(3))
    for t in range(3):
        for r in runs:
            r.step()
    for r in runs:
        r.end()


@pytest.mark.parametrize("n", [6145, 131_072, 131_073, (1 << 22) - 1, 1 << 22, (1 << 22) + 300])
def test_distinct_ids_where_the_insert_pass_changes_shape(n):
    # blocks of 256 or 512 positions, grids that claim without a load first or let the head of the batch go ahead;
    # ids of a power law, so that frequent ones meet in every block, and a batch of all distinct ones behind it
    V = 5_000_000
    import paper_2104_08542_amd as sfc
    tab = sfc.HostTable(V, 4)
    c = sfc.Cache(tab, V, n)
    order = torch.randperm(V, device="cuda:0")[:n]
    for ids in (si.zipf_ids(n, 1.05, V, 61, 0, "cuda:0"), order):
        ids = ids.clone()
        ids[n // 3] = V + 1
        c.prepare(ids); c.fetch_misses()
        st = c.stats()
        x = torch.where(ids < V, ids, -1)
        u, inv = torch.unique(x, return_inverse=True)
        at = torch.full((u.numel(),), n, device="cuda:0").scatter_reduce(0, inv, torch.arange(n, device="cuda:0"), "amin")
        rank = torch.empty_like(at)
        by = torch.argsort(at)
        rank[by] = torch.arange(u.numel(), device="cuda:0")
        assert st["n_unique"] == u.numel() and st["n_invalid"] == 1
        assert torch.equal(c.unique_ids[:u.numel()], u[by])
        assert torch.equal(c.inverse[:n].long(), rank[inv])
        c.discard()
    assert c.verify() == [0, 0, 0, 0]
    c.close(); tab.free()
