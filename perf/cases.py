"""The work that a program asks of this library, as a list of cases that can be timed and compared.

A pass of a case goes through the public binding only.  Three kinds of program:

  train    a training loop at the point where the dense model has returned its gradient: the step that
           was looked up is updated, the next batch is prepared, its missed rows are fetched and its
           model input is looked up.  With lookahead L the batch that is prepared is L steps ahead of
           the one that is looked up.  The rows that a pass returns are read after its update.
  infer    a batch that is only looked up: prepare, fetch, lookup, discard.
  exchange the common gradients of a batch, as a data-parallel program sends them to its peers.

The caches are as a long-running program has them: `prepare` runs every batch of the program's pool
once or twice (without an update), so the cache is full, evicts at its steady rate, and the first
pass is like any later one.  Ids follow a power law with exponent s over V rows (s = 0: uniform),
scattered over the row space; batches differ and come round in turn.
"""
import math

import numpy as np
import torch

import paper_2104_08542_amd as sfc

LR, EPS, ACC0, BETAS = 0.01, 1e-8, 0.1, (0.9, 0.999)


def _case(name, kind, bags, dim, vocab, cache, s, batches, optimizer="adagrad", lookahead=0, bag_hi=1,
          index="auto", bad=0.0):
    c = {"kind": kind, "bags": bags, "bag_hi": bag_hi, "dim": dim, "vocab": vocab, "cache": cache,
         "s": s, "batches": batches, "optimizer": optimizer, "lookahead": lookahead, "index": index, "bad": bad}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # online serving: a request of 32 candidates x 39 fields, the model's rows all resident
        _case("infer_32x39", "infer", 32 * 39, 16, 200_000, 200_000, 1.1, 16),
        # fine-tuning with a small batch: every call of the step is a few microseconds of work; a few ids
        # are outside the table, as raw feature ids are
        _case("train_128x39_d32", "train", 128 * 39, 32, 500_000, 50_000, 1.1, 16, bad=0.001),
        # the smallest benchmark configuration: 1024 x 39, a batch with more distinct ids than the
        # cache has rows, so some rows bypass the cache in every step
        _case("train_1024x39_bypass", "train", 1024 * 39, 16, 100_000, 10_000, 1.05, 8),
        # the second benchmark configuration: 16384 x 39, Zipf 1.1 over 1e7 rows, cache 1e6 rows
        _case("train_16384x39_d16", "train", 16384 * 39, 16, 10_000_000, 1_000_000, 1.1, 24),
        # the third (headline) configuration's batch, 65536 x 39, Zipf 1.2, dim 32, cache 1.6e6 rows of a
        # table of 1e7 (its miss rate is near that of 8e6 rows of 1e8), calls of a step in order ...
        _case("train_65536x39_d32", "train", 65536 * 39, 32, 10_000_000, 1_600_000, 1.2, 24),
        # ... and pipelined, as bench.py runs it by default: three batches in flight
        _case("train_65536x39_d32_pipelined", "train", 65536 * 39, 32, 10_000_000, 1_600_000, 1.2, 24, lookahead=2),
        # the fourth: multi-hot, 32768 x 26 bags of 1 to 20 ids, dim 64, every row resident
        _case("train_32768x26_bags_d64", "train", 32768 * 26, 64, 4_000_000, 4_000_000, 1.1, 4, bag_hi=20),
        # the paper's own training set-up: embedding size 80 with Adam; a batch with a ragged end
        _case("train_5003x39_d80_adam", "train", 5003 * 39, 80, 1_000_000, 100_000, 1.1, 16, optimizer="adam"),
        # row-wise Adagrad on wide rows, one batch ahead, table too large for the dense index in use
        _case("train_8192x26_d128_rowwise", "train", 8192 * 26, 128, 2_000_000, 400_000, 1.1, 12,
              optimizer="rowwise_adagrad", lookahead=1, index="hashed"),
        # offline scoring of bags, wide rows, all resident
        _case("infer_2048x26_bags_d128", "infer", 2048 * 26, 128, 1_000_000, 1_000_000, 1.1, 8, bag_hi=10),
        # low locality (the stress configuration's shape at a quarter of its batch): uniform ids, nearly every
        # row crosses the host link both ways
        _case("train_32768x39_uniform", "train", 32768 * 39, 16, 20_000_000, 3_000_000, 0.0, 4),
        # data-parallel: the common gradients of a headline batch
        _case("exchange_65536x39_d32", "exchange", 65536 * 39, 32, 10_000_000, 1_600_000, 1.2, 2),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["train"] * 6 + ["infer"] * 3 + ["exchange"])
    optimizer = rng.choice(["adagrad", "adagrad", "adam", "rowwise_adagrad"]) if kind == "train" else "adagrad"
    lookahead = rng.choice([0, 0, 1, 2, 3]) if kind == "train" else 0
    dim = rng.choice([8, 16, 20, 32, 48, 64, 80, 128])
    bag_hi = rng.choice([1, 1, 1, rng.randint(2, 20)])
    bags = logint(1000, 2_500_000)
    bags = min(bags, 80_000_000 // dim // (lookahead + 1), 5_000_000 // (1 + bag_hi))
    uniform = rng.random() < 0.15
    if uniform:
        bags = min(bags, 400_000 // (1 + bag_hi))
    s = 0.0 if uniform else round(rng.uniform(1.03, 1.3), 3)
    state = sfc.state_floats(optimizer, dim)
    vocab = logint(20_000, min(10_000_000, 2_000_000_000 // (4 * (dim + state))))
    while math.gcd(vocab, _A) != 1:
        vocab += 1
    cache = int(vocab * rng.choice([1.0, 0.3, 0.1, 0.05]))
    batches = max(2, min(16, 16_000_000 // bags // (1 + bag_hi)))
    return _case(None, kind, bags, dim, vocab, cache, s, batches, optimizer, lookahead, bag_hi,
                 rng.choice(["auto", "auto", "hashed"]), rng.choice([0.0, 0.0, 0.002]))


# ------------------------------------------------------------------------------------- inputs

_A, _B = 2654435761, 1013904223      # rank -> row: (rank * A + B) mod V, A prime


def _table(seed, index):
    """fp32 initial weight of table element `index` (= row * dim + column): mean 0, about 0.01 wide."""
    h = index * -7046029254386353131 + (seed * 2685821657736338717 + 1442695040888963407) % (1 << 62)
    h = (h ^ ((h >> 30) & 0x3FFFFFFFF)) * -4658895280553007687
    h = (h ^ ((h >> 27) & 0x1FFFFFFFFF)) * -7723592293110705685
    s = (h & 0xFFFF) + ((h >> 16) & 0xFFFF) + ((h >> 32) & 0xFFFF)
    return (s - 98302).to(torch.float32) * 3e-7


def _batch(case, seed, k, dev):
    """(ids, offsets or None) of batch k of the pool, on `dev`."""
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 1000003 + 2 * k + 1)
    off, n = None, case["bags"]
    if case["bag_hi"] > 1:
        lens = torch.randint(1, case["bag_hi"] + 1, (case["bags"],), generator=g, device=dev)
        off = torch.zeros(case["bags"] + 1, dtype=torch.int64, device=dev)
        off[1:] = torch.cumsum(lens, 0)
        n = int(off[-1])
    V, s = case["vocab"], case["s"]
    u = torch.rand(n, generator=g, device=dev, dtype=torch.float64)
    if s:
        a, b = 0.5 ** (1 - s), (V + 0.5) ** (1 - s)
        rank = torch.round((a + u * (b - a)) ** (1 / (1 - s))).clamp_(1, V).to(torch.int64) - 1
        ids = (rank * _A + _B) % V
    else:
        ids = (u * V).to(torch.int64).clamp_(max=V - 1)
    if case["bad"]:
        ids[torch.rand(n, generator=g, device=dev) < case["bad"]] = V + 12345
    return ids, off


def _grad(case, seed, k, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(seed * 1000003 + 2 * k + 500000)
    return torch.randn(case["bags"], case["dim"], generator=g, device=dev)


def _warm_steps(case):
    """Batches that a program has been through before the first pass."""
    return case["batches"] * (1 if case["cache"] >= case["vocab"] else 2)


class _State:
    pass


def prepare(case, seed):
    dev = torch.device("cuda:0")
    st = _State()
    st.case = case
    D, V, L, B = case["dim"], case["vocab"], case["lookahead"], case["batches"]
    # the Host table, filled in place: [weights | optimizer state] per row
    st.table = sfc.HostTable(V, D, optimizer=case["optimizer"])
    stride = D + sfc.state_floats(case["optimizer"], D)
    whole = torch.as_strided(st.table.w_t, (V - 1, stride), (stride, 1))
    per = max(1, (1 << 25) // D)
    block = torch.empty(min(per, V), stride, device=dev)
    block[:, D:] = 0.0 if case["optimizer"] == "adam" else ACC0
    for r0 in range(0, V, per):
        r1 = min(V, r0 + per)
        block[:r1 - r0, :D] = _table(seed, torch.arange(r0 * D, r1 * D, device=dev)).view(r1 - r0, D)
        whole[r0:min(r1, V - 1)].copy_(block[:min(r1, V - 1) - r0])
    st.table.w_t[V - 1].copy_(block[(V - 1) % per, :D])      # (the view of the weights ends here)
    st.table.acc_t[V - 1].copy_(block[(V - 1) % per, D:])
    st.pool = [_batch(case, seed, k, dev) for k in range(B)]
    st.grads = [_grad(case, seed, k, dev) for k in range(2)]
    st.out = torch.empty(case["bags"], D, device=dev)
    max_ids = case["bags"] * case["bag_hi"]
    st.cache = sfc.Cache(st.table, case["cache"], max_ids, case["bags"], lr=LR, eps=EPS, lookahead=L, betas=BETAS,
                         index_kind=sfc.SFC_INDEX_HASHED if case["index"] == "hashed" else sfc.SFC_INDEX_AUTO)
    for b in st.cache.bufs:          # what lies beyond a batch's ids stays as it is here
        for t in (b.unique_ids, b.inverse, b.slot):
            t.zero_()
    for k in range(_warm_steps(case)):
        st.cache.prepare(*st.pool[k % B])
        st.cache.fetch_misses()
        st.cache.lookup(st.out)
        st.cache.discard()
    st.next = 0                      # batch of the pool that is prepared next
    if case["kind"] == "train":      # the pipeline is full and the oldest step has been looked up
        for _ in range(L + 1):
            _load(st)
        st.cache.lookup(st.out)
        st.flip = 0
    elif case["kind"] == "exchange":
        _load(st)
        st.cache.lookup(st.out)
        st.common = torch.zeros(max_ids, D, device=dev)
    torch.cuda.synchronize()
    return st


def _load(st):
    """Prepares and fetches the next batch; the ids, virtual ids and slots it was given."""
    k = st.next % len(st.pool)
    st.next += 1
    b = st.cache.prepare(*st.pool[k])
    st.cache.fetch_misses()
    return b.unique_ids, b.inverse, b.slot


def run(st):
    kind = st.case["kind"]
    if kind == "train":
        st.flip ^= 1
        st.cache.backward_update(st.grads[1 - st.flip])
        ids, inverse, slot = _load(st)
        return {"rows": st.cache.lookup(st.out), "ids": ids, "inverse": inverse, "slot": slot}
    if kind == "infer":
        ids, inverse, slot = _load(st)
        rows = st.cache.lookup(st.out)
        st.cache.discard()
        return {"rows": rows, "ids": ids, "inverse": inverse, "slot": slot}
    return {"common": st.cache.segment_sum(st.grads[0], st.common)}


# ------------------------------------------------------------------------------------- what it takes

def _positions(case):
    return case["bags"] * (1 + case["bag_hi"]) / 2


def _unique(case):
    """Expected distinct ids of a batch: the sum of 1 - (1 - p)^n over the ranks, on a grid in log rank."""
    n, V, s = _positions(case), case["vocab"], case["s"]
    if not s:
        return V * -math.expm1(-n / V)
    edge = np.unique(np.round(np.exp(np.linspace(0, math.log(V + 1), 4000))))
    mass = (edge[:-1] - 0.5) ** (1 - s) - (edge[1:] - 0.5) ** (1 - s)
    mass /= 0.5 ** (1 - s) - (V + 0.5) ** (1 - s)
    count = edge[1:] - edge[:-1]
    return float(np.sum(count * -np.expm1(-n * mass / count)))


def work(case):
    """Ids in, virtual ids and slots out, every row of the batch once, the model input out; an update reads
    the gradient once and reads and writes every row with its state.  What a step moves over the host link
    depends on the cache's history and is not counted."""
    n, U, D = _positions(case), _unique(case), case["dim"]
    S = sfc.state_floats(case["optimizer"], D)
    rows, ends = 4 * case["bags"] * D, 8 * case["bags"] * (case["bag_hi"] > 1)
    if case["kind"] == "exchange":
        return {"bytes": rows + 4 * n + 4 * U * D, "flops": n * D}
    bytes_, flops = 8 * n + ends + 4 * n + 12 * U + 4 * U * D + rows, n * D
    if case["kind"] == "train":
        bytes_ += rows + 8 * U * (D + S)
        flops += n * D + 6 * U * D
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """fp32 rows: one update and, in bags, up to 20 fp32 additions; common gradients are summed wider
    than fp32 and rounded once.  Ids, virtual ids and slots are whole numbers and stay the same."""
    if case["kind"] == "infer" and case["bag_hi"] == 1:
        return "exact"
    return {"rel": 4e-7, "max": 1e-5, "differ": 0.0}


def exact(case, seed):
    """The floating outputs of the first pass in 64 bits, in plain torch; None for ids and slots."""
    dev, D, V, B = torch.device("cuda:0"), case["dim"], case["vocab"], case["batches"]
    first = _warm_steps(case)                   # steps before the one that is updated (or looked up)

    def bag_of(off, n):
        if off is None:
            return torch.arange(n, device=dev)
        return torch.repeat_interleave(torch.arange(case["bags"], device=dev), off[1:] - off[:-1])

    def weights(ids):
        at = ids.view(-1, 1) * D + torch.arange(D, device=dev)
        return _table(seed, at.reshape(-1)).view(-1, D).double()

    def first_seen(ids):
        """(distinct ids in order of first appearance, an id outside the table as -1; index per position)"""
        ids = torch.where(ids < V, ids, -1)
        u, inv = torch.unique(ids, return_inverse=True)
        at = torch.full((u.numel(),), ids.numel(), device=dev)
        at.scatter_reduce_(0, inv, torch.arange(ids.numel(), device=dev), "amin")
        order = torch.argsort(at)
        rank = torch.empty_like(order)
        rank[order] = torch.arange(order.numel(), device=dev)
        return u[order], rank[inv]

    def common(k, grad):
        ids, off = _batch(case, seed, k, dev)
        u, inv = first_seen(ids)
        bag = bag_of(off, ids.numel())
        sums = torch.zeros(u.numel(), D, dtype=torch.float64, device=dev)
        for p0 in range(0, ids.numel(), 1 << 21):
            p1 = min(ids.numel(), p0 + (1 << 21))
            sums.index_add_(0, inv[p0:p1], grad[bag[p0:p1]].double())
        return u, sums

    if case["kind"] == "exchange":
        sums = common(0, _grad(case, seed, 0, dev))[1]
        rows = torch.zeros(case["bags"] * case["bag_hi"], D, dtype=torch.float64, device=dev)
        rows[:sums.shape[0]] = sums
        return {"common": rows}
    if case["kind"] == "train":
        # batches 0 .. L are open and batch 0 is updated; batch 1 is then looked up
        u, g = common(0, _grad(case, seed, 0, dev))
        w = weights(u.clamp(min=0))
        if case["optimizer"] == "adagrad":
            w -= LR * g / ((ACC0 + g * g).sqrt() + EPS)
        elif case["optimizer"] == "adam":
            (b1, b2), t = BETAS, first + 1
            m, v = (1 - b1) * g / (1 - b1 ** t), (1 - b2) * g * g / (1 - b2 ** t)
            w -= LR * m / (v.sqrt() + EPS)
        else:
            w -= LR * g / ((ACC0 + (g * g).mean(1, keepdim=True)).sqrt() + EPS)
        new = torch.full((V,), -1, dtype=torch.int64, device=dev)
        new[u[u >= 0]] = torch.nonzero(u >= 0).view(-1)
        ids, off = _batch(case, seed, 1 % B, dev)
    else:
        ids, off = _batch(case, seed, 0, dev)
    bag = bag_of(off, ids.numel())
    rows = torch.zeros(case["bags"], D, dtype=torch.float64, device=dev)
    for p0 in range(0, ids.numel(), 1 << 21):
        part = ids[p0:p0 + (1 << 21)]
        inside = part < V
        safe = torch.where(inside, part, 0)
        x = weights(safe)
        if case["kind"] == "train":
            at = new[safe]
            x = torch.where((at >= 0).view(-1, 1), w[at.clamp(min=0)], x)
        rows.index_add_(0, bag[p0:p0 + (1 << 21)], x * inside.view(-1, 1))
    return {"rows": rows, "ids": None, "inverse": None, "slot": None}
