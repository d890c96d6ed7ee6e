"""The work that users of this library have it do, as sized cases: what is kept in hand, one pass, and what a pass cannot
do without.

A case is a dict of plain values whose "kind" names the program it runs:

  sum2        one Apply, forward: the sum of two digits (inference of the smallest program)
  sum_ops     a Sum-N program written operator by operator: Apply by Apply forward, then the reverse sweep
  sum_fold    a Sum-N training step through the fold call: forward, -log p[target], gradients of all digits
  merged      Apply, Filter and Union of a hashed function, forward and backward in one call (symbol counts in fours)
  pipeline    the same three operators called one by one, any symbol counts
  dtkp_fold   a Sum-N program under top-k proofs, forward, or with the gradient of the input facts
  reach       single-source reachability on a grid, a fixed number of rounds, forward and backward
  product     a Product-N training step, operator by operator (symbol sets that grow to thousands)
  hwf         the formula pipeline (Filter, Apply per position, evaluation), forward and backward, under either provenance

Inputs are made on the GPU from the seed with the laws of the repository's workloads: softmax of normal logits for class
probabilities, Beta(2,2) for edges, N(0,1) upstream gradients.  Function tables belong to the program, not to its inputs:
they are made once and kept.
"""
import functools
import math

import numpy as np
import torch

import workloads as W
from paper_2410_03348_amd import binding as dol

DEV = "cuda"


def listed():
    return [
        # the paper's mini-batch of 64 through the smallest program: one launch, latency only
        dict(name="sum2_b64", kind="sum2", batch=64),
        # the same mini-batch through a program written operator by operator: nine calls
        dict(name="sum5_per_operator_b64", kind="sum_ops", batch=64, digits=5),
        # the headline training step at its stated batch
        dict(name="sum15_train_b4096", kind="sum_fold", batch=4096, digits=15),
        # the same at a batch that fills the card: the largest case
        dict(name="sum15_train_b524288", kind="sum_fold", batch=524288, digits=15),
        # a generic function of 64 x 64 symbols, merged call, at its stated batch
        dict(name="hashed64x64_train_b16384", kind="merged", batch=16384, na=64, nb=64, n_out=256),
        # a generic function whose symbol counts and batch are nobody's round numbers, operator by operator
        dict(name="hashed50x37_operators_b10007", kind="pipeline", batch=10007, na=50, nb=37, n_out=201),
        # top-3 proofs at the stated batch, inference
        dict(name="dtkp_sum5_k3_b1024", kind="dtkp_fold", batch=1024, digits=5, k=3, train=False),
        # more proofs, more facts, training
        dict(name="dtkp_sum6_k5_train_b12000", kind="dtkp_fold", batch=12000, digits=6, k=5, train=True),
        # the paper's 32 x 32 grid
        dict(name="grid32_r64_b256", kind="reach", batch=256, side=32, rounds=64),
        # combinatorial explosion: 23 410 symbols at the end
        dict(name="product16_train_b256", kind="product", batch=256, digits=16),
        # formulas of seven positions under top-3 proofs at the paper's mini-batch
        dict(name="hwf7_dtkp_k3_b64", kind="hwf", batch=64, length=7, provenance="dtkp", k=3),
        # and under add-mult probabilities
        dict(name="hwf7_damp_b200", kind="hwf", batch=200, length=7, provenance="damp", k=0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["sum2", "sum_ops", "sum_fold", "merged", "pipeline", "dtkp_fold", "reach", "product", "hwf"])
    if kind == "sum2":
        return dict(kind=kind, batch=_log_int(rng, 1, 1 << 22))
    if kind == "sum_ops":
        n = rng.randint(3, 12)
        return dict(kind=kind, batch=_log_int(rng, 16, 30000 // n), digits=n)
    if kind == "sum_fold":
        n = rng.randint(2, 15)
        return dict(kind=kind, batch=_log_int(rng, 64, 524288), digits=n)
    if kind == "merged":
        na, nb = 4 * rng.randint(4, 16), 4 * rng.randint(4, 16)
        return dict(kind=kind, batch=_log_int(rng, 256, 131072), na=na, nb=nb, n_out=4 * rng.randint(8, min(64, na * nb // 8)))
    if kind == "pipeline":
        na, nb = _log_int(rng, 12, 150), _log_int(rng, 12, 150)
        return dict(kind=kind, batch=_log_int(rng, 64, min(32768, (1 << 26) // (na * nb))), na=na, nb=nb,
                    n_out=_log_int(rng, 16, min(400, na * nb // 4)))
    if kind == "dtkp_fold":
        n, k = rng.randint(2, 6), rng.choice([1, 3, 5, 7])
        return dict(kind=kind, batch=_log_int(rng, 64, 72000 // (n * max(k, 2)) * 4), digits=n, k=k, train=rng.random() < 0.5)
    if kind == "reach":
        side = rng.randint(8, 32)
        return dict(kind=kind, batch=_log_int(rng, 16, 1024), side=side, rounds=rng.randint(side, 64))
    if kind == "product":
        n = rng.randint(4, 16)
        return dict(kind=kind, batch=_log_int(rng, 16, 256), digits=n)
    provenance = rng.choice(["damp", "dtkp"])
    return dict(kind="hwf", batch=_log_int(rng, 16, 64 if provenance == "dtkp" else 200), length=rng.choice([5, 7]),
                provenance=provenance, k=rng.choice([1, 3]) if provenance == "dtkp" else 0)


# ---- function tables (the symbol side of a program)

@functools.lru_cache(maxsize=None)
def _sum_tables(n):
    """Tables of the left fold of a sum of n digits, one per Apply."""
    tables, syms, digit = [], np.arange(10, dtype=np.int32), np.arange(10, dtype=np.int32)
    for _ in range(1, n):
        tables.append(dol.FnTable.create_dense(syms[:, None] + digit[None, :]))
        syms = tables[-1].out_syms
    return tables


def _hashed(na, nb, n_out):
    """A pseudo-random function of na x nb symbols that produces every one of n_out symbols, and a predicate on these."""
    ids = W.hashed_table(17, na, nb, n_out).reshape(-1)
    ids[np.argsort(W.splitmix64(18, np.arange(na * nb)), kind="stable")[:n_out]] = np.arange(n_out)
    return ids.reshape(na, nb), W.keep_mask(19, n_out)


@functools.lru_cache(maxsize=None)
def _hashed_table(na, nb, n_out):
    ids, keep = _hashed(na, nb, n_out)
    return dol.FnTable.create_dense(ids), keep


@functools.lru_cache(maxsize=None)
def _grid_table(side):
    i, j, o = W.grid_reach_triples(side)
    return dol.FnTable.create_sparse(side * side, int(j.max()) + 1, i, j, o)


_product_ids = functools.lru_cache(maxsize=None)(W.product_stage_tables)
_hwf_ids = functools.lru_cache(maxsize=None)(W.hwf_symbol_tables)


@functools.lru_cache(maxsize=None)
def _product_tables(n):
    return [dol.FnTable.create_dense(t) for t in _product_ids(n)[2]]


@functools.lru_cache(maxsize=None)
def _hwf_tables(length):
    _, tables, _, final_map = _hwf_ids(length)
    return [dol.FnTable.create_dense(t) for t in tables], dol.FnkTable.create_dense(final_map)


# ---- inputs

def _softmax(gen, shape, sigma=1.0):
    return torch.softmax(torch.randn(shape, generator=gen, device=DEV) * sigma, dim=-1)


def _targets(gen, n, batch):
    return torch.randint(0, n, (batch,), generator=gen, device=DEV, dtype=torch.int32)


def _like(d):
    return torch.empty((d.batch, d.n_sym), device=DEV)


# ---- programs

class Sum2:
    def __init__(self, c, gen):
        B, digit = c["batch"], np.arange(10)
        self.table, = _sum_tables(2)
        self.a, self.b = dol.Dist(digit, _softmax(gen, (B, 10))), dol.Dist(digit, _softmax(gen, (B, 10)))
        self.out = dol.Dist.empty(self.table.out_syms, B)

    def run(self):
        dol.apply2(self.a, self.b, self.table, None, self.out)
        return self.out.prob

    @staticmethod
    def work(c):
        return c["batch"] * 4 * 39, c["batch"] * 200


class FoldByOperators:
    """apply2 from Distribution to Distribution, the loss gradient, and the vector-Jacobian products backwards."""

    def __init__(self, c, gen, tables, sym):
        B, self.tables = c["batch"], tables
        n = len(self.tables) + 1
        self.p = _softmax(gen, (n, B, 10), math.sqrt(2.0))
        self.digits = [dol.Dist(sym, self.p[t]) for t in range(n)]
        self.accs = [self.digits[0]] + [dol.Dist.empty(t.out_syms, B) for t in self.tables]
        self.target = _targets(gen, self.accs[-1].n_sym, B)
        self.grad_p = torch.empty_like(self.p)
        self.g_acc = [self.grad_p[0]] + [_like(d) for d in self.accs[1:]]
        self.records = [dol.OpRecord(dol.OP_APPLY2, self.accs[t], self.digits[t + 1], self.accs[t + 1], f=f)
                        for t, f in enumerate(self.tables)]

    def run(self):
        for t, f in enumerate(self.tables):
            dol.apply2(self.accs[t], self.digits[t + 1], f, None, self.accs[t + 1])
        dol.nll_grad(self.accs[-1], self.target, self.g_acc[-1])
        for t in range(len(self.tables), 0, -1):
            dol.backward(self.records[t - 1], self.g_acc[t], self.g_acc[t - 1], self.grad_p[t])
        return self.accs[-1].prob, self.grad_p


class SumOps(FoldByOperators):
    def __init__(self, c, gen):
        super().__init__(c, gen, _sum_tables(c["digits"]), np.arange(10))

    @staticmethod
    def work(c):
        return SumFold.work(c)


class Product(FoldByOperators):
    def __init__(self, c, gen):
        super().__init__(c, gen, _product_tables(c["digits"]), _product_ids(c["digits"])[1][0])

    @staticmethod
    def work(c):
        # every Distribution's tags pass between two calls; the digits, their gradients and the targets once
        stages = [len(s) for s in _product_ids(c["digits"])[1]]
        inner = sum(stages[1:])
        return c["batch"] * 4 * (20 * c["digits"] + 4 * inner + 1), c["batch"] * 2 * 3 * 10 * sum(stages[:-1])


class SumFold:
    def __init__(self, c, gen):
        B, n = c["batch"], c["digits"]
        self.p = _softmax(gen, (n, B, 10), math.sqrt(2.0))
        tables = _sum_tables(n)
        self.out = dol.Dist.empty(tables[-1].out_syms, B)
        self.grad_p = torch.empty_like(self.p)
        self.fold = dol.Fold([dol.Dist(np.arange(10), self.p[t]) for t in range(n)], tables, out=self.out,
                             target_col=_targets(gen, self.out.n_sym, B), grad_inputs=list(self.grad_p))

    def run(self):
        dol.fold_apply2(self.fold)
        return self.out.prob, self.grad_p

    @staticmethod
    def work(c):
        n = c["digits"]
        wide = [9 * t + 1 for t in range(1, n + 1)]                                   # symbols after t digits
        # a target's gradient reaches 9 (n - t) + 1 symbols of the sum of t digits, and no more than there are
        seen = [min(9 * t + 1, 9 * (n - t) + 1) for t in range(1, n + 1)]
        macs = 10 * sum(wide[:-1]) + 10 * sum(seen[:-1]) + 10 * sum(seen[1:])
        return c["batch"] * 4 * (20 * n + wide[-1] + 1), c["batch"] * 2 * macs


class Merged:
    def __init__(self, c, gen):
        B, na, nb, n = c["batch"], c["na"], c["nb"], c["n_out"]
        table, keep = _hashed_table(na, nb, n)
        a, b = dol.Dist(np.arange(na), _softmax(gen, (B, na))), dol.Dist(np.arange(nb), _softmax(gen, (B, nb)))
        other = dol.Dist(np.arange(n), _softmax(gen, (B, n)))
        made = dol.Dist(table.out_syms, None, batch=B)
        self.out = dol.Dist.empty(dol.filter_union_plan(made, keep, other), B)
        self.g = torch.randn((B, self.out.n_sym), generator=gen, device=DEV)
        self.grads = [_like(d) for d in (a, b, other)]
        self.merge = dol.ApplyMerge(a, b, table, keep, other, self.out, torch.empty(B, dtype=torch.int32, device=DEV))

    def run(self):
        dol.apply2_filter_union_forward_backward(self.merge, self.g, *self.grads)
        return self.out.prob, self.grads

    @staticmethod
    def work(c):
        na, nb, n = c["na"], c["nb"], c["n_out"]
        kept = int(_hashed(na, nb, n)[1][_hashed(na, nb, n)[0]].sum())               # tuples whose symbol passes the filter
        return c["batch"] * 4 * (2 * (na + nb + n) + 2 * n), c["batch"] * 2 * 3 * kept


class Pipeline:
    def __init__(self, c, gen):
        B, na, nb, n = c["batch"], c["na"], c["nb"], c["n_out"]
        self.table, self.keep = _hashed_table(na, nb, n)
        self.a, self.b = dol.Dist(np.arange(na), _softmax(gen, (B, na))), dol.Dist(np.arange(nb), _softmax(gen, (B, nb)))
        self.other = dol.Dist(np.arange(n), _softmax(gen, (B, n)))
        self.made = dol.Dist.empty(self.table.out_syms, B)
        self.kept = dol.Dist.empty(dol.filter_plan(self.made, self.keep), B)
        self.out = dol.Dist.empty(dol.union_plan(self.kept, self.other), B)
        self.g = torch.randn((B, self.out.n_sym), generator=gen, device=DEV)
        self.g_made, self.g_kept, self.g_a, self.g_b, self.g_other = (
            _like(d) for d in (self.made, self.kept, self.a, self.b, self.other))
        self.rec_apply = dol.OpRecord(dol.OP_APPLY2, self.a, self.b, self.made, f=self.table)
        self.rec_filter = dol.OpRecord(dol.OP_FILTER, self.made, None, self.kept, pred_mask=self.keep)
        self.rec_union = dol.OpRecord(dol.OP_UNION, self.kept, self.other, self.out)

    def run(self):
        dol.apply2(self.a, self.b, self.table, None, self.made)
        dol.filter(self.made, self.keep, None, self.kept)
        dol.union(self.kept, self.other, None, self.out)
        dol.backward(self.rec_union, self.g, self.g_kept, self.g_other)
        dol.backward(self.rec_filter, self.g_kept, self.g_made, None)
        dol.backward(self.rec_apply, self.g_made, self.g_a, self.g_b)
        return self.made.prob, self.kept.prob, self.out.prob, self.g_a, self.g_b, self.g_other

    @staticmethod
    def work(c):
        na, nb, n = c["na"], c["nb"], c["n_out"]
        kept = int(_hashed(na, nb, n)[1].sum())
        # per call: operands in, results out
        forward = (na + nb + n) + (n + kept) + (kept + 2 * n)
        backward = (n + 2 * kept + 2 * n) + (kept + n) + (2 * na + 2 * nb + n)
        return c["batch"] * 4 * (forward + backward), c["batch"] * 2 * 3 * na * nb


class DtkpSum:
    def __init__(self, c, gen):
        B, n, k = c["batch"], c["digits"], c["k"]
        self.fact_prob = _softmax(gen, (B, n, 10)).reshape(B, 10 * n)
        self.prov = dol.Prov(dol.DTKP, k, self.fact_prob, np.arange(10 * n) // 10)
        tables = _sum_tables(n)
        self.out = dol.Dist.empty(tables[-1].out_syms, B, k=k)
        self.grad = torch.empty_like(self.fact_prob) if c["train"] else None
        digits = [dol.Dist(np.arange(10), torch.empty((B, 10), device=DEV)) for _ in range(n)]
        self.fold = dol.DtkpFold(digits, [10 * t + np.arange(10) for t in range(n)], tables, self.out,
                                 target_col=_targets(gen, self.out.n_sym, B) if c["train"] else None, grad_fact_prob=self.grad)

    def run(self):
        dol.dtkp_fold_apply2(self.fold, self.prov)
        got = [self.out.proof_mask, self.out.proof_prob, self.out.prob]
        return got if self.grad is None else got + [self.grad]

    @staticmethod
    def work(c):
        n, k = c["digits"], c["k"]
        candidates = sum(10 * (9 * t + 1) * (1 if t == 1 else k) for t in range(1, n))  # one product each
        rows = (9 * n + 1) * (12 * k + 4) + 4 * 10 * n + ((4 * 10 * n + 4) if c["train"] else 0)
        return c["batch"] * rows, c["batch"] * candidates


class Reach:
    def __init__(self, c, gen):
        B, self.rounds = c["batch"], c["rounds"]
        self.table = _grid_table(c["side"])
        n, edges = self.table.na, self.table.nb - 1
        p = torch.ones((B, edges + 1), device=DEV)                                    # the last symbol: stay, tag 1
        p[:, :edges] = torch.rand((B, edges, 3), generator=gen, device=DEV).median(dim=-1).values
        r0 = torch.zeros((B, n), device=DEV)
        r0[:, 0] = 1.0
        self.edges, self.r0 = dol.Dist(np.arange(edges + 1), p), dol.Dist(np.arange(n), r0)
        self.g = torch.randn((B, n), generator=gen, device=DEV)
        self.out, self.g_edges = dol.Dist.empty(np.arange(n), B), torch.empty_like(p)
        self.every = dol.iterate_ckpt_every(self.table, B, self.rounds)
        n_ck = dol.iterate_ckpt_count(self.rounds, self.every)
        self.ckpt = torch.empty((n_ck, B, n), device=DEV) if n_ck else None

    def run(self):
        dol.iterate_apply2_backward(self.r0, self.edges, self.table, self.rounds, self.every, self.out, self.ckpt, None,
                                    self.g, None, self.g_edges)
        return self.out.prob, self.g_edges

    @staticmethod
    def work(c):
        side = c["side"]
        n, edges = side * side, 2 * side * (side - 1)
        return c["batch"] * 4 * (3 * n + 2 * (edges + 1)), c["batch"] * c["rounds"] * 2 * 3 * (2 * edges + n)


class Hwf:
    def __init__(self, c, gen):
        B, L, k = c["batch"], c["length"], c["k"]
        self.dtkp = c["provenance"] == "dtkp"
        self.tables, self.final = _hwf_tables(L)
        self.p = _softmax(gen, (B, L, 14))
        self.grad_p = torch.empty_like(self.p)
        self.keep = [(np.arange(14) < 10 if t % 2 == 0 else np.arange(14) >= 10).astype(np.uint8) for t in range(L)]
        self.pos = [dol.Dist(np.arange(14), self.p[:, t, :]) for t in range(L)]
        kept = [dol.filter_plan(self.pos[t], self.keep[t]) for t in range(L)]
        at = np.concatenate([[0], np.cumsum([len(s) for s in kept])])
        self.facts = [np.arange(at[t], at[t + 1], dtype=np.int32) for t in range(L)]
        fact_prob = torch.empty((B, int(at[-1])), device=DEV)
        self.g_fact = torch.empty_like(fact_prob)
        self.prov = None
        if self.dtkp:                    # the kept classes are the input facts
            self.xs = [dol.Dist(kept[t], fact_prob[:, at[t]:at[t + 1]]) for t in range(L)]
            self.g_x = [self.g_fact[:, at[t]:at[t + 1]] for t in range(L)]
            self.prov = dol.Prov(dol.DTKP, k, fact_prob, np.concatenate([np.full(len(s), t) for t, s in enumerate(kept)]))
            first = dol.Dist.empty(kept[0], B, k=k)
        else:
            self.xs = [dol.Dist.empty(kept[t], B) for t in range(L)]
            self.g_x = [_like(d) for d in self.xs]
            first = self.xs[0]
        self.accs = [first] + [dol.Dist.empty(t.out_syms, B, k=k) for t in self.tables]
        self.out = dol.Dist.empty(self.final.out_syms, B, k=k)
        self.g = torch.randn((B, self.out.n_sym), generator=gen, device=DEV)
        self.g_acc = [self.g_x[0]] + [_like(d) for d in self.accs[1:]] if not self.dtkp else None
        self.rec_filter = [dol.OpRecord(dol.OP_FILTER, self.pos[t], None, self.xs[t], pred_mask=self.keep[t]) for t in range(L)]
        self.rec_apply = [dol.OpRecord(dol.OP_APPLY2, self.accs[t], self.xs[t + 1], self.accs[t + 1], f=f)
                          for t, f in enumerate(self.tables)] if not self.dtkp else None

    def run(self):
        for t, d in enumerate(self.pos):
            dol.filter(d, self.keep[t], None, self.xs[t])
        if self.dtkp:
            dol.dtkp_init(self.accs[0], self.facts[0], self.prov)
            for t, f in enumerate(self.tables):
                dol.dtkp_apply2_input(self.accs[t], self.facts[t + 1], f, self.prov, self.accs[t + 1])
        else:
            for t, f in enumerate(self.tables):
                dol.apply2(self.accs[t], self.xs[t + 1], f, None, self.accs[t + 1])
        dol.apply_k([self.accs[-1]], self.final, self.prov, self.out)
        if self.dtkp:
            dol.dtkp_backward(self.out, self.prov, self.g, self.g_fact)
        else:
            dol.apply_k_backward([self.accs[-1]], self.final, self.out, self.g, [self.g_acc[-1]])
            for t in range(len(self.tables), 0, -1):
                dol.backward(self.rec_apply[t - 1], self.g_acc[t], self.g_acc[t - 1], self.g_x[t])
        for t in range(len(self.pos)):
            dol.backward(self.rec_filter[t], self.g_x[t], self.grad_p[:, t, :], None)
        got = [self.out.prob, self.grad_p]
        return got + [self.out.proof_mask, self.out.proof_prob] if self.dtkp else got

    @staticmethod
    def work(c):
        states, tables, values, _ = _hwf_ids(c["length"])
        L, k, n = c["length"], c["k"], [len(s) for s in states]
        kept = sum(10 if t % 2 == 0 else 4 for t in range(L))
        tuples = sum(t.size for t in tables) + n[-1]
        filters = 4 * 2 * (14 * L + kept)
        if c["provenance"] == "dtkp":    # every state's proofs out and in again, the result's proofs and tags, the facts
            moved = 12 * k * 2 * sum(n) + 4 * sum(n) + (12 * k + 4) * 2 * len(values) + 4 * len(values) + 8 * kept
            return c["batch"] * (filters + moved), c["batch"] * tuples * k
        moved = 4 * (4 * sum(n) + 2 * len(values) + 4 * kept)
        return c["batch"] * (filters + moved), c["batch"] * 2 * 3 * tuples


_KINDS = dict(sum2=Sum2, sum_ops=SumOps, sum_fold=SumFold, merged=Merged, pipeline=Pipeline, dtkp_fold=DtkpSum, reach=Reach,
              product=Product, hwf=Hwf)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return _KINDS[case["kind"]](case, gen)


def run(state):
    return state.run()


def work(case):
    moved, operations = _KINDS[case["kind"]].work(case)
    return {"bytes": moved, "flops": operations}


def tolerance(case):
    # float32 tags and gradients throughout, sums of up to some thousand terms; proof masks are whole numbers and exact
    return {"rel": 1e-5, "max": 2e-4}
