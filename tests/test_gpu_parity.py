"""Parity of the HIP library against the CPU oracle, element by element, through the C ABI (needs an MI355X).

Floating-point bar: |gpu - oracle| <= 1e-7 + 1e-5 * |oracle| (oracle accumulates in float64).
Integer / index / proof-mask bar: bit-exact.
Stress cases with unnormalised tags use a one-signed upstream gradient: a float32 sum of mixed-sign terms of order 1
cannot meet an absolute 1e-7 where it cancels to ~0, whatever the kernel.
"""
import os
import subprocess
import sys

import numpy as np
import pytest

import oracle
import workloads as W
from oracle import programs as OP

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03348_amd import programs
    return programs


@pytest.fixture(scope="module")
def dol():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2410_03348_amd import binding
    return binding


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def assert_close(got, want, what=""):
    got = np.asarray(got, np.float64)
    want = np.asarray(want, np.float64)
    assert got.shape == want.shape, (what, got.shape, want.shape)
    err = np.abs(got - want)
    tol = 1e-7 + 1e-5 * np.abs(want)
    bad = err > tol
    assert not bad.any(), "%s: %d of %d outside tolerance, worst excess %g at %s" % (
        what, int(bad.sum()), bad.size, float((err - tol).max()), np.unravel_index(np.argmax(err - tol), err.shape))


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


# ---------------------------------------------------------------- config 1

@pytest.mark.parametrize("batch", [64, 1, 257])
def test_config1_sum2(gp, batch):
    w = W.config1(batch=batch, seed=batch)
    ref = OP.sum2_fwd(w)
    prog = gp.Sum2Forward(w)
    prog.forward()
    out = prog.out
    np.testing.assert_array_equal(out.sym_ids, ref["syms"])
    assert_close(host(out.prob), ref["out"], "sum2")


# ---------------------------------------------------------------- config 2

@pytest.mark.parametrize("batch,n", [(4096, 15), (300, 15), (37, 4), (1, 2)])
def test_config2_sum_chain(gp, batch, n):
    w = W.config2(batch=batch, n_digits=n, seed=n)
    ref = OP.sum_chain_fwd_bwd(w)
    prog = gp.SumChain(w)
    prog.step()
    np.testing.assert_array_equal(prog.accs[-1].sym_ids, ref["syms"])
    for t in range(1, n):
        assert_close(host(prog.accs[t].prob), ref["accs"][t], "chain stage %d" % t)
    assert_close(host(prog.g_acc[-1]), ref["g_out"], "loss gradient")
    assert_close(host(prog.grad_p), ref["grad_p"], "chain grad")


@pytest.mark.parametrize("batch,n", [(4096, 15), (301, 15), (37, 4), (1, 2), (64, 32), (6401, 15), (8192, 6)])
def test_config2_fused_fold(gp, batch, n):
    """dol_fold_apply2: the same results as the chain of per-operator calls, and as the oracle.  The two largest batches
    take the form of the kernel that keeps the reverse sweep's operands in registers."""
    w = W.config2(batch=batch, n_digits=n, seed=n + 100)
    ref = OP.sum_chain_fwd_bwd(w)
    prog = gp.SumChainFused(w)
    prog.step()
    np.testing.assert_array_equal(prog.out.sym_ids, ref["syms"])
    assert_close(host(prog.out.prob), ref["out"], "fold forward")
    assert_close(host(prog.grad_p), ref["grad_p"], "fold grad")
    chain = gp.SumChain(w)
    chain.step()
    np.testing.assert_array_equal(host(prog.out.prob), host(chain.accs[-1].prob))    # same arithmetic, bit for bit


@pytest.mark.parametrize("batch,n,pad", [(1, 1, 0), (5, 3, 0), (1000, 19, 0), (4099, 136, 0), (333, 2050, 0), (70, 19, 5)])
def test_nll_grad(dol, batch, n, pad):
    """dol_nll_grad: -1 / max(p[target], FLT_MIN) at the target, zero elsewhere; rows that are not a multiple of 16 bytes,
    a last workgroup with fewer rows, a padded tensor (the element-wise kernel), a tag of zero."""
    p = W.uniform01(3, batch * n).astype(np.float32).reshape(batch, n)
    target = (np.arange(batch) * 7 % n).astype(np.int32)
    p[0, target[0]] = 0.0
    buf = torch.full((batch, n + pad), 9.0, device="cuda")
    buf[:, :n] = dev(p)
    grad = torch.full((batch, n + pad), 7.0, device="cuda")
    dol.nll_grad(dol.Dist(np.arange(n), buf[:, :n]), dev(target), grad[:, :n])
    want = np.zeros((batch, n), np.float32)
    want[np.arange(batch), target] = np.float32(-1.0) / np.maximum(p[np.arange(batch), target], np.float32(1.17549435e-38))
    got = host(grad)
    np.testing.assert_array_equal(got[:, :n] != 0, want != 0)
    assert_close(got[:, :n], want, "nll gradient")
    assert np.all(got[:, n:] == 7.0)


@pytest.mark.parametrize("widths", [[7, 3, 10, 16, 2], [5, 1, 9, 4, 13, 6, 11]])
@pytest.mark.parametrize("B", [77, 6203])
def test_fused_fold_with_clamping_and_explicit_gradient(dol, B, widths):
    """Unnormalised tags drive several stages over 1; the fold must gate exactly like the per-operator path.
    Also: explicit upstream gradient, padded leading dimensions, mixed operand widths, forward-only call.  The larger
    batch takes the kernel's other form (history in registers); the second list of widths covers second operands of
    1, 4, 6, 9, 11 and 13 symbols (how the lanes share out a short operand's gradient sums depends on that count)."""
    ins = [(W.uniform01(10 + t, B * n) * 0.9).astype(np.float32).reshape(B, n) for t, n in enumerate(widths)]
    syms = [np.arange(n, dtype=np.int32) for n in widths]
    tabs, tris, accs, cur = [], [], [ins[0]], syms[0]
    for t in range(1, len(widths)):
        tab = W.sum_table(cur, syms[t])
        tri = oracle.dense_to_triples(tab)
        cur, o = oracle.damp_apply2_fwd(tri, tab.shape[0], tab.shape[1], accs[-1], ins[t])
        tabs.append(tab); tris.append(tri); accs.append(o)
    assert (accs[-1] == 1.0).any() and (accs[2] == 1.0).any()
    g = np.abs(W.normal(5, B * cur.size)).astype(np.float32).reshape(B, -1)
    want, gr = [None] * len(widths), g
    for t in range(len(widths) - 1, 0, -1):
        gr, want[t] = oracle.damp_apply2_bwd(tris[t - 1], tabs[t - 1].shape[0], tabs[t - 1].shape[1], accs[t - 1], ins[t], gr)
    want[0] = gr
    pad = 3
    d_in = []
    for t, n in enumerate(widths):
        buf = torch.zeros((B, n + pad), device="cuda")
        buf[:, :n] = dev(ins[t])
        d_in.append(dol.Dist(syms[t], buf[:, :n]))
    ftabs = [dol.FnTable.create_dense(t) for t in tabs]
    out = dol.Dist.empty(cur, B)
    gbuf = torch.zeros((B, cur.size + 5), device="cuda")
    gbuf[:, :cur.size] = dev(g)
    gins = [torch.full((B, n + pad), 7.0, device="cuda") for n in widths]
    gins[2] = None                                   # a skipped gradient
    dol.fold_apply2(dol.Fold(d_in, ftabs, out=out, grad_out=gbuf[:, :cur.size], grad_inputs=gins))
    assert_close(host(out.prob), accs[-1], "fold forward (clamped)")
    np.testing.assert_array_equal(host(out.prob) == 1.0, accs[-1] == 1.0)
    for t, n in enumerate(widths):
        if gins[t] is None:
            continue
        assert_close(host(gins[t])[:, :n], want[t], "fold grad %d" % t)
        assert np.all(host(gins[t])[:, n:] == 7.0)
    out2 = dol.Dist.empty(cur, B)
    dol.fold_apply2(dol.Fold(d_in, ftabs, out=out2))                  # forward only
    np.testing.assert_array_equal(host(out2.prob), host(out.prob))
    hashed = dol.FnTable.create_dense(W.hashed_table(1, widths[0], widths[1], 9))
    with pytest.raises(dol.DolError) as ei:
        dol.fold_apply2(dol.Fold(d_in[:2], [hashed], out=dol.Dist.empty(hashed.out_syms, B)))
    assert ei.value.status == 5


def _row_of_mass(key, B, width, mass):
    """[B, width] tags in [0, 1] whose rows sum to about mass[s] (as far as tags of at most 1 allow)."""
    p = W.uniform01(key, B * width).reshape(B, width).astype(np.float64) + 0.05
    p = p / p.sum(axis=1, keepdims=True) * mass[:, None]
    return np.minimum(p, 1.0).astype(np.float32)


@pytest.mark.parametrize("loss", ["target", "grad_out"])
@pytest.mark.parametrize("n", [2, 3, 15])
@pytest.mark.parametrize("B", [77, 6203])
def test_fused_fold_with_masses_on_either_side_of_one(dol, B, n, loss):
    """Operands that Union left above mass 1 and Filter below it: a later operand of small mass, or of none at all, does not
    undo an earlier stage's clamp.  Neighbouring samples share a pattern of masses four at a time (calm: normalised;
    an overflow made up for later; a row of zeros first, in the middle or last), and in every fifth four the patterns are
    mixed.  The larger batch takes the kernel's form with the history in registers."""
    patterns = {0: np.ones(n), 1: np.ones(n), 2: np.ones(n), 3: np.ones(n), 4: np.ones(n), 5: np.full(n, 1.3)}
    patterns[1][0], patterns[1][1:] = 1.8, np.where(np.arange(1, n) % 2 == 1, 1.6, 0.4)
    patterns[2][1:], patterns[2][1] = 0.9, 0.0
    patterns[3][0], patterns[3][1:], patterns[3][n // 2] = 1.8, 1.5, 0.0
    patterns[4][0], patterns[4][1:], patterns[4][n - 1] = 1.8, 1.5, 0.0
    s = np.arange(B)
    which = np.where((s // 4) % 5 == 4, s % 6, (s // 4) % 6)
    mass = np.stack([patterns[k] for k in range(6)])[which]
    ins = [_row_of_mass(30 + t, B, 10, mass[:, t]) for t in range(n)]
    first = which == 1                                    # the largest tags where the sums have to be clamped
    ins[0][first] = 0.0
    ins[0][first, :2] = 0.9
    if n <= 3:
        ins[1][first] = 0.0
        ins[1][first, :2] = 0.8
    if n == 3:
        ins[2][first] = 0.0
        ins[2][first, :2] = np.array([0.3, 0.2], np.float32)
    syms = np.arange(10, dtype=np.int32)
    tabs, tris, accs, cur, kept = [], [], [ins[0]], syms, np.ones(B, bool)
    for t in range(1, n):
        tab = W.sum_table(cur, syms)
        tri = oracle.dense_to_triples(tab)
        cur, o, _, pre = oracle.damp_apply2_fwd(tri, tab.shape[0], tab.shape[1], accs[-1], ins[t], want_pre=True)
        tabs.append(tab); tris.append(tri); accs.append(o)
        # a stage's ten float32 multiply-adds err by at most 10 x 6e-8 of a sum, 15 stages by 1e-5: closer to 1 the oracle's
        # running sums and the kernel's may lie on different sides of it
        kept &= (np.abs(pre - 1.0) > 1e-5).all(axis=1)
    assert kept.mean() > 0.9
    at_one = np.stack([(o == 1.0).any(axis=1) for o in accs[1:]]).any(axis=0)
    small = ins[0].max(axis=1) * np.maximum(np.prod([x.sum(axis=1) for x in ins[1:]], axis=0), 1.0) <= 0.999
    whole = np.add.reduceat(np.where(small, 1, 0), np.arange(0, B, 4)) == np.minimum(4, B - np.arange(0, B, 4))
    if n > 2:                                             # clamps that the product of all masses does not show, in whole fours
        assert (at_one & small & np.repeat(whole, 4)[:B]).any()
    assert (~at_one).any() and at_one.any()
    out = dol.Dist.empty(cur, B)
    gins = [torch.full((B, 10), 7.0, device="cuda") for _ in range(n)]
    d_in = [dol.Dist(syms, dev(x)) for x in ins]
    ftabs = [dol.FnTable.create_dense(t) for t in tabs]
    if loss == "target":
        target = np.argmax(accs[-1] - 0.01 * W.uniform01(3, accs[-1].size).reshape(accs[-1].shape), axis=1).astype(np.int32)
        target[accs[-1].max(axis=1) < 1e-3] = -1          # (nothing to be likely: no gradient)
        g = np.zeros((B, cur.size), np.float32)
        ok = target >= 0
        g[ok, target[ok]] = np.float32(-1.0) / accs[-1][ok, target[ok]].astype(np.float32)
        dol.fold_apply2(dol.Fold(d_in, ftabs, out=out, target_col=dev(target), grad_inputs=gins))
    else:
        g = np.abs(W.normal(5, B * cur.size)).astype(np.float32).reshape(B, -1)
        dol.fold_apply2(dol.Fold(d_in, ftabs, out=out, grad_out=dev(g), grad_inputs=gins))
    want, gr = [None] * n, g
    for t in range(n - 1, 0, -1):
        gr, want[t] = oracle.damp_apply2_bwd(tris[t - 1], tabs[t - 1].shape[0], tabs[t - 1].shape[1], accs[t - 1], ins[t], gr)
    want[0] = gr
    assert_close(host(out.prob)[kept], accs[-1][kept], "fold forward")
    np.testing.assert_array_equal(host(out.prob)[kept] == 1.0, accs[-1][kept] == 1.0)
    for t in range(n):
        assert_close(host(gins[t])[kept], want[t][kept], "fold grad %d" % t)


@pytest.mark.parametrize("B", [5, 8203])
@pytest.mark.parametrize("kind", ["calm", "large", "clamped"])
@pytest.mark.parametrize("widths", [[10] * 15, [3, 10], [255, 16], [40, 1, 16, 16], [1, 1, 2], [16] * 9, [7] * 18, [2, 13, 1, 5, 16, 3, 9, 9, 9], [10] * 24],
                         ids=lambda w: "%dx%d" % (len(w), max(w)))
def test_fold_code_for_chain_shapes(dol, widths, kind, B):
    """The code written for a chain: blocks of every width and changes between them, short operands of 1 to 16 symbols, rows
    that wait in LDS, rows apart by different distances,
    targets on either end and outside, a target of probability 0.  calm: no sum reaches 1, the late stages count from the
    target; large: the same with a first operand so small that the others' sums may exceed 2, where they do not; clamped:
    sums beyond 1.  A third of the samples, the last ones among them, are looked at.
    Tolerance: the bar of 1e-5 relative (sums of non-negative terms and products with one upstream value, under a target and with
    an explicit gradient of one sign: a term's roundings, one a stage and one an addition behind it, mostly cancel)."""
    n, look = len(widths), np.unique(np.concatenate([np.arange(0, B, 3), np.arange(max(0, B - 9), B)]))
    scale = {"calm": np.ones(n), "large": np.r_[0.9 / 3.0 ** (n - 1), np.full(n - 1, 3.0)], "clamped": np.r_[1.0, np.where(np.arange(1, n) % 2, 1.7, 0.6)]}[kind]
    ins = []
    for t, m in enumerate(widths):
        x = W.uniform01(60 + t, B * m).reshape(B, m) + 0.01
        ins.append((x / x.sum(axis=1, keepdims=True) * scale[t] * 0.998 ** (1.0 / n)).astype(np.float32))
    if kind == "clamped" and widths[0] > 1:
        ins[0][:, 1:], ins[0][:, 0] = 0.0, 1.0
        for t in range(1, n):
            ins[t][1::2, 1:] = 0.0
            ins[t][1::2, 0] = scale[t]
    ins[-1][2, :] = 0.0
    syms = [np.arange(m, dtype=np.int32) for m in widths]
    tabs, tris, accs, cur, kept = [], [], [ins[0][look]], syms[0], np.ones(look.size, bool)
    for t in range(1, n):
        tabs.append(W.sum_table(cur, syms[t]))
        tris.append(oracle.dense_to_triples(tabs[-1]))
        cur, o, _, pre = oracle.damp_apply2_fwd(tris[-1], tabs[-1].shape[0], tabs[-1].shape[1], accs[-1], ins[t][look], want_pre=True)
        accs.append(o)
        kept &= (np.abs(pre - 1.0) > 2e-5).all(axis=1) | (kind != "clamped")
    assert kept.mean() > 0.4
    d_in, gins = [], []
    for t, m in enumerate(widths):
        pad = (0, 3, 3, 1)[t % 4]
        buf = torch.zeros((B, m + pad), device="cuda")
        buf[:, :m] = dev(ins[t])
        d_in.append(dol.Dist(syms[t], buf[:, :m]))
        gins.append(torch.full((B, m + pad), 7.0, device="cuda"))
    ftabs, out = [dol.FnTable.create_dense(t) for t in tabs], dol.Dist.empty(cur, B)
    target = (W.uniform01(9, B) * cur.size).astype(np.int32)
    target[0], target[1], target[3], target[4] = 0, cur.size - 1, -1, cur.size
    assert np.all(accs[-1][look == 2] == 0.0)
    g_t = np.zeros((look.size, cur.size), np.float32)
    for r, s in enumerate(look):
        if 0 <= target[s] < cur.size:
            p32 = np.float32(accs[-1][r, target[s]])
            g_t[r, target[s]] = np.float32(-1.0) / np.maximum(p32, np.float32(1.17549435e-38))
    g_x = (np.abs(W.normal(5, B * cur.size)) + 0.1).astype(np.float32).reshape(B, -1)
    for which in ("target", "grad_out"):
        for g in gins:
            g.fill_(7.0)
        if which == "target":
            dol.fold_apply2(dol.Fold(d_in, ftabs, out=out, target_col=dev(target), grad_inputs=gins))
        else:
            dol.fold_apply2(dol.Fold(d_in, ftabs, out=out, grad_out=dev(g_x), grad_inputs=gins))
        want, gr = [None] * n, (g_t if which == "target" else g_x[look])
        for t in range(n - 1, 0, -1):
            gr, want[t] = oracle.damp_apply2_bwd(tris[t - 1], tabs[t - 1].shape[0], tabs[t - 1].shape[1], accs[t - 1], ins[t][look], gr)
        want[0] = gr
        got = host(out.prob)[look]
        assert np.all(np.abs(got - accs[-1])[kept] <= 1e-5 * accs[-1][kept] + 1e-37)
        np.testing.assert_array_equal(got[kept] == 1.0, accs[-1][kept] == 1.0)
        for t, m in enumerate(widths):
            x = host(gins[t])
            assert np.all(x[:, m:] == 7.0)
            bad = np.abs(x[look, :m] - want[t]) > 1e-5 * np.abs(want[t]) + 1e-30
            assert not bad[kept].any(), "%s: grad %d" % (which, t)


def test_fold_code_serves_all_strides(dol, monkeypatch, tmp_path):
    """A chain's code is built twice at most, for rows of like inputs at one distance and for any, whatever distances and batches
    follow, and gives the same bits."""
    monkeypatch.setenv("DOL_JIT_DUMP_DIR", str(tmp_path))
    widths, builds = [9, 11, 11, 11], 0
    syms, tabs, cur = [np.arange(m, dtype=np.int32) for m in widths], [], np.arange(widths[0], dtype=np.int32)
    for t in range(1, len(widths)):
        tabs.append(dol.FnTable.create_dense(W.sum_table(cur, syms[t])))
        cur = tabs[-1].out_syms
    for B in (70, 9000):
        target, first = dev((W.uniform01(19, B) * cur.size).astype(np.int32)), None
        for pads in ((0, 0, 0, 0), (2, 2, 2, 2), (0, 1, 2, 3), (3, 0, 0, 5), (0, 4, 0, 0)):
            ins, gins = [], []
            for t, m in enumerate(widths):
                buf = torch.zeros((B, m + pads[t]), device="cuda")
                buf[:, :m] = dev(W.uniform01(70 + t, B * m).reshape(B, m).astype(np.float32) * (1.9 / m))
                ins.append(dol.Dist(syms[t], buf[:, :m]))
                gins.append(torch.zeros((B, m + pads[t]), device="cuda"))
            out = dol.Dist.empty(cur, B)
            fold = dol.Fold(ins, tabs, out=out, target_col=target, grad_inputs=gins)
            assert dol.fold_kernel(fold) == "damp_fold_chain_kernel"
            dol.fold_apply2(fold)
            for f in tmp_path.iterdir():
                builds += 1
                f.unlink()
            got = [host(out.prob)] + [host(g)[:, :m] for g, m in zip(gins, widths)]
            first = first or got
            for x, y in zip(got, first):
                np.testing.assert_array_equal(x, y)
    assert builds == 2


NO_COMPILER = r"""
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np, torch
import workloads as W
from paper_2410_03348_amd import binding as dol

def apply2(f, a, b, g):
    da, db, out = dol.Dist(np.arange(f.na), a), dol.Dist(np.arange(f.nb), b), dol.Dist.empty(f.out_syms, a.shape[0])
    dol.apply2(da, db, f, None, out)
    ga, gb = torch.empty_like(a), torch.empty_like(b)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), g, ga, gb)
    return out.prob, ga, gb

whole = dol.FnTable.create_dense(W.hashed_table(65, 16, 16, 32))
try:
    apply2(whole, torch.rand(64, 16, device="cuda"), torch.rand(64, 16, device="cuda"), torch.rand(64, whole.n_out, device="cuda"))
    sys.exit("the compiler was there")
except RuntimeError:
    pass
f, B, few = dol.FnTable.create_dense(W.hashed_table(65, 63, 61, 255)), 4400, 4300
assert f.kernel_at(False, B) == "damp_table_fwd_kernel" and f.kernel_at(False, few) != "damp_table_fwd_kernel"
x = [torch.rand(B, n, device="cuda") * s for n, s in ((63, 0.1), (61, 0.1), (f.n_out, 1.0))]
for _ in range(2):
    for got, want in zip(apply2(f, *x), apply2(f, *(t[:few].contiguous() for t in x))):
        assert torch.equal(got[:few], want)
for n in (4, 18):
    sym, tabs, cur, p = np.arange(10, dtype=np.int32), [], np.arange(10, dtype=np.int32), torch.softmax(torch.randn(n, 70, 10, device="cuda"), -1)
    for t in range(1, n):
        tabs.append(dol.FnTable.create_dense(W.sum_table(cur, sym)))
        cur = tabs[-1].out_syms
    ins, grads = [dol.Dist(sym, p[t]) for t in range(n)], torch.zeros_like(p)
    out, g = dol.Dist.empty(cur, 70), torch.rand(70, cur.size, device="cuda")
    fold = dol.Fold(ins, tabs, out=out, grad_out=g, grad_inputs=list(grads))
    assert dol.fold_kernel(fold) == "damp_fold_chain_kernel"
    dol.fold_apply2(fold)
    accs, want = [ins[0]], torch.zeros_like(p)
    for t in range(1, n):
        accs.append(dol.Dist.empty(tabs[t - 1].out_syms, 70))
        dol.apply2(accs[-2], ins[t], tabs[t - 1], None, accs[-1])
    for t in range(n - 1, 0, -1):
        ga = want[0] if t == 1 else torch.empty(70, accs[t - 1].n_sym, device="cuda")
        dol.backward(dol.OpRecord(dol.OP_APPLY2, accs[t - 1], ins[t], accs[t], f=tabs[t - 1]), g, ga, want[t])
        g = ga
    torch.testing.assert_close(out.prob, accs[-1].prob, rtol=1e-5, atol=1e-7)
    torch.testing.assert_close(grads, want, rtol=1e-5, atol=1e-7)
print("served")
"""


def test_calls_that_have_other_kernels_need_no_compiler(tmp_path):
    """With a run-time compiler that fails, folds and tables of ragged rows run in the kernels that were built ahead; a table that
    has always had generated code for these rows says what failed."""
    stub = tmp_path / "stub.c"
    stub.write_text("int hiprtcCompileProgram(void *p, int n, const char **o) { return 6; }")      # HIPRTC_ERROR_COMPILATION
    so = str(tmp_path / "stub.so")
    subprocess.run([os.environ.get("CC", "gcc"), "-shared", "-fPIC", "-o", so, str(stub)], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    run = subprocess.run([sys.executable, "-c", NO_COMPILER, so], capture_output=True, text=True, cwd=root, timeout=100)
    assert run.returncode == 0 and "served" in run.stdout, run.stdout + run.stderr


# ---------------------------------------------------------------- config 3

@pytest.mark.parametrize("batch,na,nb,n_out", [(16384, 64, 64, 256), (1000, 64, 64, 256), (129, 17, 33, 40), (3, 5, 2, 300)])
def test_config3_hashed_pipeline(gp, batch, na, nb, n_out):
    w = W.config3(batch=batch, na=na, nb=nb, n_out=n_out, seed=7)
    ref = OP.hashed_pipeline_fwd_bwd(w)
    prog = gp.HashedPipeline(w)
    prog.step()
    np.testing.assert_array_equal(prog.o1.sym_ids, ref["s1"])
    np.testing.assert_array_equal(prog.o2.sym_ids, ref["s2"])
    np.testing.assert_array_equal(prog.o3.sym_ids, ref["s3"])
    assert_close(host(prog.o1.prob), ref["o1"], "apply")
    np.testing.assert_array_equal(host(prog.o2.prob), host(prog.o1.prob)[:, prog.pred.astype(bool)])
    assert_close(host(prog.o3.prob), ref["o3"], "union")
    assert_close(host(prog.g2), ref["g2"], "union bwd a")
    assert_close(host(prog.gp2), ref["gp2"], "union bwd b")
    assert_close(host(prog.g1), ref["g1"], "filter bwd")
    assert_close(host(prog.ga), ref["ga"], "apply bwd a")
    assert_close(host(prog.gb), ref["gb"], "apply bwd b")


@pytest.mark.parametrize("batch,na,nb,n_out", [(16384, 64, 64, 256), (1000, 64, 64, 256), (129, 17, 33, 40), (3, 5, 2, 300)])
def test_config3_fused_filter_union(gp, batch, na, nb, n_out):
    """dol_filter_union and its backward: the same results as filter then union, without the filtered tensor."""
    w = W.config3(batch=batch, na=na, nb=nb, n_out=n_out, seed=9)
    ref = OP.hashed_pipeline_fwd_bwd(w)
    prog = gp.HashedPipelineFused(w)
    prog.step()
    np.testing.assert_array_equal(prog.o3.sym_ids, ref["s3"])
    assert_close(host(prog.o3.prob), ref["o3"], "filter-union")
    assert_close(host(prog.gp2), ref["gp2"], "filter-union bwd b")
    assert_close(host(prog.g1), ref["g1"], "filter-union bwd a")
    assert_close(host(prog.ga), ref["ga"], "apply bwd a")
    assert_close(host(prog.gb), ref["gb"], "apply bwd b")
    per_op = gp.HashedPipeline(w)
    per_op.step()
    np.testing.assert_array_equal(host(prog.o3.prob), host(per_op.o3.prob))
    np.testing.assert_array_equal(host(prog.g1), host(per_op.g1))
    np.testing.assert_array_equal(host(prog.gp2), host(per_op.gp2))


@pytest.mark.parametrize("batch,na,nb,n_out,scale", [(16384, 64, 64, 256, 1.0), (16421, 64, 64, 256, 6.0), (12301, 64, 64, 256, 6.0), (1000, 64, 64, 256, 1.0), (333, 64, 64, 256, 12.0),
                                                      (65, 32, 16, 64, 9.0), (1, 16, 16, 8, 1.0), (200, 64, 64, 128, 30.0),
                                                      (130, 4, 64, 8, 3.0)])
def test_config3_apply_filter_union_in_one_launch(gp, dol, batch, na, nb, n_out, scale):
    """dol_apply2_filter_union and its reverse: the results of dol_apply2 + dol_filter_union + two dol_backward calls
    (bit for bit) and of the oracle.  scale > 1 multiplies the tags (capped at 1) so that sums of the Apply and of the
    union land on both sides of the clamp: those tiles re-derive every decision."""
    w = W.config3(batch=batch, na=na, nb=nb, n_out=n_out, seed=11)
    if scale != 1.0:
        for key in ("pa", "pb", "p2"):
            w.arrays[key] = np.minimum(w[key] * np.float32(scale), np.float32(1.0))
        w.arrays["g"] = np.abs(w["g"])         # one-signed upstream gradient: see the tolerance note in the module docstring
    ref = OP.hashed_pipeline_fwd_bwd(w)
    prog = gp.HashedPipelineMerged(w)
    prog.step()
    np.testing.assert_array_equal(prog.o3.sym_ids, ref["s3"])
    assert_close(host(prog.o3.prob), ref["o3"], "apply-filter-union")
    np.testing.assert_array_equal(host(prog.o3.prob) == 1.0, ref["o3"] == 1.0)
    assert_close(host(prog.gp2), ref["gp2"], "apply-filter-union grad c")
    assert_close(host(prog.ga), ref["ga"], "apply-filter-union grad a")
    assert_close(host(prog.gb), ref["gb"], "apply-filter-union grad b")
    # some clamp acted in a sample <=> the saved word says so
    both = np.isin(ref["s3"], ref["s2"])
    o2_in_3 = np.zeros_like(ref["o3"], dtype=np.float32)
    o2_in_3[:, both] = ref["o2"]
    pre32 = oracle.damp_apply2_fwd(oracle.dense_to_triples(w["table"]), na, nb, w["pa"], w["pb"], want_pre=True)[2]
    acted = (pre32 > 1.0).any(axis=1) | (((o2_in_3 + w["p2"].astype(np.float32)) > np.float32(1.0)) & both[None, :]).any(axis=1)
    np.testing.assert_array_equal(host(prog.saved) != 0, acted)
    per_op = gp.HashedPipelineFused(w)
    per_op.step()
    np.testing.assert_array_equal(host(prog.o3.prob), host(per_op.o3.prob))
    np.testing.assert_array_equal(host(prog.gp2), host(per_op.gp2))
    assert_close(host(prog.ga), host(per_op.ga).astype(np.float64), "one launch against three: grad a")
    assert_close(host(prog.gb), host(per_op.gb).astype(np.float64), "one launch against three: grad b")
    # without the saved words every tile re-derives its decisions: same results; accumulate adds
    m2 = dol.ApplyMerge(prog.a, prog.b, prog.table, prog.pred, prog.p2, prog.o3, None)
    ga, gb, gc = prog.ga.clone(), prog.gb.clone(), prog.gp2.clone()
    dol.apply2_filter_union_backward(m2, prog.g3, ga, gb, gc, accumulate=7)
    assert_close(host(ga), 2.0 * host(prog.ga).astype(np.float64), "accumulated grad a")
    assert_close(host(gb), 2.0 * host(prog.gb).astype(np.float64), "accumulated grad b")
    assert_close(host(gc), 2.0 * host(prog.gp2).astype(np.float64), "accumulated grad c")
    dol.apply2_filter_union_backward(m2, prog.g3, None, gb, None)
    np.testing.assert_array_equal(host(gb), host(prog.gb))


@pytest.mark.parametrize("batch,na,nb,n_out", [(3072, 32, 16, 64), (3073, 32, 16, 64), (7, 12, 20, 36), (3, 64, 64, 512)])
def test_merged_calls_on_either_side_of_a_workgroup_per_sample(gp, dol, batch, na, nb, n_out):
    """dol_apply2_filter_union both ways, in two calls and in one, at the batch up to which a sample gets a workgroup and above
    it (tiles), for the smallest and widest symbol sets: against the oracle, clamps acting in many samples."""
    w = W.config3(batch=batch, na=na, nb=nb, n_out=n_out, seed=31)
    for key in ("pa", "pb", "p2"):
        w.arrays[key] = np.minimum(w[key] * np.float32(6.0), np.float32(1.0))
    w.arrays["g"] = np.abs(w["g"])
    ref = OP.hashed_pipeline_fwd_bwd(w)
    for one in (False, True):
        prog = gp.HashedPipelineMerged(w, one_launch=one)
        prog.step()
        np.testing.assert_array_equal(host(prog.o3.prob) == 1.0, ref["o3"] == 1.0)
        for got, want in ((prog.o3.prob, ref["o3"]), (prog.ga, ref["ga"]), (prog.gb, ref["gb"]), (prog.gp2, ref["gp2"])):
            assert_close(host(got), want, "merged, one launch %s" % one)
        assert n_out == 512 or host(prog.saved).any()


@pytest.mark.parametrize("clamps", [False, True])
@pytest.mark.parametrize("batch,na,nb,n_out,nc,shift", [
    (3100, 64, 60, 512, 512, 0),        # the widest result
    (8200, 16, 20, 132, 132, 0),        # eight wavefronts; a last group of one piece
    (16390, 12, 16, 36, 100, 0),        # four wavefronts; the second Distribution has symbols that the Apply has not
    (8200, 16, 20, 132, 64, 96),        # symbols of one side only, on both sides
    (16390, 64, 64, 256, 192, 96),      # .. and rows too long to stay in registers
    (16390, 64, 64, 256, 256, 0),       # eight wavefronts above 256 tiles of an aligned plan
    (22599, 64, 64, 256, 256, 0),       # .. and four, rows staged again
    (16390, 56, 56, 200, 200, 0),       # what both passes want is asked for behind the sums
    (16390, 16, 20, 132, 64, 96),       # four wavefronts, rows kept, symbols of one side only
    (3100, 16, 20, 132, 64, 96),        # .. in tiles of 32 samples
    (8199, 64, 64, 256, 192, 96),       # eight wavefronts, rows staged again
    (3100, 64, 64, 256, 192, 96),       # .. in tiles of 32 samples
    (3137, 64, 64, 64, 64, 0),          # eight wavefronts either way, many tuples to a symbol
    (8200, 64, 60, 512, 512, 0),        # the widest result in four wavefronts
    (8200, 16, 64, 320, 320, 0),        # a wide result in eight
])
def test_merged_call_in_one_launch_equals_the_two_calls(dol, batch, na, nb, n_out, nc, shift, clamps):
    """dol_apply2_filter_union_forward_backward against its two halves, bit for bit: with the result's symbols those of the
    second Distribution and not, in every build for a batch, where no clamp acts and where some samples' do, gradients written, added to
    and left out.  Some samples, at the edges of tiles among them, against the oracle, with a one-signed upstream gradient."""
    ids = W.hashed_table(29, na, nb, n_out)
    if n_out <= na * nb:
        ids.reshape(-1)[:n_out] = np.arange(n_out)
    keep = W.keep_mask(30, n_out)
    keep[:shift] = np.arange(shift) % 2                    # (the call takes rows of whole fours)
    x = [(W.uniform01(k, batch * m) / m).astype(np.float32).reshape(batch, m) for k, m in ((1, na), (2, nb), (3, nc))]
    if clamps:
        for t in x:
            t[::37] = np.minimum(t[::37] * t.shape[1], 1.0)
    f = dol.FnTable.create_dense(ids)
    a, b, c = dol.Dist(np.arange(na), dev(x[0])), dol.Dist(np.arange(nb), dev(x[1])), dol.Dist(np.arange(nc) + shift, dev(x[2]))
    made = dol.Dist(f.out_syms, None, batch=batch)
    n3 = len(dol.filter_union_plan(made, keep, c))
    g = dev(W.normal(6, batch * n3).astype(np.float32).reshape(batch, n3))

    def run(one, accumulate, with_gc):
        out = dol.Dist.empty(dol.filter_union_plan(made, keep, c), batch)
        grads = [torch.full((batch, m), 0.5, device="cuda") for m in (na, nb, nc)]
        if not with_gc:
            grads[2] = None
        saved = torch.full((batch,), -1, dtype=torch.int32, device="cuda")
        m = dol.ApplyMerge(a, b, f, keep, c, out, saved)
        if one:
            dol.apply2_filter_union_forward_backward(m, g, *grads, accumulate=accumulate)
        else:
            dol.apply2_filter_union(m)
            dol.apply2_filter_union_backward(m, g, *grads, accumulate=accumulate)
        return [out.prob, saved] + [t for t in grads if t is not None]

    for accumulate, with_gc in ((0, True), (7, True), (0, False)):
        want = run(False, accumulate, with_gc)
        assert bool(host(want[1]).any()) == clamps
        for got, w in zip(run(True, accumulate, with_gc), want):
            np.testing.assert_array_equal(host(got), host(w))
    g = g.abs()
    got = run(True, 0, True)
    look = np.r_[0, 1, 31:34, 63:66, 37 * 40, batch - 2, batch - 1]
    tri, (xa, xb, xc), gl = oracle.dense_to_triples(ids), (t[look] for t in x), host(g)[look]
    syms, made_l = oracle.damp_apply2_fwd(tri, na, nb, xa, xb)
    kept = oracle.damp_filter_fwd(keep[syms], made_l)
    _, ia, ib = oracle.union_plan(oracle.filter_plan(syms, keep[syms])[0], np.arange(nc, dtype=np.int32) + shift)
    g_kept, gc = oracle.damp_union_bwd(ia, ib, kept, xc, gl)
    ga, gb = oracle.damp_apply2_bwd(tri, na, nb, xa, xb, oracle.damp_filter_bwd(keep[syms], g_kept))
    for name, i, ref in (("result", 0, oracle.damp_union_fwd(ia, ib, kept, xc)), ("grad a", 2, ga), ("grad b", 3, gb), ("grad c", 4, gc)):
        assert_close(host(got[i])[look], ref, name)


@pytest.mark.parametrize("nc", [16000, 40332, 40336, 60000])
def test_merged_calls_with_a_wide_second_distribution(dol, nc):
    """The second Distribution has far more symbols than the table produces: rows of more than 64 KB, the widest that a
    workgroup's LDS holds beside the table's rows (158 KB), the next wider one and one far beyond, at a small batch."""
    B, na, nb, n_out = 5, 16, 12, 32
    ids, keep = W.hashed_table(3, na, nb, n_out), W.keep_mask(4, n_out)
    keep[:8] = [1, 0] * 4
    tri = oracle.dense_to_triples(ids)
    pa, pb, pc = ((W.uniform01(k, B * n) * 0.5).astype(np.float32).reshape(B, n) for k, n in ((1, na), (2, nb), (5, nc)))
    s1, o1 = oracle.damp_apply2_fwd(tri, na, nb, pa, pb)
    assert s1.size == n_out
    s2, _ = oracle.filter_plan(s1, keep)
    o2 = oracle.damp_filter_fwd(keep, o1)
    sc = np.arange(nc, dtype=np.int32) + 8                 # (the table's first symbols are not among them)
    s3, ia, ib = oracle.union_plan(s2, sc)
    assert s3.size == nc + 4
    o3 = oracle.damp_union_fwd(ia, ib, o2, pc)
    g = np.abs(W.normal(6, B * s3.size)).astype(np.float32).reshape(B, -1)
    g2, gc = oracle.damp_union_bwd(ia, ib, o2, pc, g)
    ga, gb = oracle.damp_apply2_bwd(tri, na, nb, pa, pb, oracle.damp_filter_bwd(keep, g2))
    f = dol.FnTable.create_dense(ids)
    a, b, c = dol.Dist(np.arange(na), dev(pa)), dol.Dist(np.arange(nb), dev(pb)), dol.Dist(sc, dev(pc))
    out = dol.Dist.empty(s3, B)
    grads = [torch.empty((B, n), device="cuda") for n in (na, nb, nc)]
    m = dol.ApplyMerge(a, b, f, keep, c, out, torch.empty(B, dtype=torch.int32, device="cuda"))
    for one in (False, True):
        for t in [out.prob] + grads:
            t.fill_(-3.0)
        if one:
            dol.apply2_filter_union_forward_backward(m, dev(g), *grads)
        else:
            dol.apply2_filter_union(m)
            dol.apply2_filter_union_backward(m, dev(g), *grads)
        np.testing.assert_array_equal(host(out.prob) == 1.0, o3 == 1.0)
        for got, want in zip([out.prob] + grads, (o3, ga, gb, gc)):
            assert_close(host(got), want, "merged with %d symbols, one launch %s" % (nc, one))


@pytest.mark.parametrize("batch", [40, 3072, 3073])
def test_merged_calls_treat_a_nan_as_the_operators_do(dol, batch):
    """A tag that is no number: the merged calls clamp, mark and gate what dol_apply2 followed by dol_filter_union does, in the
    form for small batches and in the tiles, and a NaN of one symbol reaches no column that has no tuple with it."""
    na, nb, n = 16, 8, 64
    ids, keep = W.hashed_table(23, na, nb, n), np.ones(n, np.uint8)
    ids.reshape(-1)[:n] = np.arange(n)                     # (every symbol is produced; columns of one to some tuples)
    ids[na - 1] = np.arange(nb)                            # (a's last symbol: only what c does not have)
    keep[::4] = 0
    x = [(W.uniform01(k, batch * m) * 0.4).astype(np.float32).reshape(batch, m) for k, m in ((1, na), (2, nb), (3, n))]
    for where, (arr, col) in enumerate(((0, 0), (0, na - 1), (1, 0), (1, nb - 1), (2, 7), (2, 40))):
        x[arr][where::16, col] = np.nan                    # (most samples have none)
    f = dol.FnTable.create_dense(ids)
    a, b, c = dol.Dist(np.arange(na), dev(x[0])), dol.Dist(np.arange(nb), dev(x[1])), dol.Dist(np.arange(n) + n // 2, dev(x[2]))
    made = dol.Dist.empty(f.out_syms, batch)
    out = dol.Dist.empty(dol.filter_union_plan(made, keep, c), batch)
    g = np.abs(W.normal(6, batch * out.n_sym)).astype(np.float32).reshape(batch, -1)
    want = [torch.empty((batch, m), device="cuda") for m in (na, nb, n)]
    g_made = torch.empty((batch, n), device="cuda")
    dol.apply2(a, b, f, None, made)
    dol.filter_union(made, keep, c, None, out)
    dol.backward(dol.OpRecord(dol.OP_FILTER_UNION, made, c, out, pred_mask=keep), dev(g), g_made, want[2])
    dol.backward(dol.OpRecord(dol.OP_APPLY2, a, b, made, f=f), g_made, want[0], want[1])
    want, want_out = [host(t) for t in want], host(out.prob)
    assert np.isnan(want[0]).any() and np.isnan(want[1]).any() and np.isnan(want_out).any()
    clean = ~np.stack([np.isnan(t).any(axis=1) for t in x]).any(axis=0)
    assert 0 < clean.sum() < batch and not any(np.isnan(t[clean]).any() for t in want)
    has = np.zeros((n, nb), bool)                          # a NaN of b's first symbol clamps the columns it is in
    has[ids.reshape(-1), np.tile(np.arange(nb), na)] = True
    assert not has[:, 0].all()
    lone = dol.Dist.empty(out.sym_ids, batch)
    got = [torch.empty((batch, m), device="cuda") for m in (na, nb, n)]
    saved = torch.empty(batch, dtype=torch.int32, device="cuda")
    for one in (False, True):
        m = dol.ApplyMerge(a, b, f, keep, c, lone, saved)
        for t in [lone.prob] + got:
            t.fill_(-3.0)
        if one:
            dol.apply2_filter_union_forward_backward(m, dev(g), *got)
        else:
            dol.apply2_filter_union(m)
            dol.apply2_filter_union_backward(m, dev(g), *got)
        np.testing.assert_array_equal(host(lone.prob), want_out)
        assert (host(saved)[np.isnan(x[0]).any(axis=1) | np.isnan(x[1]).any(axis=1)] != 0).all()
        for t, w in zip(got, want):
            t = host(t)
            np.testing.assert_array_equal(np.isnan(t), np.isnan(w))
            assert_close(np.nan_to_num(t), np.nan_to_num(w), "merged with NaN, one launch %s" % one)


@pytest.mark.parametrize("batch,scale", [(16384, 1.0), (16421, 6.0), (12301, 6.0), (333, 12.0), (64, 1.0), (1, 1.0)])
def test_config3_forward_and_backward_in_one_launch(gp, dol, batch, scale):
    """dol_apply2_filter_union_forward_backward: the results of the two separate calls, bit for bit (clamp words included),
    with samples in which clamps act (scale > 1) and without."""
    w = W.config3(batch=batch, seed=21)
    if scale != 1.0:
        for key in ("pa", "pb", "p2"):
            w.arrays[key] = np.minimum(w[key] * np.float32(scale), np.float32(1.0))
    two = gp.HashedPipelineMerged(w)
    two.step()
    one = gp.HashedPipelineMerged(w, one_launch=True)
    assert len(one.launches) == 1
    for t in (one.o3.prob, one.ga, one.gb, one.gp2):
        t.fill_(-3.0)
    one.saved.fill_(-3)
    one.step()
    np.testing.assert_array_equal(host(one.o3.prob), host(two.o3.prob))
    np.testing.assert_array_equal(host(one.saved), host(two.saved))
    np.testing.assert_array_equal(host(one.ga), host(two.ga))
    np.testing.assert_array_equal(host(one.gb), host(two.gb))
    np.testing.assert_array_equal(host(one.gp2), host(two.gp2))
    if scale != 1.0:
        assert host(one.saved).any()
    ref = OP.hashed_pipeline_fwd_bwd(w)
    assert_close(host(one.o3.prob), ref["o3"], "one-launch forward")
    if scale == 1.0:                          # (mixed-sign gradients over unnormalised tags cannot meet the absolute bar)
        assert_close(host(one.ga), ref["ga"], "one-launch grad a")
        assert_close(host(one.gp2), ref["gp2"], "one-launch grad c")
    with pytest.raises(dol.DolError) as ei:   # the backward pass of this call needs the clamp words
        dol.apply2_filter_union_forward_backward(dol.ApplyMerge(one.a, one.b, one.table, one.pred, one.p2, one.o3, None), one.g3,
                                                 one.ga, one.gb, one.gp2)
    assert ei.value.status == 1


def test_apply_filter_union_rejects_what_it_cannot_take(dol):
    w = W.config3(batch=8, na=17, nb=33, n_out=40, seed=3)                     # symbol counts that are not multiples of 4
    f = dol.FnTable.create_dense(w["table"])
    a, b = dol.Dist(np.arange(17), dev(w["pa"])), dol.Dist(np.arange(33), dev(w["pb"]))
    c = dol.Dist(np.arange(40), dev(w["p2"]))
    pred = np.ones(f.n_out, np.uint8)
    out = dol.Dist.empty(dol.filter_union_plan(dol.Dist(f.out_syms, None, batch=8), pred, c), 8)
    with pytest.raises(dol.DolError) as ei:
        dol.apply2_filter_union(dol.ApplyMerge(a, b, f, pred, c, out))
    assert ei.value.status == 5


def test_filter_union_edge_cases(dol):
    """Everything dropped, nothing dropped, disjoint and empty second operand, padded rows, clamped sums, accumulate."""
    B = 37
    sd = np.array([1, 4, 6, 8, 9], np.int32)
    sc = np.array([0, 4, 9, 12], np.int32)
    a = (W.uniform01(1, B * 5) * 0.9).astype(np.float32).reshape(B, 5)
    c = (W.uniform01(2, B * 4) * 0.9).astype(np.float32).reshape(B, 4)
    g_all = np.abs(W.normal(3, B * 9)).astype(np.float32).reshape(B, 9)
    for pred in ([1, 1, 1, 1, 1], [0, 0, 0, 0, 0], [0, 1, 0, 1, 1], [1, 0, 1, 0, 0]):
        pred = np.array(pred, np.uint8)
        kept, fa = oracle.filter_plan(sd, pred)[0], np.ascontiguousarray(a[:, pred.astype(bool)])
        usyms, ia, ib = oracle.union_plan(kept, sc)
        want = oracle.damp_union_fwd(ia, ib, fa, c)
        ta = torch.zeros((B, 8), device="cuda"); ta[:, :5] = dev(a)            # padded rows
        da, dc = dol.Dist(sd, ta[:, :5]), dol.Dist(sc, dev(c))
        np.testing.assert_array_equal(dol.filter_union_plan(da, pred, dc), usyms)
        out = dol.Dist.empty(usyms, B)
        dol.filter_union(da, pred, dc, None, out)
        assert_close(host(out.prob), want, "filter-union %s" % pred)
        np.testing.assert_array_equal(host(out.prob) == 1.0, want == 1.0)
        g = g_all[:, :usyms.size]
        wfa, wc = oracle.damp_union_bwd(ia, ib, fa, c, g)
        wa = np.zeros((B, 5), np.float32); wa[:, pred.astype(bool)] = wfa
        ga, gc = torch.full((B, 8), 3.0, device="cuda"), torch.zeros((B, 4), device="cuda")
        rec = dol.OpRecord(dol.OP_FILTER_UNION, da, dc, out, pred_mask=pred)
        dol.backward(rec, dev(g), ga, gc)
        assert_close(host(ga)[:, :5], wa, "filter-union bwd a %s" % pred)
        assert np.all(host(ga)[:, 5:] == 3.0)
        assert_close(host(gc), wc, "filter-union bwd c %s" % pred)
        dol.backward(dol.OpRecord(dol.OP_FILTER_UNION, da, dc, out, pred_mask=pred, accumulate=2), dev(g), None, gc)
        assert_close(host(gc), 2.0 * wc.astype(np.float64), "filter-union bwd c accumulated")
    empty = dol.Dist(np.zeros(0, np.int32), torch.zeros((B, 0), device="cuda"))
    da = dol.Dist(sd, dev(a))
    out = dol.Dist.empty(dol.filter_union_plan(da, np.ones(5, np.uint8), empty), B)
    dol.filter_union(da, np.ones(5, np.uint8), empty, None, out)
    np.testing.assert_array_equal(host(out.prob), a)


# ---------------------------------------------------------------- config 4

@pytest.mark.parametrize("batch,n,k", [(1024, 5, 3), (130, 5, 1), (65, 4, 8), (7, 3, 5), (1, 2, 2)])
def test_config4_dtkp_sum(gp, dol, batch, n, k):
    w = W.config4(batch=batch, n_digits=n, k=k, seed=k)
    ref = OP.dtkp_sum_chain(w)
    prog = gp.DtkpSumChain(w)
    prog.step()
    for t in range(1, n):
        syms, m, pp, pr = ref["stages"][t - 1]
        d = prog.accs[t]
        np.testing.assert_array_equal(d.sym_ids, syms)
        np.testing.assert_array_equal(host(d.proof_mask).view(np.uint64), m, err_msg="masks stage %d" % t)
        np.testing.assert_array_equal(host(d.proof_prob), pp, err_msg="proof probs stage %d" % t)
        assert_close(host(d.prob), pr, "tag prob stage %d" % t)
    # gradient of -log Pr(target sum) w.r.t. the digit probabilities through the kept proofs
    last = prog.accs[-1]
    S = last.n_sym
    target = (W.splitmix64(77, np.arange(batch)) % np.uint64(S)).astype(np.int64)
    g = np.zeros((batch, S), np.float32)
    g[np.arange(batch), target] = -1.0 / np.maximum(ref["prob"][np.arange(batch), target], np.float32(1e-30))
    want = oracle.dtkp_prob_bwd(ref["mask"], w["fact_prob"], g)
    gpad = torch.zeros((batch, S + 3), device="cuda")             # a padded gradient tensor
    gpad[:, :S] = dev(g)
    gf = torch.empty((batch, 10 * n), device="cuda")
    dol.dtkp_backward(last, prog.prov, gpad, gf)
    assert_close(host(gf), want, "dtkp gradient of the digit probabilities")
    with pytest.raises(dol.DolError) as ei:                        # the per-operator backward does not take DTKP
        dol.backward(dol.OpRecord(dol.OP_APPLY2, prog.accs[0], prog.digits[1], prog.accs[1], f=prog.tables[0],
                                  prov=prog.prov), gpad, None, None)
    assert ei.value.status == 5


@pytest.mark.parametrize("batch,n,k", [(1024, 5, 3), (130, 5, 1), (65, 4, 8), (7, 3, 5), (1, 2, 2), (3, 6, 2)])
def test_config4_fused_dtkp_fold(gp, dol, batch, n, k):
    """dol_dtkp_fold_apply2: initialisation + all applies (+ the gradient of -log Pr(target)) in one launch."""
    w = W.config4(batch=batch, n_digits=n, k=k, seed=k + 10)
    ref = OP.dtkp_sum_chain(w)
    prog = gp.DtkpSumChainFused(w, with_gradient=True)
    prog.step()
    np.testing.assert_array_equal(prog.out.sym_ids, ref["syms"])
    np.testing.assert_array_equal(host(prog.out.proof_mask).view(np.uint64), ref["mask"])
    np.testing.assert_array_equal(host(prog.out.proof_prob), ref["pprob"])
    assert_close(host(prog.out.prob), ref["prob"], "fused dtkp tag prob")
    S = ref["syms"].size
    target = np.arange(batch) % S
    g = np.zeros((batch, S), np.float32)
    g[np.arange(batch), target] = -1.0 / np.maximum(ref["prob"][np.arange(batch), target], np.float32(1.17549435e-38))
    assert_close(host(prog.grad_fact), oracle.dtkp_prob_bwd(ref["mask"], w["fact_prob"], g), "fused dtkp gradient")
    per_op = gp.DtkpSumChain(w)
    per_op.step()
    np.testing.assert_array_equal(host(prog.out.proof_mask), host(per_op.accs[-1].proof_mask))
    np.testing.assert_array_equal(host(prog.out.proof_prob), host(per_op.accs[-1].proof_prob))
    np.testing.assert_array_equal(host(prog.out.prob), host(per_op.accs[-1].prob))
    # an explicit upstream gradient instead of a target; forward only
    gsym = W.normal(5, batch * S).astype(np.float32).reshape(batch, S)
    gf = torch.empty((batch, 10 * n), device="cuda")
    out2 = dol.Dist.empty(ref["syms"], batch, k=k)
    dol.dtkp_fold_apply2(dol.DtkpFold(prog.digits, prog.facts, prog.tables, out2, grad_out=dev(gsym), grad_fact_prob=gf), prog.prov)
    assert_close(host(gf), oracle.dtkp_prob_bwd(ref["mask"], w["fact_prob"], gsym), "fused dtkp gradient, explicit")
    out3 = dol.Dist.empty(ref["syms"], batch, k=k)
    dol.dtkp_fold_apply2(dol.DtkpFold(prog.digits, prog.facts, prog.tables, out3), prog.prov)
    np.testing.assert_array_equal(host(out3.proof_mask), host(prog.out.proof_mask))


@pytest.mark.parametrize("k", [1, 3, 8])
def test_fused_dtkp_fold_when_a_stage_brings_no_new_facts(dol, k):
    """The fused fold with inputs whose facts are not new to the fold: facts below the ones already in the proofs (the
    product over ascending facts is then redone, not continued), an input given twice (the same fact is idempotent, a
    rival of it excludes the proof), an input that shares its exclusion group with an earlier one under other facts,
    and one with new facts again.  Against the oracle's operator-by-operator composition, bit for bit."""
    batch, nv = 70, 4
    fact_sets = [8 + np.arange(nv), 4 + np.arange(nv), 8 + np.arange(nv), np.arange(nv), 12 + np.arange(nv), 16 + np.arange(nv)]
    n_facts = 20
    grp = (np.arange(n_facts) // nv).astype(np.int32)
    grp[16:20] = grp[0:4]                    # the last input's facts are rivals of the fourth input's
    fp = W.uniform01(77, batch * n_facts).astype(np.float32).reshape(batch, n_facts)
    fp[:, 5] = fp[:, 6]                      # equal probabilities: ties decided by the masks
    fp[3] = 0.0
    sym = np.arange(nv, dtype=np.int32)
    m, pp, pr = oracle.dtkp_init(fact_sets[0].astype(np.int32), fp, k)
    syms, tables = sym, []
    for t in range(1, len(fact_sets)):
        dm, _, _ = oracle.dtkp_init(fact_sets[t].astype(np.int32), fp, k)
        tab = W.sum_table(syms, sym)
        syms, m, pp, pr = oracle.dtkp_apply2(oracle.dense_to_triples(tab), syms.size, nv, k, grp, fp, m, dm)
        tables.append(dol.FnTable.create_dense(tab))
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    digits = [dol.Dist(sym, torch.empty((batch, nv), device="cuda")) for _ in fact_sets]
    out = dol.Dist.empty(syms, batch, k=k)
    g = W.normal(9, batch * syms.size).astype(np.float32).reshape(batch, -1)
    gf = torch.empty((batch, n_facts), device="cuda")
    dol.dtkp_fold_apply2(dol.DtkpFold(digits, [f.astype(np.int32) for f in fact_sets], tables, out, grad_out=dev(g), grad_fact_prob=gf), prov)
    np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), m)
    np.testing.assert_array_equal(host(out.proof_prob), pp)
    assert_close(host(out.prob), pr, "fold tag prob")
    assert_close(host(gf), oracle.dtkp_prob_bwd(m, fp, g), "fold gradient")


@pytest.mark.parametrize("draw", ["four", "apart"])
@pytest.mark.parametrize("batch", [1, 6])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8])
def test_fused_dtkp_fold_list_merge_with_ties(dol, k, batch, draw):
    """The fused fold where every input brings new facts, for every list length: probabilities from four values only (equal
    probabilities inside a list, between lists and on either side of the k-th place, zeros among them), Distributions of
    10, 100 and 109 symbols (in place up to 64, two buffers above), a last workgroup that is not full.  apart: no fact has its
    neighbour's probability in every other sample, so that columns are ranked first, and all have it in the rest."""
    sym = np.arange(10, dtype=np.int32)
    fp = (W.splitmix64(k, np.arange(batch * 40)) % np.uint64(4)).astype(np.float32).reshape(batch, 40) / 4
    if draw == "apart":
        fp[::2] = np.array([0.25, 0.5, 0.0, 0.75, 0.5], np.float32)[np.arange(40) % 5]
        fp[1::2] = 0.25
    grp = (np.arange(40) // 10).astype(np.int32)
    for tabs in ([sym[:, None] * 10 + sym[None, :]] + [None, None], [None, None, None]):
        m, pp, pr = oracle.dtkp_init(sym, fp, k)
        syms, tables = sym, []
        for t, tab in enumerate(tabs):
            tab = W.sum_table(syms, sym) if tab is None else tab.astype(np.int32)
            dm, _, _ = oracle.dtkp_init(10 * (t + 1) + sym, fp, k)
            syms, m, pp, pr = oracle.dtkp_apply2(oracle.dense_to_triples(tab), syms.size, 10, k, grp, fp, m, dm)
            tables.append(dol.FnTable.create_dense(tab))
        digits = [dol.Dist(sym, torch.empty((batch, 10), device="cuda")) for _ in range(4)]
        out = dol.Dist.empty(syms, batch, k=k)
        gf = torch.empty((batch, 40), device="cuda")
        target = (np.arange(batch) * 5 % syms.size).astype(np.int32)
        dol.dtkp_fold_apply2(dol.DtkpFold(digits, [10 * t + sym for t in range(4)], tables, out, target_col=dev(target),
                                          grad_fact_prob=gf), dol.Prov(dol.DTKP, k, dev(fp), grp))
        np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), m)
        np.testing.assert_array_equal(host(out.proof_prob), pp)
        assert_close(host(out.prob), pr, "fold tag prob")
        g = np.zeros((batch, syms.size), np.float32)
        g[np.arange(batch), target] = -1.0 / np.maximum(pr[np.arange(batch), target], np.float32(1.17549435e-38))
        assert_close(host(gf), oracle.dtkp_prob_bwd(m, fp, g), "fold gradient")


@pytest.mark.parametrize("shared", [0, 1])
@pytest.mark.parametrize("k", [1, 2, 3, 5, 8])
def test_fused_dtkp_fold_where_two_proofs_are_equally_probable(dol, k, shared):
    """Facts of which two of one input, or of two inputs, have one probability in some samples, so that single columns have ties: at
    the last place, inside the list, in the last stage and before it, in columns of more candidates than lanes.  shared: every
    input gives one fact to two of its symbols, so that a proof comes twice.  Against the oracle's composition, bit for bit."""
    batch, nv, n = 37, 10, 4
    n_facts = n * nv
    fp = W.uniform01(171 + k, batch * n_facts).astype(np.float32).reshape(batch, n_facts)
    fp[::3, 12], fp[::3, 4], fp[1::6, 33] = fp[::3, 17], fp[::3, 25], 0.0
    facts = [(nv * t + np.arange(nv)).astype(np.int32) for t in range(n)]
    if shared:
        for f in facts:
            f[6] = f[2]
    grp = (np.arange(n_facts) // nv).astype(np.int32)
    sym = np.arange(nv, dtype=np.int32)
    m, _, _ = oracle.dtkp_init(facts[0], fp, k)
    syms, tables = sym, []
    for t in range(1, n):
        dm, _, _ = oracle.dtkp_init(facts[t], fp, k)
        tab = W.sum_table(syms, sym) // (2 if t == 2 else 1)
        syms, m, pp, pr = oracle.dtkp_apply2(oracle.dense_to_triples(tab), syms.size, nv, k, grp, fp, m, dm)
        tables.append(dol.FnTable.create_dense(tab))
    out = dol.Dist.empty(syms, batch, k=k)
    digits = [dol.Dist(sym, torch.empty((batch, nv), device="cuda")) for _ in range(n)]
    dol.dtkp_fold_apply2(dol.DtkpFold(digits, facts, tables, out), dol.Prov(dol.DTKP, k, dev(fp), grp))
    np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), m)
    np.testing.assert_array_equal(host(out.proof_prob), pp)
    assert_close(host(out.prob), pr, "fold tag prob")


@pytest.mark.parametrize("k", [1, 3, 5, 7])
def test_fused_dtkp_fold_where_many_columns_have_ties(dol, k):
    """Samples with no, one, several and all columns of a stage to be ranked by their masks, facts of different probabilities all the
    same: products of powers of two, products that underflow.  Against the oracle's composition, bit for bit."""
    batch, nv, n = 48, 10, 4
    n_facts = n * nv
    fp = W.uniform01(57 + k, batch * n_facts).astype(np.float32).reshape(batch, n_facts)
    for r in range(batch - 12):
        for f in range(r % 12):
            fp[r, nv + 3 * f % 30] = fp[r, nv + (3 * f + 17) % 30]
    fp[-12:-6] = np.float32(2.0) ** -(1 + np.arange(n_facts) % nv)
    fp[-6:] = fp[-6:] ** 60
    facts = [(nv * t + np.arange(nv)).astype(np.int32) for t in range(n)]
    grp = (np.arange(n_facts) // nv).astype(np.int32)
    sym = np.arange(nv, dtype=np.int32)
    m, _, _ = oracle.dtkp_init(facts[0], fp, k)
    syms, tables = sym, []
    for t in range(1, n):
        dm, _, _ = oracle.dtkp_init(facts[t], fp, k)
        tab = W.sum_table(syms, sym)
        syms, m, pp, pr = oracle.dtkp_apply2(oracle.dense_to_triples(tab), syms.size, nv, k, grp, fp, m, dm)
        tables.append(dol.FnTable.create_dense(tab))
    out = dol.Dist.empty(syms, batch, k=k)
    digits = [dol.Dist(sym, torch.empty((batch, nv), device="cuda")) for _ in range(n)]
    dol.dtkp_fold_apply2(dol.DtkpFold(digits, facts, tables, out), dol.Prov(dol.DTKP, k, dev(fp), grp))
    np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), m)
    np.testing.assert_array_equal(host(out.proof_prob), pp)
    assert_close(host(out.prob), pr, "fold tag prob")


@pytest.mark.parametrize("batch,n_sym,n_facts,k", [(1, 1, 1, 1), (1, 1100, 63, 3), (3, 64, 8, 2), (40, 65, 9, 3), (300, 130, 41, 5), (2, 63, 7, 8)])
def test_dtkp_gradient_of_any_number_of_facts(dol, batch, n_sym, n_facts, k):
    """The facts in whole and broken eights, one workgroup to a sample and several, one wavefront and all, facts of probability 0 among
    them.  Against the oracle (1e-5: a sum of at most n_sym * k products and one division)."""
    pick = W.splitmix64(91 + n_facts, np.arange(3 * batch * n_sym * k)).reshape(batch, n_sym, k, 3) % np.uint64(n_facts)
    masks = np.bitwise_or.reduce(np.uint64(1) << pick, axis=-1)
    masks[:, ::5, k - 1] = oracle.ABSENT
    for x in range(1, k):                       # (no proof twice in a list)
        for y in range(x):
            masks[..., x] = np.where(masks[..., x] == masks[..., y], oracle.ABSENT, masks[..., x])
    fp = (0.02 + 0.3 * W.uniform01(92, batch * n_facts)).astype(np.float32).reshape(batch, n_facts)
    fp[::2, n_facts // 2] = 0.0
    prob = np.ones(masks.shape, np.float32)
    for f in range(n_facts):
        prob = np.where((masks >> np.uint64(f)) & np.uint64(1) == 1, prob * fp[:, f, None, None], prob)
    prob[masks == oracle.ABSENT] = 0.0
    g = W.normal(93, batch * n_sym).astype(np.float32).reshape(batch, n_sym)
    dist = dol.Dist.empty(np.arange(n_sym, dtype=np.int32), batch, k=k)
    dist.proof_mask.copy_(dev(masks.view(np.int64)))
    dist.proof_prob.copy_(dev(prob))
    gf = torch.full((batch, n_facts), 7.0, device="cuda")
    dol.dtkp_backward(dist, dol.Prov(dol.DTKP, k, dev(fp), None), dev(g), gf)
    assert_close(host(gf), oracle.dtkp_prob_bwd(masks, fp, g), "dtkp gradient")


@pytest.mark.parametrize("k", [1, 3, 8])
@pytest.mark.parametrize("columns,longest", [(32, 4), (32, 5), (31, 6), (33, 6), (37, 7), (62, 6), (63, 9), (2, 90), (1, 5)])
def test_fused_dtkp_fold_whose_lanes_help(dol, k, columns, longest):
    """Stages of fewer columns than lanes, at the edge of a wavefront's half and of all of it, columns of one tuple and of up to `longest`
    (odd and even, more candidates than lanes), so that a column is one lane's or two lanes' work, some with ties; for few samples
    and, the same ones over and over, for many.  Against the oracle's composition, bit for bit."""
    nv, batch = (16, 12, 10), 9
    n_facts = sum(nv)
    first = np.cumsum((0,) + nv[:2])
    fp = W.uniform01(33 + 7 * columns + longest, batch * n_facts).astype(np.float32).reshape(batch, n_facts)
    fp[::4, 20], fp[::4, 3] = fp[::4, 24], fp[::4, 9]
    facts = [(f + np.arange(m)).astype(np.int32) for f, m in zip(first, nv)]
    grp = np.repeat(np.arange(3), nv).astype(np.int32)
    lengths = np.minimum(longest, 1 + np.arange(columns) % longest) if columns > 2 else np.array([longest, 3][:columns])
    lengths[columns // 2] = longest
    m, _, _ = oracle.dtkp_init(facts[0], fp, k)
    tables, n_cur = [], nv[0]
    for t in (1, 2):
        room = n_cur * nv[t]
        n_out, per = (columns, lengths) if lengths.sum() <= room else (room // 3, np.full(room // 3, 3))
        tab = np.full(room, -1, np.int32)
        tab[np.argsort(W.uniform01(5 + t, room), kind="stable")[:per.sum()]] = np.repeat(np.arange(n_out), per)
        tab = tab.reshape(n_cur, nv[t])
        dm, _, _ = oracle.dtkp_init(facts[t], fp, k)
        syms, m, pp, pr = oracle.dtkp_apply2(oracle.dense_to_triples(tab), n_cur, nv[t], k, grp, fp, m, dm)
        tables.append(dol.FnTable.create_dense(tab))
        n_cur = syms.size
    for tiles in (1, 345):
        out = dol.Dist.empty(syms, batch * tiles, k=k)
        ins = [dol.Dist(np.arange(n, dtype=np.int32), torch.empty((batch * tiles, n), device="cuda")) for n in nv]
        dol.dtkp_fold_apply2(dol.DtkpFold(ins, facts, tables, out), dol.Prov(dol.DTKP, k, dev(np.tile(fp, (tiles, 1))), grp))
        np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), np.tile(m, (tiles, 1, 1)))
        np.testing.assert_array_equal(host(out.proof_prob), np.tile(pp, (tiles, 1, 1)))
        assert_close(host(out.prob), np.tile(pr, (tiles, 1)), "fold tag prob")


def digit_fold(dol, n, k, batch, modulo=0, last=0, seed=1):
    """A fold over n digits: sums, or sums modulo `modulo`, the last stage spread over `last` columns; the call and its provenance."""
    sym = np.arange(10, dtype=np.int32)
    syms, tables = sym, []
    for t in range(1, n):
        ids = W.sum_table(syms, sym)
        ids = ids % modulo if modulo else ids
        if last and t == n - 1:
            ids = (np.arange(ids.size) * 7 % last).reshape(ids.shape)
        tables.append(dol.FnTable.create_dense(ids.astype(np.int32)))
        syms = tables[-1].out_syms
    fp = dev(W.uniform01(seed, batch * 10 * n).astype(np.float32).reshape(batch, 10 * n))
    digits = [dol.Dist(sym, torch.empty((batch, 10), device="cuda")) for _ in range(n)]
    fold = dol.DtkpFold(digits, [10 * t + sym for t in range(n)], tables, dol.Dist.empty(syms, batch, k=k))
    return fold, dol.Prov(dol.DTKP, k, fp, np.arange(10 * n) // 10)


@pytest.mark.parametrize("n,k,batch,modulo,last,many", [
    (6, 5, 3073, 0, 0, True), (6, 5, 3072, 0, 0, False),        # three samples to a SIMD
    (3, 5, 4096, 0, 0, False), (6, 3, 4096, 32, 0, False), (6, 3, 4096, 33, 0, True), (4, 1, 4096, 0, 0, True),   # help for more than 32 columns
    (5, 1, 4096, 50, 300, False), (5, 2, 4096, 50, 300, True),  # a workgroup less for the shares' LDS, and as many
    (6, 7, 4096, 0, 0, True), (6, 8, 4096, 0, 0, False), (6, 8, 4096, 36, 100, True)])    # for the registers, and where LDS allows three either way
def test_fused_dtkp_fold_looks_shares_up_where_that_pays(dol, n, k, batch, modulo, last, many):
    """The build with looked-up shares is taken where a stage of more than 32 columns is helped and no workgroup of a unit is lost."""
    fold, prov = digit_fold(dol, n, k, batch, modulo, last)
    assert dol.dtkp_fold_kernel(fold, prov) == "dtkp_fold_kernel<%d, %s>" % (k, "true" if many else "false")
    fold.c.out.contents.n_sym += 1
    assert dol.dtkp_fold_kernel(fold, prov) == ""


def fold_of_few_and_many(dol, fp, grp, facts, ids, k, tiles, many):
    """A fold over the ids of its stages (-1: no column), of few samples and of the same ones `tiles` times over: masks and probabilities
    against the oracle's composition, the gradients of both losses of the many against those of the few, all bit for bit.  many:
    whether the call then takes the build whose lanes look their shares up."""
    batch, n_facts = fp.shape
    sizes = [f.size for f in facts]
    m = oracle.dtkp_init(facts[0], fp, k)[0]
    syms, tables = np.arange(sizes[0]), []
    for t, tab in enumerate(ids, 1):
        tab = np.ascontiguousarray(tab, np.int32)
        assert tab.shape == (syms.size, sizes[t])
        dm = oracle.dtkp_init(facts[t], fp, k)[0]
        syms, m, pp, pr = oracle.dtkp_apply2(oracle.dense_to_triples(tab), syms.size, sizes[t], k, grp, fp, m, dm)
        tables.append(dol.FnTable.create_dense(tab))
    S = syms.size
    target = (np.arange(batch) * 7 % S).astype(np.int32)
    g = W.normal(k + S, batch * S).astype(np.float32).reshape(batch, S)
    few = []
    for r in (1, tiles):
        ins = [dol.Dist(np.arange(x, dtype=np.int32), torch.empty((batch * r, x), device="cuda")) for x in sizes]
        prov = dol.Prov(dol.DTKP, k, dev(np.tile(fp, (r, 1))), grp)
        out = dol.Dist.empty(syms, batch * r, k=k)
        for loss in ({}, dict(target_col=dev(np.tile(target, r))), dict(grad_out=dev(np.tile(g, (r, 1))))):
            gf = torch.full((batch * r, n_facts), 7.0, device="cuda") if loss else None
            fold = dol.DtkpFold(ins, facts, tables, out, grad_fact_prob=gf, **loss)
            assert dol.dtkp_fold_kernel(fold, prov) == "dtkp_fold_kernel<%d, %s>" % (k, "true" if many and r > 1 else "false")
            out.proof_mask.fill_(5), out.proof_prob.fill_(5.0), out.prob.fill_(5.0)
            dol.dtkp_fold_apply2(fold, prov)
            np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64).reshape(r, batch, S, k), np.broadcast_to(m, (r,) + m.shape))
            np.testing.assert_array_equal(host(out.proof_prob).reshape(r, batch, S, k), np.broadcast_to(pp, (r,) + pp.shape))
            assert_close(host(out.prob), np.tile(pr, (r, 1)), "fold tag prob")
            if loss and r == 1:
                few.append(host(gf).view(np.int32))
            elif loss:
                want = few.pop(0)
                np.testing.assert_array_equal(host(gf).view(np.int32).reshape(r, batch, n_facts), np.broadcast_to(want, (r,) + want.shape))


def facts_of_all_kinds(n, nv, seed):
    """Samples' fact probabilities: without equal ones, with one and two equal pairs (some columns to be ranked by their masks), powers of two
    and products that underflow (most columns), all the same, of four values and certain ones, a fact of probability -0 (every column
    candidate by candidate)."""
    n_facts = n * nv
    fp = W.uniform01(seed, 20 * n_facts).astype(np.float32).reshape(20, n_facts)
    fp[4:10, nv + 2], fp[7:10, 4] = fp[4:10, 2 * nv + 7], fp[7:10, nv + 5]
    fp[10:12] = np.float32(2.0) ** -(1 + np.arange(n_facts) % nv)
    fp[12:14] = fp[12:14] ** 60
    fp[14] = np.float32(0.1)
    fp[15:17] = np.asarray((0.5, 0.25, 1.0, 0.0), np.float32)[(fp[15:17] * 4).astype(int)]
    fp[17] = np.arange(n_facts) % nv == 3
    fp[18, 12] = -0.0
    return fp


@pytest.mark.parametrize("n,k", [(5, 1), (5, 2), (5, 3), (5, 4), (6, 5), (6, 6), (6, 7), (5, 8)])
def test_fused_dtkp_fold_of_few_and_many_samples(dol, n, k):
    """Sum programs both ways in both builds of the fold: few samples, and the same ones over and over so that lanes look their shares up."""
    fp = facts_of_all_kinds(n, 10, 300 + k)
    sym, syms, ids = np.arange(10, dtype=np.int32), np.arange(10, dtype=np.int32), []
    for t in range(1, n):
        ids.append(W.sum_table(syms, sym))
        syms = np.unique(ids[-1])
    facts = [10 * t + sym for t in range(n)]
    fold_of_few_and_many(dol, fp, np.arange(10 * n) // 10, facts, ids, k, 160, k < 8)


@pytest.mark.parametrize("k", [2, 3, 5, 7])
def test_fused_dtkp_fold_of_many_samples_with_stages_of_every_kind(dol, k):
    """Stages that lanes help with beside one whose facts are not new (the first input's once more) and a last one of more columns than
    lanes, which leaves every wavefront two buffers; two symbols of an input by one fact, so that a proof comes twice."""
    fp = facts_of_all_kinds(5, 10, 320 + k)
    sym, syms, ids = np.arange(10, dtype=np.int32), np.arange(10, dtype=np.int32), []
    for t in range(1, 6):
        tab = W.sum_table(syms, sym)
        ids.append((np.arange(tab.size) * 7 % 120).reshape(tab.shape) if t == 5 else tab)
        syms = np.unique(ids[-1])
    facts = [10 * t + sym for t in (0, 1, 2, 3, 0, 4)]
    facts[2] = facts[2].copy()
    facts[2][6] = facts[2][2]
    fold_of_few_and_many(dol, fp, np.arange(50) // 10, facts, ids, k, 160, True)


@pytest.mark.parametrize("k", [1, 3, 5, 7, 8])
@pytest.mark.parametrize("long,columns,helpers", [((9,), 63, 1), ((9, 9), 62, 2), ((8,) * 27, 37, 27), ((8,) * 31, 33, 31), ((12,) * 20, 20, 20), ((7,), 32, 1),
                                                   ((90, 40), 2, 1), ((9,) * 2, 63, 0), ((6,), 64, 0)])
def test_fused_dtkp_fold_with_few_long_columns(dol, k, long, columns, helpers):
    """The longest columns of a stage are as many as the wavefront has lanes to spare, one fewer, one more (nobody helps then), and more
    than half of the columns; in the first stage (one proof to a symbol) and, by columns of the same lengths or one that takes nearly
    all tuples, in the second."""
    nv = (16, 16, 10)
    rest = [1 + c % 3 for c in range(columns - len(long))]
    lengths = np.array((list(long) + rest))[np.argsort(W.uniform01(columns, columns), kind="stable")]
    assert lengths.sum() <= nv[0] * nv[1]
    # what the plan works out: columns of more than `most` tuples get a helper
    most = (lengths.max() + 1) // 2
    while columns + (lengths > most).sum() > 64:
        most += 1
    assert (helpers and (lengths > most).sum() == helpers and lengths.max() - most >= 2) or (not helpers and lengths.max() - most < 2)
    ids, n_cur = [], nv[0]
    for t in (1, 2):
        room = n_cur * nv[t]
        per = lengths if lengths.sum() <= room else np.array([room - 3, 3])
        tab = np.full(room, -1, np.int32)
        tab[np.argsort(W.uniform01(15 + t, room), kind="stable")[:per.sum()]] = np.repeat(np.arange(per.size), per)
        ids.append(tab.reshape(n_cur, nv[t]))
        n_cur = per.size
    first = np.cumsum((0,) + nv[:2])
    facts = [(f + np.arange(m)).astype(np.int32) for f, m in zip(first, nv)]
    fp = W.uniform01(43 + columns, 9 * sum(nv)).astype(np.float32).reshape(9, sum(nv))
    fp[::4, 20], fp[::4, 3] = fp[::4, 24], fp[::4, 9]
    fold_of_few_and_many(dol, fp, np.repeat(np.arange(3), nv).astype(np.int32), facts, ids, k, 345, helpers and columns > 32 and k < 8)


# ---------------------------------------------------------------- config 5

@pytest.mark.parametrize("batch,side,rounds", [(256, 32, 64), (33, 7, 20), (2, 3, 5)])
def test_config5_grid_reach(gp, batch, side, rounds):
    w = W.config5(batch=batch, side=side, rounds=rounds, seed=side)
    ref = OP.grid_reach_fwd_bwd(w)
    prog = gp.GridReach(w)
    prog.step()
    hist = host(prog.hist)
    assert_close(hist, ref["hist"], "reach history")
    # the clamp decisions: saturated entries agree exactly
    np.testing.assert_array_equal(hist == 1.0, ref["hist"] == 1.0)
    assert_close(host(prog.grad_p), ref["grad_p"], "reach grad")


@pytest.mark.parametrize("batch,side,rounds", [(256, 32, 64), (33, 7, 20), (2, 3, 5), (5, 4, 1), (3, 3, 0)])
def test_config5_fused_iteration(gp, dol, batch, side, rounds):
    """dol_iterate_apply2 / dol_iterate_backward: all rounds in one launch, same results as round-by-round calls."""
    w = W.config5(batch=batch, side=side, rounds=rounds, seed=side + 1)
    ref = OP.grid_reach_fwd_bwd(w)
    prog = gp.GridReachFused(w, ckpt_every=0)
    prog.step()
    hist = host(prog.hist)
    assert_close(hist, ref["hist"], "fused reach history")
    np.testing.assert_array_equal(hist == 1.0, ref["hist"] == 1.0)
    assert_close(host(prog.grad_p), ref["grad_p"], "fused reach grad")
    if rounds:
        per_round = gp.GridReach(w)
        per_round.step()
        np.testing.assert_array_equal(hist, host(per_round.hist))          # same arithmetic, bit for bit
    g0 = torch.empty((batch, side * side), device="cuda")
    dol.iterate_backward(prog.edges, prog.table, rounds, prog.hist, prog.g_out, g0, None)
    if rounds == 0:
        np.testing.assert_array_equal(host(g0), w["g"])
    with pytest.raises(dol.DolError) as ei:                                 # a table that is not square
        f = dol.FnTable.create_dense(W.sum_table(range(4), range(3)))
        dol.iterate_apply2(dol.Dist(np.arange(4), torch.ones((2, 4), device="cuda")),
                           dol.Dist(np.arange(3), torch.ones((2, 3), device="cuda")), f, 2,
                           torch.empty((3, 2, 4), device="cuda"))
    assert ei.value.status == 5


@pytest.mark.parametrize("batch,side,rounds,every", [(256, 32, 64, 8), (256, 32, 64, 16), (33, 7, 20, 6), (33, 7, 20, 1),
                                                      (2, 3, 5, 5), (2, 3, 5, 9), (5, 4, 1, 3), (3, 3, 0, 2), (7, 32, 64, 30), (9, 32, 64, 32)])
def test_config5_checkpointed_iteration(gp, dol, batch, side, rounds, every):
    """dol_iterate_apply2_ckpt / dol_iterate_backward_ckpt: only the last round and a checkpoint every `every` rounds
    leave the chip; the reverse sweep replays the rounds in between.  Same results as the oracle, and bit for bit
    those of the sweeps that keep the whole history."""
    w = W.config5(batch=batch, side=side, rounds=rounds, seed=side + 2)
    ref = OP.grid_reach_fwd_bwd(w)
    prog = gp.GridReachFused(w, ckpt_every=every)
    prog.step()
    out = host(prog.out.prob)
    assert_close(out, ref["hist"][-1], "checkpointed reach result")
    np.testing.assert_array_equal(out == 1.0, ref["hist"][-1] == 1.0)
    assert_close(host(prog.grad_p), ref["grad_p"], "checkpointed reach grad")
    n_ck = dol.iterate_ckpt_count(rounds, every)
    assert n_ck == max(0, -(-rounds // every) - 1)
    assert 1 <= dol.iterate_ckpt_every(prog.table, batch, rounds) <= max(rounds, 1)
    for x in range(n_ck):                                                   # the checkpoints are rounds of the history
        assert_close(host(prog.ckpt[x]), ref["hist"][(x + 1) * every], "checkpoint %d" % x)
    full = gp.GridReachFused(w, ckpt_every=0)
    full.step()
    np.testing.assert_array_equal(out, host(full.hist[rounds]))
    np.testing.assert_array_equal(host(prog.g_e), host(full.g_e))
    g0a, g0b = torch.empty((batch, side * side), device="cuda"), torch.empty((batch, side * side), device="cuda")
    dol.iterate_backward_ckpt(prog.r0, prog.edges, prog.table, rounds, every, prog.ckpt, prog.g_out, g0a, None)
    dol.iterate_backward(full.edges, full.table, rounds, full.hist, full.g_out, g0b, None)
    np.testing.assert_array_equal(host(g0a), host(g0b))
    with pytest.raises(dol.DolError) as ei:
        dol.iterate_apply2_ckpt(prog.r0, prog.edges, prog.table, rounds, 0, prog.out, prog.ckpt)
    assert ei.value.status == 1


@pytest.mark.parametrize("batch,side,rounds,every", [(256, 32, 64, 22), (256, 32, 64, 32), (33, 7, 20, 6), (5, 4, 1, 8), (40, 12, 30, 30), (3, 3, 7, 2),
                                                      (600, 7, 20, 6), (520, 32, 11, 8)])
def test_config5_iteration_in_one_launch(gp, dol, batch, side, rounds, every):
    """dol_iterate_apply2_backward: both sweeps in one launch (in two, issued by the one call, for batches above 512).  With an upstream gradient: bit for bit the results of
    the two separate calls.  With a target node per sample (loss = -log r[target]): against the oracle's sweeps fed
    the gradient of that loss at the oracle's own result."""
    w = W.config5(batch=batch, side=side, rounds=rounds, seed=side + 3)
    two = gp.GridReachFused(w, ckpt_every=every)
    two.step()
    one = gp.GridReachFused(w, ckpt_every=every, one_launch=True)
    assert len(one.launches) == (1 if batch <= 512 else 2)
    one.step()
    np.testing.assert_array_equal(host(one.out.prob), host(two.out.prob))
    np.testing.assert_array_equal(host(one.g_e), host(two.g_e))
    if one.ckpt is not None:
        np.testing.assert_array_equal(host(one.ckpt), host(two.ckpt))
    n = side * side
    g0a, g0b = torch.empty((batch, n), device="cuda"), torch.empty((batch, n), device="cuda")
    dol.iterate_apply2_backward(one.r0, one.edges, one.table, rounds, every, one.out, one.ckpt, None, one.g_out, g0a, None)
    dol.iterate_backward_ckpt(two.r0, two.edges, two.table, rounds, every, two.ckpt, two.g_out, g0b, None)
    np.testing.assert_array_equal(host(g0a), host(g0b))
    # a target node per sample
    ref = OP.grid_reach_fwd_bwd(w)
    near = np.array([r * side + c for r in range(side) for c in range(side) if r + c <= rounds], np.int32)   # reachable in time
    target = near[np.arange(batch) * 7 % near.size]
    r_t = ref["hist"][-1][np.arange(batch), target]
    assert (r_t > 0).all()
    g = np.zeros((batch, n), np.float32)
    g[np.arange(batch), target] = -1.0 / np.maximum(r_t, np.float32(1.17549435e-38))
    wd = {k: w[k] for k in ("side", "edge_u", "edge_v", "src", "rounds", "p")}
    wd["g"] = g
    want = OP.grid_reach_fwd_bwd(wd)["grad_p"]
    ge = torch.empty_like(one.g_e)
    dol.iterate_apply2_backward(one.r0, one.edges, one.table, rounds, every, one.out, one.ckpt, dev(target), None, None, ge)
    assert_close(host(one.out.prob), ref["hist"][-1], "one-launch reach result")
    assert_close(host(ge)[:, :w["p"].shape[1]], want, "one-launch reach grad from a target")
    for args in ((None, None), (dev(target), one.g_out)):
        with pytest.raises(dol.DolError) as ei:
            dol.iterate_apply2_backward(one.r0, one.edges, one.table, rounds, every, one.out, one.ckpt, args[0], args[1], None, ge)
        assert ei.value.status == 1


def test_iterated_apply_passes_gradient_on_the_clamp_bound(dol):
    """Two nodes, one edge, a "stay" symbol of tag 1: with p = 0.5 the second round's sum at node 1 is exactly 1 and the
    clamp passes gradient (App. A.2), d r_2[1] / d p = 2; with p = 0.75 the clamp acts (0); with 0.25 nothing clamps (2).
    The same case pins the oracle (tests/test_oracle_reach.py)."""
    tri = (np.array([0, 0, 1, 1], np.int32), np.array([0, 1, 0, 1], np.int32), np.array([1, 0, 0, 1], np.int32))
    f = dol.FnTable.create_sparse(2, 2, *tri)
    ps = np.array([0.5, 0.75, 0.25], np.float32)
    r0 = dol.Dist(np.arange(2), dev(np.tile(np.array([[1.0, 0.0]], np.float32), (3, 1))))
    e = dol.Dist(np.arange(2), dev(np.stack([ps, np.ones(3, np.float32)], axis=1)))
    g = dev(np.tile(np.array([[0.0, 1.0]], np.float32), (3, 1)))
    hist = torch.empty((3, 3, 2), device="cuda")
    dol.iterate_apply2(r0, e, f, 2, hist)
    np.testing.assert_array_equal(host(hist[2])[:, 1], np.array([1.0, 1.0, 0.5], np.float32))
    ge = torch.empty((3, 2), device="cuda")
    dol.iterate_backward(e, f, 2, hist, g, None, ge)
    np.testing.assert_array_equal(host(ge)[:, 0], np.array([2.0, 0.0, 2.0], np.float32))
    out, ge2 = dol.Dist.empty(np.arange(2), 3), torch.empty((3, 2), device="cuda")
    ck = torch.empty((1, 3, 2), device="cuda")
    dol.iterate_apply2_ckpt(r0, e, f, 2, 1, out, ck)
    dol.iterate_backward_ckpt(r0, e, f, 2, 1, ck, g, None, ge2)
    np.testing.assert_array_equal(host(ge2), host(ge))


@pytest.mark.parametrize("batch,n_nodes,n_edges,scale", [(64, 10, 16, 0.5), (130, 12, 30, 1.0), (3, 5, 4, 0.9), (70, 16, 40, 0.3)])
def test_transitive_closure_program(gp, batch, n_nodes, n_edges, scale):
    """The recursion of App. B, Fig. 9 over a random directed graph: symbol sets grow step by step, tags pile up
    towards the clamp, gradients of Distributions used twice are summed with the accumulate flags."""
    w = W.closure_workload(batch=batch, n_nodes=n_nodes, n_edges=n_edges, scale=scale, seed=n_nodes)
    w.arrays["g"] = np.abs(w["g"])         # one-signed upstream gradient: see the tolerance note in the module docstring
    ref = OP.transitive_closure_fwd_bwd(w, W.join_triples)
    prog = gp.TransitiveClosure(w, W.join_triples)
    prog.step()
    assert len(prog.rounds) == ref["rounds"]
    np.testing.assert_array_equal(prog.out.sym_ids, ref["syms"])
    assert_close(host(prog.out.prob), ref["out"], "closure tags")
    np.testing.assert_array_equal(host(prog.out.prob) == 1.0, ref["out"] == 1.0)
    assert_close(host(prog.grad_p), ref["grad_p"], "closure gradient of the edge probabilities")


@pytest.mark.parametrize("long_a,long_b", [((5, 9), (0, 1, 2)), ((5,), (0,)), ((), (0, 1, 2))])
def test_fused_iteration_with_long_rows(dol, long_a, long_b):
    """A square table in which some symbols of either operand meet more than 64 tuples: the fused sweeps sum the
    first two such rows with the whole workgroup and leave the others to single threads."""
    na, nb, B, rounds = 150, 80, 9, 5
    ti, tj, to = [], [], []
    for j in long_b:                                   # symbol j of e combines with every symbol of r
        for i in range(na):
            ti.append(i); tj.append(j); to.append((i * (2 * j + 1) + j) % na)
    for i in long_a:                                   # symbol i of r combines with every remaining symbol of e
        for j in range(3, nb):
            ti.append(i); tj.append(j); to.append((i + 3 * j) % na)
    for i in range(20, 140):                           # a few ordinary tuples
        ti.append(i); tj.append(3 + i % 70); to.append((i + 1) % na)
    order = np.lexsort((tj, ti))
    tri = tuple(np.asarray(x, np.int32)[order] for x in (ti, tj, to))
    assert np.unique(tri[2]).size == na
    r0 = (W.uniform01(1, B * na) * 0.3).astype(np.float32).reshape(B, na)
    r0[:, 7] = 1.0                                     # stays on the clamp in every round
    e = (W.uniform01(2, B * nb) * 0.02).astype(np.float32).reshape(B, nb)
    e[:, 0] = 1.0
    hist = [r0]
    for t in range(rounds):
        hist.append(oracle.damp_apply2_fwd(tri, na, nb, hist[-1], e)[1])
    g = np.abs(W.normal(3, B * na)).astype(np.float32).reshape(B, na)
    want_ge = np.zeros((B, nb), np.float64)
    gr = g
    for t in reversed(range(rounds)):
        gr, ge = oracle.damp_apply2_bwd(tri, na, nb, hist[t], e, gr)
        want_ge += ge
    f = dol.FnTable.create_sparse(na, nb, *tri)
    d0, de = dol.Dist(np.arange(na), dev(r0)), dol.Dist(np.arange(nb), dev(e))
    dh = torch.empty((rounds + 1, B, na), device="cuda")
    dol.iterate_apply2(d0, de, f, rounds, dh)
    got = host(dh)
    assert_close(got, np.stack(hist), "iterated apply")
    np.testing.assert_array_equal(got == 1.0, np.stack(hist) == 1.0)
    g0, ge = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.iterate_backward(de, f, rounds, dh, dev(g), g0, ge)
    assert_close(host(g0), gr, "iterated apply: gradient of r0")
    assert_close(host(ge), want_ge, "iterated apply: gradient of e")
    # the shares of d loss / d e meet in a fixed order: a second run and the checkpointed sweeps give the same bits
    g0b, geb = torch.empty_like(g0), torch.empty_like(ge)
    dol.iterate_backward(de, f, rounds, dh, dev(g), g0b, geb)
    np.testing.assert_array_equal(host(ge), host(geb))
    np.testing.assert_array_equal(host(g0), host(g0b))
    for every in (2, 3, 7):
        out = dol.Dist.empty(np.arange(na), B)
        n_ck = dol.iterate_ckpt_count(rounds, every)
        ck = torch.empty((n_ck, B, na), device="cuda") if n_ck else None
        dol.iterate_apply2_ckpt(d0, de, f, rounds, every, out, ck)
        np.testing.assert_array_equal(host(out.prob), got[-1])
        g0c, gec = torch.empty_like(g0), torch.empty_like(ge)
        dol.iterate_backward_ckpt(d0, de, f, rounds, every, ck, dev(g), g0c, gec)
        np.testing.assert_array_equal(host(gec), host(ge))
        np.testing.assert_array_equal(host(g0c), host(g0))


@pytest.mark.parametrize("B,na", [(5, 300), (5, 700), (520, 700)])
def test_fused_iteration_with_six_tuples_per_symbol(dol, B, na):
    """Every column and every row of the table holds six tuples: the builds that keep six tuples in registers, without
    tail loops, in each launch shape (one symbol per thread; 1024 threads; two symbols per thread for the larger
    batch, whose combined call issues its two sweeps as two launches)."""
    nb, rounds, every = 40, 10, 4
    i = np.repeat(np.arange(na, dtype=np.int32), 6)
    d = np.tile(np.arange(6, dtype=np.int32), na)
    ti, tj, to = i, (i + 5 * d) % nb, (i + np.array([0, 1, 7, 31, 100, 211], np.int32)[d]) % na
    order = np.lexsort((tj, ti))
    tri = tuple(x[order].astype(np.int32) for x in (ti, tj, to))
    assert np.bincount(tri[2], minlength=na).max() == 6 and np.bincount(tri[0]).max() == 6
    r0 = (W.uniform01(1, B * na) * 0.5).astype(np.float32).reshape(B, na)
    r0[:, 3] = 1.0
    e = (W.uniform01(2, B * nb) * 0.45).astype(np.float32).reshape(B, nb)
    hist = [r0]
    for t in range(rounds):
        hist.append(oracle.damp_apply2_fwd(tri, na, nb, hist[-1], e)[1])
    assert (hist[-1] == 1.0).any() and (hist[-1] < 1.0).any()
    g = np.abs(W.normal(3, B * na)).astype(np.float32).reshape(B, na)
    want_ge, gr = np.zeros((B, nb), np.float64), g
    for t in reversed(range(rounds)):
        gr, ge = oracle.damp_apply2_bwd(tri, na, nb, hist[t], e, gr)
        want_ge += ge
    f = dol.FnTable.create_sparse(na, nb, *tri)
    d0, de = dol.Dist(np.arange(na), dev(r0)), dol.Dist(np.arange(nb), dev(e))
    n_ck = dol.iterate_ckpt_count(rounds, every)
    out, ck = dol.Dist.empty(np.arange(na), B), torch.empty((n_ck, B, na), device="cuda")
    g0, ge = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.iterate_apply2_ckpt(d0, de, f, rounds, every, out, ck)
    dol.iterate_backward_ckpt(d0, de, f, rounds, every, ck, dev(g), g0, ge)
    assert_close(host(out.prob), hist[-1], "six tuples: result")
    np.testing.assert_array_equal(host(out.prob) == 1.0, hist[-1] == 1.0)
    assert_close(host(g0), gr, "six tuples: gradient of r0")
    assert_close(host(ge), want_ge, "six tuples: gradient of e")
    out2, ck2 = dol.Dist.empty(np.arange(na), B), torch.empty_like(ck)
    g0b, geb = torch.empty_like(g0), torch.empty_like(ge)
    dol.iterate_apply2_backward(d0, de, f, rounds, every, out2, ck2, None, dev(g), g0b, geb)
    for a, b in ((out2.prob, out.prob), (ck2, ck), (g0b, g0), (geb, ge)):
        np.testing.assert_array_equal(host(a), host(b))


@pytest.mark.parametrize("B,w,h", [(3, 2, 2), (3, 64, 2), (2, 33, 31), (5, 5, 40), (2, 2, 512), (300, 7, 9), (800, 22, 22), (600, 32, 3),
                                   (1030, 9, 17), (2, 64, 32), (2, 65, 3)])
def test_fused_iteration_over_a_grid(dol, B, w, h):
    """Tables of a full w x h grid with a "stay" tuple per node: strips of one, two and four nodes, bands that fill a wavefront
    and bands that do not, last strips of one node, samples beside each other on a unit; symbols of e with one tuple, a few,
    more than four and more than a wavefront."""
    na, rounds, every = w * h, 9, 4
    x, y = np.arange(na) % w, np.arange(na) // w
    ti, tj, to, nb = [np.arange(na)], [np.zeros(na, np.int64)], [np.arange(na)], 1
    for dx, dy, share in ((1, 0, na), (-1, 0, 7), (0, 1, 3), (0, -1, 1)):       # so many nodes share a symbol of e
        ok = (x + dx >= 0) & (x + dx < w) & (y + dy >= 0) & (y + dy < h)
        ti.append(np.arange(na)[ok])
        to.append(np.arange(na)[ok] + dx + w * dy)
        tj.append(nb + (np.arange(na)[ok] * 5) // share % (na // share + 1))
        nb = int(tj[-1].max()) + 2
    ti, tj, to = (np.concatenate(v) for v in (ti, tj, to))
    order = np.lexsort((tj, ti))
    tri = tuple(np.asarray(v, np.int32)[order] for v in (ti, tj, to))
    r0 = (W.uniform01(1, B * na) * 0.9).astype(np.float32).reshape(B, na)
    r0[:, 1] = 1.0
    e = (W.uniform01(2, B * nb) * 0.45).astype(np.float32).reshape(B, nb)
    n_ref = min(B, 4)
    hist = [r0[-n_ref:]]
    for t in range(rounds):
        hist.append(oracle.damp_apply2_fwd(tri, na, nb, hist[-1], e[-n_ref:])[1])
    g = np.abs(W.normal(3, B * na)).astype(np.float32).reshape(B, na)
    want_ge, gr = np.zeros((n_ref, nb), np.float64), g[-n_ref:]
    for t in reversed(range(rounds)):
        gr, ge = oracle.damp_apply2_bwd(tri, na, nb, hist[t], e[-n_ref:], gr)
        want_ge += ge
    f = dol.FnTable.create_sparse(na, nb, *tri)
    d0, de = dol.Dist(np.arange(na), dev(r0)), dol.Dist(np.arange(nb), dev(e))
    dh = torch.empty((rounds + 1, B, na), device="cuda")
    dol.iterate_apply2(d0, de, f, rounds, dh)
    step = dol.Dist(np.arange(na), dev(r0))
    for t in range(rounds):                            # the rounds are those of as many calls, bit for bit
        nxt = dol.Dist.empty(np.arange(na), B)
        dol.apply2(step, de, f, None, nxt)
        torch.testing.assert_close(dh[t + 1], nxt.prob, rtol=0, atol=0)
        step = nxt
    g0, ge = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.iterate_backward(de, f, rounds, dh, dev(g), g0, ge)
    assert_close(host(g0)[-n_ref:], gr, "grid: gradient of r0")
    assert_close(host(ge)[-n_ref:], want_ge, "grid: gradient of e")
    n_ck = dol.iterate_ckpt_count(rounds, every)
    out, ck = dol.Dist.empty(np.arange(na), B), torch.empty((n_ck, B, na), device="cuda")
    g0b, geb = torch.empty_like(g0), torch.empty_like(ge)
    dol.iterate_apply2_ckpt(d0, de, f, rounds, every, out, ck)
    dol.iterate_backward_ckpt(d0, de, f, rounds, every, ck, dev(g), g0b, geb)
    out2, ck2, g0c, gec = dol.Dist.empty(np.arange(na), B), torch.empty_like(ck), torch.empty_like(g0), torch.empty_like(ge)
    dol.iterate_apply2_backward(d0, de, f, rounds, every, out2, ck2, None, dev(g), g0c, gec)
    for a, b in ((out.prob, dh[-1]), (ck[0], dh[every]), (g0b, g0), (geb, ge), (out2.prob, out.prob), (ck2, ck), (g0c, g0), (gec, ge)):
        torch.testing.assert_close(a, b, rtol=0, atol=0)


@pytest.mark.parametrize("w,h,every,rounds", [(32, 32, 33, 34), (32, 32, 33, 66), (32, 32, 32, 71), (32, 32, 1, 3), (8, 8, 68, 69), (8, 8, 67, 140),
                                              (64, 20, 17, 34), (64, 20, 16, 23), (8, 8, 4, 10), (8, 8, 9, 20), (16, 16, 24, 41)])
def test_both_sweeps_with_a_segment_in_registers(dol, w, h, every, rounds):
    """dol_iterate_apply2_backward of a small batch, whose last segment but one waits in registers: segments of as many rounds as
    fit there and fewer, of odd and even counts, a last segment of one round, segments before them; strips of one, two and four
    nodes.  Bit for bit what the two calls give."""
    na, B = w * h, 3
    x, y = np.arange(na) % w, np.arange(na) // w
    ti, tj = [np.arange(na)], [np.zeros(na, np.int64)]
    to = [np.arange(na)]
    for d, (dx, dy) in enumerate(((1, 0), (-1, 0), (0, 1), (0, -1))):
        ok = (x + dx >= 0) & (x + dx < w) & (y + dy >= 0) & (y + dy < h)
        ti.append(np.arange(na)[ok]), to.append(np.arange(na)[ok] + dx + w * dy), tj.append(np.full(ok.sum(), d + 1))
    ti, tj, to = (np.concatenate(v) for v in (ti, tj, to))
    order = np.lexsort((tj, ti))
    f = dol.FnTable.create_sparse(na, 5, *(np.asarray(v, np.int32)[order] for v in (ti, tj, to)))
    d0 = dol.Dist(np.arange(na), dev((W.uniform01(1, B * na) * 0.9).astype(np.float32).reshape(B, na)))
    de = dol.Dist(np.arange(5), dev((W.uniform01(2, B * 5) * 0.3).astype(np.float32).reshape(B, 5)))
    g = dev(W.normal(3, B * na).astype(np.float32).reshape(B, na))
    ck = torch.empty((dol.iterate_ckpt_count(rounds, every), B, na), device="cuda")
    got = []
    for one_call in (False, True):
        out, g0, ge = dol.Dist.empty(np.arange(na), B), torch.empty((B, na), device="cuda"), torch.empty((B, 5), device="cuda")
        ck.fill_(7.0)
        if one_call:
            dol.iterate_apply2_backward(d0, de, f, rounds, every, out, ck, None, g, g0, ge)
        else:
            dol.iterate_apply2_ckpt(d0, de, f, rounds, every, out, ck)
            dol.iterate_backward_ckpt(d0, de, f, rounds, every, ck, g, g0, ge)
        got.append([host(t) for t in (out.prob, ck, g0, ge)])
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("side,rounds,every,batch,want", [
    (32, 64, 32, 256, "damp_iterate_grid_fwd_bwd_kept_kernel"), (32, 64, 32, 257, "damp_iterate_grid_fwd_bwd_kernel"),
    (24, 100, 34, 20, "damp_iterate_grid_fwd_bwd_kept_kernel"), (24, 100, 50, 20, "damp_iterate_grid_fwd_bwd_kernel"),      # 34 rounds fit the registers
    (8, 10, 10, 20, "damp_iterate_grid_fwd_bwd_kernel")])                                                                    # one segment
def test_programs_name_the_kernel_of_both_sweeps(gp, dol, side, rounds, every, batch, want):
    """The launch of a reachability program carries the name of the kernel that the library runs for its sizes."""
    prog = gp.GridReachFused(W.config5(batch=batch, side=side, rounds=rounds, seed=5), ckpt_every=every, one_launch=True)
    assert [l.kernel for l in prog.launches] == [want] == [dol.iterate_kernel(prog.table, batch, rounds, every)]


def test_fused_iteration_with_more_than_1024_symbols(dol):
    """Four symbols of the first operand per thread (the widest build of the fused sweeps)."""
    na, nb, B, rounds = 1100, 40, 3, 4
    i = np.arange(na, dtype=np.int32)
    ti = np.concatenate([i, i]); tj = np.concatenate([np.zeros(na, np.int32), 1 + i % 39])
    to = np.concatenate([i, (i * 7 + 3) % na]).astype(np.int32)
    order = np.lexsort((tj, ti))
    tri = tuple(x[order].astype(np.int32) for x in (ti, tj, to))
    r0 = (W.uniform01(1, B * na) * 0.3).astype(np.float32).reshape(B, na)
    r0[:, 11] = 1.0
    e = (W.uniform01(2, B * nb) * 0.3).astype(np.float32).reshape(B, nb)
    e[:, 0] = 1.0
    hist = [r0]
    for t in range(rounds):
        hist.append(oracle.damp_apply2_fwd(tri, na, nb, hist[-1], e)[1])
    g = np.abs(W.normal(3, B * na)).astype(np.float32).reshape(B, na)
    want_ge, gr = np.zeros((B, nb), np.float64), g
    for t in reversed(range(rounds)):
        gr, ge = oracle.damp_apply2_bwd(tri, na, nb, hist[t], e, gr)
        want_ge += ge
    f = dol.FnTable.create_sparse(na, nb, *tri)
    d0, de = dol.Dist(np.arange(na), dev(r0)), dol.Dist(np.arange(nb), dev(e))
    dh = torch.empty((rounds + 1, B, na), device="cuda")
    dol.iterate_apply2(d0, de, f, rounds, dh)
    got = host(dh)
    assert_close(got, np.stack(hist), "iterated apply, 1100 symbols")
    np.testing.assert_array_equal(got == 1.0, np.stack(hist) == 1.0)
    g0, ge = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.iterate_backward(de, f, rounds, dh, dev(g), g0, ge)
    assert_close(host(g0), gr, "iterated apply, 1100 symbols: gradient of r0")
    assert_close(host(ge), want_ge, "iterated apply, 1100 symbols: gradient of e")
    out = dol.Dist.empty(np.arange(na), B)
    ck = torch.empty((1, B, na), device="cuda")
    dol.iterate_apply2_ckpt(d0, de, f, rounds, 2, out, ck)
    np.testing.assert_array_equal(host(out.prob), got[-1])
    g0c, gec = torch.empty_like(g0), torch.empty_like(ge)
    dol.iterate_backward_ckpt(d0, de, f, rounds, 2, ck, dev(g), g0c, gec)
    np.testing.assert_array_equal(host(gec), host(ge))
    np.testing.assert_array_equal(host(g0c), host(g0))


def test_backward_of_tables_with_long_rows(dol):
    """A table whose rows hold hundreds of tuples (one symbol of b combines with every symbol of a)."""
    na, B = 300, 20
    i = np.arange(na, dtype=np.int32)
    tri = (np.concatenate([i, i]), np.concatenate([np.zeros(na, np.int32), np.ones(na, np.int32)]),
           np.concatenate([i % 7, 7 + i % 5]))
    order = np.lexsort((tri[1], tri[0]))
    tri = tuple(x[order].astype(np.int32) for x in tri)
    a = W.softmax_rows(W.normal(1, B * na).reshape(B, na))
    b = (W.uniform01(2, B * 2)).astype(np.float32).reshape(B, 2)
    syms, want = oracle.damp_apply2_fwd(tri, na, 2, a, b)
    f = dol.FnTable.create_sparse(na, 2, *tri)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(2), dev(b))
    do = dol.Dist.empty(syms, B)
    dol.apply2(da, db, f, None, do)
    assert_close(host(do.prob), want, "long-row apply")
    g = np.abs(W.normal(3, B * syms.size)).astype(np.float32).reshape(B, -1)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f), dev(g), ga, gb)
    wa, wb = oracle.damp_apply2_bwd(tri, na, 2, a, b, g)
    assert_close(host(ga), wa, "long-row bwd a")
    assert_close(host(gb), wb, "long-row bwd b")


# ---------------------------------------------------------------- operators on their own: edge cases

def test_apply_with_rejected_tuples_and_padding(dol):
    na, nb, B = 9, 6, 70
    tab = W.hashed_table(3, na, nb, 11)
    tab[0, :] = -1                     # symbol 0 of a never admitted
    tab[4, 2] = -1
    a = W.softmax_rows(W.normal(1, B * na).reshape(B, na))
    b = W.softmax_rows(W.normal(2, B * nb).reshape(B, nb))
    tri = oracle.dense_to_triples(tab)
    syms, want = oracle.damp_apply2_fwd(tri, na, nb, a, b)
    f = dol.FnTable.create_dense(tab)
    np.testing.assert_array_equal(f.out_syms, syms)
    # padded leading dimensions on every tensor
    ta = torch.zeros((B, na + 3), device="cuda"); ta[:, :na] = dev(a)
    tb = torch.zeros((B, nb + 5), device="cuda"); tb[:, :nb] = dev(b)
    to = torch.full((B, f.n_out + 2), -7.0, device="cuda")
    da, db, do = dol.Dist(np.arange(na), ta[:, :na]), dol.Dist(np.arange(nb), tb[:, :nb]), dol.Dist(syms, to[:, :f.n_out])
    assert da.ld == na + 3 and do.ld == f.n_out + 2
    dol.apply2(da, db, f, None, do)
    assert_close(host(to)[:, :f.n_out], want, "apply padded")
    assert np.all(host(to)[:, f.n_out:] == -7.0)          # padding untouched
    g = W.normal(9, B * f.n_out).astype(np.float32).reshape(B, -1)
    tg = torch.zeros((B, f.n_out + 2), device="cuda"); tg[:, :f.n_out] = dev(g)
    ga = torch.full((B, na + 3), 5.0, device="cuda")
    gb = torch.full((B, nb + 5), 5.0, device="cuda")
    rec = dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f)
    dol.backward(rec, tg, ga, gb)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    assert_close(host(ga)[:, :na], wa, "bwd a padded")
    assert_close(host(gb)[:, :nb], wb, "bwd b padded")
    assert np.all(host(ga)[:, 0] == 0) and np.all(host(ga)[:, na:] == 5.0) and np.all(host(gb)[:, nb:] == 5.0)
    # accumulate flags add to what is there
    rec2 = dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f, accumulate=3)
    dol.backward(rec2, tg, ga, gb)
    assert_close(host(ga)[:, :na], 2 * wa.astype(np.float64), "bwd a accumulated")
    assert_close(host(gb)[:, :nb], 2 * wb.astype(np.float64), "bwd b accumulated")


def test_clamp_decisions_match_oracle(dol):
    """Tags large enough that many columns exceed 1: values clamp, gradients gate, decisions agree bit for bit."""
    na, nb, B = 12, 12, 200
    tab = W.hashed_table(5, na, nb, 6)
    a = (W.uniform01(1, B * na) * 0.4).astype(np.float32).reshape(B, na)
    b = (W.uniform01(2, B * nb) * 0.4).astype(np.float32).reshape(B, nb)
    # exact boundary cases: rows 0..2 make column sums of exactly 0.875, 1.0, 1.125
    for r, tot in enumerate((0.875, 1.0, 1.125)):
        a[r] = 0; b[r] = 0
        a[r, 0] = 1.0; b[r, 0] = tot
    tri = oracle.dense_to_triples(tab)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    assert 0.2 < (pre32 > 1).mean() < 0.8
    f = dol.FnTable.create_dense(tab)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    do = dol.Dist.empty(syms, B)
    dol.apply2(da, db, f, None, do)
    got = host(do.prob)
    assert_close(got, want, "clamped apply")
    np.testing.assert_array_equal(got == 1.0, pre32 >= 1.0)
    g = W.normal(3, B * syms.size).astype(np.float32).reshape(B, -1)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f), dev(g), ga, gb)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    assert_close(host(ga), wa, "gated bwd a")
    assert_close(host(gb), wb, "gated bwd b")


@pytest.mark.parametrize("na,nb,n_out,B,scale", [(12, 12, 8, 200, 0.4), (64, 64, 256, 130, 0.7), (128, 4, 16, 64, 0.25),
                                                  (16, 128, 100, 257, 0.2), (4, 4, 4, 4160, 1.0), (64, 64, 256, 64, 0.05)])
def test_hashed_tables_in_lds_with_clamping(dol, na, nb, n_out, B, scale):
    """Hashed tables whose sizes are multiples of four (whole tiles of 64 samples go through the LDS kernels, the
    remainder through the direct ones), some tuples rejected, tags scaled so that columns land on both sides of
    the clamp (the last case: all far below it); rows 0..2 hit 0.875 / 1.0 / 1.125 exactly."""
    tab = W.hashed_table(7, na, nb, n_out)
    tab[1, :] = -1
    tab[na - 1, nb // 2] = -1
    a = (W.uniform01(1, B * na) * scale).astype(np.float32).reshape(B, na)
    b = (W.uniform01(2, B * nb) * scale).astype(np.float32).reshape(B, nb)
    for r, tot in enumerate((0.875, 1.0, 1.125)):
        a[r] = 0; b[r] = 0
        a[r, 0] = 1.0; b[r, 0] = tot
    tri = oracle.dense_to_triples(tab)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    f = dol.FnTable.create_dense(tab)
    if syms.size % 4 == 0:                 # operand rows that fit in registers: code written for the table; else LDS gathers
        kind = "table" if max(na, nb) <= 64 else "lds"
        assert f.kernel_fwd == "damp_%s_fwd_kernel" % kind and f.kernel_bwd == "damp_%s_bwd_kernel" % kind
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    do = dol.Dist.empty(syms, B)
    dol.apply2(da, db, f, None, do)
    got = host(do.prob)
    assert_close(got, want, "lds apply")
    np.testing.assert_array_equal(got == 1.0, pre32 >= 1.0)
    g = np.abs(W.normal(3, B * syms.size)).astype(np.float32).reshape(B, -1)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f), dev(g), ga, gb)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    assert_close(host(ga), wa, "lds bwd a")
    assert_close(host(gb), wb, "lds bwd b")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f, accumulate=3), dev(g), ga, gb)
    assert_close(host(ga), 2.0 * wa.astype(np.float64), "lds bwd a accumulated")
    assert_close(host(gb), 2.0 * wb.astype(np.float64), "lds bwd b accumulated")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f, accumulate=1), dev(g), ga, None)     # one side only
    assert_close(host(ga), 3.0 * wa.astype(np.float64), "lds bwd a alone")


@pytest.mark.parametrize("na,nb,B", [(127, 10, 300), (10, 10, 65), (1, 3, 70), (200, 16, 130), (5, 7, 64), (70, 1, 33),
                                      (9, 17, 40), (64, 4, 129), (300, 10, 50), (257, 2, 9), (256, 16, 5)])
def test_sum_tables_with_clamping(dol, na, nb, B):
    """Sum-shaped tables of every supported width, with unnormalised tags so that many columns exceed 1 and the
    backward pass has to re-derive the clamp decisions; rows 0..2 hit 0.875 / 1.0 / 1.125 exactly."""
    check_sum_table(dol, na, nb, B)


@pytest.mark.parametrize("na,nb,B", [(127, 10, 16384 + 37), (19, 10, 16384), (17, 16, 20001), (192, 16, 16385), (64, 4, 16401),
                                      (70, 1, 16390), (100, 8, 16384 + 63), (37, 3, 16387), (118, 10, 32768), (10, 10, 16389),
                                      (3, 16, 16400), (1, 1, 16385), (16, 2, 16384), (127, 10, 40005), (30, 10, 70001)])
def test_sum_tables_at_batches_that_fill_the_chip(dol, na, nb, B):
    """The same at batches where a lane owns a sample and a workgroup a tile of 64: whole tiles and a ragged last
    one, tiles that must re-derive the clamp decisions and (the second half of the batch) tiles that need not."""
    check_sum_table(dol, na, nb, B, calm_from=B // 2, kernel="rows")


def check_sum_table(dol, na, nb, B, calm_from=None, kernel=None):
    tab = W.sum_table(range(na), range(nb))
    x = min(1.0, 2.2 / np.sqrt(min(na, nb)))        # column sums of min(na, nb) terms scatter around 1
    a = (W.uniform01(na, B * na) * x).astype(np.float32).reshape(B, na)
    b = (W.uniform01(nb + 100, B * nb) * x).astype(np.float32).reshape(B, nb)
    for r, tot in enumerate((0.875, 1.0, 1.125)):
        a[r] = 0; b[r] = 0
        a[r, na - 1] = 1.0; b[r, 0] = tot
    a[3] *= 0.01                       # a sample far below the clamp takes the shortcut
    if calm_from is not None:
        a[calm_from:] *= 0.01
    tri = oracle.dense_to_triples(tab)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    f = dol.FnTable.create_dense(tab)
    if kernel:
        assert f.kernel_at(False, B).startswith("damp_conv_fwd_%s_kernel" % (kernel if na > 16 else "small")), f.kernel_at(False, B)
        assert f.kernel_at(True, B).startswith("damp_conv_bwd_%s_kernel" % kernel), f.kernel_at(True, B)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    do = dol.Dist.empty(syms, B)
    dol.apply2(da, db, f, None, do)
    got = host(do.prob)
    assert_close(got, want, "sum apply")
    np.testing.assert_array_equal(got == 1.0, pre32 >= 1.0)
    # one-signed upstream gradient: with tags of order 1 a float32 sum of mixed-sign terms cannot meet an
    # absolute 1e-7 where it cancels to ~0, whatever the kernel; the clamp decisions are what is under test here
    g = np.abs(W.normal(3, B * syms.size)).astype(np.float32).reshape(B, -1)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f), dev(g), ga, gb)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    assert_close(host(ga), wa, "sum bwd a")
    assert_close(host(gb), wb, "sum bwd b")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f, accumulate=3), dev(g), ga, gb)
    assert_close(host(ga), 2.0 * wa.astype(np.float64), "sum bwd a accumulated")
    assert_close(host(gb), 2.0 * wb.astype(np.float64), "sum bwd b accumulated")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f), dev(g), None, gb)      # one side only
    assert_close(host(gb), wb, "sum bwd b alone")


@pytest.mark.parametrize("B", [3, 70])
def test_tuple_list_backward_with_the_gradient_row_staged(dol, B):
    """A sparse table of 700 x 600 symbols onto 400 with a long row in either operand, tags large enough to put many
    results on the clamp: dol_backward through the kernel that works out the gated gradient row once per sample, with
    accumulation, one-sided calls and the decisions on the clamp compared with the oracle's."""
    na, nb, S = 700, 600, 400
    ti, tj, to = [], [], []
    for i in range(na):                                 # a few tuples per symbol of a
        for d in range(3):
            ti.append(i); tj.append((i * 7 + d * 131) % (nb - 1) + 1); to.append((i * 3 + d * 17) % S)
    for j in range(1, nb):                              # row 5 of a meets every symbol of b, symbol 0 of b every symbol of a
        ti.append(5); tj.append(j); to.append((j * 11) % S)
    for i in range(na):
        ti.append(i); tj.append(0); to.append((i * 13 + 1) % S)
    keys = sorted(set(zip(ti, tj)))
    first = {}
    for i, j, o in zip(ti, tj, to):
        first.setdefault((i, j), o)
    tri = tuple(np.asarray(x, np.int32) for x in ([k[0] for k in keys], [k[1] for k in keys], [first[k] for k in keys]))
    a = (W.uniform01(1, B * na) * 0.9).astype(np.float32).reshape(B, na)
    b = (W.uniform01(2, B * nb) * 0.5).astype(np.float32).reshape(B, nb)
    b[:, 0] = 1.0
    f = dol.FnTable.create_sparse(na, nb, *tri)
    assert f.kernel_bwd == "damp_apply2_bwd_staged_kernel", f.kernel_bwd
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    assert (pre32 > 1.0).mean() > 0.1 and (pre32 <= 1.0).mean() > 0.1
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    do = dol.Dist.empty(syms, B)
    dol.apply2(da, db, f, None, do)
    np.testing.assert_array_equal(host(do.prob) == 1.0, pre32 >= 1.0)
    g = np.abs(W.normal(3, B * syms.size)).astype(np.float32).reshape(B, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    rec = dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f)
    dol.backward(rec, dev(g), ga, gb)
    assert_close(host(ga), wa, "staged bwd a")
    assert_close(host(gb), wb, "staged bwd b")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, do, f=f, accumulate=3), dev(g), ga, gb)
    assert_close(host(ga), 2.0 * wa.astype(np.float64), "staged bwd a accumulated")
    assert_close(host(gb), 2.0 * wb.astype(np.float64), "staged bwd b accumulated")
    ga2, gb2 = torch.empty_like(ga), torch.empty_like(gb)
    dol.backward(rec, dev(g), ga2, None)
    dol.backward(rec, dev(g), None, gb2)
    ga3, gb3 = torch.empty_like(ga), torch.empty_like(gb)
    dol.backward(rec, dev(g), ga3, gb3)
    np.testing.assert_array_equal(host(ga2), host(ga3))            # a fixed summation order: the same bits on every run
    np.testing.assert_array_equal(host(gb2), host(gb3))


def test_union_and_filter_edge_cases(dol):
    B = 50
    sa, sb = np.array([1, 4, 6, 8, 9], np.int32), np.array([0, 4, 9, 12], np.int32)
    a = (W.uniform01(4, B * 5) * 0.9).astype(np.float32).reshape(B, 5)
    b = (W.uniform01(5, B * 4) * 0.9).astype(np.float32).reshape(B, 4)
    a[0, 1], b[0, 1] = 0.5, 0.5          # a+b == 1 exactly: passes gradient
    a[1, 1], b[1, 1] = 0.75, 0.5         # clamps
    da, db = dol.Dist(sa, dev(a)), dol.Dist(sb, dev(b))
    syms = dol.union_plan(da, db)
    want_syms, ia, ib = oracle.union_plan(sa, sb)
    np.testing.assert_array_equal(syms, want_syms)
    do = dol.Dist.empty(syms, B)
    dol.union(da, db, None, do)
    assert_close(host(do.prob), oracle.damp_union_fwd(ia, ib, a, b), "union")
    g = W.normal(6, B * syms.size).astype(np.float32).reshape(B, -1)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    dol.backward(dol.OpRecord(dol.OP_UNION, da, db, do), dev(g), ga, gb)
    wa, wb = oracle.damp_union_bwd(ia, ib, a, b, g)
    np.testing.assert_array_equal(host(ga), wa)
    np.testing.assert_array_equal(host(gb), wb)
    # union with an empty Distribution is the identity
    de = dol.Dist(np.empty(0, np.int32), torch.empty((B, 0), device="cuda"))
    d2 = dol.Dist.empty(dol.union_plan(da, de), B)
    dol.union(da, de, None, d2)
    np.testing.assert_array_equal(host(d2.prob), a)
    # filter: all kept = identity, none kept = empty result, and the transpose
    d3 = dol.Dist.empty(sa, B)
    dol.filter(da, np.ones(5, np.uint8), None, d3)
    np.testing.assert_array_equal(host(d3.prob), a)
    assert dol.filter_plan(da, np.zeros(5, np.uint8)).size == 0
    d4 = dol.Dist(np.empty(0, np.int32), torch.empty((B, 0), device="cuda"))
    dol.filter(da, np.zeros(5, np.uint8), None, d4)
    pred = np.array([1, 0, 0, 1, 1], np.uint8)
    d5 = dol.Dist.empty(dol.filter_plan(da, pred), B)
    dol.filter(da, pred, None, d5)
    np.testing.assert_array_equal(host(d5.prob), oracle.damp_filter_fwd(pred, a))
    g5 = W.normal(7, B * 3).astype(np.float32).reshape(B, 3)
    gi = torch.full((B, 5), 9.0, device="cuda")
    dol.backward(dol.OpRecord(dol.OP_FILTER, da, None, d5, pred_mask=pred), dev(g5), gi, None)
    np.testing.assert_array_equal(host(gi), oracle.damp_filter_bwd(pred, g5))


def test_empty_batch_and_errors(dol):
    f = dol.FnTable.create_dense(W.sum_table(range(3), range(3)))
    e3 = dol.Dist(np.arange(3), torch.empty((0, 3), device="cuda"))
    e5 = dol.Dist(f.out_syms, torch.empty((0, 5), device="cuda"))
    dol.apply2(e3, e3, f, None, e5)                       # batch 0 is legal
    a = dol.Dist(np.arange(3), torch.ones((2, 3), device="cuda"))
    wrong = dol.Dist(np.arange(4), torch.ones((2, 4), device="cuda"))
    out = dol.Dist.empty(f.out_syms, 2)
    out.prob.fill_(-3.0)
    with pytest.raises(dol.DolError) as ei:
        dol.apply2(a, wrong, f, None, out)
    assert ei.value.status == 2 and "table" in str(ei.value)
    assert np.all(host(out.prob) == -3.0)                  # outputs untouched on error
    with pytest.raises(dol.DolError) as ei:
        dol.FnTable.create_sparse(2, 2, [0, 0], [1, 1], [5, 6])       # a function has one value per tuple
    assert ei.value.status == 1
    with pytest.raises(dol.DolError) as ei:
        dol.FnTable.create_sparse(2, 2, [0, 2], [1, 1], [5, 6])       # index outside the operand
    assert ei.value.status == 2
    none = dol.FnTable.create_dense(np.full((3, 3), -1, np.int32))     # nothing admitted: empty result, zero gradients
    assert none.n_out == 0
    o0 = dol.Dist(np.empty(0, np.int32), torch.empty((2, 0), device="cuda"))
    dol.apply2(a, a, none, None, o0)
    ga = torch.full((2, 3), 4.0, device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, a, a, o0, f=none), torch.empty((2, 0), device="cuda"), ga, None)
    assert np.all(host(ga) == 0)
    prov = dol.Prov(dol.DTKP, 3, torch.ones((2, 4), device="cuda"), None)
    with pytest.raises(dol.DolError) as ei:
        dol.backward(dol.OpRecord(dol.OP_APPLY2, a, a, out, f=f, prov=prov), out.prob, ga, None)
    assert ei.value.status == 5


@pytest.mark.parametrize("n", [1, 5, 1000])
def test_results_under_other_symbols_are_refused(dol, n):
    """out.sym_ids are compared with what the table produces, to the last one, whichever call makes the result; without any they pass."""
    f = dol.FnTable.create_dense(3 * np.arange(n, dtype=np.int32)[:, None])
    a, one = dol.Dist(np.arange(n), torch.full((2, n), 0.5, device="cuda")), dol.Dist(np.arange(1), torch.ones((2, 1), device="cuda"))
    prov = dol.Prov(dol.DTKP, 2, torch.full((2, 3), 0.5, device="cuda"), None)
    pa = dol.Dist.empty(np.arange(n), 2, k=2)
    dol.dtkp_init(pa, np.zeros(n, np.int32), prov)
    calls = (lambda out: dol.apply2(a, one, f, None, out), lambda out: dol.dtkp_apply2_input(pa, np.array([1], np.int32), f, prov, out))
    for call in calls:
        call(dol.Dist.empty(f.out_syms, 2, k=2))
        for at in {0, n // 2, n - 1}:
            ids = f.out_syms.copy()
            ids[at] += 1
            out = dol.Dist.empty(ids, 2, k=2)
            out.prob.fill_(-3.0)
            with pytest.raises(dol.DolError) as ei:
                call(out)
            assert ei.value.status == 1 and "out.sym_ids[%d] = %d, the table produces %d" % (at, ids[at], f.out_syms[at]) in str(ei.value)
            assert np.all(host(out.prob) == -3.0)
        out = dol.Dist.empty(f.out_syms, 2, k=2)
        out.c.sym_ids = None
        call(out)


def test_dtkp_general_conjunction_union_filter(dol):
    """k x k conjunction with overlapping fact sets, exclusion groups, then union and filter under DTKP."""
    B, k, n_facts = 40, 3, 12
    fp = W.uniform01(11, B * n_facts).astype(np.float32).reshape(B, n_facts)
    grp = np.array([0, 0, 0, 1, 1, 1, 2, 3, 4, 5, 6, 7], np.int32)
    d_fp = dev(fp)
    prov = dol.Prov(dol.DTKP, k, d_fp, grp)
    # two stages of apply so that the second sees multi-proof tags on both sides
    s0, s1 = np.arange(3, dtype=np.int32), np.arange(3, dtype=np.int32)
    tabs = [W.hashed_table(21, 3, 3, 4), W.hashed_table(22, 3, 3, 4)]
    facts = [[0, 1, 6], [3, 4, 7], [2, 8, 9], [5, 10, 11]]
    o_m = [oracle.dtkp_init(f, fp, k) for f in facts]
    g_d = []
    for f in facts:
        d = dol.Dist.empty(np.arange(3), B, k=k)
        dol.dtkp_init(d, f, prov)
        g_d.append(d)
    for x in range(4):
        np.testing.assert_array_equal(host(g_d[x].proof_mask).view(np.uint64), o_m[x][0])
        np.testing.assert_array_equal(host(g_d[x].proof_prob), o_m[x][1])
        np.testing.assert_array_equal(host(g_d[x].prob), o_m[x][2])
    mids_o, mids_g = [], []
    for x, tab in enumerate(tabs):
        tri = oracle.dense_to_triples(tab)
        so, om, op, opr = oracle.dtkp_apply2(tri, 3, 3, k, grp, fp, o_m[2 * x][0], o_m[2 * x + 1][0])
        f = dol.FnTable.create_dense(tab)
        out = dol.Dist.empty(f.out_syms, B, k=k)
        dol.apply2(g_d[2 * x], g_d[2 * x + 1], f, prov, out)
        np.testing.assert_array_equal(out.sym_ids, so)
        np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), om)
        np.testing.assert_array_equal(host(out.proof_prob), op)
        assert_close(host(out.prob), opr, "dtkp apply")
        mids_o.append((so, om, op, opr)); mids_g.append(out)
    # k x k conjunction of the two multi-proof results (facts of groups 0 and 1 overlap across sides)
    na, nb = mids_o[0][0].size, mids_o[1][0].size
    tab2 = W.hashed_table(23, na, nb, 5)
    tri2 = oracle.dense_to_triples(tab2)
    so, om, op, opr = oracle.dtkp_apply2(tri2, na, nb, k, grp, fp, mids_o[0][1], mids_o[1][1])
    f2 = dol.FnTable.create_dense(tab2)
    out2 = dol.Dist.empty(f2.out_syms, B, k=k)
    dol.apply2(mids_g[0], mids_g[1], f2, prov, out2)
    np.testing.assert_array_equal(host(out2.proof_mask).view(np.uint64), om)
    np.testing.assert_array_equal(host(out2.proof_prob), op)
    assert_close(host(out2.prob), opr, "dtkp k x k apply")
    assert (om[:, :, 1] != oracle.ABSENT).any()
    # union of the two mid results (their symbol lists overlap)
    usyms, ia, ib = oracle.union_plan(mids_o[0][0], mids_o[1][0])
    um, up, upr = oracle.dtkp_union(ia, ib, mids_o[0][1], mids_o[0][2], mids_o[1][1], mids_o[1][2])
    uo = dol.Dist.empty(dol.union_plan(mids_g[0], mids_g[1]), B, k=k)
    np.testing.assert_array_equal(uo.sym_ids, usyms)
    dol.union(mids_g[0], mids_g[1], prov, uo)
    np.testing.assert_array_equal(host(uo.proof_mask).view(np.uint64), um)
    np.testing.assert_array_equal(host(uo.proof_prob), up)
    assert_close(host(uo.prob), upr, "dtkp union")
    # gradient of the k x k result's and the union's tag probabilities w.r.t. the facts (uniform fact probabilities
    # put several symbols over 1, so the clamp gate is exercised; proofs share facts across slots)
    for name, dist, masks, prob in (("k x k", out2, om, opr), ("union", uo, um, upr)):
        gsym = W.normal(31, B * masks.shape[1]).astype(np.float32).reshape(B, -1)
        want = oracle.dtkp_prob_bwd(masks, fp, gsym)
        gf = torch.full((B, n_facts), 7.0, device="cuda")
        dol.dtkp_backward(dist, prov, dev(gsym), gf)
        assert_close(host(gf), want, "dtkp gradient, " + name)
    assert (upr == 1.0).any() and (upr < 1.0).any()
    # filter
    pred = (np.arange(usyms.size) % 2 == 0).astype(np.uint8)
    fm, fpp, fpr = oracle.dtkp_filter(pred, um, up, upr)
    fo = dol.Dist.empty(dol.filter_plan(uo, pred), B, k=k)
    dol.filter(uo, pred, prov, fo)
    np.testing.assert_array_equal(host(fo.proof_mask).view(np.uint64), fm)
    np.testing.assert_array_equal(host(fo.proof_prob), fpp)
    np.testing.assert_array_equal(host(fo.prob), fpr)


@pytest.mark.parametrize("which", ["chain", "fold", "hashed", "hashed-fused", "dtkp-fold", "reach-fused", "reach-one-launch", "hashed-merged", "hashed-one-launch", "product",
                                   "formula-damp", "formula-dtkp"])
def test_hip_graph_replay_matches_eager(gp, which):
    """Every entry point issues only asynchronous launches once its symbol-side plans exist, so a whole step can be
    captured; replays (with eager work and synchronisations between them) equal the eager result."""
    if which == "chain":
        prog = gp.SumChain(W.config2(batch=512, n_digits=6, seed=5)); key = lambda: prog.grad_p
    elif which == "fold":
        prog = gp.SumChainFused(W.config2(batch=512, n_digits=6, seed=5)); key = lambda: prog.grad_p
    elif which == "hashed":
        prog = gp.HashedPipeline(W.config3(batch=320, seed=5)); key = lambda: prog.ga
    elif which == "hashed-fused":
        prog = gp.HashedPipelineFused(W.config3(batch=320, seed=5)); key = lambda: prog.ga
    elif which == "hashed-merged":
        prog = gp.HashedPipelineMerged(W.config3(batch=320, seed=5)); key = lambda: prog.ga
    elif which == "hashed-one-launch":
        prog = gp.HashedPipelineMerged(W.config3(batch=320, seed=5), one_launch=True); key = lambda: prog.ga
    elif which == "reach-one-launch":
        prog = gp.GridReachFused(W.config5(batch=16, side=8, rounds=12, seed=5), one_launch=True); key = lambda: prog.grad_p
    elif which == "dtkp-fold":
        prog = gp.DtkpSumChainFused(W.config4(batch=200, seed=5), with_gradient=True); key = lambda: prog.grad_fact
    elif which == "product":
        prog = gp.ProductChain(W.product_workload(batch=40, n_digits=7, seed=5)); key = lambda: prog.grad_p
    elif which == "formula-damp":
        prog = gp.HwfPipeline(W.hwf_workload(batch=24, length=5, seed=5), "damp"); key = lambda: prog.grad_p
    elif which == "formula-dtkp":
        prog = gp.HwfPipeline(W.hwf_workload(batch=24, length=5, seed=5), "dtkp"); key = lambda: prog.grad_p
    else:
        prog = gp.GridReachFused(W.config5(batch=16, side=8, rounds=12, seed=5)); key = lambda: prog.grad_p
    prog.step()
    eager = host(key()).copy()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        prog.step()
    torch.cuda.current_stream().wait_stream(s)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        prog.step()
    for _ in range(3):
        key().fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        np.testing.assert_array_equal(host(key()), eager)


# ---------------------------------------------------------------- large batches: sampled rows against the oracle

def _rows_of(w, idx, per_sample):
    """A sub-workload holding only the samples `idx` (samples are independent, so the oracle can run on them alone)."""
    arrays = {}
    for name, arr in w.arrays.items():
        axis = per_sample.get(name)
        arrays[name] = arr if axis is None else np.ascontiguousarray(np.take(arr, idx, axis=axis))
    params = dict(w.params, batch=len(idx))
    return W.Workload(w.name, params, arrays)


def _sample_rows(batch, n=48):
    picks = (W.splitmix64(batch, np.arange(n, dtype=np.uint64)) % np.uint64(batch)).astype(np.int64)
    return np.unique(np.concatenate([[0, 1, 63, 64, batch // 2, batch - 2, batch - 1], picks]))


@pytest.mark.parametrize("cfg,batch", [(2, 200003), (3, 70001), (4, 50021), (5, 1031)])
def test_large_batches_sampled_rows(gp, cfg, batch):
    """The launch shapes of the B-scaled bench variants (odd batches, many tiles per workgroup, grids of 10^5
    workgroups): rows sampled over the whole batch against the oracle run on those samples alone."""
    w = W.make_config(cfg, batch=batch, seed=11)
    idx = _sample_rows(batch)
    if cfg == 2:
        prog = gp.SumChainFused(w)
        prog.step()
        ref = OP.sum_chain_fwd_bwd(_rows_of(w, idx, dict(p=1, target=0)))
        assert_close(host(prog.out.prob)[idx], ref["out"], "fold forward, sampled rows")
        assert_close(host(prog.grad_p)[:, idx], ref["grad_p"], "fold gradient, sampled rows")
    elif cfg == 3:
        ref = OP.hashed_pipeline_fwd_bwd(_rows_of(w, idx, dict(pa=0, pb=0, p2=0, g=0)))
        for cls in (gp.HashedPipelineMerged, gp.HashedPipelineFused):     # the bench's two launches; Apply, then Filter + Union
            prog = cls(w)
            prog.step()
            assert_close(host(prog.o3.prob)[idx], ref["o3"], "hashed pipeline forward, sampled rows")
            assert_close(host(prog.ga)[idx], ref["ga"], "hashed pipeline grad a, sampled rows")
            assert_close(host(prog.gb)[idx], ref["gb"], "hashed pipeline grad b, sampled rows")
            assert_close(host(prog.gp2)[idx], ref["gp2"], "hashed pipeline grad p2, sampled rows")
            del prog
    elif cfg == 4:
        prog = gp.DtkpSumChainFused(w)
        prog.step()
        ref = OP.dtkp_sum_chain(_rows_of(w, idx, dict(p=1, fact_prob=0)))
        np.testing.assert_array_equal(host(prog.out.proof_mask).view(np.uint64)[idx], ref["mask"])
        np.testing.assert_array_equal(host(prog.out.proof_prob)[idx], ref["pprob"])
        assert_close(host(prog.out.prob)[idx], ref["prob"], "dtkp fold, sampled rows")
    else:
        ref = OP.grid_reach_fwd_bwd(_rows_of(w, idx, dict(p=0, g=0)))
        for one_launch in (True, False):                                   # the bench's single launch; the two sweeps apart
            prog = gp.GridReachFused(w, one_launch=one_launch)
            prog.step()
            assert_close(host(prog.out.prob)[idx], ref["r"], "reachability, sampled rows")
            assert_close(host(prog.grad_p)[idx], ref["grad_p"], "reachability gradient, sampled rows")
            del prog


# ---------------------------------------------------------------- Apply over K Distributions, unary Apply, ApplyIf

def _rand_table(seed, shape, n_ids, drop_every=0):
    t = (W.splitmix64(seed, np.arange(int(np.prod(shape)))) % np.uint64(n_ids)).astype(np.int32).reshape(shape)
    if drop_every:
        t.reshape(-1)[::drop_every] = -1
    return t


@pytest.mark.parametrize("shape,n_ids,scale,batch", [
    ((37,), 6, 1.0, 300), ((37,), 6, 9.0, 45),                      # unary, second one clamps
    ((10, 10), 19, 1.0, 129), ((10, 10, 10), 28, 1.0, 513),         # sums of two and three digits
    ((9, 5, 7), 40, 3.2, 200), ((4, 3, 5, 4), 23, 1.0, 77), ((3, 2, 3, 2, 3), 11, 2.0, 64),
    ((2, 3, 2, 2, 3, 2), 9, 1.0, 33), ((300, 4, 3), 500, 1.0, 1000), ((2100,), 2100, 1.0, 3)])
def test_apply_k_damp_forward_and_backward(dol, shape, n_ids, scale, batch):
    K = len(shape)
    if n_ids in (19, 28):      # digit sums
        table = np.zeros(shape, np.int32)
        for l in range(K):
            table = table + np.arange(10).reshape([-1 if m == l else 1 for m in range(K)])
        table = table.astype(np.int32)
    else:
        table = _rand_table(300 + K, shape, n_ids, drop_every=5)
    ins = [(W.softmax_rows(W.normal(310 + l, batch * n).reshape(batch, n)) * scale).astype(np.float32)
           for l, n in enumerate(shape)]
    idx, to = oracle.dense_to_tuples(table)
    syms, want, pre32, _ = oracle.damp_applyk_fwd(idx, to, ins, want_pre=True)
    f = dol.FnkTable.create_dense(table)
    np.testing.assert_array_equal(f.out_syms, syms)
    if K == 1:      # rows of fewer than 2 048 tags stay with the cached gathers
        want_names = ("damp_apply1_fwd_kernel", "damp_apply1_bwd_kernel") if shape[0] < 2048 else \
                     ("damp_apply1_fwd_staged_kernel", "damp_apply1_bwd_staged_kernel")
    else:
        want_names = ("damp_applyk_fwd_kernel<%d>" % K, "damp_applyk_bwd_kernel<%d>" % K)
    assert (f.kernel_fwd, f.kernel_bwd) == want_names
    lds = [n + (3 if l % 2 else 0) for l, n in enumerate(shape)]       # some operands with padded rows
    d_in = []
    for x, n, ld in zip(ins, shape, lds):
        buf = torch.zeros((batch, ld), device="cuda")
        buf[:, :n] = dev(x)
        d_in.append(dol.Dist(np.arange(n), buf[:, :n]))
    out = dol.Dist.empty(f.out_syms, batch)
    dol.apply_k(d_in, f, None, out)
    assert_close(host(out.prob), want, "apply_k forward")
    if scale > 1.0:
        assert (pre32 > 1).any() and (pre32 < 1).any()
    sign = np.float32(1.0) if scale > 1.0 else None
    g = W.normal(320, batch * syms.size).astype(np.float32).reshape(batch, -1)
    if sign is not None:
        g = np.abs(g)
    wants = oracle.damp_applyk_bwd(idx, to, ins, g)
    grads = [torch.full((batch, ld), 5.0, device="cuda") for ld in lds]
    skip = 1 if K >= 3 else None
    dol.apply_k_backward(d_in, f, out, dev(g), [None if l == skip else gr for l, gr in enumerate(grads)])
    for l, n in enumerate(shape):
        got = host(grads[l])
        if l == skip:
            assert np.all(got == 5.0)
            continue
        assert_close(got[:, :n], wants[l], "apply_k grad of operand %d" % l)
        assert np.all(got[:, n:] == 5.0)


@pytest.mark.parametrize("batch", [3, 300])
def test_wide_operand_rows_staged_in_lds(dol, batch):
    """Unary and binary Apply over operand rows of thousands of tags (the kernels that copy a sample's rows into LDS
    and gather there): a few workgroups per sample at batch 3, one at batch 300; padded rows whose starts fall off
    16-byte boundaries; columns of every length from 1 up, one of them long enough for the wavefront kernel; tags
    scaled so that columns clamp, with pre exactly 1 (gradient passes) and pre > 1 (blocked) in sample 0."""
    # ---- unary
    n_in, n_ids = 5001, 700
    table = _rand_table(6100, (n_in,), n_ids, drop_every=9)
    table[:200:2] = 5                                                  # 100 symbols on one column
    x = (W.softmax_rows(W.normal(6101, batch * n_in).reshape(batch, n_in)) * 700.0).astype(np.float32)
    x[0, :] = 0.125                                                    # columns of 8 symbols sum to exactly 1
    idx, to = oracle.dense_to_tuples(table)
    syms, want, pre32, _ = oracle.damp_applyk_fwd(idx, to, [x], want_pre=True)
    assert (pre32[0] == 1).any() and (pre32 > 1).any() and (pre32 < 1).any()
    f = dol.FnkTable.create_dense(table)
    assert (f.kernel_fwd, f.kernel_bwd) == ("damp_apply1_fwd_staged_kernel", "damp_apply1_bwd_staged_kernel")
    buf = torch.zeros((batch, n_in + 3), device="cuda")
    buf[:, :n_in] = dev(x)
    d_in = [dol.Dist(np.arange(n_in), buf[:, :n_in])]
    out = dol.Dist.empty(f.out_syms, batch)
    dol.apply_k(d_in, f, None, out)
    assert_close(host(out.prob), want, "wide unary forward")
    g = np.abs(W.normal(6102, batch * syms.size).astype(np.float32).reshape(batch, -1)) + np.float32(0.5)
    (wx,) = oracle.damp_applyk_bwd(idx, to, [x], g)
    gx = torch.full((batch, n_in + 3), 5.0, device="cuda")
    dol.apply_k_backward(d_in, f, out, dev(g), [gx])
    got = host(gx)
    np.testing.assert_array_equal(got[:, :n_in], wx)                   # each entry is a gradient entry or 0
    assert np.all(got[:, n_in:] == 5.0)
    assert (wx[0] == 0).any() and (wx[0] != 0).any()
    # ---- binary
    na, nb = 3000, 20
    table2 = _rand_table(6110, (na, nb), 9000, drop_every=7)
    table2[:90, 0] = 17                                                # a long column
    a = (W.softmax_rows(W.normal(6111, batch * na).reshape(batch, na)) * (na * 1.2)).astype(np.float32)
    b = (W.softmax_rows(W.normal(6112, batch * nb).reshape(batch, nb)) * 3.0).astype(np.float32)
    tri = oracle.dense_to_triples(table2)
    syms2, want2, pre2, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    assert (pre2 > 1).any() and (pre2 < 1).any()
    f2 = dol.FnTable.create_dense(table2)
    assert f2.kernel_fwd == "damp_apply2_fwd_staged_kernel"
    abuf = torch.zeros((batch, na + 1), device="cuda")
    abuf[:, :na] = dev(a)
    bbuf = torch.zeros((batch, nb + 2), device="cuda")
    bbuf[:, :nb] = dev(b)
    da, db = dol.Dist(np.arange(na), abuf[:, :na]), dol.Dist(np.arange(nb), bbuf[:, :nb])
    out2 = dol.Dist.empty(f2.out_syms, batch)
    dol.apply2(da, db, f2, None, out2)
    np.testing.assert_array_equal(out2.sym_ids, syms2)
    assert_close(host(out2.prob), want2, "wide binary forward")
    np.testing.assert_array_equal(host(out2.prob) == 1.0, pre2 >= 1.0)
    # ---- binary with a short second operand: the per-j map kernels with the long row (forward) and the gated
    # gradient row (backward) in LDS; columns where some j occurs twice go through their tuple lists
    nb3 = 7
    table3 = _rand_table(6120, (na, nb3), 2500, drop_every=7)
    b3 = (W.softmax_rows(W.normal(6122, batch * nb3).reshape(batch, nb3)) * 1.1).astype(np.float32)
    tri3 = oracle.dense_to_triples(table3)
    syms3, want3, pre3, _ = oracle.damp_apply2_fwd(tri3, na, nb3, a, b3, want_pre=True)
    assert (pre3 > 1).any() and (pre3 < 1).any()
    f3 = dol.FnTable.create_dense(table3)
    assert (f3.kernel_fwd, f3.kernel_bwd) == ("damp_byj_fwd_staged_kernel", "damp_byj_bwd_row_kernel")
    db3 = dol.Dist(np.arange(nb3), dev(b3))
    out3 = dol.Dist.empty(f3.out_syms, batch)
    dol.apply2(da, db3, f3, None, out3)
    assert_close(host(out3.prob), want3, "wide per-j forward")
    np.testing.assert_array_equal(host(out3.prob) == 1.0, pre3 >= 1.0)
    g3 = np.abs(W.normal(6123, batch * syms3.size).astype(np.float32).reshape(batch, -1)) + np.float32(0.5)
    wa3, wb3 = oracle.damp_apply2_bwd(tri3, na, nb3, a, b3, g3)
    ga3 = torch.full((batch, na + 1), 5.0, device="cuda")
    gb3 = torch.empty((batch, nb3), device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db3, out3, f=f3), dev(g3), ga3, gb3)
    assert_close(host(ga3)[:, :na], wa3, "wide per-j grad a")
    assert_close(host(gb3), wb3, "wide per-j grad b")
    assert np.all(host(ga3)[:, na:] == 5.0)


@pytest.mark.parametrize("na,nb,n_out,clamped", [(20000, 10, 40449, 0.01), (20000, 10, 40450, 0.01), (45000, 3, 45001, 0.0), (41003, 4, 41002, 0.5), (60000, 16, 60000, 0.01)])
def test_result_rows_wider_than_lds_backward(dol, na, nb, n_out, clamped):
    """Gradients of a table with a short second operand whose result row is the widest that fits LDS, the next wider one, and
    of up to 60 000 symbols: no column, some and many at the clamp, a long column among them."""
    B = 2
    i = np.repeat(np.arange(na, dtype=np.int64), nb)
    j = np.tile(np.arange(nb), na)
    o = (i * n_out // na + W.splitmix64(77, np.arange(i.size)).astype(np.int64) % 5) % n_out
    o[np.argsort(W.splitmix64(78, np.arange(i.size)), kind="stable")[:n_out]] = np.arange(n_out)     # (every symbol is produced)
    o[(i < 40) & (o != 7)] = 7                                # a long column
    tri = tuple(x.astype(np.int32) for x in (i, j, o))
    a = (W.uniform01(1, B * na) * 0.2).astype(np.float32).reshape(B, na)
    if clamped:
        a[:, ::max(1, int(1 / clamped))] = 1.0
    b = (W.uniform01(2, B * nb) * 0.3 + 0.7).astype(np.float32).reshape(B, nb)
    if not clamped:
        a, b = a * np.float32(0.01), b * np.float32(0.01)
    syms, want, pre32, pre64 = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    assert ((pre32 > 1).mean() > clamped / 2) if clamped else not (pre32 > 1).any()
    f = dol.FnTable.create_sparse(na, nb, *tri)
    assert f.kernel_bwd == ("damp_byj_bwd_row_kernel" if syms.size <= 40447 else "damp_byj_bwd_global_kernel")
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(syms, B)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "forward")
    np.testing.assert_array_equal(host(out.prob) == 1.0, pre32 >= 1.0)
    g = (np.abs(W.normal(901, B * syms.size)) + 0.5).astype(np.float32).reshape(B, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    assert_close(host(ga), wa, "backward a")
    assert_close(host(gb), wb, "backward b")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f, accumulate=3), dev(g), ga, gb)
    assert_close(host(ga), 2.0 * wa.astype(np.float64), "backward a accumulated")
    assert_close(host(gb), 2.0 * wb.astype(np.float64), "backward b accumulated")


@pytest.mark.parametrize("nb", [10, 20])
@pytest.mark.parametrize("n_out", [60, 64, 65, 200, 1700])
def test_backward_with_many_long_columns_at_the_clamp(dol, nb, n_out):
    """Columns of more than 64 tuples that sum to within a few roundings of 1, or well above it: as many as a workgroup lists,
    one more, and more than a thousand; the decision is the sequential float sum's."""
    B, per = 3, 4 if nb == 20 else 7
    na = per * n_out
    i = np.repeat(np.arange(na), nb).astype(np.int32)
    j = np.tile(np.arange(nb), na).astype(np.int32)
    o = (i % n_out).astype(np.int32)
    w = W.uniform01(70 + nb, B * na).reshape(B, per, n_out) ** 3 + 1e-6
    want_sum = 1.0 + 1e-7 * ((np.arange(n_out) * 7 + np.arange(B)[:, None] * 3) % 5 - 2)
    want_sum[:, ::6] = 1.7
    a = (w / w.sum(axis=1, keepdims=True) * want_sum[:, None, :] / nb).astype(np.float32).reshape(B, na)
    b = np.ones((B, nb), np.float32)
    tri = (i, j, o)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    assert (pre32 > 1.5).any() and ((pre32 > 1) & (pre32 < 1.1)).any() and (pre32 <= 1).any()
    f = dol.FnTable.create_sparse(na, nb, *tri)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(syms, B)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "forward")
    np.testing.assert_array_equal(host(out.prob) == 1.0, pre32 >= 1.0)
    g = (np.abs(W.normal(901, B * syms.size)) + 0.5).astype(np.float32).reshape(B, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    assert_close(host(ga), wa, "backward a")
    assert_close(host(gb), wb, "backward b")


@pytest.mark.parametrize("na,nb,n_long,n_short,B", [(36300, 20, 900, 6000, 2), (36344, 20, 3, 12000, 2), (37000, 20, 1500, 3000, 1), (37000, 4, 40, 30000, 3),
                                                    (700, 30, 90, 10, 300), (500, 12, 31, 700, 5)])
def test_forward_with_long_columns_shared_over_workgroups(dol, na, nb, n_long, n_short, B):
    """Columns of 65 to some thousand tuples among short ones, few and many of them, beside rows that leave room in LDS for a
    block of results and rows that do not; every third long column sums to within roundings of 1, where the order of
    definition decides, the others above and below."""
    r = W.splitmix64(31, np.arange(na * nb))
    i, j = np.repeat(np.arange(na), nb), np.tile(np.arange(nb), na)
    long_rows = na // 2
    n_tail = min(na - long_rows, max(1, 3 * n_short // nb))                  # rows whose tuples go to the short columns
    keep = (i < long_rows) | (i >= na - n_tail)
    i, j, r = i[keep], j[keep], r[keep]
    o = np.where(i < long_rows, i % n_long, n_long + (r % np.uint64(n_short)).astype(np.int64))
    syms, o = np.unique(o, return_inverse=True)
    tri = (i.astype(np.int32), j.astype(np.int32), o.astype(np.int32))
    lengths = np.bincount(o)
    assert (lengths[:n_long] > 64).all() and (lengths[n_long:] <= 64).all()
    b = np.ones((B, nb), np.float32)
    a = (W.uniform01(33, B * na).reshape(B, na) ** 2 + 1e-4).astype(np.float64)
    for c in range(n_long):
        rows = np.arange(c, long_rows, n_long)
        want_sum = (1.0 + 1e-7 * ((c + np.arange(B)) % 5 - 2), 1.5, 0.6)[c % 3]
        a[:, rows] *= (np.asarray(want_sum) / (a[:, rows].sum(axis=1) * nb)).reshape(-1, 1)
    a[:, long_rows:] *= 0.2
    a = a.astype(np.float32)
    _, want, pre32, pre64 = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    near = pre32[:, :n_long][:, ::3]
    assert np.abs(near - 1).max() < 1e-5 and (near > 1).any() and (near <= 1).any()
    f = dol.FnTable.create_sparse(na, nb, *tri)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(f.out_syms, B)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "forward")
    np.testing.assert_array_equal(host(out.prob) == 1.0, pre32 >= 1.0)


def test_apply_k_two_operands_equal_apply2_bit_for_bit(dol):
    B = 150
    table = W.hashed_table(41, 30, 20, 64)
    a = (W.softmax_rows(W.normal(42, B * 30).reshape(B, 30)) * 2).astype(np.float32)
    b = (W.softmax_rows(W.normal(43, B * 20).reshape(B, 20)) * 2).astype(np.float32)
    da, db = dol.Dist(np.arange(30), dev(a)), dol.Dist(np.arange(20), dev(b))
    f2, fk = dol.FnTable.create_dense(table), dol.FnkTable.create_dense(table)
    np.testing.assert_array_equal(f2.out_syms, fk.out_syms)
    o2, ok = dol.Dist.empty(f2.out_syms, B), dol.Dist.empty(fk.out_syms, B)
    dol.apply2(da, db, f2, None, o2)
    dol.apply_k([da, db], fk, None, ok)
    np.testing.assert_array_equal(host(o2.prob), host(ok.prob))


def test_apply_if_table(dol):
    B, na, nb = 90, 12, 9
    table = W.hashed_table(51, na, nb, 16)
    cond = ((np.arange(na)[:, None] + np.arange(nb)[None, :]) % 3 != 1)
    a = W.softmax_rows(W.normal(52, B * na).reshape(B, na))
    b = W.softmax_rows(W.normal(53, B * nb).reshape(B, nb))
    tri = oracle.dense_to_triples(np.where(cond, table, -1))
    syms, want = oracle.damp_apply2_fwd(tri, na, nb, a, b)
    g = W.normal(54, B * syms.size).astype(np.float32).reshape(B, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    junk = np.where(cond, table, -7).astype(np.int32)               # entries the condition rejects are never read
    f = dol.FnTable.create_if(junk, cond)
    np.testing.assert_array_equal(f.out_syms, syms)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(f.out_syms, B)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "apply_if forward")
    ga, gb = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    assert_close(host(ga), wa, "apply_if grad a")
    assert_close(host(gb), wb, "apply_if grad b")
    with pytest.raises(dol.DolError):
        dol.FnTable.create_if(np.full((2, 2), -1, np.int32), np.ones((2, 2), np.uint8))


@pytest.mark.parametrize("k", [1, 3, 8])
def test_apply_k_dtkp(dol, k):
    """Three operands with multi-proof tags and exclusion groups, then a unary Apply that merges symbols."""
    B, nv = 60, 4
    fp = np.concatenate([W.softmax_rows(W.normal(60 + t, B * nv).reshape(B, nv)) for t in range(4)], axis=1)
    grp = np.repeat(np.arange(4), nv).astype(np.int32)
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    o_tags, g_tags = [], []
    for t in range(4):
        o_tags.append(oracle.dtkp_init(np.arange(nv) + nv * t, fp, k)[0])
        d = dol.Dist.empty(np.arange(nv), B, k=k)
        dol.dtkp_init(d, np.arange(nv) + nv * t, prov)
        g_tags.append(d)
    # operand 0: sum of slots 0 and 1 (several proofs per symbol)
    sum_t = np.add.outer(np.arange(nv), np.arange(nv)).astype(np.int32)
    s0, m0, p0, _ = oracle.dtkp_apply2(oracle.dense_to_triples(sum_t), nv, nv, k, grp, fp, o_tags[0], o_tags[1])
    f0 = dol.FnTable.create_dense(sum_t)
    a = dol.Dist.empty(f0.out_syms, B, k=k)
    dol.apply2(g_tags[0], g_tags[1], f0, prov, a)
    table = _rand_table(70, (s0.size, nv, nv), 9, drop_every=6)
    idx, to = oracle.dense_to_tuples(table)
    syms, om, op, opr = oracle.dtkp_applyk(idx, to, k, grp, fp, [m0, o_tags[2], o_tags[3]])
    f = dol.FnkTable.create_dense(table)
    np.testing.assert_array_equal(f.out_syms, syms)
    out = dol.Dist.empty(f.out_syms, B, k=k)
    dol.apply_k([a, g_tags[2], g_tags[3]], f, prov, out)
    np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), om)
    np.testing.assert_array_equal(host(out.proof_prob), op)
    assert_close(host(out.prob), opr, "dtkp apply_k")
    # the same call with the operands' stored proof probabilities withheld
    bare = [dol.Dist(d.sym_ids, d.prob, d.proof_mask, None) for d in (a, g_tags[2], g_tags[3])]
    out_b = dol.Dist.empty(f.out_syms, B, k=k)
    dol.apply_k(bare, f, prov, out_b)
    np.testing.assert_array_equal(host(out_b.proof_mask).view(np.uint64), om)
    np.testing.assert_array_equal(host(out_b.proof_prob), op)
    # unary Apply over the result
    f1 = (np.arange(syms.size) % 3).astype(np.int32)
    f1[2] = -1
    idx1, to1 = oracle.dense_to_tuples(f1)
    s1, m1, p1, pr1 = oracle.dtkp_applyk(idx1, to1, k, grp, fp, [om])
    fu = dol.FnkTable.create_dense(f1)
    np.testing.assert_array_equal(fu.out_syms, s1)
    out1 = dol.Dist.empty(fu.out_syms, B, k=k)
    dol.apply_k([out], fu, prov, out1)
    np.testing.assert_array_equal(host(out1.proof_mask).view(np.uint64), m1)
    np.testing.assert_array_equal(host(out1.proof_prob), p1)
    assert_close(host(out1.prob), pr1, "dtkp unary apply")
    if k > 1:
        assert (m1[:, :, 1] != oracle.ABSENT).any()


def test_apply_k_argument_errors_and_empty(dol):
    with pytest.raises(dol.DolError):
        dol.FnkTable([3, 3], [[0, 0], [0, 0]], [1, 2])              # one index tuple twice
    with pytest.raises(dol.DolError):
        dol.FnkTable([3, 3], [[0, 3]], [1])                         # position outside the operand
    with pytest.raises(dol.DolError):
        dol.FnkTable([2] * 7, np.zeros((1, 7), np.int32), [1])      # too many operands
    f = dol.FnkTable.create_dense(np.arange(6, dtype=np.int32).reshape(2, 3))
    a, b = dol.Dist(np.arange(2), torch.ones((4, 2), device="cuda")), dol.Dist(np.arange(3), torch.ones((4, 3), device="cuda"))
    with pytest.raises(dol.DolError) as ei:
        dol.apply_k([a, b], f, None, dol.Dist.empty(np.arange(5), 4))
    assert ei.value.status == 2
    with pytest.raises(dol.DolError):
        dol.apply_k([b, a], f, None, dol.Dist.empty(f.out_syms, 4))
    with pytest.raises(dol.DolError):
        dol.apply_k([a], f, None, dol.Dist.empty(f.out_syms, 4))
    none = dol.FnkTable.create_dense(np.full((2, 3), -1, np.int32))
    assert none.n_out == 0
    o0 = dol.Dist.empty(none.out_syms, 4)
    dol.apply_k([a, b], none, None, o0)
    ga = torch.full((4, 2), 3.0, device="cuda")
    dol.apply_k_backward([a, b], none, o0, torch.empty((4, 0), device="cuda"), [ga, None])
    assert np.all(host(ga) == 0)
    e = dol.Dist.empty(f.out_syms, 0)
    dol.apply_k([dol.Dist(np.arange(2), torch.ones((0, 2), device="cuda")), dol.Dist(np.arange(3), torch.ones((0, 3), device="cuda"))], f, None, e)


@pytest.mark.parametrize("n", [2047, 2048, 40445, 40448, 40449])
@pytest.mark.parametrize("lengths", [[1], [2, 1], [1, 2, 3, 4, 5, 127, 128, 129, 255], [1024, 1025, 7]], ids=lambda x: "-".join(map(str, x)))
@pytest.mark.parametrize("B", [1, 70, 300])
def test_unary_apply_of_wide_rows(dol, n, lengths, B):
    """Unary Apply, forward and backward, on either side of the shortest and longest rows that are staged in LDS: columns of one to
    a thousand symbols (two to a word of the lists; 128 are the most that a lane sums), short lists and long ones in their
    kernels, a last chunk that is not full, rejected symbols, rows of other strides, columns at the clamp and beyond.
    Tolerance: the bar of 1e-5; where a sum of at most 128 tags is exactly 1 or beyond it, the decision is the oracle's."""
    col, c = np.full(n, -1, np.int32), 0
    place, at = W.splitmix64(5, np.arange(n)).argsort(kind="stable"), 0
    while at < n - 5:
        take = min(lengths[c % len(lengths)], n - 5 - at)
        col[place[at:at + take]] = 3 * c
        at, c = at + take, c + 1
    x = (W.uniform01(8, B * n).reshape(B, n) * (1.2 / np.bincount(col[col >= 0])[np.maximum(col, 0)])).astype(np.float32)
    x[0] = 0.0
    x[0, col == 0] = 1.0                                         # a sum of exactly 1, or of more
    kept = np.nonzero(col >= 0)[0]
    look = np.unique(np.r_[0:min(B, 6), B - 1])
    syms, want, _, pre = oracle.damp_applyk_fwd(kept[:, None], col[kept], [x[look]], want_pre=True)
    g = W.normal(9, B * syms.size).astype(np.float32).reshape(B, -1)
    want_g, = oracle.damp_applyk_bwd(kept[:, None], col[kept], [x[look]], g[look])
    f = dol.FnkTable.create_dense(col)
    buf, gbuf, out = torch.zeros((B, n + 3), device="cuda"), torch.zeros((B, n + 3), device="cuda"), torch.full((B, syms.size + 5), 7.0, device="cuda")
    buf[:, :n] = dev(x)
    d, o = dol.Dist(np.arange(n), buf[:, :n]), dol.Dist(syms, out[:, :syms.size])
    dol.apply_k([d], f, None, o)
    dol.apply_k_backward([d], f, o, dev(g), [gbuf])
    got, got_g = host(out)[look], host(gbuf)[look, :n]
    assert np.all(got[:, syms.size:] == 7.0)
    assert_close(got[:, :syms.size], want, "unary forward")
    sure = np.abs(pre - 1.0) > (0 if max(lengths) <= 128 else 1e-4)
    np.testing.assert_array_equal((got[:, :syms.size] == 1.0)[sure], (want == 1.0)[sure])
    passes = np.ones((look.size, n), bool)
    passes[:, kept] = sure[:, np.searchsorted(syms, col[kept])] | (pre == 1.0)[:, np.searchsorted(syms, col[kept])]
    np.testing.assert_array_equal(got_g[passes], want_g.astype(np.float32)[passes])


@pytest.mark.parametrize("n", [2100, 9000, 40000])
@pytest.mark.parametrize("lengths", [[40, 64], [66, 100, 127, 128], [129, 600, 1000], [1023, 1024, 1025, 1500], [1900]], ids=lambda x: "-".join(map(str, x)))
@pytest.mark.parametrize("B", [3, 70])
def test_unary_apply_decides_long_columns_in_their_order(dol, n, lengths, B):
    """Columns of 40 to 1 900 symbols, as a lane, 16 lanes, a wavefront and a workgroup sum them, that add up to within a few roundings
    of 1 on both sides, or well above it: which ones the clamp acts on, and whose gradients pass, is the sequential float32 sum's
    to say, without exception."""
    col, c, at = np.full(n, -1, np.int32), 0, 0
    place = W.splitmix64(51, np.arange(n)).argsort(kind="stable")
    while at + lengths[c % len(lengths)] <= n:
        take = lengths[c % len(lengths)]
        col[place[at:at + take]] = c
        at, c = at + take, c + 1
    kept = np.nonzero(col >= 0)[0]
    w = W.uniform01(52, B * n).reshape(B, n) ** 3 + 1e-6
    sums = np.stack([np.bincount(col[kept], weights=w[r, kept], minlength=c) for r in range(B)])
    want_sum = 1.0 + 1e-7 * ((np.arange(c) * 7 + np.arange(B)[:, None] * 3) % 7 - 3)
    want_sum[:, ::6] = 1.7
    x = np.where(col >= 0, w * (want_sum / sums)[:, np.maximum(col, 0)], 0.3).astype(np.float32)
    syms, want, pre32, _ = oracle.damp_applyk_fwd(kept[:, None], col[kept], [x], want_pre=True)
    g = (np.abs(W.normal(53, B * c)) + 0.5).astype(np.float32).reshape(B, c)
    want_g, = oracle.damp_applyk_bwd(kept[:, None], col[kept], [x], g)
    assert c == 1 or ((pre32 > 1) & (pre32 < 1.1)).any() and (pre32 < 1).any()
    f = dol.FnkTable.create_dense(col)
    d, o, gx = dol.Dist(np.arange(n), dev(x)), dol.Dist.empty(syms, B), torch.full((B, n), 5.0, device="cuda")
    dol.apply_k([d], f, None, o)
    dol.apply_k_backward([d], f, o, dev(g), [gx])
    assert_close(host(o.prob), want, "forward")
    np.testing.assert_array_equal(host(o.prob) == 1.0, pre32 >= 1.0)
    np.testing.assert_array_equal(host(gx), want_g.astype(np.float32))


@pytest.mark.parametrize("length", [66, 100, 128, 129, 600, 1000])
def test_unary_apply_of_wide_rows_keeps_its_precision(dol, length):
    """Columns of more than 64 symbols, below the clamp: 64 partial sums, or blocks of about 16 symbols, leave no more than some ten
    roundings on the way to a result, whose errors average out to less than one rounding's largest, 2^-24, root mean square
    (measured 0.42e-7; one symbol after the other 1.1e-7 at 66 and 1.6e-7 at 128)."""
    n, B = 40000 // length * length, 20
    col = np.repeat(np.arange(n // length), length)[W.splitmix64(54, np.arange(n)).argsort(kind="stable")].astype(np.int32)
    x = (W.uniform01(55, B * n) / length).astype(np.float32).reshape(B, n)
    f = dol.FnkTable.create_dense(col)
    o = dol.Dist.empty(f.out_syms, B)
    dol.apply_k([dol.Dist(np.arange(n), dev(x))], f, None, o)
    want = np.stack([np.bincount(col, weights=x[r].astype(np.float64)) for r in range(B)])
    err = host(o.prob).astype(np.float64) / want - 1.0
    assert np.sqrt((err ** 2).mean()) < 2.0 ** -24


# ---------------------------------------------------------------- Product-N fold (irregular growing symbol sets)

@pytest.mark.parametrize("batch,n", [(64, 4), (256, 8), (33, 11)])
def test_product_chain(gp, batch, n):
    """The fold of Fig. 2 with f = x * y: tables without structure, a zero column that every row feeds (summed by a
    wavefront once it is long), operand rows longer than a thread's share in the backward pass."""
    w = W.product_workload(batch=batch, n_digits=n, seed=n)
    ref = OP.product_chain_fwd_bwd(w)
    prog = gp.ProductChain(w)
    prog.step()
    np.testing.assert_array_equal(prog.accs[-1].sym_ids, ref["syms"])
    for t in range(1, n):
        assert_close(host(prog.accs[t].prob), ref["accs"][t], "product stage %d" % t)
    assert_close(host(prog.g_acc[-1]), ref["g_out"], "loss gradient")
    assert_close(host(prog.grad_p), ref["grad_p"], "product chain grad")


def test_long_column_near_the_clamp_takes_the_defining_order(dol):
    """A column of 3000 tuples whose sum lies within rounding of 1: the clamp decision (seen through backward) must be
    the one of the sequential float sum, on either side of 1."""
    B, na = 48, 3000
    table = np.zeros((na, 1), np.int32)                      # every symbol maps to 0: one long column
    a = W.uniform01(81, B * na).astype(np.float32).reshape(B, na)
    a = (a / a.sum(1, keepdims=True, dtype=np.float64)).astype(np.float32)       # rows sum to 1 up to rounding
    a[::3] *= np.float32(1.0 + 2e-7)
    b = np.ones((B, 1), np.float32)
    tri = oracle.dense_to_triples(table)
    syms, want, pre32, pre64 = oracle.damp_apply2_fwd(tri, na, 1, a, b, want_pre=True)
    assert (pre32 > 1).any() and (pre32 <= 1).any() and np.abs(pre64 - 1).max() < 1e-5
    g = np.ones((B, 1), np.float32)
    wa, wb = oracle.damp_apply2_bwd(tri, na, 1, a, b, g)
    f = dol.FnTable.create_dense(table)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(1), dev(b))
    out = dol.Dist.empty(f.out_syms, B)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "long column forward")
    ga, gb = torch.empty((B, na), device="cuda"), torch.empty((B, 1), device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    np.testing.assert_array_equal(host(ga), wa)              # 0 or 1 per sample: the decision itself
    assert_close(host(gb), wb, "long column grad b")


# ---------------------------------------------------------------- formula pipeline (filter -> chained apply -> unary apply)

@pytest.mark.parametrize("batch,length", [(64, 7), (33, 5), (5, 1)])
def test_formula_pipeline_damp(gp, batch, length):
    w = W.hwf_workload(batch=batch, length=length, seed=length)
    ref = OP.hwf_pipeline_damp(w)
    prog = gp.HwfPipeline(w, "damp")
    prog.step()
    np.testing.assert_array_equal(prog.out.sym_ids, ref["syms"])
    for t in range(1, length):
        assert_close(host(prog.accs[t].prob), ref["accs"][t], "formula stage %d" % t)
    assert_close(host(prog.out.prob), ref["out"], "formula values")
    assert_close(host(prog.grad_p), ref["grad_p"], "formula grad")


@pytest.mark.parametrize("batch,length,k", [(64, 7, 3), (20, 5, 1), (9, 3, 8)])
def test_formula_pipeline_dtkp(gp, batch, length, k):
    w = W.hwf_workload(batch=batch, length=length, k=k, seed=40 + length)
    ref = OP.hwf_pipeline_dtkp(w)
    prog = gp.HwfPipeline(w, "dtkp")
    prog.step()
    np.testing.assert_array_equal(host(prog.fact_prob), ref["fact_prob"])
    for t in range(1, length):
        m, pp, pr = ref["stages"][t - 1]
        np.testing.assert_array_equal(host(prog.accs[t].proof_mask).view(np.uint64), m)
        np.testing.assert_array_equal(host(prog.accs[t].proof_prob), pp)
    np.testing.assert_array_equal(host(prog.out.proof_mask).view(np.uint64), ref["mask"])
    np.testing.assert_array_equal(host(prog.out.proof_prob), ref["pprob"])
    assert_close(host(prog.out.prob), ref["prob"], "formula value probabilities")
    assert_close(host(prog.gfact), ref["gfact"], "formula fact gradient")
    assert_close(host(prog.grad_p), ref["grad_p"], "formula class gradient")


def test_apply_k_long_columns(dol):
    """Columns of hundreds to thousands of tuples (summed by a wavefront): a unary map onto one symbol whose sum lies
    within rounding of 1, where the clamp decision must still be the sequential float sum's, and a three-operand
    function with two images."""
    B, n = 40, 3000
    x = W.uniform01(91, B * n).astype(np.float32).reshape(B, n)
    x = (x / x.sum(1, keepdims=True, dtype=np.float64)).astype(np.float32)
    x[::3] *= np.float32(1.0 + 2e-7)
    idx, to = oracle.dense_to_tuples(np.zeros(n, np.int32))
    syms, want, pre32, pre64 = oracle.damp_applyk_fwd(idx, to, [x], want_pre=True)
    assert (pre32 > 1).any() and (pre32 <= 1).any() and np.abs(pre64 - 1).max() < 1e-5
    (wg,) = oracle.damp_applyk_bwd(idx, to, [x], np.ones((B, 1), np.float32))
    f = dol.FnkTable.create_dense(np.zeros(n, np.int32))
    d = dol.Dist(np.arange(n), dev(x))
    out = dol.Dist.empty(f.out_syms, B)
    dol.apply_k([d], f, None, out)
    assert_close(host(out.prob), want, "long unary column")
    gx = torch.empty((B, n), device="cuda")
    dol.apply_k_backward([d], f, out, torch.ones((B, 1), device="cuda"), [gx])
    np.testing.assert_array_equal(host(gx), wg)
    # three operands, two images: columns of about 500 tuples, one side of them over 1
    shape = (40, 5, 5)
    table = _rand_table(95, shape, 2)
    ins = [(W.softmax_rows(W.normal(96 + l, B * m).reshape(B, m)) * (1.3 if l == 0 else 1.0)).astype(np.float32)
           for l, m in enumerate(shape)]
    idx, to = oracle.dense_to_tuples(table)
    syms, want, pre32, _ = oracle.damp_applyk_fwd(idx, to, ins, want_pre=True)
    g = np.abs(W.normal(99, B * 2)).astype(np.float32).reshape(B, 2)
    wants = oracle.damp_applyk_bwd(idx, to, ins, g)
    f3 = dol.FnkTable.create_dense(table)
    d3 = [dol.Dist(np.arange(m), dev(v)) for m, v in zip(shape, ins)]
    out3 = dol.Dist.empty(f3.out_syms, B)
    dol.apply_k(d3, f3, None, out3)
    assert_close(host(out3.prob), want, "long three-operand columns")
    grads = [torch.empty((B, m), device="cuda") for m in shape]
    dol.apply_k_backward(d3, f3, out3, dev(g), grads)
    for l in range(3):
        assert_close(host(grads[l]), wants[l], "long three-operand grad %d" % l)


def test_short_second_operand_tables_near_the_clamp(dol):
    """f(i, j) = i + 2j over 800 x 4 symbols: columns of four tuples whose defining order (ascending i) is the
    reverse of the order the per-j kernel adds them in, with sums within rounding of 1; clamp decisions (seen
    through backward) must be those of the defining order."""
    B, na, nb = 96, 800, 4
    table = (np.arange(na)[:, None] + 2 * np.arange(nb)[None, :]).astype(np.int32)
    a = np.ones((B, na), np.float32)
    b = W.softmax_rows(W.normal(71, B * nb).reshape(B, nb))
    b[::4] *= np.float32(1.0 + 1.2e-7)
    tri = oracle.dense_to_triples(table)
    syms, want, pre32, pre64 = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    inner = pre32[:, 6:na]
    assert (inner > 1).any() and (inner <= 1).any() and np.abs(pre64[:, 6:na] - 1).max() < 1e-6
    g = np.abs(W.normal(72, B * syms.size)).astype(np.float32).reshape(B, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    f = dol.FnTable.create_dense(table)
    assert f.kernel_fwd == "damp_byj_fwd_kernel" and f.kernel_bwd == "damp_byj_bwd_kernel"
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(f.out_syms, B)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "per-j forward")
    ga, gb = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    assert_close(host(ga), wa, "per-j grad a")
    assert_close(host(gb), wb, "per-j grad b")


@pytest.mark.parametrize("na,nb", [(767, 3), (769, 8), (1023, 9), (1025, 10), (2047, 16), (2049, 4), (2305, 10)])
def test_dense_map_blocks(dol, na, nb):
    """f(i, j) = i + 2j: rows and columns on either side of a whole number of blocks of 256 map entries, maps of 4, 8, 10 and 16
    rows; gradients written and added."""
    B = 3
    table = (np.arange(na)[:, None] + 2 * np.arange(nb)[None, :]).astype(np.int32)
    a, b = W.softmax_rows(W.normal(73, B * na).reshape(B, na)), W.softmax_rows(W.normal(74, B * nb).reshape(B, nb))
    tri = oracle.dense_to_triples(table)
    syms, want = oracle.damp_apply2_fwd(tri, na, nb, a, b)[:2]
    g = np.abs(W.normal(75, B * syms.size)).astype(np.float32).reshape(B, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    f = dol.FnTable.create_dense(table)
    assert "byj" in f.kernel_at(False, B) and "byj" in f.kernel_at(True, B)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(f.out_syms, B)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "forward")
    rec = dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f)
    ga, gb = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.backward(rec, dev(g), ga, gb)
    assert_close(host(ga), wa, "grad a")
    assert_close(host(gb), wb, "grad b")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f, accumulate=3), dev(g), ga, gb)
    assert_close(host(ga), 2 * wa, "grad a, added")
    assert_close(host(gb), 2 * wb, "grad b, added")


@pytest.mark.parametrize("grows", [True, False])
@pytest.mark.parametrize("na,nb,B", [(600, 3, 2), (2047, 10, 3), (2049, 8, 40), (8193, 16, 2), (18001, 10, 5)])
def test_dense_maps_in_and_out_of_the_defining_order(dol, na, nb, B, grows):
    """f(i, j) = i + 3j, whose columns' tuples have j falling as i rises, and i - 3j, where it rises; the last j maps every i to one
    symbol, a column that a workgroup sums where it has more than 512 tuples.  One second tag is infinite: columns without it stay
    finite.  Where j falls the sums are those of the defining order, float32 for float32; the long column's tolerance is the bar."""
    table = (np.arange(na)[:, None] + (3 if grows else -3) * np.arange(nb)[None, :] + 3 * nb).astype(np.int32)
    table[:, nb - 1] = na + 6 * nb
    a = W.softmax_rows(W.normal(76, B * na).reshape(B, na)) * np.float32(na / 3.0)      # columns on both sides of the clamp
    b = W.softmax_rows(W.normal(77, B * nb).reshape(B, nb))
    b[:, nb - 1] = 0.7 / na * 3.0
    b[1, 0] = np.inf
    tri = oracle.dense_to_triples(table)
    syms, want, pre32, pre64 = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    f = dol.FnTable.create_dense(table)
    assert "byj" in f.kernel_at(False, B)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(f.out_syms, B)
    dol.apply2(da, db, f, None, out)
    got = host(out.prob)
    assert (want[1] < 1).any() and np.isinf(pre32[1]).any() and (want[0] == 1).any()
    assert_close(got, want, "forward")
    np.testing.assert_array_equal(got[:, :-1] == 1.0, pre32[:, :-1] >= 1.0)
    if grows:
        np.testing.assert_array_equal(got[:, :-1], np.minimum(pre32[:, :-1], np.float32(1)))


@pytest.mark.parametrize("na,nb", [(1200, 8), (2060, 3), (4098, 10), (12300, 16)])
@pytest.mark.parametrize("n_long", [1, 2, 3])
@pytest.mark.parametrize("B", [1, 70, 300])
def test_dense_maps_with_one_and_several_long_columns(dol, na, nb, n_long, B):
    """The first second-operand symbol maps the first operand to one, two or three symbols only, columns that a workgroup sums, of
    unequal lengths: one is asked for ahead where it is long enough for that, several are shared out over a sample's parts.
    Some samples' long columns lie at the clamp.  Tolerance: the bar."""
    i, j = np.arange(na)[:, None], np.arange(nb)[None, :]
    table = np.where(j == 0, 10 ** 6 + np.minimum(i * 2 * n_long // (na + na // 2), n_long - 1), i + j).astype(np.int32)
    a = (W.uniform01(86, B * na) * (2.0 / na)).astype(np.float32).reshape(B, na)
    b = W.uniform01(87, B * nb).astype(np.float32).reshape(B, nb)
    b[::3, 0] = 1.6 * n_long
    look = np.unique(np.r_[0:min(B, 4), B - 1])
    tri = oracle.dense_to_triples(table)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a[look], b[look], want_pre=True)
    f = dol.FnTable.create_dense(table)
    assert "byj" in f.kernel_at(False, B) or na == 1200
    out = dol.Dist.empty(f.out_syms, B)
    dol.apply2(dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b)), f, None, out)
    assert_close(host(out.prob)[look], want, "forward")
    np.testing.assert_array_equal(host(out.prob)[look] == 1.0, pre32 >= 1.0)


def lane_tree(x, pairs_first):
    """The sum over the last axis as lanes exchange them: neighbours first, or the lane half of them away first.  float32."""
    while x.shape[-1] > 1:
        x = x[..., 0::2] + x[..., 1::2] if pairs_first else x[..., :x.shape[-1] // 2] + x[..., x.shape[-1] // 2:]
    return x[..., 0]


def fma32(a, b, c):
    """float32 fused multiply-add; exact before the one rounding for factors of 16 bits and sums of less than 2^20 times their unit."""
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


@pytest.mark.parametrize("na,nb,B", [(250, 10, 3), (257, 3, 2), (1000, 10, 2), (1011, 4, 5), (1009, 9, 2)])
def test_dense_map_sums_keep_their_order(dol, na, nb, B):
    """The short operand's gradient bit for bit: a lane's rows 64 apart, four at a time, neighbouring lanes' sums first, then rows
    of 16, halves and wavefronts in order, each wavefront 256 rows."""
    ids = (W.splitmix64(61 + na, np.arange(na * nb)) % np.uint64(2 * na)).astype(np.int32).reshape(na, nb)
    f = dol.FnTable.create_dense(ids)
    assert f.kernel_at(True, B).startswith("damp_byj_bwd"), f.kernel_at(True, B)
    bits = lambda seed, n: (W.splitmix64(seed, np.arange(n)) % np.uint64(1 << 16)).astype(np.float32)
    a = bits(1, B * na).reshape(B, na) * np.float32(2.0 ** -26)
    b = bits(2, B * nb).reshape(B, nb) * np.float32(2.0 ** -16)
    g = (bits(3, B * f.n_out).reshape(B, f.n_out) - np.float32(32768.0)) * np.float32(2.0 ** -12)
    da, db, out = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b)), dol.Dist.empty(f.out_syms, B)
    dol.apply2(da, db, f, None, out)
    assert float(out.prob.max()) < 1.0
    ga, gb = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    rows = -(-na // 256) * 256
    v, av = np.zeros((B, nb, rows), np.float32), np.zeros((B, 1, rows), np.float32)
    v[:, :, :na] = np.moveaxis(g[:, np.searchsorted(f.out_syms, ids)], 2, 1)
    av[:, 0, :na] = a
    v, av = v.reshape(B, nb, -1, 4, 64), av.reshape(B, 1, -1, 4, 64)
    acc = np.zeros((B, nb, rows // 256, 64), np.float32)
    for x in range(4):
        acc = fma32(v[:, :, :, x], np.broadcast_to(av[:, :, :, x], acc.shape), acc)
    shares = lane_tree(acc, True)
    want = np.zeros((B, nb), np.float32)
    for w in range(shares.shape[-1]):
        want = want + shares[..., w]
    np.testing.assert_array_equal(host(gb), want)


@pytest.mark.parametrize("na,B", [(19, 64), (28, 16), (100, 80)])
def test_sum_table_sums_keep_their_order(dol, na, B):
    """The same for a table of sums, whose samples have 32 lanes each (in whole tiles: what is left of a batch is summed in stretches)."""
    nb = 10
    f = dol.FnTable.create_dense(np.add.outer(np.arange(na), np.arange(nb)).astype(np.int32))
    assert f.kernel_at(True, B).startswith("damp_conv_bwd_tile_kernel"), f.kernel_at(True, B)
    bits = lambda seed, n: (W.splitmix64(seed, np.arange(n)) % np.uint64(1 << 16)).astype(np.float32)
    a = bits(4, B * na).reshape(B, na) * np.float32(2.0 ** -24)
    b = bits(5, B * nb).reshape(B, nb) * np.float32(2.0 ** -20)
    g = (bits(6, B * f.n_out).reshape(B, f.n_out) - np.float32(32768.0)) * np.float32(2.0 ** -12)
    da, db, out = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b)), dol.Dist.empty(f.out_syms, B)
    dol.apply2(da, db, f, None, out)
    ga, gb = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    rows = -(-na // 32) * 32
    acc = np.zeros((B, nb, 32), np.float32)
    for i0 in range(0, rows, 32):
        live = np.arange(i0, min(i0 + 32, na))
        for j in range(nb):
            acc[:, j, :live.size] = fma32(g[:, live + j], a[:, live], acc[:, j, :live.size])
    np.testing.assert_array_equal(host(gb), lane_tree(acc, True))


@pytest.mark.parametrize("batch,n_sym,n_facts,k", [(2, 60, 63, 1), (3, 1100, 9, 2), (300, 130, 41, 3), (1, 2500, 17, 5)])
def test_dtkp_gradient_sums_keep_their_order(dol, batch, n_sym, n_facts, k):
    """The top-k gradient bit for bit: a lane's symbols ascending, the lane 32 away first, the nearest last, wavefronts in order, every share
    divided by the fact's probability (1/2, so that the quotient is exact)."""
    masks = (np.uint64(1) << (W.splitmix64(71 + n_facts, np.arange(2 * batch * n_sym * k)).reshape(2, batch, n_sym, k) % np.uint64(n_facts)))
    masks = masks[0] | masks[1]
    masks[:, ::7, k - 1] = oracle.ABSENT
    prob = (W.uniform01(72, masks.size).astype(np.float32).reshape(masks.shape) * np.float32(0.9 / k))
    prob[masks == oracle.ABSENT] = 0.0
    g = W.normal(73, batch * n_sym).astype(np.float32).reshape(batch, n_sym)
    dist = dol.Dist.empty(np.arange(n_sym, dtype=np.int32), batch, k=k)
    dist.proof_mask.copy_(dev(masks.view(np.int64)))
    dist.proof_prob.copy_(dev(prob))
    gf = torch.empty((batch, n_facts), device="cuda")
    dol.dtkp_backward(dist, dol.Prov(dol.DTKP, k, torch.full((batch, n_facts), 0.5, device="cuda"), None), dev(g), gf)
    waves = max(1, min(16, -(-n_sym // 64)))
    steps = -(-n_sym // (64 * waves))
    coef, held = np.zeros((batch, steps * waves * 64, k), np.float32), np.zeros((batch, steps * waves * 64, k), np.uint64)
    coef[:, :n_sym] = g[:, :, None] * prob
    held[:, :n_sym] = np.where(masks == oracle.ABSENT, np.uint64(0), masks)
    coef, held = coef.reshape(batch, steps, waves, 64, k), held.reshape(batch, steps, waves, 64, k)
    want = np.zeros((batch, n_facts), np.float32)
    for j in range(n_facts):
        acc = np.zeros((batch, waves, 64), np.float32)
        for t in range(steps):
            for x in range(k):
                acc = acc + np.where((held[:, t, :, :, x] >> np.uint64(j)) & np.uint64(1) == 1, coef[:, t, :, :, x], np.float32(0.0))
        shares = lane_tree(acc, False)
        for w in range(waves):
            want[:, j] = want[:, j] + shares[:, w] * np.float32(2.0)
    np.testing.assert_array_equal(host(gf), want)


@pytest.mark.parametrize("nb", [4, 16, 40])
@pytest.mark.parametrize("extra,batch", [(0, 3), (57, 1), (4096, 2), (4097, 300)])
def test_workgroup_per_sample_kernels(dol, nb, extra, batch):
    """The kernels that give a sample a workgroup: columns of every kind of length (a lane each up to 64 tuples, a wavefront,
    the workgroup above 512), result rows on either side of a block of 4 096 columns and of a part per workgroup, rows that
    are not multiples of four.  A column's tags sum to within a few roundings of 1, so its clamp decision, seen through the
    backward pass, must be the sequential float sum's; one long column hides its tail behind a large first term."""
    lengths = [1, 2, 3, 4, 5, 16, 17, 63, 64, 65, 130, 511, 512, 513, 1500] + [4 if nb <= 16 else 1 + c % 3 for c in range(extra)]
    total = sum(lengths)
    col = np.repeat(np.arange(len(lengths)), lengths).astype(np.int32)
    first = np.repeat(np.cumsum([0] + lengths[:-1]), lengths)
    i = np.arange(total, dtype=np.int32)
    j = ((i - first) % nb).astype(np.int32)
    w = W.uniform01(900 + nb, batch * total).reshape(batch, total) ** 3 + 1e-9
    w[:, first[col == 14][0]] *= 1e4
    sums = np.add.reduceat(w, np.unique(first), axis=1)
    a = (w / sums[:, col] * (1.0 + 1e-7 * ((np.arange(len(lengths)) * 7 + np.arange(batch)[:, None] * 3) % 5 - 2))[:, col]).astype(np.float32)
    b = np.ones((batch, nb), np.float32)
    tri = (i, j, col)
    syms, want, pre32, pre64 = oracle.damp_apply2_fwd(tri, total, nb, a, b, want_pre=True)
    assert (pre32 > 1).any() and (pre32 <= 1).any() and np.abs(pre64 - 1).max() < 1e-5
    f = dol.FnTable.create_sparse(total, nb, *tri)
    da, db = dol.Dist(np.arange(total), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(f.out_syms, batch)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "forward")
    np.testing.assert_array_equal(host(out.prob) == 1.0, pre32 >= 1.0)
    g = (np.abs(W.normal(901, batch * syms.size)) + 0.5).astype(np.float32).reshape(batch, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, total, nb, a, b, g)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    rec = dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f)
    dol.backward(rec, dev(g), ga, gb)
    assert_close(host(ga), wa, "backward a")
    assert_close(host(gb), wb, "backward b")
    rec3 = dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f, accumulate=3)
    dol.backward(rec3, dev(g), ga, gb)
    assert_close(host(ga), 2.0 * wa.astype(np.float64), "backward a accumulated")
    assert_close(host(gb), 2.0 * wb.astype(np.float64), "backward b accumulated")


@pytest.mark.parametrize("na,nb,n_ids,batch", [(50, 37, 201, 4097), (13, 12, 30, 8200), (101, 10, 226, 8193)])
def test_tiles_of_64_samples_at_large_batches(dol, na, nb, n_ids, batch):
    """The kernels over tiles of 64 samples, which serve tables of this size above 4 096 (8 192) samples: ragged symbol counts
    and a last tile that is not full, columns on either side of the clamp."""
    tab = W.hashed_table(61, na, nb, n_ids)
    tab[0, :] = -1
    a = (W.uniform01(62, batch * na) * 0.5).astype(np.float32).reshape(batch, na)
    b = (W.uniform01(63, batch * nb) * 0.8).astype(np.float32).reshape(batch, nb)
    tri = oracle.dense_to_triples(tab)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    f = dol.FnTable.create_dense(tab)
    assert f.kernel_at(False, batch) == "damp_lds_fwd_kernel" and f.kernel_at(True, batch) == "damp_lds_bwd_kernel"
    assert f.kernel_at(False, 64) != f.kernel_at(False, batch)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(syms, batch)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "tiles forward")
    np.testing.assert_array_equal(host(out.prob) == 1.0, pre32 >= 1.0)
    g = np.abs(W.normal(64, batch * syms.size)).astype(np.float32).reshape(batch, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    assert_close(host(ga), wa, "tiles backward a")
    assert_close(host(gb), wb, "tiles backward b")


@pytest.mark.parametrize("na,nb,n_ids,batch", [(63, 61, 255, 8193), (50, 37, 201, 10007), (5, 64, 66, 53000), (64, 6, 64, 45001), (33, 47, 1023, 16390),
                                               (29, 64, 5, 9101), (50, 40, 129, 17000), (63, 61, 330, 5001)])
def test_generated_tables_of_any_symbol_counts(dol, na, nb, n_ids, batch):
    """The code written for a table whose rows are not whole 16-byte pieces: every remainder of each count, result rows of one
    to sixteen groups, last tiles of which the words are no whole pieces, every build (up to 8 192 and 16 384 samples and above), columns
    on either side of the clamp, a sample of NaN and one of infinities, accumulation and one-sided calls."""
    tab = W.hashed_table(65, na, nb, n_ids)
    f = dol.FnTable.create_dense(tab)
    assert f.kernel_at(False, batch) == "damp_table_fwd_kernel" and f.kernel_at(True, batch) == "damp_table_bwd_kernel"
    a = (W.uniform01(66, batch * na) * (2.0 * n_ids / (na * nb))).astype(np.float32).reshape(batch, na)
    b = W.uniform01(67, batch * nb).astype(np.float32).reshape(batch, nb)
    a[1::4] *= 2.2                                # (long columns all lie near half the scale)
    a[batch // 3] *= 1e-3
    odd = [64, 65]
    a[64, 1], b[65, 2] = np.nan, np.inf
    look = np.unique(np.concatenate([np.arange(0, batch, max(1, batch // 700)), np.arange(batch - 70, batch), np.arange(0, 70)]))
    look = look[~np.isin(look, odd)]
    tri = oracle.dense_to_triples(tab)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a[look], b[look], want_pre=True)
    da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
    buf = torch.full((batch * syms.size + 16,), -3.0, device="cuda")          # (nothing past the last row is written)
    out = dol.Dist(syms, buf[:batch * syms.size].view(batch, syms.size))
    dol.apply2(da, db, f, None, out)
    got = host(out.prob)
    assert_close(got[look], want, "forward")
    np.testing.assert_array_equal(got[look] == 1.0, pre32 >= 1.0)
    assert np.all(host(buf[batch * syms.size:]) == -3.0) and (want == 1.0).any() and (want < 1.0).any()
    # (a sum with NaN or infinity in it is clamped to 1, wherever the kernels meet it)
    hit = np.zeros(syms.size, bool)
    for c in np.searchsorted(syms, np.unique(tab[1][tab[1] >= 0])):
        hit[c] = True
    np.testing.assert_array_equal(got[64][hit], 1.0)
    g = np.abs(W.normal(68, batch * syms.size)).astype(np.float32).reshape(batch, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a[look], b[look], g[look])
    rec = dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f)
    ga, gb = torch.full_like(da.prob, 5.0), torch.full_like(db.prob, 5.0)
    dol.backward(rec, dev(g), ga, gb)
    assert_close(host(ga)[look], wa, "backward a")
    assert_close(host(gb)[look], wb, "backward b")
    only = torch.full_like(db.prob, 5.0)
    dol.backward(rec, dev(g), None, only)
    np.testing.assert_array_equal(host(only)[look], host(gb)[look])
    acc = dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f, accumulate=3)
    once_a, once_b = host(ga)[look].astype(np.float64), host(gb)[look].astype(np.float64)
    dol.backward(acc, dev(g), ga, gb)
    assert_close(host(ga)[look], 2.0 * once_a, "backward a accumulated")
    assert_close(host(gb)[look], 2.0 * once_b, "backward b accumulated")


@pytest.mark.parametrize("na,nb,n_ids", [(13, 12, 30), (50, 37, 201), (101, 10, 226), (101, 10, 9), (226, 10, 442), (442, 10, 785), (100, 100, 50),
                                         (128, 30, 700), (30, 30, 2), (64, 64, 32), (16, 16, 200)])
def test_a_result_does_not_depend_on_the_batch_it_is_in(dol, na, nb, n_ids):
    """Tables that are served by tiles in large batches and by a workgroup per sample in small ones: every bit of a sample's
    result is the same, for short and long columns, sums on either side of the clamp and infinities and NaN among the tags."""
    B, few = 8200, 37
    f = dol.FnTable.create_dense(W.hashed_table(71, na, nb, n_ids))
    assert f.kernel_at(False, B) in ("damp_lds_fwd_kernel", "damp_table_fwd_kernel")
    a = torch.from_numpy((W.uniform01(72, B * na) ** 4 * (6.0 * n_ids / (na * nb))).astype(np.float32).reshape(B, na)).cuda()
    b = torch.from_numpy(W.uniform01(73, B * nb).astype(np.float32).reshape(B, nb)).cuda()
    a[few - 1, 1], a[few - 2, 0] = float("nan"), float("inf")
    whole = dol.Dist.empty(f.out_syms, B)
    dol.apply2(dol.Dist(np.arange(na), a), dol.Dist(np.arange(nb), b), f, None, whole)
    for first in (0, B - few):
        part = dol.Dist.empty(f.out_syms, few)
        dol.apply2(dol.Dist(np.arange(na), a[first:first + few].contiguous()), dol.Dist(np.arange(nb), b[first:first + few].contiguous()), f, None, part)
        np.testing.assert_array_equal(host(part.prob).view(np.int32), host(whole.prob[first:first + few].contiguous()).view(np.int32))
    p = host(whole.prob)
    assert (p < 1.0).any() and (p == 1.0).any()


@pytest.mark.parametrize("na,nb,n_ids,large", [(50, 37, 201, 0), (63, 61, 255, 16385), (61, 5, 77, 0), (33, 47, 1023, 0), (63, 63, 1021, 0)])
def test_ragged_rows_keep_their_bits_where_generated_code_takes_over(dol, na, nb, n_ids, large):
    """The first batch that generated code serves and the last one below it, a few samples, and a batch of another build: every
    bit of a sample's result is the same, sums on either side of the clamp and samples with NaN and infinity among them."""
    f = dol.FnTable.create_dense(W.hashed_table(74, na, nb, n_ids))
    at = (1 << 24) // (na * nb)
    assert f.kernel_at(False, at) == "damp_table_fwd_kernel" and f.kernel_at(False, at - 1) != "damp_table_fwd_kernel"
    B = max(at, large)
    a = torch.from_numpy((W.uniform01(75, B * na) ** 4 * (6.0 * n_ids / (na * nb))).astype(np.float32).reshape(B, na)).cuda()
    b = torch.from_numpy(W.uniform01(76, B * nb).astype(np.float32).reshape(B, nb)).cuda()
    a[5, 1], a[6, 0], b[7, 2] = float("nan"), float("inf"), float("inf")

    def run(n):
        out = dol.Dist.empty(f.out_syms, n)
        dol.apply2(dol.Dist(np.arange(na), a[:n].contiguous()), dol.Dist(np.arange(nb), b[:n].contiguous()), f, None, out)
        return host(out.prob).view(np.int32)

    whole = run(B)
    for n in (at, at - 1, 37):
        np.testing.assert_array_equal(run(n), whole[:n])
    p = whole.view(np.float32)
    assert (p < 1.0).any() and (p == 1.0).any()


def test_ragged_backward_goes_by_samples_a_little_longer(dol):
    """Result rows of hundreds of symbols, whose reverse pass no other tile serves: a workgroup per sample past the line at
    which forward passes take generated code, and generated code above."""
    f = dol.FnTable.create_dense(W.hashed_table(81, 63, 63, 1021))
    at = (1 << 24) // (63 * 63) + 1
    assert f.kernel_at(False, at) == "damp_table_fwd_kernel" and f.kernel_at(True, at) == "damp_apply2_bwd_staged_kernel"
    assert f.kernel_at(True, 8456) == "damp_table_bwd_kernel"


@pytest.mark.parametrize("na,nb,n_ids,backward", [(63, 63, 1021, True), (128, 128, 200, False), (300, 8, 20, False), (13, 12, 30, False), (100, 100, 50, True),
                                                  (32, 40, 128, True), (20, 20, 20, True)])
def test_both_sides_of_the_choice_between_tiles_and_a_workgroup_per_sample(dol, na, nb, n_ids, backward):
    """The last batch that goes by samples and the first one in tiles: one such place for a table, the earlier the more work
    its samples are, and the same results on both sides."""
    tab = W.hashed_table(81, na, nb, n_ids)
    f = dol.FnTable.create_dense(tab)
    tiles = f.kernel_at(backward, 100000)
    assert tiles.startswith(("damp_lds_", "damp_table_"))
    by_sample = [f.kernel_at(backward, batch) != tiles for batch in range(1, 8300)]
    few = by_sample.index(False)
    assert few > 256 and not any(by_sample[few:])
    for batch in (few, few + 1):
        a = (W.uniform01(82, batch * na) * (2.0 * n_ids / (na * nb))).astype(np.float32).reshape(batch, na)
        b = W.uniform01(83, batch * nb).astype(np.float32).reshape(batch, nb)
        tri = oracle.dense_to_triples(tab)
        syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
        da, db = dol.Dist(np.arange(na), dev(a)), dol.Dist(np.arange(nb), dev(b))
        out = dol.Dist.empty(syms, batch)
        dol.apply2(da, db, f, None, out)
        assert_close(host(out.prob), want, "forward")
        np.testing.assert_array_equal(host(out.prob) == 1.0, pre32 >= 1.0)
        if backward:
            g = np.abs(W.normal(84, batch * syms.size)).astype(np.float32).reshape(batch, -1)
            wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
            ga, gb = torch.empty_like(da.prob), torch.empty_like(db.prob)
            dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
            assert_close(host(ga), wa, "backward a")
            assert_close(host(gb), wb, "backward b")


def test_more_samples_than_one_launch_has_workgroups(dol):
    """A workgroup per sample for one sample more than a launch of 2^32 - 1 threads holds at 1 024 threads each: the samples
    around the border and at both ends."""
    B, na, nb, n_ids = (1 << 22), 700, 1, 5
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 30 GB of GPU memory")
    tab = W.hashed_table(91, na, nb, n_ids)
    f = dol.FnTable.create_dense(tab)
    assert not f.kernel_at(False, B).startswith(("damp_lds", "damp_table", "damp_conv"))
    rows = (W.uniform01(92, 1024 * na) * 0.01).astype(np.float32).reshape(1024, na)
    a = dev(rows).repeat(B // 1024, 1)
    b = torch.ones(B, nb, device="cuda")
    tri = oracle.dense_to_triples(tab)
    g = np.abs(W.normal(93, 1024 * n_ids)).astype(np.float32).reshape(1024, -1)
    _, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, rows, np.ones((1024, nb), np.float32), want_pre=True)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, rows, np.ones((1024, nb), np.float32), g)
    da, db = dol.Dist(np.arange(na), a), dol.Dist(np.arange(nb), b)
    out = dol.Dist(f.out_syms, torch.full((B, f.n_out), -1.0, device="cuda"))
    dol.apply2(da, db, f, None, out)
    ga, gb = torch.full_like(a, -1.0), torch.full_like(b, -1.0)
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g).repeat(B // 1024, 1), ga, gb)
    for first in (0, B - 1024):                     # (the border lies in the last 1 024)
        assert_close(host(out.prob[first:first + 1024]), want, "forward")
        assert_close(host(ga[first:first + 1024]), wa, "backward a")
        assert_close(host(gb[first:first + 1024]), wb, "backward b")


# ---------------------------------------------------------------- seeded random tables over every kernel choice

@pytest.mark.parametrize("seed", range(24))
def test_random_tables_differential(dol, seed):
    """Random table shapes, densities, image counts, batch sizes and paddings (drawn from a seeded stream), so that
    every kernel the library can pick for dol_apply2 / dol_backward (LDS gather, per-j maps with and without the
    workgroup-per-sample backward, tuple lists, wavefront columns and rows) meets the oracle on shapes nobody chose
    by hand.  One-signed upstream gradient (see the module docstring)."""
    r = W.splitmix64(5000 + seed, np.arange(16)).astype(np.uint64)
    pick = lambda k, lo, hi: int(lo + r[k] % np.uint64(hi - lo + 1))
    na = [pick(0, 1, 40), pick(0, 100, 700), pick(0, 1025, 3000)][seed % 3]
    nb = [pick(1, 1, 16), pick(1, 17, 60), pick(1, 1, 4)][(seed // 3) % 3]
    n_ids = max(1, [pick(2, 1, 8), pick(2, na // 2 + 1, na + nb), pick(2, 2 * na, 3 * na)][(seed // 9) % 3])
    batch = pick(3, 1, 70)
    table = (W.splitmix64(6000 + seed, np.arange(na * nb)) % np.uint64(n_ids)).astype(np.int32).reshape(na, nb)
    drop = pick(4, 0, 3)
    if drop:
        table.reshape(-1)[::drop + 1] = -1
    scale = [1.0, 1.0, float(max(1.0, 0.7 * n_ids))][pick(5, 0, 2)]
    a = (W.softmax_rows(W.normal(7000 + seed, batch * na).reshape(batch, na)) * scale).astype(np.float32)
    b = W.softmax_rows(W.normal(8000 + seed, batch * nb).reshape(batch, nb))
    tri = oracle.dense_to_triples(table)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, na, nb, a, b, want_pre=True)
    g = np.abs(W.normal(9000 + seed, batch * max(syms.size, 1))).astype(np.float32).reshape(batch, -1)[:, :syms.size]
    g = np.ascontiguousarray(g)
    wa, wb = oracle.damp_apply2_bwd(tri, na, nb, a, b, g)
    f = dol.FnTable.create_dense(table)
    np.testing.assert_array_equal(f.out_syms, syms)
    pad = pick(6, 0, 5)
    abuf = torch.zeros((batch, na + pad), device="cuda")
    abuf[:, :na] = dev(a)
    da, db = dol.Dist(np.arange(na), abuf[:, :na]), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(f.out_syms, batch)
    dol.apply2(da, db, f, None, out)
    what = "seed %d: %d x %d -> %d, batch %d, %s / %s" % (seed, na, nb, syms.size, batch, f.kernel_fwd, f.kernel_bwd)
    assert_close(host(out.prob), want, what + " forward")
    ga = torch.full((batch, na + pad), 3.0, device="cuda")
    gb = torch.empty((batch, nb), device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    assert_close(host(ga)[:, :na], wa, what + " grad a")
    assert np.all(host(ga)[:, na:] == 3.0)
    assert_close(host(gb), wb, what + " grad b")


@pytest.mark.parametrize("seed", range(8))
def test_random_tables_differential_dtkp(dol, seed):
    """The same under DTKP-AM: multi-proof operands (results of earlier applies over shared exclusion groups), few
    images so that columns run from a handful to hundreds of tuples (thread and wavefront kernels), k from 1 to 5;
    also the K-operand call on the same table."""
    r = W.splitmix64(5100 + seed, np.arange(8)).astype(np.uint64)
    k = [1, 2, 3, 5][seed % 4]
    B, nv = int(3 + r[0] % np.uint64(40)), 6
    fp = np.concatenate([W.softmax_rows(W.normal(5200 + seed * 4 + t, B * nv).reshape(B, nv)) for t in range(4)], axis=1)
    grp = np.repeat(np.arange(4), nv).astype(np.int32)
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    o_ops, g_ops = [], []
    for side in range(2):
        n_mid = int(8 + r[1 + side] % np.uint64(25))
        tab = (W.splitmix64(5300 + seed * 2 + side, np.arange(nv * nv)) % np.uint64(n_mid)).astype(np.int32).reshape(nv, nv)
        m0 = oracle.dtkp_init(np.arange(nv) + nv * (2 * side), fp, k)[0]
        m1 = oracle.dtkp_init(np.arange(nv) + nv * (2 * side + 1), fp, k)[0]
        s, m, p, _ = oracle.dtkp_apply2(oracle.dense_to_triples(tab), nv, nv, k, grp, fp, m0, m1)
        d0, d1 = dol.Dist.empty(np.arange(nv), B, k=k), dol.Dist.empty(np.arange(nv), B, k=k)
        dol.dtkp_init(d0, np.arange(nv) + nv * (2 * side), prov)
        dol.dtkp_init(d1, np.arange(nv) + nv * (2 * side + 1), prov)
        ft = dol.FnTable.create_dense(tab)
        d = dol.Dist.empty(ft.out_syms, B, k=k)
        dol.apply2(d0, d1, ft, prov, d)
        o_ops.append((s, m)); g_ops.append(d)
    na, nb = o_ops[0][0].size, o_ops[1][0].size
    n_ids = int(1 + r[3] % np.uint64(6))
    table = (W.splitmix64(5400 + seed, np.arange(na * nb)) % np.uint64(n_ids)).astype(np.int32).reshape(na, nb)
    table.reshape(-1)[::7] = -1
    tri = oracle.dense_to_triples(table)
    syms, om, op, opr = oracle.dtkp_apply2(tri, na, nb, k, grp, fp, o_ops[0][1], o_ops[1][1])
    f = dol.FnTable.create_dense(table)
    out = dol.Dist.empty(f.out_syms, B, k=k)
    dol.apply2(g_ops[0], g_ops[1], f, prov, out)
    np.testing.assert_array_equal(out.sym_ids, syms)
    np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), om)
    np.testing.assert_array_equal(host(out.proof_prob), op)
    assert_close(host(out.prob), opr, "dtkp random table, seed %d" % seed)
    fk = dol.FnkTable.create_dense(table)
    outk = dol.Dist.empty(fk.out_syms, B, k=k)
    dol.apply_k(g_ops, fk, prov, outk)
    np.testing.assert_array_equal(host(outk.proof_mask).view(np.uint64), om)
    np.testing.assert_array_equal(host(outk.proof_prob), op)
    gsym = W.normal(5500 + seed, B * syms.size).astype(np.float32).reshape(B, -1)
    want = oracle.dtkp_prob_bwd(om, fp, gsym)
    gf = torch.empty((B, fp.shape[1]), device="cuda")
    dol.dtkp_backward(out, prov, dev(gsym), gf)
    assert_close(host(gf), want, "dtkp random table gradient, seed %d" % seed)


@pytest.mark.parametrize("batch,n", [(1, 1), (3, 5), (65, 63), (4100, 64), (2, 65), (700, 196), (9, 256), (33, 257), (5, 513), (3, 1200), (20000, 3)])
@pytest.mark.parametrize("pad", [0, 3])
def test_filter_and_union_of_any_width(dol, batch, n, pad):
    """Filter, Union and their reverse over rows of every kind of width and stride (several rows side by side in a workgroup,
    several workgroups side by side on a row), overwriting and accumulating, with either gradient left out."""
    def rows(seed, m):
        x = torch.zeros((batch, m + pad), device="cuda")
        x[:, :m] = dev((W.uniform01(seed, batch * m) * 0.8).astype(np.float32).reshape(batch, m))
        return x[:, :m]
    keep = (W.splitmix64(5, np.arange(n)) % np.uint64(3) > 0).astype(np.uint8)
    keep[-1] = 1
    a = dol.Dist(np.arange(n), rows(1, n))
    kept = dol.Dist(dol.filter_plan(a, keep), rows(2, int(keep.sum())))
    dol.filter(a, keep, None, kept)
    at = torch.as_tensor(np.flatnonzero(keep), device="cuda")
    assert torch.equal(kept.prob, a.prob[:, at])
    g, ga = rows(3, kept.n_sym), rows(4, n)
    want = torch.zeros_like(a.prob)
    want[:, at] = g
    for acc in (0, 1):
        before = ga.clone()
        dol.backward(dol.OpRecord(dol.OP_FILTER, a, None, kept, pred_mask=keep, accumulate=acc), g, ga, None)
        assert torch.equal(ga, before + want if acc else want)
    # union with symbols that overlap a's in part
    sb = np.arange(n // 2, n // 2 + n + 2)
    b = dol.Dist(sb, rows(6, sb.size))
    u = dol.Dist(dol.union_plan(a, b), rows(7, n // 2 + n + 2))
    dol.union(a, b, None, u)
    lo, m = n // 2, n - n // 2
    total = torch.zeros((batch, u.n_sym), device="cuda")
    total[:, :n] = a.prob
    total[:, lo:] += b.prob
    both = torch.zeros(u.n_sym, dtype=torch.bool, device="cuda")
    both[lo:lo + m] = True
    assert torch.equal(u.prob, torch.where(both, total.clamp(max=1.0), total))
    g, ga, gb = rows(8, u.n_sym), rows(9, n), rows(10, sb.size)
    gate = torch.where(both & (total > 1.0), torch.zeros_like(g), g)
    for acc in (0, 1, 2, 3):
        before = (ga.clone(), gb.clone())
        dol.backward(dol.OpRecord(dol.OP_UNION, a, b, u, accumulate=acc), g, ga, gb)
        assert torch.equal(ga, before[0] + gate[:, :n] if acc & 1 else gate[:, :n])
        assert torch.equal(gb, before[1] + gate[:, lo:] if acc & 2 else gate[:, lo:])
    for x, y in ((rows(11, n), None), (None, rows(12, sb.size))):
        dol.backward(dol.OpRecord(dol.OP_UNION, a, b, u), g, x, y)
        assert torch.equal(x, gate[:, :n]) if x is not None else torch.equal(y, gate[:, lo:])


@pytest.mark.parametrize("batch,n", [(1, 64), (70, 40), (5, 300), (600, 200), (3, 1100)])
@pytest.mark.parametrize("kept_at", ["none", "first", "last", "every 70th"])
def test_filter_backward_where_few_columns_have_a_source(dol, batch, n, kept_at):
    """Wavefronts of columns of which none, one or a few were kept; the fused filter-union's reverse beside it, and tags of NaN
    and infinity in the operand, which no dropped column may pick up."""
    keep = np.zeros(n, np.uint8)
    keep[{"none": [], "first": [0], "last": [n - 1], "every 70th": list(range(0, n, 70))}[kept_at]] = 1
    a = dol.Dist(np.arange(n), dev((W.uniform01(1, batch * n) * 0.8).astype(np.float32).reshape(batch, n)))
    a.prob[:, keep == 0] = float("nan")
    kept = dol.Dist.empty(np.flatnonzero(keep), batch) if keep.any() else dol.Dist(np.empty(0, np.int32), torch.empty((batch, 0), device="cuda"))
    at = torch.as_tensor(np.flatnonzero(keep), device="cuda")
    g = dev(W.normal(2, batch * kept.n_sym).astype(np.float32).reshape(batch, -1))
    want = torch.zeros_like(a.prob)
    want[:, at] = g
    ga = torch.full_like(a.prob, float("nan"))
    for acc in (0, 1):
        dol.backward(dol.OpRecord(dol.OP_FILTER, a, None, kept, pred_mask=keep, accumulate=acc), g, ga, None)
        assert torch.equal(ga, (1 + acc) * want)
    c = dol.Dist(np.arange(n // 2, n // 2 + n), dev((W.uniform01(3, batch * n) * 0.8).astype(np.float32).reshape(batch, n)))
    u = dol.Dist.empty(dol.filter_union_plan(a, keep, c), batch)
    dol.filter_union(a, keep, c, None, u)
    g = dev(W.normal(4, batch * u.n_sym).astype(np.float32).reshape(batch, -1))
    gc = torch.full_like(c.prob, float("nan"))
    dol.backward(dol.OpRecord(dol.OP_FILTER_UNION, a, c, u, pred_mask=keep), g, ga, gc)
    pos = {int(x): i for i, x in enumerate(u.sym_ids)}
    wa, wc = torch.zeros_like(a.prob), g[:, [pos[int(x)] for x in c.sym_ids]].clone()
    for x in np.flatnonzero(keep):
        gx = g[:, pos[int(x)]].clone()
        if x >= n // 2:
            over = a.prob[:, x] + c.prob[:, x - n // 2] > 1.0
            gx[over] = 0.0
            wc[over, x - n // 2] = 0.0
        wa[:, x] = gx
    assert torch.equal(ga, wa) and torch.equal(gc, wc)


@pytest.mark.parametrize("batch,lengths", [(1, (4, 5)), (1, (16, 17)), (3, (1, 16, 17, 64, 65, 5, 4)), (9, (1025, 2, 1024, 65, 64, 17, 40, 33, 3, 5, 4, 7)), (5, (1500,) + (20,) * 33)])
def test_dtkp_columns_of_every_length(dol, batch, lengths):
    """A lane, 4 lanes, 16, a wavefront and a workgroup per column in one launch: lengths on both sides of each limit, groups of
    columns that do not fill their workgroup, a second operand given by its facts and by its lists, and a unary function."""
    k, nb, n_facts = 3, 6, 24
    n = sum(lengths)
    na = -(-n // nb)
    fp = W.uniform01(41, batch * n_facts).astype(np.float32).reshape(batch, n_facts)
    grp = np.concatenate([np.arange(18), np.full(6, 18)]).astype(np.int32)
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    # first operand: up to k proofs of two facts per symbol (a table of 18 x 18 onto its symbols)
    pair = (W.splitmix64(42, np.arange(18 * 18)) % np.uint64(na)).astype(np.int32).reshape(18, 18)
    pair.reshape(-1)[:min(na, 324)] = np.arange(min(na, 324))
    one = oracle.dtkp_init(np.arange(18), fp, k)
    syms, am, ap, _ = oracle.dtkp_apply2(oracle.dense_to_triples(pair), 18, 18, k, grp, fp, one[0], one[0])
    which = np.arange(na) % syms.size                  # (symbols past those repeat them)
    am, ap = np.ascontiguousarray(am[:, which]), np.ascontiguousarray(ap[:, which])
    fact_b = np.arange(18, 24, dtype=np.int32)
    bm = oracle.dtkp_init(fact_b, fp, k)
    col = np.repeat(np.arange(len(lengths)), lengths)[np.argsort(W.splitmix64(43, np.arange(n)))].astype(np.int32)
    table = np.full(na * nb, -1, np.int32)
    table[:n] = col
    so, om, op, opr = oracle.dtkp_apply2(oracle.dense_to_triples(table.reshape(na, nb)), na, nb, k, grp, fp, am, bm[0])
    f = dol.FnTable.create_dense(table.reshape(na, nb))
    a = dol.Dist(np.arange(na), torch.zeros((batch, na), device="cuda"), dev(am.view(np.int64)), dev(ap))
    b = dol.Dist.empty(np.arange(nb), batch, k=k)
    dol.dtkp_init(b, fact_b, prov)
    for call in (lambda out: dol.apply2(a, b, f, prov, out), lambda out: dol.dtkp_apply2_input(a, fact_b, f, prov, out)):
        out = dol.Dist.empty(f.out_syms, batch, k=k)
        call(out)
        np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), om)
        np.testing.assert_array_equal(host(out.proof_prob), op)
        assert_close(host(out.prob), opr, "dtkp columns")
    # a unary function with the same columns
    m1, p1 = np.ascontiguousarray(am[:, np.arange(n) % na]), np.ascontiguousarray(ap[:, np.arange(n) % na])
    idx, to = oracle.dense_to_tuples(col)
    s1, um, up, upr = oracle.dtkp_applyk(idx, to, k, grp, fp, [m1])
    fu = dol.FnkTable.create_dense(col)
    x = dol.Dist(np.arange(n), torch.zeros((batch, n), device="cuda"), dev(m1.view(np.int64)), dev(p1))
    out = dol.Dist.empty(fu.out_syms, batch, k=k)
    dol.apply_k([x], fu, prov, out)
    np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), um)
    np.testing.assert_array_equal(host(out.proof_prob), up)
    assert_close(host(out.prob), upr, "dtkp unary columns")


@pytest.mark.parametrize("k", [1, 2, 4, 5])
@pytest.mark.parametrize("apart", [False, True])
@pytest.mark.parametrize("values", [None, (0.5, 0.25, 1.0, 0.0), (0.5, 1e-30, 3e-39, 1.0)], ids=["random", "equal", "tiny"])
def test_dtkp_columns_ranked_by_keys(dol, k, values, apart):
    """Columns of 1 to 70 tuples (a lane, four, 16 and a wavefront) where a list is ranked by probability and origin alone, on
    both sides of the longest such list: probabilities all different, drawn from four values (equal ones within a lane, between
    lanes and on the cut, proofs of probability 0), and so small that products underflow.  apart: the same where the first
    facts' neighbours differ in every other sample, which lets columns with equal probabilities be ranked all the same."""
    lengths, batch, nb, n_facts = (1, 2, 3, 4, 5, 8, 16, 17, 40, 64, 65, 70, 1, 4, 12), 6, 6, 30
    n = sum(lengths)
    na = -(-n // nb)
    fp = W.uniform01(141, batch * n_facts).astype(np.float32).reshape(batch, n_facts)
    if values is not None:
        fp = np.asarray(values, np.float32)[(fp * len(values)).astype(int)]
    if apart:
        fp[::2, :8] = np.asarray(values or (0.5, 0.25), np.float32)[np.arange(8) % 2]
    grp = np.concatenate([np.arange(24), np.full(6, 24)]).astype(np.int32)
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    pair = (W.splitmix64(142, np.arange(24 * 24)) % np.uint64(na)).astype(np.int32).reshape(24, 24)
    pair.reshape(-1)[:na] = np.arange(na)
    one = oracle.dtkp_init(np.arange(24), fp, k)
    _, am, ap, _ = oracle.dtkp_apply2(oracle.dense_to_triples(pair), 24, 24, k, grp, fp, one[0], one[0])
    fact_b = np.arange(24, 30, dtype=np.int32)
    bm = oracle.dtkp_init(fact_b, fp, k)
    col = np.repeat(np.arange(len(lengths)), lengths)[np.argsort(W.splitmix64(143, np.arange(n)))].astype(np.int32)
    table = np.full(na * nb, -1, np.int32)
    table[:n] = col
    _, om, op, opr = oracle.dtkp_apply2(oracle.dense_to_triples(table.reshape(na, nb)), na, nb, k, grp, fp, am, bm[0])
    f = dol.FnTable.create_dense(table.reshape(na, nb))
    a = dol.Dist(np.arange(na), torch.zeros((batch, na), device="cuda"), dev(am.view(np.int64)), dev(ap))
    out = dol.Dist.empty(f.out_syms, batch, k=k)
    dol.dtkp_apply2_input(a, fact_b, f, prov, out)
    np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), om)
    np.testing.assert_array_equal(host(out.proof_prob), op)
    assert_close(host(out.prob), opr, "ranked by keys")
    m1, p1 = np.ascontiguousarray(am[:, np.arange(n) % na]), np.ascontiguousarray(ap[:, np.arange(n) % na])
    idx, to = oracle.dense_to_tuples(col)
    _, um, up, upr = oracle.dtkp_applyk(idx, to, k, grp, fp, [m1])
    x = dol.Dist(np.arange(n), torch.zeros((batch, n), device="cuda"), dev(m1.view(np.int64)), dev(p1))
    fu = dol.FnkTable.create_dense(col)
    got = dol.Dist.empty(fu.out_syms, batch, k=k)
    dol.apply_k([x], fu, prov, got)
    np.testing.assert_array_equal(host(got.proof_mask).view(np.uint64), um)
    np.testing.assert_array_equal(host(got.proof_prob), up)
    assert_close(host(got.prob), upr, "unary, ranked by keys")
    x.proof_prob[x.proof_mask == -1] = 0.7          # what an absent proof's probability says counts for nothing
    dol.apply_k([x], fu, prov, got)
    np.testing.assert_array_equal(host(got.proof_mask).view(np.uint64), um)
    np.testing.assert_array_equal(host(got.proof_prob), up)


@pytest.mark.parametrize("k,batch", [(1, 1200), (3, 400), (3, 433), (4, 290), (5, 231), (8, 140)])
def test_dtkp_columns_in_sets_of_samples(dol, k, batch):
    """Batches whose lists exceed the L2s are worked on in sets of samples, the last one larger: each sample's results are those of
    the same sample in a batch of one set."""
    lengths = [3000, 90, 70, 40, 17, 16, 9, 5] * 2 + [4] * 30 + [3] * 40 + [2] * 300 + [1] * 1200
    na, nb, n_facts, part = 1001, 10, 24, 25
    n, S = sum(lengths), len(lengths)
    assert n <= na * nb and batch * (S + na) * 12 * k > 32 << 20
    fp = W.uniform01(151, batch * n_facts).astype(np.float32).reshape(batch, n_facts)
    grp = np.concatenate([np.arange(14), np.full(10, 14)]).astype(np.int32)
    table = np.full(na * nb, -1, np.int32)
    col = np.repeat(np.arange(S), lengths).astype(np.int32)
    table[np.argsort(W.splitmix64(152, np.arange(na * nb)))[:n]] = col
    f = dol.FnTable.create_dense(table.reshape(na, nb))
    final = (W.splitmix64(153, np.arange(S)) % np.uint64(400)).astype(np.int32)
    fu = dol.FnkTable.create_dense(final)
    fact_b = np.arange(14, 24, dtype=np.int32)
    gen = torch.Generator(device="cuda").manual_seed(154)
    bits = torch.randint(0, 14, (batch, na, k), generator=gen, device="cuda")
    am = torch.sort(torch.bitwise_or(torch.ones_like(bits) << bits, torch.ones_like(bits) << (bits * 5 + 3) % 14), -1).values
    ap = torch.rand((batch, na, k), generator=gen, device="cuda")

    def run(s0, s1):
        prov = dol.Prov(dol.DTKP, k, dev(fp[s0:s1]), grp)
        a = dol.Dist(np.arange(na), torch.zeros((s1 - s0, na), device="cuda"), am[s0:s1].contiguous(), ap[s0:s1].contiguous())
        out = dol.Dist.empty(f.out_syms, s1 - s0, k=k)
        dol.dtkp_apply2_input(a, fact_b, f, prov, out)
        end = dol.Dist.empty(fu.out_syms, s1 - s0, k=k)
        dol.apply_k([out], fu, prov, end)
        return out.proof_mask, out.proof_prob, out.prob, end.proof_mask, end.proof_prob, end.prob

    whole = run(0, batch)
    parts = [run(s, min(s + part, batch)) for s in range(0, batch, part)]
    for x, got in enumerate(whole):
        assert torch.equal(got, torch.cat([p[x] for p in parts])), x


@pytest.mark.parametrize("k", [1, 3])
def test_dtkp_apply2_input_equals_init_then_apply2(dol, k):
    """The second operand given by its facts: bit for bit what dol_dtkp_init + dol_apply2 give, on a table with
    columns of every length, a first operand with several proofs per symbol, shared exclusion groups."""
    B, nv = 50, 6
    fp = np.concatenate([W.softmax_rows(W.normal(5600 + t, B * nv).reshape(B, nv)) for t in range(3)], axis=1)
    grp = np.repeat(np.arange(3), nv).astype(np.int32)
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    d0, d1, d2 = (dol.Dist.empty(np.arange(nv), B, k=k) for _ in range(3))
    for t, d in enumerate((d0, d1, d2)):
        dol.dtkp_init(d, np.arange(nv) + nv * t, prov)
    tab = (W.splitmix64(5700, np.arange(nv * nv)) % np.uint64(9)).astype(np.int32).reshape(nv, nv)
    ft = dol.FnTable.create_dense(tab)
    a = dol.Dist.empty(ft.out_syms, B, k=k)
    dol.apply2(d0, d1, ft, prov, a)
    # second operand: the facts of slot 2 in a permuted order, one of them used by two symbols, one fact of slot 1
    fact_b = np.array([14, 12, 17, 12, 13, 15, 16, 7], np.int32)
    table = (W.splitmix64(5800, np.arange(a.n_sym * fact_b.size)) % np.uint64(4)).astype(np.int32).reshape(a.n_sym, -1)
    table.reshape(-1)[::5] = -1
    f = dol.FnTable.create_dense(table)
    b = dol.Dist.empty(np.arange(fact_b.size), B, k=k)
    dol.dtkp_init(b, fact_b, prov)
    want, got = dol.Dist.empty(f.out_syms, B, k=k), dol.Dist.empty(f.out_syms, B, k=k)
    dol.apply2(a, b, f, prov, want)
    dol.dtkp_apply2_input(a, fact_b, f, prov, got)
    np.testing.assert_array_equal(host(got.proof_mask), host(want.proof_mask))
    np.testing.assert_array_equal(host(got.proof_prob), host(want.proof_prob))
    np.testing.assert_array_equal(host(got.prob), host(want.prob))
    # and against the oracle's composition
    am = oracle.dtkp_apply2(oracle.dense_to_triples(tab), nv, nv, k, grp, fp,
                            oracle.dtkp_init(np.arange(nv), fp, k)[0], oracle.dtkp_init(np.arange(nv) + nv, fp, k)[0])[1]
    _, om, op, opr = oracle.dtkp_apply2(oracle.dense_to_triples(table), a.n_sym, fact_b.size, k, grp, fp, am,
                                        oracle.dtkp_init(fact_b, fp, k)[0])
    np.testing.assert_array_equal(host(got.proof_mask).view(np.uint64), om)
    np.testing.assert_array_equal(host(got.proof_prob), op)
    with pytest.raises(dol.DolError):
        dol.dtkp_apply2_input(a, np.full(fact_b.size, 18, np.int32), f, prov, got)


@pytest.mark.parametrize("facts", ["new", "mixed"])
@pytest.mark.parametrize("na,nb,S,B", [(5, 3, 1, 3), (31, 1, 31, 77), (128, 1, 128, 9), (130, 2, 129, 20), (36, 64, 700, 5), (36, 65, 300, 11), (4, 9, 1, 130)])
@pytest.mark.parametrize("k", [1, 3, 4])
def test_dtkp_input_columns_at_the_edges_of_workgroups(dol, k, na, nb, S, B, facts):
    """The second operand given by its facts, over columns of one tuple and of a few, workgroups that end in another sample and
    samples of many to a workgroup, up to 64 symbols whose facts wait in LDS and one more; facts above all others, and facts
    held already, below others and rivals.  Bit for bit what dol_dtkp_init + dol_apply2 give."""
    n0, n1, low = 12, 12, 24
    n_facts = 60
    fp = W.uniform01(6100 + na, B * n_facts).astype(np.float32).reshape(B, n_facts)
    fp[:, 3] = fp[:, 5]                                     # (equal proofs now and then)
    grp = np.concatenate([np.repeat(np.arange(4), 6), np.full(n_facts - low, 9)]).astype(np.int32)
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    d0, d1 = dol.Dist.empty(np.arange(n0), B, k=k), dol.Dist.empty(np.arange(n1), B, k=k)
    dol.dtkp_init(d0, np.arange(n0), prov)
    dol.dtkp_init(d1, np.arange(n1) + n0, prov)
    first = dol.FnTable.create_dense((np.arange(n0 * n1) * 7 % na).astype(np.int32).reshape(n0, n1))
    a = dol.Dist.empty(first.out_syms, B, k=k)
    assert a.n_sym == na
    dol.apply2(d0, d1, first, prov, a)
    fact_b = (low + np.arange(nb) * 5 % (n_facts - low) if facts == "new" else np.arange(nb) * 11 % n_facts).astype(np.int32)
    ids = (W.splitmix64(6200, np.arange(na * nb)) % np.uint64(S)).astype(np.int32)
    ids[np.argsort(W.splitmix64(6300, np.arange(na * nb)), kind="stable")[:S]] = np.arange(S)
    f = dol.FnTable.create_dense(ids.reshape(na, nb))
    assert f.out_syms.size == S
    b = dol.Dist.empty(np.arange(nb), B, k=k)
    dol.dtkp_init(b, fact_b, prov)
    want, got = dol.Dist.empty(f.out_syms, B, k=k), dol.Dist.empty(f.out_syms, B, k=k)
    dol.apply2(a, b, f, prov, want)
    dol.dtkp_apply2_input(a, fact_b, f, prov, got)
    np.testing.assert_array_equal(host(got.proof_mask), host(want.proof_mask))
    np.testing.assert_array_equal(host(got.proof_prob), host(want.proof_prob))
    np.testing.assert_array_equal(host(got.prob), host(want.prob))


@pytest.mark.parametrize("values", [None, (0.5, 0.25, 1.0, 0.0)], ids=["random", "equal"])
@pytest.mark.parametrize("facts", ["new", "mixed"])
@pytest.mark.parametrize("nb", [64, 65])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6])
def test_dtkp_input_over_lists_in_any_order(dol, k, nb, facts, values):
    """An operand whose proofs lie in no order, with absent ones before and between them (of any probability), joined to facts that
    are new to all proofs of a wavefront, and to facts held already, below others and rivals; columns of one tuple and of every
    kind of length, on both sides of the longest lists ranked by keys, facts in LDS and not.  Against the oracle, bit for bit."""
    lengths = (1, 2, 3, 4, 5, 15, 16, 17, 64, 65, 70) + (1,) * 70
    batch, low, n_facts, n = 5, 24, 60, sum(lengths)
    na = -(-n // nb)
    fp = W.uniform01(151 + nb, batch * n_facts).astype(np.float32).reshape(batch, n_facts)
    if values is not None:
        fp[1:] = np.asarray(values, np.float32)[(fp[1:] * len(values)).astype(int)]
    grp = np.concatenate([np.repeat(np.arange(4), 6), np.full(n_facts - low, 9)]).astype(np.int32)
    # a proof: one fact of some of the four groups
    pick = W.splitmix64(152, np.arange(batch * na * k * 4)).reshape(batch, na, k, 4) % np.uint64(9)
    am = np.bitwise_or.reduce(np.where(pick < 6, np.uint64(1) << (pick % np.uint64(6) + np.uint64(6) * np.arange(4, dtype=np.uint64)), np.uint64(0)), axis=-1)
    am[W.uniform01(153, am.size).reshape(am.shape) < 0.2] = oracle.ABSENT
    am[am == 0] = oracle.ABSENT
    for x in range(1, k):                       # (no proof twice in a list)
        for y in range(x):
            am[..., x] = np.where(am[..., x] == am[..., y], oracle.ABSENT, am[..., x])
    ap = np.ones(am.shape, np.float32)
    for f in range(low):
        ap = np.where((am >> np.uint64(f)) & np.uint64(1) == 1, ap * fp[:, f, None, None], ap)
    ap[am == oracle.ABSENT] = 0.7
    fact_b = (low + np.arange(nb) * 5 % (n_facts - low) if facts == "new" else np.arange(nb) * 11 % n_facts).astype(np.int32)
    col = np.repeat(np.arange(len(lengths)), lengths)[np.argsort(W.splitmix64(154, np.arange(n)))].astype(np.int32)
    table = np.full(na * nb, -1, np.int32)
    table[:n] = col
    table = table.reshape(na, nb)
    bm = oracle.dtkp_init(fact_b, fp, k)[0]
    _, om, op, opr = oracle.dtkp_apply2(oracle.dense_to_triples(table), na, nb, k, grp, fp, am, bm)
    f = dol.FnTable.create_dense(table)
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    a = dol.Dist(np.arange(na), torch.zeros((batch, na), device="cuda"), dev(am.view(np.int64)), dev(ap))
    b = dol.Dist.empty(np.arange(nb), batch, k=k)
    dol.dtkp_init(b, fact_b, prov)
    for call in (lambda out: dol.dtkp_apply2_input(a, fact_b, f, prov, out), lambda out: dol.apply2(a, b, f, prov, out)):
        out = dol.Dist.empty(f.out_syms, batch, k=k)
        call(out)
        np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), om)
        np.testing.assert_array_equal(host(out.proof_prob), op)
        assert_close(host(out.prob), opr, "lists in any order")


@pytest.mark.parametrize("k,nv", [(1, 6), (3, 6), (3, 20), (8, 12)])
def test_dtkp_gradient_with_impossible_facts(dol, k, nv):
    """Fact probabilities of exactly 0 and far below 1e-30 in some samples: there the product of a proof's other facts
    cannot come from dividing the proof's probability, so the kernel multiplies them out.  nv = 20 gives 400 result
    symbols (several wavefronts per sample, a ragged last group of 64); the padded gradient tensor has ld > n_sym."""
    B = 70
    fp = np.concatenate([W.softmax_rows(W.normal(5900 + t, B * nv).reshape(B, nv)) for t in range(3)], axis=1)
    fp[::3, 1:nv] = 0.0                                            # kept lists there must take impossible proofs
    fp[1::5, nv + 1] = np.float32(1e-36)
    fp[2::7, 2 * nv + 3] = np.float32(1e-41)                       # subnormal
    fp[5, :] = 0.0                                                 # every proof of this sample is impossible
    fp = np.ascontiguousarray(fp, np.float32)
    grp = np.repeat(np.arange(3), nv).astype(np.int32)
    prov = dol.Prov(dol.DTKP, k, dev(fp), grp)
    d = [dol.Dist.empty(np.arange(nv), B, k=k) for _ in range(3)]
    for t in range(3):
        dol.dtkp_init(d[t], np.arange(nv) + nv * t, prov)
    # a: pairs of (slot 0, slot 1) facts folded onto few symbols, so that symbols keep several proofs
    tab = (W.splitmix64(5950, np.arange(nv * nv)) % np.uint64(nv)).astype(np.int32).reshape(nv, nv)
    ft = dol.FnTable.create_dense(tab)
    a = dol.Dist.empty(ft.out_syms, B, k=k)
    dol.apply2(d[0], d[1], ft, prov, a)
    # out: one symbol per (a symbol, slot 2 fact)
    table = np.arange(a.n_sym * nv, dtype=np.int32).reshape(a.n_sym, nv)
    f = dol.FnTable.create_dense(table)
    out = dol.Dist.empty(f.out_syms, B, k=k)
    dol.apply2(a, d[2], f, prov, out)
    inits = [oracle.dtkp_init(np.arange(nv) + nv * t, fp, k)[0] for t in range(3)]
    _, am, _, _ = oracle.dtkp_apply2(oracle.dense_to_triples(tab), nv, nv, k, grp, fp, inits[0], inits[1])
    _, om, op, opr = oracle.dtkp_apply2(oracle.dense_to_triples(table), a.n_sym, nv, k, grp, fp, am, inits[2])
    np.testing.assert_array_equal(host(out.proof_mask).view(np.uint64), om)
    np.testing.assert_array_equal(host(out.proof_prob), op)
    S = om.shape[1]
    gsym = W.normal(5960 + k, B * S).astype(np.float32).reshape(B, S)
    want = oracle.dtkp_prob_bwd(om, fp, gsym)
    assert np.abs(want[::3, 1:nv]).max() > 0                       # the zero facts do receive gradient
    gpad = torch.zeros((B, S + 5), device="cuda")
    gpad[:, :S] = dev(gsym)
    gf = torch.full((B, fp.shape[1]), 3.0, device="cuda")
    dol.dtkp_backward(out, prov, gpad, gf)
    assert_close(host(gf), want, "dtkp gradient with impossible facts, k=%d" % k)


@pytest.mark.parametrize("m,nb,batch", [(1, 1, 5), (16, 16, 257), (7, 3, 256), (16, 1, 1000), (10, 10, 255), (3, 16, 513)])
def test_sum_shaped_apply_with_short_first_operand(dol, m, nb, batch):
    """The thread-per-sample forward kernel: every width up to 16, whole and partial tiles of 256 samples, tags that
    clamp; backward (through the tile / loop kernels) on the same result."""
    a = (W.uniform01(100 + m, batch * m) * 0.9).astype(np.float32).reshape(batch, m)
    b = (W.uniform01(200 + nb, batch * nb) * 0.9).astype(np.float32).reshape(batch, nb)
    table = W.sum_table(np.arange(m), np.arange(nb))
    tri = oracle.dense_to_triples(table)
    syms, want, pre32, _ = oracle.damp_apply2_fwd(tri, m, nb, a, b, want_pre=True)
    f = dol.FnTable.create_dense(table)
    assert f.kernel_fwd.startswith("damp_conv_fwd_small_kernel")
    da, db = dol.Dist(np.arange(m), dev(a)), dol.Dist(np.arange(nb), dev(b))
    out = dol.Dist.empty(f.out_syms, batch)
    dol.apply2(da, db, f, None, out)
    assert_close(host(out.prob), want, "short first operand forward")
    if min(m, nb) >= 3:
        assert (pre32 > 1).any()
    g = np.abs(W.normal(300 + m, batch * syms.size)).astype(np.float32).reshape(batch, -1)
    wa, wb = oracle.damp_apply2_bwd(tri, m, nb, a, b, g)
    ga, gb = torch.empty((batch, m), device="cuda"), torch.empty((batch, nb), device="cuda")
    dol.backward(dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f), dev(g), ga, gb)
    assert_close(host(ga), wa, "short first operand grad a")
    assert_close(host(gb), wb, "short first operand grad b")


def test_first_call_of_a_generated_kernel_while_capturing(dol):
    """A graph may be recorded from the very first call: a table of 30 x 21 symbols whose kernels are made at that moment, both
    directions, and a sum of 20 digits, which the generated fold takes."""
    B, na, nb = 30000, 30, 21
    f = dol.FnTable.create_dense(_rand_table(81, (na, nb), 77))
    da, db = dol.Dist(np.arange(na), dev(W.softmax_rows(W.normal(82, B * na).reshape(B, na)))), dol.Dist(
        np.arange(nb), dev(W.softmax_rows(W.normal(83, B * nb).reshape(B, nb))))
    out = dol.Dist.empty(f.out_syms, B)
    g = dev(W.normal(84, B * out.n_sym).reshape(B, -1).astype(np.float32))
    ga, gb = torch.empty((B, na), device="cuda"), torch.empty((B, nb), device="cuda")
    rec = dol.OpRecord(dol.OP_APPLY2, da, db, out, f=f)
    p = dev(W.softmax_rows(W.normal(85, 20 * 40 * 10).reshape(-1, 10)).reshape(20, 40, 10))
    tables, syms = [], np.arange(10, dtype=np.int32)
    for _ in range(19):
        tables.append(dol.FnTable.create_dense(syms[:, None] + np.arange(10, dtype=np.int32)[None, :]))
        syms = tables[-1].out_syms
    total, grads = dol.Dist.empty(syms, 40), torch.empty_like(p)
    fold = dol.Fold([dol.Dist(np.arange(10), p[t]) for t in range(20)], tables, out=total,
                    target_col=torch.arange(40, device="cuda", dtype=torch.int32), grad_inputs=list(grads))

    def step():
        dol.apply2(da, db, f, None, out)
        dol.backward(rec, g, ga, gb)
        dol.fold_apply2(fold)

    results = (out.prob, ga, gb, total.prob, grads)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    step()
    want = [x.clone() for x in results]
    for _ in range(3):
        for x in results:
            x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for x, y in zip(results, want):
            assert torch.equal(x, y)
