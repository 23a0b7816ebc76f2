"""GPU parity of single kernels at the sizes where their tiling can go wrong, against fp64 arithmetic or the CPU oracle."""
import numpy as np
import pytest

from oracle import abs_oracle as O
from paper_2406_13936_amd import workloads as W

pytestmark = pytest.mark.gpu

EPS32 = 2.0 ** -24      # half a unit in the last place of fp32 (round to nearest), relative
EPSBF = 2.0 ** -9       # the same for bf16


def _A():
    import paper_2406_13936_amd as A
    return A


# The 256 x 256 tile's pipelined main loop reads two k-tiles of 64 ahead: reductions of one, two, three, an odd number of
# k-tiles and ragged last k-tiles, with row and column remainders (K of the inner products = fin, of the gradient = b).
@pytest.mark.parametrize("b,fin,fout", [(1030, 8, 1032), (1024, 64, 1024), (1025, 72, 1100 // 8 * 8), (1100, 136, 1048),
                                        (1031, 264, 1024), (257, 1032, 1040), (330, 1024, 1096), (1027, 1088, 1160)])
def test_large_tile_contractions_at_the_edges_of_the_reduction(b, fin, fout):
    import torch
    A = _A()
    M = 16 if b < 1024 else 2        # (the large tile is taken for short reductions only if it fills the chip)
    g = torch.Generator().manual_seed(b + fin)
    a = torch.randn((M, b, fin), generator=g).to(torch.bfloat16)
    d = torch.randn((M, b, fout), generator=g).to(torch.bfloat16)
    res, n, q, gbar = A.layer_stats([a.cuda()], [d.cuda()], want_per_sample=True, want_gbar=True)
    for m in (0, M - 1):
        a64, d64 = a[m].double().numpy(), d[m].double().numpy()
        G, Gabs = d64.T @ a64 / b, np.abs(d64).T @ np.abs(a64) / b
        # a sum of b products in fp32, any order: (b + 1) roundings of at most the sum of magnitudes; one more for 1 / b
        err = np.abs(gbar[m].cpu().numpy().reshape(fout, fin) - G)
        assert (err <= (b + 2) * EPS32 * Gabs).all(), (m, err.max())
        want = (d64 * (a64 @ G.T)).sum(1)
        # Gbar rounded to bf16 as the operand, then fin products and fout products summed in fp32
        bound = (EPSBF * (1 + 2 ** -8) + (b + fin + fout + 4) * EPS32) * (np.abs(d64) * (np.abs(a64) @ Gabs.T)).sum(1)
        assert (np.abs(q[m].cpu().numpy() - want) <= bound).all(), m
        # (the bound above cannot tell a wrong entry of a long sum: the spread of the differences does)
        assert np.linalg.norm(q[m].cpu().numpy() - want) <= 1e-3 * np.linalg.norm(want), m
        np.testing.assert_allclose(n[m].cpu().numpy(), (a64 ** 2).sum(1) * (d64 ** 2).sum(1), rtol=(fin + fout + 4) * EPS32)
        assert abs(res[m].gbar_sq - (G ** 2).sum()) <= 1e-5 * (G ** 2).sum()


# Forward and backward-data in the same tile: reductions of 72 (two k-tiles, ragged), 1032 (17 k-tiles) and 10 / 130 classes.
@pytest.mark.parametrize("dims,act", [((72, 1032, 1040, 130), W.ACT_GELU), ((64, 1048, 1024, 10), W.ACT_RELU)])
def test_large_tile_step_at_the_edges_of_the_reduction(dims, act):
    A = _A()
    b, M = 1030, 2
    w = W.Workload("edges", dims, act, True, W.PREC_BF16, N=2048, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SHB, lr=0.05,
                   momentum=0.9, test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=5)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, momentum=w.momentum, mixed=True, want_ip=True)
    try:
        for h in range(2):
            idx = W.step_indices(w, 0, h, b)
            rep.local_step(idx, w.lr)
            g = rep.inner_product_test(w.theta)
            orc.local_step(idx, w.lr)
            for m in range(M):
                s = orc.stats[m]
                for got, want in ((g[m].sum_sq, s["S1"]), (g[m].gbar_sq, s["S2"]), (g[m].sum_q, s["S4"]),
                                  (g[m].sum_q2, s["S3"]), (g[m].loss_sum, s["loss_sum"])):
                    assert abs(got - want) <= 2e-3 * abs(want), (h, m, got, want)
                grad = rep.get_grad(m).astype(np.float64)
                assert np.linalg.norm(grad - orc.grads[m]) <= 2e-3 * np.linalg.norm(orc.grads[m]), (h, m)
                p = rep.get_params(m).astype(np.float64)
                assert np.abs(p - orc.x[m]).max() <= 1e-3 * np.abs(orc.x[m]).max()
        assert rep.guard_intact()
    finally:
        rep.close()


# Launches of few 32 x 32 tiles: row and column remainders of the 32 x 32 (forward, logits) and 32 x 64 (backward-data)
# tiles, reductions shorter than a wave's first chunk (8), a chunk with a remainder (72, 264) and more than one trip (1096).
@pytest.mark.parametrize("dims,act,b", [((8, 40, 3), W.ACT_RELU, 2), ((72, 8, 16, 2), W.ACT_GELU, 31),
                                        ((264, 72, 104, 130), W.ACT_GELU, 33), ((1096, 136, 10), W.ACT_NONE, 65),
                                        ((40, 1096, 64, 33), W.ACT_RELU, 32),
                                        # the last layer's bias gradient: summed in one launch up to b = 128, 16 columns a block
                                        ((64, 72, 16), W.ACT_RELU, 128), ((64, 72, 17), W.ACT_GELU, 128),
                                        ((64, 72, 16), W.ACT_GELU, 129), ((64, 72, 100), W.ACT_RELU, 129)])
def test_small_launches_at_the_edges_of_their_tiles(dims, act, b):
    A = _A()
    M = 3
    w = W.Workload("edges", dims, act, True, W.PREC_BF16, N=512, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.05,
                   test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=7)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, mixed=True, want_ip=True, gram_max_b=256)
    try:
        for h in range(2):
            idx = W.step_indices(w, 0, h, b)
            rep.local_step(idx, w.lr)
            g = rep.inner_product_test(w.theta)
            orc.local_step(idx, w.lr)
            for m in range(M):
                s = orc.stats[m]
                for got, want in ((g[m].sum_sq, s["S1"]), (g[m].gbar_sq, s["S2"]), (g[m].loss_sum, s["loss_sum"])):
                    assert abs(got - want) <= 2e-3 * abs(want), (h, m, got, want)
                grad = rep.get_grad(m).astype(np.float64)
                assert np.linalg.norm(grad - orc.grads[m]) <= 2e-3 * np.linalg.norm(orc.grads[m]), (h, m)
                K = dims[-1]
                assert np.linalg.norm(grad[-K:] - orc.grads[m][-K:]) <= 2e-3 * np.linalg.norm(orc.grads[m][-K:]), (h, m)
                p = rep.get_params(m).astype(np.float64)
                assert np.abs(p - orc.x[m]).max() <= 1e-3 * np.abs(orc.x[m]).max()
        assert rep.guard_intact()
    finally:
        rep.close()


# fp32 contractions: 16-, 32- and 64-wide tiles with remainders, k-steps of 256 / 128 / 32 with remainders on either side of a
# step, the bias sums beside the weight gradient, and a reduction long enough over few tiles to be split (b = 4099).
@pytest.mark.parametrize("dims,b,M", [((33, 2), 2, 1), ((257, 17), 255, 3), ((256, 10), 257, 4), ((130, 40, 5), 513, 2),
                                      ((520, 136, 70), 300, 8), ((31, 3), 4099, 1)])
def test_fp32_step_at_the_edges_of_its_tiles(dims, b, M):
    A = _A()
    act = W.ACT_GELU if len(dims) > 2 else W.ACT_NONE
    w = W.Workload("edges", dims, act, True, W.PREC_F32, N=512, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.05,
                   test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=9)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, want_ip=True)
    try:
        idx = W.step_indices(w, 0, 0, b)
        rep.local_step(idx, w.lr)
        g = rep.inner_product_test(w.theta)
        orc.local_step(idx, w.lr)
        for m in range(M):
            s = orc.stats[m]
            # fp32 sums of up to 4099 products: (terms + layers) * 2^-24 of their magnitudes at worst, 1e-4 with room
            for got, want in ((g[m].sum_sq, s["S1"]), (g[m].gbar_sq, s["S2"]), (g[m].sum_q2, s["S3"]), (g[m].loss_sum, s["loss_sum"])):
                assert abs(got - want) <= 1e-4 * abs(want), (m, got, want)
            grad, K = rep.get_grad(m).astype(np.float64), dims[-1]
            assert np.linalg.norm(grad - orc.grads[m]) <= 1e-5 * np.linalg.norm(orc.grads[m]), m
            assert np.linalg.norm(grad[-K:] - orc.grads[m][-K:]) <= 1e-5 * np.linalg.norm(orc.grads[m][-K:]), m
        assert rep.guard_intact()
    finally:
        rep.close()


# Statistics alone with the batch gradient not asked for, in an aligned buffer (written by the launches that form it), in one
# that is not 16-byte aligned and in one that overlaps an input (both filled at the end): the same values in all four.
@pytest.mark.parametrize("M,b,ins,outs", [(1, 2, (8,), (8,)), (3, 300, (72, 136), (136, 40)), (2, 1030, (264,), (1032,))])
def test_statistics_alone_deliver_the_same_gradient_into_any_buffer(M, b, ins, outs):
    import ctypes as C
    import torch
    A = _A()
    g = torch.Generator().manual_seed(b)
    a = [torch.randn((M, b, i), generator=g).to(torch.bfloat16).cuda() for i in ins]
    d = [torch.randn((M, b, o), generator=g).to(torch.bfloat16).cuda() for o in outs]
    res0, n0, q0, _ = A.layer_stats(a, d, want_per_sample=True)
    res1, n1, q1, gbar = A.layer_stats(a, d, want_per_sample=True, want_gbar=True)
    key = lambda r: (r.sum_sq, r.gbar_sq, r.sum_q, r.sum_q2)  # noqa: E731
    assert [key(r) for r in res0] == [key(r) for r in res1] and torch.equal(n0, n1) and torch.equal(q0, q1)
    at = 0
    for l, (i, o) in enumerate(zip(ins, outs)):
        a64, d64 = a[l].double().cpu(), d[l].double().cpu()
        G = d64.transpose(1, 2).contiguous() @ a64 / b
        Gabs = d64.abs().transpose(1, 2).contiguous() @ a64.abs() / b
        got = gbar[:, at:at + i * o].cpu().double().view(M, o, i)
        assert ((got - G).abs() <= (b + 2) * EPS32 * Gabs).all()
        at += i * o
    want = (gbar.double() ** 2).sum(1).cpu().numpy()      # (fp32 sums of four squares, then double)
    np.testing.assert_allclose([r.gbar_sq for r in res1], want, rtol=8 * EPS32)
    lib, L = A.load_library(), len(ins)
    Wsum = at
    words = M * Wsum + M * b * (max(ins) + max(outs)) + 64
    for lead in (1, 0):                                    # one float past an aligned address; in front of the first input
        buf = torch.zeros(words, dtype=torch.float32, device="cuda")
        ins_c, outs_c = (C.c_int * L)(*ins), (C.c_int * L)(*outs)
        first = a[0]
        if lead == 0:
            first = buf[4:4 + a[0].numel() // 2 + 1].view(torch.bfloat16)[:a[0].numel()].view(a[0].shape)
            first.copy_(a[0])
        nbytes = C.c_size_t(0)
        assert lib.abs_layer_stats_workspace_bytes(L, ins_c, outs_c, M, b, C.byref(nbytes)) == 0
        ws = torch.empty(nbytes.value + 256, dtype=torch.uint8, device="cuda")
        ap = (C.c_void_p * L)(*[t.data_ptr() for t in [first] + a[1:]])
        dp = (C.c_void_p * L)(*[t.data_ptr() for t in d])
        out = (A.TestResult * M)()
        st = torch.cuda.current_stream().cuda_stream
        assert lib.abs_layer_stats(L, ins_c, outs_c, M, b, ap, dp, (ws.data_ptr() + 255) // 256 * 256, nbytes.value, st, out,
                                   None, None, buf.data_ptr() + 4 * lead) == 0
        torch.cuda.synchronize()
        assert [key(r) for r in out] == [key(r) for r in res1]
        assert torch.equal(buf[lead:lead + M * Wsum].view(M, Wsum), gbar)


# The softmax head inside the logits' launch: classes at the edges of its lanes (2, 16 / 17, 32 / 33, the latter of each pair in a
# launch of its own in one precision or both), rows beyond a tile, workers with batches of their own.
@pytest.mark.parametrize("prec,K,sizes", [(p, K, s) for p in (W.PREC_F32, W.PREC_BF16) for K in (2, 16, 17, 32, 33)
                                          for s in ((33, 33), (2, 47))])
def test_softmax_head_at_the_edges_of_its_lanes(prec, K, sizes):
    A = _A()
    M, b, d = len(sizes), max(sizes), 40
    w = W.Workload("head", (d, K), W.ACT_NONE, True, prec, N=256, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.05,
                   test=W.TEST_NORM, data="teacher_mlp", seed=11)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    try:
        idx = W.step_indices(w, 0, 0, b)
        rep.local_step_ragged([idx[m][:s] for m, s in enumerate(sizes)], 0.0)
        res = rep.norm_test(0.5)
        rnd = O.bf16_round if prec == W.PREC_BF16 else (lambda v: np.asarray(v, np.float64))
        Wm, bias = x0[:d * K].reshape(K, d).astype(np.float64), x0[d * K:].astype(np.float64)
        tol = 1e-3 if prec == W.PREC_BF16 else 1e-5      # delta rounded to bf16 near a tie: single entries move by 2^-9
        for m, s in enumerate(sizes):
            a = np.asarray(rnd(X[idx[m][:s]]), np.float64)
            z = a @ np.asarray(rnd(Wm), np.float64).T + bias
            lab = y[idx[m][:s]]
            mx = z.max(1, keepdims=True)
            p = np.exp(z - mx)
            loss = (np.log(p.sum(1)) + mx[:, 0] - z[np.arange(s), lab]).sum()
            p /= p.sum(1, keepdims=True)
            p[np.arange(s), lab] -= 1.0
            delta = np.asarray(rnd(p), np.float64)
            n = (delta ** 2).sum(1) * ((a ** 2).sum(1) + 1.0)
            assert abs(res[m].loss_sum - loss) <= 1e-5 * loss
            assert abs(res[m].sum_sq - n.sum()) <= tol * n.sum()
            G = np.concatenate([(delta.T @ a / s).ravel(), delta.mean(0)])
            got = rep.get_grad(m).astype(np.float64)
            assert np.linalg.norm(got - G) <= tol * np.linalg.norm(G)
        assert rep.guard_intact()
    finally:
        rep.close()


# fp32 weight gradients of long batches over few tiles are cut into slices, whatever tile the launch takes (64 x 64: 100 x 1024
# outputs of 4 replicas, 136 x 520 of 8; 32 x 32: 70 x 136, 60 x 200; 16 x 16: 10 x 256), slices with a remainder and empty ones
# (b = 2305: 9 steps of 256 in 8 slices of two); the bias gradient then comes from column sums, the step from its own launch.
@pytest.mark.parametrize("dims,b,M,opt", [((1024, 100), 2048, 4, W.OPT_SGD), ((256, 100), 2305, 16, W.OPT_SHB),
                                          ((520, 136, 70), 2050, 8, W.OPT_SGD), ((200, 60, 12), 2305, 6, W.OPT_ADAGRAD),
                                          ((256, 10), 2049, 4, W.OPT_ADAMW)])
def test_fp32_long_reductions_over_few_tiles_are_split(dims, b, M, opt):
    A = _A()
    act = W.ACT_GELU if len(dims) > 2 else W.ACT_NONE
    w = W.Workload("long", dims, act, True, W.PREC_F32, N=4096, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=opt, lr=0.05, momentum=0.9,
                   weight_decay=0.05, test=W.TEST_NORM, data="teacher_mlp", seed=13)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    try:
        rep.profile_enable(True)
        idx = W.step_indices(w, 0, 0, b)
        rep.local_step(idx, w.lr)
        assert "col_sum" in rep.profile_read()            # (un-split, the bias sums come out of the weight gradient's launch)
        rep.profile_enable(False)
        _check_fp32_step(rep, w, _fp32_oracle(w, X, y, x0), idx, (0, M - 1))
        assert rep.guard_intact()
    finally:
        rep.close()


# The optimizer step in the epilogue of the fp32 weight gradients, biases beside them: 64 x 64 tiles (136 x 520 outputs of 8
# replicas), 32 x 32 (100 x 136) and 16 x 16 (the narrow net), with remainders; the second step starts from non-zero state.
@pytest.mark.parametrize("opt", [W.OPT_SGD, W.OPT_SHB, W.OPT_ADAMW, W.OPT_ADAGRAD])
@pytest.mark.parametrize("dims,sizes", [((520, 136, 100), (201,) * 8), ((520, 136, 100), (201, 2, 64, 150, 33, 201, 7, 128)),
                                        ((37, 19, 5), (65, 40))])
def test_fp32_step_in_the_weight_gradient_moves_every_parameter(dims, sizes, opt):
    A = _A()
    M, b = len(sizes), max(sizes)
    w = W.Workload("step", dims, W.ACT_GELU, True, W.PREC_F32, N=1024, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=opt, lr=0.05, momentum=0.9,
                   weight_decay=0.05, test=W.TEST_NORM, data="teacher_mlp", seed=17)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    try:
        orc = _fp32_oracle(w, X, y, x0)
        for h in range(2):
            rows = [W.batch_indices(w.seed, h, 0, m, s, w.N) for m, s in enumerate(sizes)]
            if len(set(sizes)) > 1:
                rep.local_step_ragged(rows, w.lr)
            else:
                rep.local_step(np.stack(rows), w.lr)
            _check_fp32_step(rep, w, orc, rows, (0, 1, M - 1))
        assert rep.guard_intact()
    finally:
        rep.close()


def _fp32_oracle(w, X, y, x0):
    return O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, w.M, opt=w.opt, momentum=w.momentum, beta1=w.beta1, beta2=w.beta2,
                      eps=w.eps, weight_decay=w.weight_decay)


def _check_fp32_step(rep, w, orc, idx, sampled):
    """Gradient, ||gbar||^2, parameters and optimizer state after a step (already taken by `rep`) against the oracle, workers
    `sampled` only; the oracle then takes over parameters and state (a sign-like step turns a last-bit difference of a gradient
    that is noise into a step of the learning rate, which the next step's gradients would show).
    A gradient entry is a sum of b products in fp32: (b + layers) roundings of 2^-24, random in sign, of terms that largely
    cancel: 1e-5 of the largest entry leaves a factor of 10 at b = 2305.  The step adds one rounding of the parameter; sign-like
    optimizers divide the gradient by its own magnitude, so their parameters are compared where that is no rounding noise."""
    orc.local_step(idx, w.lr, only=sorted(set(sampled)))
    res = rep.norm_test(0.5)
    for m in sorted(set(sampled)):
        g, K = orc.grads[m], w.dims[-1]
        got = rep.get_grad(m).astype(np.float64)
        assert np.abs(got - g).max() <= 1e-5 * np.abs(g).max(), m
        assert np.abs(got - g)[-K:].max() <= 1e-5 * np.abs(g[-K:]).max(), m
        assert abs(res[m].gbar_sq - orc.stats[m]["S2"]) <= 1e-5 * orc.stats[m]["S2"], m
        signed = w.opt in (W.OPT_ADAMW, W.OPT_ADAGRAD)
        sel = np.abs(g) >= 1e-2 * np.abs(g).max() if signed else slice(None)
        p = rep.get_params(m).astype(np.float64)
        assert np.abs(p - orc.x[m])[sel].max() <= 1e-5 * np.abs(orc.x[m]).max(), m
        if signed:                                       # (noise or not, a step of this kind is bounded)
            assert np.abs(p - orc.x[m]).max() <= 2.1 * w.lr, m
        orc.x[m] = p
        if w.opt != W.OPT_SGD:
            v = rep.get_opt_state(m, 0).astype(np.float64)
            assert np.abs(v - orc.st[m].v).max() <= 4e-5 * np.abs(orc.st[m].v).max(), m
            orc.st[m].v = v
        if w.opt == W.OPT_ADAMW:
            mm = rep.get_opt_state(m, 1).astype(np.float64)
            assert np.abs(mm - orc.st[m].m).max() <= 4e-5 * np.abs(orc.st[m].m).max(), m
            orc.st[m].m = mm


# Launches of the bf16 weight gradients on 128 x 128 tiles, with and without the step in the epilogue: all layers in one launch on
# 128 x 128 or 64 x 128 tiles, with slices or whole, or a launch per layer; `own` of them have a launch to themselves.  The form of
# the update changes neither the launches' sums nor the parameters.
@pytest.mark.parametrize("dims,M,b,opt,own", [
    ((784, 512, 512, 10), 2, 4096, W.OPT_SHB, 3),             # long reductions in slices of unequal length: a launch each
    ((784, 768, 768, 768, 100), 4, 1101, W.OPT_ADAMW, 0),     # 480 coarse tiles: one round, whole reductions
    ((784, 512, 512, 10), 8, 1101, W.OPT_SGD, 0),             # 384 coarse tiles: 736 of 64 x 128
    ((1024, 256, 256, 256, 100), 2, 2305, W.OPT_SHB, 0),      # slices in one launch (64 x 128 tiles)
    ((512, 200, 10), 3, 2305, W.OPT_SGD, 0),                  # the same on 128 x 128 tiles, widths that are no multiple
])
def test_weight_gradient_launches_of_long_batches(dims, M, b, opt, own):
    A = _A()
    w = W.Workload("wgrad", dims, W.ACT_RELU, True, W.PREC_BF16, N=4096, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=opt, lr=0.02, momentum=0.9,
                   weight_decay=0.05, test=W.TEST_NORM, data="teacher_mlp", seed=19)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=opt, momentum=w.momentum, beta1=w.beta1, beta2=w.beta2, eps=w.eps,
                     weight_decay=w.weight_decay, mixed=True)
    idx = W.step_indices(w, 0, 0, b)
    orc.local_step(idx, w.lr, only=[M - 1])
    g = orc.grads[M - 1]
    params = []
    for fused in (True, False):
        rep = A.Replicas.from_workload(w, X, y, x0)
        try:
            rep.set_fused_update(fused)
            rep.profile_enable(True)
            rep.local_step(idx, w.lr)
            names = [n for n in rep.profile_read() if n.startswith("gemm_wgrad_")]
            rep.profile_enable(False)
            assert sum(not n.endswith("_L0") for n in names) == own, names
            res = rep.norm_test(0.5)
            assert abs(res[M - 1].gbar_sq - orc.stats[M - 1]["S2"]) <= 2e-3 * orc.stats[M - 1]["S2"]
            p = rep.get_params(M - 1)
            got = rep.get_grad(M - 1).astype(np.float64)
            assert np.linalg.norm(got - g) <= 2e-3 * np.linalg.norm(g)
            at = 0                                            # layer by layer: a small one would drown in the norm of all
            for fin, fout in zip(dims[:-1], dims[1:]):
                for size in (fin * fout, fout):
                    part = slice(at, at + size)
                    assert np.linalg.norm(got[part] - g[part]) <= 4e-3 * np.linalg.norm(g[part]), (fin, fout, size)
                    at += size
            sel = np.abs(g) >= 1e-2 * np.abs(g).max() if opt == W.OPT_ADAMW else slice(None)
            assert np.abs(p - orc.x[M - 1])[sel].max() <= 1e-3 * np.abs(orc.x[M - 1]).max()
            params.append((p, rep.get_params(0), got))
            assert rep.guard_intact()
        finally:
            rep.close()
    for a, c in zip(*params):
        assert np.array_equal(a, c)


# Around the largest launches that take the 32-row tiles (32 x 32 tiles over all replicas: forward and logits 512, logits of more
# than 32 classes 384, backward-data 1024): the last size on them, the first beyond, against the oracle.
@pytest.mark.parametrize("dims,M,b,fwd,logits,bwd", [
    ((64, 512, 256, 10), 8, 128, "32x32", "32x32", "32x64"),      # 512 / 256, 32 tiles
    ((64, 512, 256, 10), 8, 129, "64x128", "32x32", "32x64"),     # 640
    ((64, 512, 512, 100), 8, 256, "64x128", "32x32", "32x64"),    # 1024; logits 256
    ((64, 264, 512, 100), 12, 256, "64x128", "32x32", "32x64"),   # 864 / 1536; logits 384
    ((64, 512, 512, 100), 8, 289, "64x128", "32x32", "64x128"),   # 1280; logits 320
    ((64, 512, 512, 100), 8, 417, "64x128", "64x128", "64x128"),  # 1792; logits 448
    ((64, 1024, 64, 10), 32, 32, "64x128", "32x32", "64x128"),   # 1024, one row of tiles; 32
])
def test_edge_of_the_small_launches(dims, M, b, fwd, logits, bwd):
    A = _A()
    w = W.Workload("small", dims, W.ACT_RELU, True, W.PREC_BF16, N=1024, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.05,
                   test=W.TEST_NORM, data="teacher_mlp", seed=23)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, mixed=True)
    try:
        rep.profile_enable(True)
        idx = W.step_indices(w, 0, 0, b)
        rep.local_step(idx, w.lr)
        names = set(rep.profile_read())
        rep.profile_enable(False)
        # (layer 1 for the forward, the middle one for backward-data)
        assert {"gemm_fwd_%s_L1" % fwd, "gemm_logits_%s_L3" % logits, "gemm_bwd_%s_L2" % bwd} <= names, names
        res = rep.norm_test(0.5)
        orc.local_step(idx, w.lr, only=[0, M - 1])
        for m in (0, M - 1):
            s = orc.stats[m]
            for got, want in ((res[m].sum_sq, s["S1"]), (res[m].gbar_sq, s["S2"]), (res[m].loss_sum, s["loss_sum"])):
                assert abs(got - want) <= 2e-3 * abs(want), (m, got, want)
            grad = rep.get_grad(m).astype(np.float64)
            assert np.linalg.norm(grad - orc.grads[m]) <= 2e-3 * np.linalg.norm(orc.grads[m]), m
        assert rep.guard_intact()
    finally:
        rep.close()


# What the per-kernel profile says of a launch: the layer where only one is in it, the tile that ran, the bytes of what it stores.
def test_profile_names_the_launch_and_counts_its_bytes():
    A = _A()

    def profile(dims, prec, M, b):
        w = W.Workload("prof", dims, W.ACT_RELU, True, prec, N=256, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.05,
                       test=W.TEST_NORM, data="teacher_mlp", seed=29)
        X, y = W.make_dataset(w)
        rep = A.Replicas.from_workload(w, X, y, W.make_x0(w))
        try:
            rep.profile_enable(True)
            rep.local_step(W.step_indices(w, 0, 0, b), w.lr)
            return rep.profile_read()
        finally:
            rep.close()

    p = profile((64, 136, 40), W.PREC_BF16, 2, 300)
    assert {n for n in p if "wgrad" in n} == {"gemm_wgrad_128x64_L1", "gemm_wgrad_64x128_L2"}
    p = profile((256, 136, 40), W.PREC_BF16, 2, 300)
    assert {n for n in p if "wgrad" in n} == {"gemm_wgrad_64x128_L0"}
    p = profile((256, 136, 40), W.PREC_BF16, 2, 100)
    assert {n for n in p if "wgrad" in n} == {"gemm_wgrad_64x256_L0"}
    p = profile((64, 10), W.PREC_BF16, 3, 50)
    # operands; rows of 16 stored signals, index, label, norm and loss
    assert p["gemm_logits_32x32_L1"]["bytes"] == 3 * ((50 + 10) * 64 * 2 + 50 * (16 * 2 + 16))
    p = profile((64, 10), W.PREC_F32, 3, 50)
    assert p["gemm_logits_128x128_L1"]["bytes"] == 3 * ((50 + 10) * 64 * 4 + 50 * (16 * 4 + 16))
    assert p["gemm_wgrad_128x128_L1"]["bytes"] == 3 * ((10 + 64) * 50 * 4 + 640 * (8 + 4))      # gradient stored beside the step


# Nets of more layers than a shared weight-gradient launch holds (eight): on the short-batch tiles (b = 200), whole reductions on
# 64 x 128 tiles (b = 300, 960 and, around the batch from which slices are weighed, 961) and slices (b = 1100), two steps, with and
# without the step in the epilogue.  Ten layers of bf16 roundings lie between input and gradient: a unit on a tie moves a
# sample's signal by 2^-8 of itself, a few ties per layer and sample; the norms of whole layers stay within 1e-2.
@pytest.mark.parametrize("b", [200, 300, 960, 961, 1100])
@pytest.mark.parametrize("fused", [True, False])
def test_weight_gradients_of_more_layers_than_one_launch_holds(b, fused):
    A = _A()
    dims, M = (128,) * 10 + (10,), 3
    w = W.Workload("deep", dims, W.ACT_GELU, True, W.PREC_BF16, N=2048, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SHB, lr=0.05, momentum=0.9,
                   test=W.TEST_NORM, data="teacher_mlp", seed=31)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, momentum=w.momentum, mixed=True)
    try:
        rep.set_fused_update(fused)
        for h in range(2):
            idx = W.step_indices(w, 0, h, b)
            rep.local_step(idx, w.lr)
            res = rep.norm_test(0.5)
            orc.local_step(idx, w.lr, only=[0, M - 1])
            for m in (0, M - 1):
                g, s = orc.grads[m], orc.stats[m]
                for got, want in ((res[m].sum_sq, s["S1"]), (res[m].gbar_sq, s["S2"]), (res[m].loss_sum, s["loss_sum"])):
                    assert abs(got - want) <= 5e-3 * abs(want), (h, m, got, want)
                got, at = rep.get_grad(m).astype(np.float64), 0
                for fin, fout in zip(dims[:-1], dims[1:]):
                    for size in (fin * fout, fout):
                        part = slice(at, at + size)
                        assert np.linalg.norm(got[part] - g[part]) <= 1e-2 * np.linalg.norm(g[part]), (h, m, at)
                        at += size
                p, v = rep.get_params(m).astype(np.float64), rep.get_opt_state(m, 0).astype(np.float64)
                assert np.abs(p - orc.x[m]).max() <= 1e-3 * np.abs(orc.x[m]).max(), (h, m)
                assert np.linalg.norm(v - orc.st[m].v) <= 1e-2 * np.linalg.norm(orc.st[m].v), (h, m)
                orc.x[m], orc.st[m].v = p, v
        assert rep.guard_intact()
    finally:
        rep.close()


# fp32 weight gradients over long batches: products follow one another for at most 128 samples before their sum is put down, so the
# rounding error does not grow with the batch.  2^-24 is one rounding: the gradient (signals of 1024-long sums included) lies within
# 4.5 of them of its 64-bit value in norm; one chain over the batch drifts by sqrt(b) / 3 of them (9 at b = 1024, 18 at 4096).
@pytest.mark.parametrize("dims,b,roundings", [((784, 10), 1024, 4.5), ((784, 10), 4096, 4.5), ((520, 136, 100), 2048, 7), ((100, 64, 7), 256, 4.5),
                                              ((1024, 256, 100), 1024, 9)])
def test_fp32_weight_gradients_do_not_lose_precision_over_the_batch(dims, b, roundings):
    A = _A()
    act = W.ACT_GELU if len(dims) > 2 else W.ACT_NONE
    w = W.Workload("prec", dims, act, True, W.PREC_F32, N=4096, M=4, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.05, test=W.TEST_NORM,
                   data="teacher_mlp" if len(dims) > 2 else "mixture", seed=101)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, w.M, opt=w.opt)
    try:
        idx = W.step_indices(w, 0, 0, b)
        rep.local_step(idx, w.lr)
        orc.local_step(idx, w.lr, only=[0, 3])
        err = [np.linalg.norm(rep.get_grad(m).astype(np.float64) - orc.grads[m]) / np.linalg.norm(orc.grads[m]) for m in (0, 3)]
        assert max(err) <= roundings * EPS32, err
    finally:
        rep.close()


# Layers of 256 x 256 tiles: up to 512 samples, and up to 1536 where the tiles are many, the step in the epilogue takes smaller
# tiles than the separate update, and MFMAs of another shape; both add the products of an entry in the same order, so the
# parameters and the gradient formed on demand equal those of the separate update.
@pytest.mark.parametrize("b,M,opt,tile", [(257, 2, W.OPT_SHB, "64x128"), (512, 2, W.OPT_SGD, "64x128"), 
                                          (513, 16, W.OPT_ADAMW, "128x256"), (1536, 16, W.OPT_ADAGRAD, "128x256"),
                                          (1537, 16, W.OPT_SHB, "256x256")])
def test_wide_layers_take_the_same_step_in_either_form_of_the_update(b, M, opt, tile):
    A = _A()
    w = W.Workload("wide", (1024, 1032, 1024, 10), W.ACT_RELU, True, W.PREC_BF16, N=1024, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=opt,
                   lr=0.02, momentum=0.9, weight_decay=0.05, test=W.TEST_NORM, data="teacher_mlp", seed=5)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    out = []
    for fused in (True, False):
        rep = A.Replicas.from_workload(w, X, y, x0)
        try:
            rep.set_fused_update(fused)
            rep.profile_enable(True)
            rep.local_step(W.step_indices(w, 0, 0, b), w.lr)
            names = [n for n in rep.profile_read() if n.startswith("gemm_wgrad_")]
            rep.profile_enable(False)
            assert not fused or any(n.startswith("gemm_wgrad_" + tile) for n in names), names
            res = rep.norm_test(0.5)
            out.append((rep.get_params(M - 1), rep.get_grad(M - 1)))
            assert abs(res[M - 1].gbar_sq - np.sum(out[-1][1].astype(np.float64) ** 2)) <= 1e-5 * res[M - 1].gbar_sq
            assert rep.guard_intact()
        finally:
            rep.close()
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])


# The same edges as in the two tests of large tiles above, over so many workers that the launches take 256 x 256 tiles.
@pytest.mark.parametrize("b,fin,fout,M,both", [(1030, 8, 1032, 16, False), (1024, 64, 1024, 16, False), (1025, 72, 1096, 14, False),
                                               (257, 1032, 1040, 14, False), (1027, 1088, 1160, 12, True), (1031, 1024, 1024, 13, True)])
def test_large_tile_contractions_over_many_workers(b, fin, fout, M, both):
    import torch
    A = _A()
    g = torch.Generator(device="cuda").manual_seed(b + fin)
    a = torch.randn((M, b, fin), device="cuda", generator=g).to(torch.bfloat16)
    d = torch.randn((M, b, fout), device="cuda", generator=g).to(torch.bfloat16)
    res, n, q, gbar = A.layer_stats([a], [d], want_per_sample=True, want_gbar=True)
    for m in (0, M // 2, M - 1):
        a64, d64 = a[m].double(), d[m].double()
        G, Gabs = d64.T @ a64 / b, d64.abs().T @ a64.abs() / b
        # bounds as in test_large_tile_contractions_at_the_edges_of_the_reduction
        assert bool(((gbar[m].reshape(fout, fin).double() - G).abs() <= (b + 2) * EPS32 * Gabs).all()), m
        want = (d64 * (a64 @ G.T)).sum(1)
        bound = (EPSBF * (1 + 2 ** -8) + (b + fin + fout + 4) * EPS32) * (d64.abs() * (a64.abs() @ Gabs.T)).sum(1)
        err = (q[m].double() - want).abs()
        assert bool((err <= bound).all()) and float(err.norm() / want.norm()) <= 1e-3, m
        norms = (a64 ** 2).sum(1) * (d64 ** 2).sum(1)
        assert bool(((n[m].double() - norms).abs() <= (fin + fout + 4) * EPS32 * norms).all()), m
        assert abs(res[m].gbar_sq - float((G ** 2).sum())) <= 1e-5 * float((G ** 2).sum()), m


@pytest.mark.parametrize("dims,act,b,M,classes", [((72, 1032, 1040, 130), W.ACT_GELU, 1030, 10, ("fwd", "bwd", "ipdot")),
                                                  ((64, 1048, 1024, 10), W.ACT_RELU, 1030, 10, ("fwd", "bwd", "ipdot")),
                                                  ((72, 2048, 264, 10), W.ACT_GELU, 257, 16, ("fwd", "bwd", "ipdot")),   # row 2 of tiles: one sample
                                                  ((136, 200, 136, 10), W.ACT_RELU, 2500, 16, ("fwd", "bwd", "ipdot"))])  # one column of tiles
def test_large_tile_step_over_many_workers(dims, act, b, M, classes):
    A = _A()
    w = W.Workload("edges", dims, act, True, W.PREC_BF16, N=2048, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SHB, lr=0.05,
                   momentum=0.9, test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=5)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, momentum=w.momentum, mixed=True, want_ip=True)
    try:
        idx = W.step_indices(w, 0, 0, b)
        rep.profile_enable(True)
        rep.local_step(idx, w.lr)
        names = rep.profile_read()
        rep.profile_enable(False)
        for c in classes:
            assert any(x.startswith("gemm_%s_256x256" % c) for x in names), (c, sorted(names))
        g = rep.inner_product_test(w.theta)
        orc.local_step(idx, w.lr, only=[0, M - 1])
        for m in (0, M - 1):
            s = orc.stats[m]
            for got, want in ((g[m].sum_sq, s["S1"]), (g[m].gbar_sq, s["S2"]), (g[m].sum_q, s["S4"]),
                              (g[m].sum_q2, s["S3"]), (g[m].loss_sum, s["loss_sum"])):
                assert abs(got - want) <= 2e-3 * abs(want), (m, got, want)
            grad = rep.get_grad(m).astype(np.float64)
            assert np.linalg.norm(grad - orc.grads[m]) <= 2e-3 * np.linalg.norm(orc.grads[m]), m
            p = rep.get_params(m).astype(np.float64)
            assert np.abs(p - orc.x[m]).max() <= 1e-3 * np.abs(orc.x[m]).max()
        assert rep.guard_intact()
    finally:
        rep.close()


# Bias gradients and per-sample statistics in front of a weight-gradient launch: 64 and 256 columns to a block (more than 16
# partials a column, or not), the last layer summed directly up to 1024 samples (16 classes) or 256 (more), sample blocks of 64,
# workers with batches of their own; every form of the update and the separate statistics agree.
@pytest.mark.parametrize("dims,sizes", [((784, 264, 16), [1024] * 2), ((784, 264, 16), [1025] * 2), ((136, 520, 264, 17), [256, 65, 2]),
                                        ((136, 520, 264, 17), [257, 129, 64]), ((64, 72, 40, 100), [33] * 3), ((64, 136, 10), [2300] * 4)])
def test_the_end_of_a_step_in_front_of_the_weight_gradients(dims, sizes):
    A = _A()
    M, cap = len(sizes), max(sizes)
    out = []
    for fused, mask in ((True, 1), (False, 1), (True, 3)):
        w = W.Workload("tail", dims, W.ACT_GELU, True, W.PREC_BF16, N=2048, M=M, H=1, rounds=1, b0=cap, b_cap=cap, opt=W.OPT_SHB, lr=0.05,
                       momentum=0.9, test=W.TEST_IP if mask == 3 else W.TEST_NORM, theta=0.9, data="teacher_mlp", seed=7)
        X, y = W.make_dataset(w)
        x0 = W.make_x0(w)
        rep = A.Replicas.from_workload(w, X, y, x0)
        orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, momentum=w.momentum, mixed=True)
        try:
            rep.set_fused_update(fused)
            idx = W.step_indices(w, 0, 0, cap)
            rows = [idx[m][:s] for m, s in enumerate(sizes)]
            if len(set(sizes)) == 1:
                rep.local_step(idx, w.lr)
            else:
                rep.local_step_ragged(rows, w.lr)
            orc.local_step(rows, w.lr)
            res = rep.norm_test(0.5)
            for m in range(M):
                st = orc.stats[m]
                for got, want in ((res[m].sum_sq, st["S1"]), (res[m].gbar_sq, st["S2"]), (res[m].loss_sum, st["loss_sum"])):
                    assert abs(got - want) <= 2e-3 * abs(want), (m, got, want)
                at = 0                             # layer by layer: the bias gradients apart
                grad = rep.get_grad(m).astype(np.float64)
                for fin, fout in zip(dims[:-1], dims[1:]):
                    bias = slice(at + fin * fout, at + fin * fout + fout)
                    assert np.linalg.norm(grad[bias] - orc.grads[m][bias]) <= 4e-3 * np.linalg.norm(orc.grads[m][bias]), (m, fout)
                    at = bias.stop
            n = [rep.get_per_sample(m, sizes[m])[0] for m in range(M)]
            out.append(([rep.get_params(m) for m in range(M)], n, [(r.sum_sq, r.loss_sum) for r in res]))
            assert rep.guard_intact()
        finally:
            rep.close()
    for other in out[1:]:
        for m in range(M):
            assert np.array_equal(out[0][0][m], other[0][m]) and np.array_equal(out[0][1][m], other[1][m]), m
            np.testing.assert_allclose(out[0][2][m], other[2][m], rtol=1e-12)      # (the samples' sums in double, other blocks)


# Launches over workers with batches of their own number only the tiles that the workers have: extents at the edges of 64, 128 and
# 256 rows, outputs in bands (wider than eight 256-wide tiles), narrow logits, more workers than a wavefront has lanes.  Sample i's
# activations and signals do not depend on who else is in the batch: norms bit for bit those of a step on the whole batches.
@pytest.mark.parametrize("dims,sizes", [
    ((72, 512, 264, 100), [501, 2, 64, 65]),                                         # 64 x 128
    ((136, 520, 40), [1030, 128, 129, 1025, 2, 127, 384, 1030]),                     # 128 x 128, 128 x 64
    ((40, 2312, 264, 12), [600, 2, 256, 257, 512, 513, 255, 300]),                   # 256 x 256, in bands
    ((72, 264, 264, 100), [257, 2, 129] * 22 + [64, 300, 128, 300]),                 # 70 workers
    ((72, 1032, 1032, 100), [1024, 2, 256] * 21 + [2, 2, 513]),                      # 66 workers, the last ones short
])
def test_ragged_launches_number_the_tiles_that_there_are(dims, sizes):
    A = _A()
    M, cap = len(sizes), max(sizes)
    w = W.Workload("ragged", dims, W.ACT_GELU, True, W.PREC_BF16, N=2048, M=M, H=1, rounds=1, b0=cap, b_cap=cap, opt=W.OPT_SGD, lr=0.0,
                   test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=13)
    X, y = W.make_dataset(w)
    rep = A.Replicas.from_workload(w, X, y, W.make_x0(w))
    try:
        idx = W.step_indices(w, 0, 0, cap)
        rep.local_step(idx, 0.0)
        whole = [rep.get_per_sample(m, cap)[0] for m in range(M)]
        rep.local_step_ragged([idx[m][:s] for m, s in enumerate(sizes)], 0.0)
        res = rep.inner_product_test(0.9)
        for m, s in enumerate(sizes):
            n, q = rep.get_per_sample(m, s, want_q=True)
            assert np.array_equal(n, whole[m][:s]), m
            # sum of q_i = b <gbar, gbar rounded to bf16>: off b ||gbar||^2 by at most 2^-9 of it (and fp32 sums)
            assert abs(q.astype(np.float64).sum() - s * res[m].gbar_sq) <= 2.0 ** -8 * s * res[m].gbar_sq, m
        assert rep.guard_intact()
    finally:
        rep.close()


# The batch gather behind the tiles of the first layer or of the logits, as its own launch beyond 1024 blocks of four
# rows: gathered rows (the gradient reads them), their norms, and a first layer that reads
# the dataset, against the oracle.
@pytest.mark.parametrize("prec,dims,sizes", [
    (W.PREC_F32, (30, 7), [1024] * 4), (W.PREC_F32, (30, 7), [1025] * 4), (W.PREC_F32, (257, 33, 18), [2]), (W.PREC_F32, (100, 66, 10), [33, 2, 17]),
    (W.PREC_F32, (65, 70), [130] * 13), (W.PREC_BF16, (64, 10), [1024] * 4), (W.PREC_BF16, (64, 10), [1025] * 4), (W.PREC_BF16, (72, 10), [2]),
    (W.PREC_BF16, (136, 264, 40), [33, 2, 17]), (W.PREC_BF16, (136, 512, 10), [501] * 8),
    (W.PREC_BF16, (136, 512, 10), [501, 2, 64, 65, 500, 501, 333, 8]),
])
def test_the_gather_behind_the_tiles_of_a_contraction(prec, dims, sizes):
    A = _A()
    M, cap = len(sizes), max(sizes)
    w = W.Workload("gather", dims, W.ACT_RELU if len(dims) > 2 else W.ACT_NONE, True, prec, N=2048, M=M, H=1, rounds=1, b0=cap, b_cap=cap,
                   opt=W.OPT_SGD, lr=0.0, test=W.TEST_NORM, data="teacher_mlp", seed=19)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, mixed=prec == W.PREC_BF16)
    tol = 4e-3 if prec == W.PREC_BF16 else 1e-5      # (signals on a rounding tie of bf16; fp32 sums of at most 1025 terms)
    try:
        idx = W.step_indices(w, 0, 0, cap)
        idx[:, :2] = [0, w.N - 1]                    # the ends of the dataset
        rows = [idx[m][:s] for m, s in enumerate(sizes)]
        if len(set(sizes)) == 1:
            rep.local_step(idx, 0.0)
        else:
            rep.local_step_ragged(rows, 0.0)
        orc.local_step(rows, 0.0)
        res = rep.norm_test(0.5)
        for m in range(M):
            st, grad = orc.stats[m], rep.get_grad(m).astype(np.float64)
            for got, want in ((res[m].sum_sq, st["S1"]), (res[m].gbar_sq, st["S2"]), (res[m].loss_sum, st["loss_sum"])):
                assert abs(got - want) <= tol * abs(want), (m, got, want)
            assert np.linalg.norm(grad - orc.grads[m]) <= tol * np.linalg.norm(orc.grads[m]), m
        assert rep.guard_intact()
    finally:
        rep.close()


# The gradient that is formed on demand after a step in the weight gradients' epilogue is the one that the step applied, which the
# separate update stores: bias sums of a last layer with few column partials (b / 128) beside hidden layers with more than sixteen
# (784-512-512-100: 12 and 48), and the other way round; summed directly; workers with batches of their own.
@pytest.mark.parametrize("dims,sizes", [((784, 512, 512, 100), [1500] * 2), ((784, 512, 512, 10), [1100] * 8), ((784, 264, 16), [1025] * 2),
                                        ((72, 264, 136, 100), [2300] * 2), ((72, 264, 136, 100), [500] * 2), ((72, 264, 136, 17), [1500, 900, 2])])
def test_the_gradient_on_demand_is_the_one_that_the_step_applied(dims, sizes):
    A = _A()
    M, cap = len(sizes), max(sizes)
    w = W.Workload("demand", dims, W.ACT_RELU, True, W.PREC_BF16, N=4096, M=M, H=1, rounds=1, b0=cap, b_cap=cap, opt=W.OPT_SGD, lr=0.05,
                   test=W.TEST_NORM, data="teacher_mlp", seed=23)
    X, y = W.make_dataset(w)
    x0 = 5.0 * W.make_x0(w)                          # (probabilities from 1e-9 to 1: the sums of the signals are not exact in fp32)
    idx = W.step_indices(w, 0, 0, cap)
    out = []
    for fused in (True, False):
        rep = A.Replicas.from_workload(w, X, y, x0)
        try:
            rep.set_fused_update(fused)
            if len(set(sizes)) == 1:
                rep.local_step(idx, w.lr)
            else:
                rep.local_step_ragged([idx[m][:s] for m, s in enumerate(sizes)], w.lr)
            out.append([(rep.get_grad(m), rep.get_params(m)) for m in range(M)])
            assert rep.guard_intact()
        finally:
            rep.close()
    for m in range(M):
        assert np.array_equal(out[0][m][0], out[1][m][0]), (m, np.flatnonzero(out[0][m][0] != out[1][m][0])[:8])
        assert np.array_equal(out[0][m][1], out[1][m][1]), m


# Workers with batches of their own take the tiles that suit what these make, not the largest worker's: one long batch beside short ones
# leaves the 256 x 256 shape of forward, backward-data and inner products, weight gradients go by the mean batch if then no layer keeps it
# (of 3072 inputs the first one does, and the second stays with it).
@pytest.mark.parametrize("dims,sizes,test,gone,there", [
    ((784, 384, 384, 10), [2048] + [257] * 15, W.TEST_IP, ("fwd_256x256", "bwd_256x256", "ipdot_256x256"), ("fwd_128x128", "bwd_128x128", "ipdot_128x128")),
    ((64, 768, 776, 100), [1024] + [130] * 15, W.TEST_NORM, ("fwd_256x256", "bwd_256x256"), ("fwd_128x128", "bwd_128x128")),
    ((784, 512, 512, 10), [int(3000 * 30.0 ** (-m / 15)) for m in range(16)], W.TEST_NORM, ("wgrad_256x256",), ("fwd_256x256",)),
    ((784, 512, 512, 10), [3000] * 9 + [2000] * 7, W.TEST_NORM, (), ("fwd_256x256", "wgrad_256x256")),
    ((3072, 984, 984, 38), [2100] * 2 + [700] * 6, W.TEST_NORM, (), ("wgrad_256x256_L1", "wgrad_256x256_L2"))])
def test_ragged_launches_take_the_tiles_that_suit_their_workers(dims, sizes, test, gone, there):
    A = _A()
    M, cap = len(sizes), max(sizes)
    w = W.Workload("shapes", dims, W.ACT_RELU, True, W.PREC_BF16, N=4096, M=M, H=1, rounds=1, b0=cap, b_cap=cap, opt=W.OPT_SHB, lr=0.05,
                   momentum=0.9, test=test, theta=0.9, data="teacher_mlp", seed=31)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    idx = W.step_indices(w, 0, 0, cap)
    rows = [idx[m][:s] for m, s in enumerate(sizes)]
    orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, momentum=w.momentum, mixed=True, want_ip=test == W.TEST_IP)
    orc.local_step(rows, w.lr, only=[0, M - 1])
    grads = []
    for fused in (True, False):
        rep = A.Replicas.from_workload(w, X, y, x0)
        try:
            rep.set_fused_update(fused)
            rep.profile_enable(True)
            rep.local_step_ragged(rows, w.lr)
            names = [n for n in rep.profile_read() if n.startswith("gemm_")]
            rep.profile_enable(False)
            assert not [n for n in names for c in gone if n.startswith("gemm_" + c)], names
            assert all(any(n.startswith("gemm_" + c) for n in names) for c in there), names
            res = rep.norm_test(0.5)
            for m in (0, M - 1):
                s = orc.stats[m]
                for got, want in ((res[m].sum_sq, s["S1"]), (res[m].gbar_sq, s["S2"]), (res[m].loss_sum, s["loss_sum"])):
                    assert abs(got - want) <= 2e-3 * abs(want), (m, got, want)
                if test == W.TEST_IP:
                    assert abs(res[m].sum_q - s["S4"]) <= 2e-3 * abs(s["S4"]), m
                grad = rep.get_grad(m).astype(np.float64)
                assert np.linalg.norm(grad - orc.grads[m]) <= 2e-3 * np.linalg.norm(orc.grads[m]), m
                p = rep.get_params(m).astype(np.float64)
                assert np.abs(p - orc.x[m]).max() <= 1e-3 * np.abs(orc.x[m]).max()
            grads.append([rep.get_grad(m) for m in range(M)])
            assert rep.guard_intact()
        finally:
            rep.close()
    for m in range(M):
        assert np.array_equal(grads[0][m], grads[1][m]), m


# Sample indices outside the dataset are clamped into it, wherever a row is read from it: in fp32 and in bf16, by the first layer's 32 x 32 and
# 64 x 128 tiles, by the gather behind the tiles or in a launch of its own, by the loss head beside or behind the logits.
@pytest.mark.parametrize("prec,dims,M,b,own", [(W.PREC_F32, (30, 7), 2, 33, False), (W.PREC_F32, (257, 33, 18), 3, 66, False),
                                               (W.PREC_F32, (64, 10), 4, 1025, True), (W.PREC_BF16, (72, 10), 2, 33, False),
                                               (W.PREC_BF16, (136, 264, 40), 3, 33, False), (W.PREC_BF16, (136, 512, 10), 8, 501, False),
                                               (W.PREC_BF16, (136, 264, 100), 8, 600, True)])
def test_indices_outside_the_dataset_are_clamped(prec, dims, M, b, own):
    A = _A()
    w = W.Workload("clamp", dims, W.ACT_RELU if len(dims) > 2 else W.ACT_NONE, True, prec, N=1000, M=M, H=1, rounds=1, b0=b, b_cap=b,
                   opt=W.OPT_SGD, lr=0.05, test=W.TEST_NORM, data="teacher_mlp", seed=29)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    outside = np.array(W.step_indices(w, 0, 0, b), dtype=np.int32)
    outside[:, 1::7], outside[:, 2::7] = -1, w.N
    outside[:, 3::7], outside[:, 4::7] = np.iinfo(np.int32).min, np.iinfo(np.int32).max
    out = []
    for idx in (outside, np.clip(outside, 0, w.N - 1)):
        rep = A.Replicas.from_workload(w, X, y, x0)
        try:
            rep.profile_enable(True)
            rep.local_step(idx, w.lr)
            assert ("gather_rows" in rep.profile_read()) == own
            rep.profile_enable(False)
            res = rep.norm_test(0.5)
            out.append([(rep.get_per_sample(m, b)[0], rep.get_grad(m), rep.get_params(m), [res[m].loss_sum]) for m in range(M)])
            assert rep.guard_intact()
        finally:
            rep.close()
    for m in range(M):
        for got, want in zip(out[0][m], out[1][m]):
            assert np.array_equal(got, want), m


# The per-sample statistics count where they run: norm partials, losses and norms, four bytes each, with the weight gradients that they ride
# in front of or, with inner products, with the statistics.  72 -> 104 -> 40: partials ||a||^2 1 and 4 (forward, 32 columns each), ||delta||^2
# 2 (backward-data, 64 columns) and 1.
def test_profile_counts_the_per_sample_statistics_where_they_run():
    A = _A()
    M, b, got = 3, 33, []
    for test in (W.TEST_NORM, W.TEST_IP):
        w = W.Workload("bytes", (72, 104, 40), W.ACT_RELU, True, W.PREC_BF16, N=1024, M=M, H=1, rounds=1, b0=b, b_cap=b,
                       opt=W.OPT_SGD, lr=0.05, test=test, theta=0.9, data="teacher_mlp", seed=3)
        X, y = W.make_dataset(w)
        rep = A.Replicas.from_workload(w, X, y, W.make_x0(w))
        try:
            rep.profile_enable(True)
            rep.local_step(W.step_indices(w, 0, 0, b), w.lr)
            got.append({n: e["bytes"] for n, e in rep.profile_read().items()})
        finally:
            rep.close()
    sample = 4 * M * b * (1 + 4 + 2 + 1 + 2)
    assert got[0]["gemm_wgrad_64x256_L0"] - got[1]["gemm_wgrad_64x256_L0"] == sample
    assert got[1]["stats"] - got[0]["stats"] == sample + 4 * M * b * 2        # (and q from the Gram matrices: read and stored)


# The fp32 step of a net without hidden layers in one launch: one work-group to a replica (up to 16, 32 or 64 samples), several whose last
# one adds up, the lines between them, rows that are no multiple of 4 or of a wavefront, the most classes and features, workers with
# batches of their own (one chunk beside several); inner products in the same launch or a second one; a second step from non-zero state.
@pytest.mark.parametrize("dims,sizes,opt", [
    ((1, 2), [2, 2], W.OPT_SGD), ((3, 16), [16] * 2, W.OPT_SHB), ((16, 10), [17] * 3, W.OPT_ADAMW), ((65, 5), [32] * 2, W.OPT_ADAGRAD),
    ((257, 16), [33] * 2, W.OPT_SGD), ((512, 10), [64] * 2, W.OPT_ADAMW), ((513, 9), [64] * 2, W.OPT_SHB), ((256, 10), [65] * 4, W.OPT_SGD),
    ((1024, 16), [100] * 2, W.OPT_ADAGRAD), ((1025, 3), [129] * 2, W.OPT_SGD), ((2048, 16), [256], W.OPT_SHB), ((100, 7), [1024] * 3, W.OPT_ADAMW),
    ((100, 7), [1025] * 2, W.OPT_SGD), ((256, 10), [200, 2, 64, 65, 33, 16], W.OPT_SHB), ((30, 11), [64, 5, 40], W.OPT_SGD)])
def test_one_launch_of_a_net_without_hidden_layers(dims, sizes, opt):
    A = _A()
    M, b = len(sizes), max(sizes)
    w = W.Workload("one", dims, W.ACT_NONE, True, W.PREC_F32, N=2048, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=opt, lr=0.05, momentum=0.9,
                   weight_decay=0.05, test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=43)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    try:
        orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=opt, momentum=w.momentum, beta1=w.beta1, beta2=w.beta2, eps=w.eps,
                         weight_decay=w.weight_decay, want_ip=True)
        for h in range(2):
            rows = [W.batch_indices(w.seed, h, 0, m, s, w.N) for m, s in enumerate(sizes)]
            if len(set(sizes)) > 1:
                rep.local_step_ragged(rows, w.lr)
            else:
                rep.local_step(np.stack(rows), w.lr)
            _check_fp32_step(rep, w, orc, rows, range(M))
            res = rep.inner_product_test(0.9)
            for m in range(M):                       # sums of d, K and b fp32 products; a signal p - 1 keeps p's 2^-24, which a small one shows
                s, (n, q) = orc.stats[m], rep.get_per_sample(m, sizes[m], want_q=True)
                np.testing.assert_allclose(n, s["n"], rtol=1e-4, atol=1e-6 * s["n"].max())
                np.testing.assert_allclose(q, s["q"], rtol=1e-3, atol=1e-5 * np.abs(s["q"]).max())
                for got, want in ((res[m].sum_sq, s["S1"]), (res[m].loss_sum, s["loss_sum"]), (res[m].sum_q2, s["S3"]), (res[m].sum_q, s["S4"])):
                    assert abs(got - want) <= 1e-4 * abs(want), (m, got, want)
        assert rep.guard_intact()
    finally:
        rep.close()


# Batches below the cap that take more of its chunks than the cap itself: 16 samples each up to 128 of them, 32 or 64 beside that, so the
# scratch of a replica is not the cap's; single sizes and workers with batches of their own, one context through all of them.
@pytest.mark.parametrize("dims,cap,steps,opt", [
    ((784, 10), 130, ([65] * 4, [113] * 4, [128] * 4, [130] * 4, [16] * 4), W.OPT_SHB),
    ((512, 10), 150, ([64] * 3, [65] * 3, [128] * 3, [129] * 3, [128, 150, 17]), W.OPT_SGD),
    ((1024, 16), 224, ([97] * 2, [128, 65], [129] * 2, [128] * 2, [224] * 2), W.OPT_SGD)])
def test_one_launch_of_batches_below_the_cap(dims, cap, steps, opt):
    A = _A()
    M = len(steps[0])
    w = W.Workload("below", dims, W.ACT_NONE, True, W.PREC_F32, N=2048, M=M, H=1, rounds=1, b0=16, b_cap=cap, opt=opt, lr=0.05, momentum=0.9,
                   test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=67)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    try:
        orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=opt, momentum=w.momentum, want_ip=True)
        for h, sizes in enumerate(steps):
            rows = [W.batch_indices(w.seed, h, 0, m, s, w.N) for m, s in enumerate(sizes)]
            if len(set(sizes)) > 1:
                rep.local_step_ragged(rows, w.lr)
            else:
                rep.local_step(np.stack(rows), w.lr)
            _check_fp32_step(rep, w, orc, rows, range(M))
            res = rep.inner_product_test(0.9)
            for m in range(M):                       # (as above)
                s, (n, q) = orc.stats[m], rep.get_per_sample(m, sizes[m], want_q=True)
                np.testing.assert_allclose(n, s["n"], rtol=1e-4, atol=1e-6 * s["n"].max())
                np.testing.assert_allclose(q, s["q"], rtol=1e-3, atol=1e-5 * np.abs(s["q"]).max())
                for got, want in ((res[m].sum_sq, s["S1"]), (res[m].loss_sum, s["loss_sum"]), (res[m].sum_q2, s["S3"]), (res[m].sum_q, s["S4"])):
                    assert abs(got - want) <= 1e-4 * abs(want), (h, m, got, want)
        assert rep.guard_intact()
    finally:
        rep.close()


# Replays of a captured step of that kind, where a replica's work-groups count their arrivals: bit for bit the direct steps.
def test_replayed_steps_of_a_net_without_hidden_layers():
    import torch
    A = _A()
    w = W.Workload("replay", (100, 10), W.ACT_NONE, True, W.PREC_F32, N=1024, M=3, H=1, rounds=1, b0=40, b_cap=130, opt=W.OPT_SHB, lr=0.05,
                   momentum=0.9, test=W.TEST_IP, theta=0.9, data="mixture", seed=47)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    with torch.cuda.stream(torch.cuda.Stream()):
        ref, rep = (A.Replicas.from_workload(w, X, y, x0) for _ in range(2))
        try:
            for s, b in enumerate([130, 40, 130, 130, 40, 40, 130, 40, 130]):
                idx = W.step_indices(w, s, 0, b)
                (t1, _), (t2, _) = ref.upload_indices(idx), rep.upload_indices(idx)
                ref.local_step_dev(t1, b, w.lr)
                rep.local_step_graphed_dev(t2, b, w.lr)
                for g1, g2 in zip(ref.inner_product_test(w.theta), rep.inner_product_test(w.theta)):
                    assert (g1.sum_sq, g1.gbar_sq, g1.sum_q, g1.sum_q2, g1.loss_sum) == (g2.sum_sq, g2.gbar_sq, g2.sum_q, g2.sum_q2, g2.loss_sum), s
                assert all(np.array_equal(ref.get_params(m), rep.get_params(m)) for m in range(w.M)), s
            assert rep.graph_count() == 2
        finally:
            ref.close()
            rep.close()


# Forward, head and backward-data in one launch (nets of two to four layers on 32-row tiles, at most 32 classes): blocks of rows with one row,
# empty ones of workers with batches of their own, one and several tiles to a pass, reductions of more than one trip (1096), the most
# classes, and the first nets beyond (33 classes, five layers); batch sizes that change from step to step, so that every launch finds the
# arrivals of a differently shaped one put back; the last ones replayed from captured graphs, bit for bit the direct step.
@pytest.mark.parametrize("dims,act,steps", [
    ((8, 8, 2), W.ACT_RELU, ([2, 2], [33, 33], [33, 2], [2, 2])), ((72, 40, 32), W.ACT_GELU, ([31] * 3, [65, 32, 2], [65] * 3)),
    ((264, 72, 104, 17), W.ACT_GELU, ([33] * 2, [96, 1 + 32], [64] * 2)), ((40, 1096, 64, 8, 5), W.ACT_RELU, ([32] * 2, [40, 2], [40] * 2)),
    ((1096, 136, 520, 10), W.ACT_NONE, ([66], [7], [66])), ((72, 40, 33), W.ACT_GELU, ([33] * 2, [9, 33])),
    ((40, 24, 24, 24, 24, 6), W.ACT_RELU, ([33] * 2, [9, 33]))])
def test_passes_in_one_launch(dims, act, steps):
    import torch
    A = _A()
    M, cap = len(steps[0]), max(max(s) for s in steps)
    w = W.Workload("chain", dims, act, True, W.PREC_BF16, N=512, M=M, H=1, rounds=1, b0=cap, b_cap=cap, opt=W.OPT_SGD, lr=0.02,
                   test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=53)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    with torch.cuda.stream(torch.cuda.Stream()):
        rep, twin = (A.Replicas.from_workload(w, X, y, x0) for _ in range(2))
        orc = O.Replicas(O.Net(w.dims, w.act, True), x0, X, y, M, opt=w.opt, mixed=True, want_ip=True, gram_max_b=256)
        try:
            for h, sizes in enumerate(steps):
                rows = [W.batch_indices(w.seed, h, 0, m, s, w.N) for m, s in enumerate(sizes)]
                if len(set(sizes)) > 1:
                    rep.local_step_ragged(rows, w.lr)
                else:
                    rep.local_step(np.stack(rows), w.lr)
                orc.local_step(rows, w.lr)
                res = rep.inner_product_test(w.theta)
                for m in range(M):
                    s = orc.stats[m]
                    for got, want in ((res[m].sum_sq, s["S1"]), (res[m].gbar_sq, s["S2"]), (res[m].loss_sum, s["loss_sum"])):
                        assert abs(got - want) <= 2e-3 * abs(want), (h, m, got, want)
                    grad = rep.get_grad(m).astype(np.float64)
                    assert np.linalg.norm(grad - orc.grads[m]) <= 2e-3 * np.linalg.norm(orc.grads[m]), (h, m)
                    p = rep.get_params(m).astype(np.float64)
                    assert np.abs(p - orc.x[m]).max() <= 1e-3 * np.abs(orc.x[m]).max(), (h, m)
                    orc.x[m] = p
            for m in range(M):
                twin.set_params(m, rep.get_params(m))
            for h in range(4):
                idx = W.step_indices(w, 10 + h, 0, cap)
                (t1, _), (t2, _) = rep.upload_indices(idx), twin.upload_indices(idx)
                rep.local_step_dev(t1, cap, w.lr)
                twin.local_step_graphed_dev(t2, cap, w.lr)
                for g1, g2 in zip(rep.inner_product_test(w.theta), twin.inner_product_test(w.theta)):
                    assert (g1.sum_sq, g1.gbar_sq, g1.sum_q, g1.sum_q2, g1.loss_sum) == (g2.sum_sq, g2.gbar_sq, g2.sum_q, g2.sum_q2, g2.loss_sum), h
                assert all(np.array_equal(rep.get_params(m), twin.get_params(m)) for m in range(M)), h
            assert rep.guard_intact() and twin.guard_intact()
        finally:
            rep.close()
            twin.close()


# One replica more and the passes are launches of their own (225 and 226 blocks of 32 rows): the others' results are bit for bit the same.
@pytest.mark.parametrize("dims,act,M,b", [((16, 48, 10), W.ACT_RELU, 224, 4), ((72, 40, 32), W.ACT_GELU, 112, 33)])
def test_passes_in_one_launch_are_bitwise_the_launches_apart(dims, act, M, b):
    import ctypes as C
    A = _A()
    got = []
    for groups in (M, M + 1):
        w = W.Workload("apart", dims, act, True, W.PREC_BF16, N=512, M=groups, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SHB, lr=0.02, momentum=0.9,
                       test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=83)
        X, y = W.make_dataset(w)
        rep = A.Replicas.from_workload(w, X, y, W.make_x0(w))
        try:
            sizes = [b - m % 3 for m in range(groups)]       # (workers with batches of their own take no blocks of rows)
            host, net = (C.c_int * groups)(*sizes), (C.c_int * len(dims))(*dims)
            fits, shape = rep._lib["_ZN4absk16small_chain_fitsEiPKiiixS1_"], rep._lib["_ZN4absk20gemm_bf16_tile_shapeEiiiiPKi"]
            fits.restype = C.c_bool
            assert fits(len(dims) - 1, net, b, groups, C.c_longlong(w.N), host) == (groups == M)
            assert all(shape(0, b, d, groups, host) == 5 for d in dims[1:-1])
            for h in range(3):
                rep.local_step_ragged([W.batch_indices(w.seed, h, 0, m, n, w.N) for m, n in enumerate(sizes)], w.lr)
            res = rep.inner_product_test(w.theta)
            got.append([((r.sum_sq, r.sum_q, r.sum_q2, r.loss_sum), rep.get_per_sample(m, sizes[m], want_q=True), rep.get_grad(m), rep.get_params(m))
                        for m, r in enumerate(res[:M])])
        finally:
            rep.close()
    for m, (a, c) in enumerate(zip(*got)):
        assert a[0] == c[0], m
        assert all(np.array_equal(u, v) for u, v in zip((*a[1], *a[2:]), (*c[1], *c[2:]))), m


# A wait inside such a launch that gives up (no poll allowed, so that every tile reads what is there) is no step: every read-back says so, for the
# context that it happened in.
def test_a_wait_that_gives_up_is_an_error():
    A = _A()
    w = W.Workload("wait", (72, 40, 5), W.ACT_RELU, True, W.PREC_BF16, N=512, M=2, H=1, rounds=1, b0=33, b_cap=33, opt=W.OPT_SHB, lr=0.02,
                   momentum=0.9, test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=71)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep, other = (A.Replicas.from_workload(w, X, y, x0) for _ in range(2))
    try:
        for r in (rep, other):
            r.local_step(W.step_indices(w, 0, 0, 33), w.lr)
            r.inner_product_test(w.theta)
        rep._lib["_ZN4absk15set_chain_pollsEP7abs_ctxi"](rep._ctx, 0)
        for r in (rep, other):
            r.local_step(W.step_indices(w, 1, 0, 33), w.lr)
        for call in (lambda r: r.inner_product_test(w.theta), lambda r: r.norm_test(0.5), lambda r: r.get_params(0), lambda r: r.get_grad(1),
                     lambda r: r.get_opt_state(0), lambda r: r.get_per_sample(0, 33), lambda r: r.cross_worker_test(0.5)):
            with pytest.raises(A.AbsError, match="gave up waiting"):
                call(rep)
            call(other)
        assert rep.guard_intact()
    finally:
        rep.close()
        other.close()


# All passes of a block of rows in one work-group: blocks of 16, 32 and 64 rows, layers up to 256 and up to 512, last blocks of one row and
# full ones, the widest inputs and the most classes, widths that fill no whole wavefront, no activation and no biases, indices outside the
# dataset; and the first nets beyond (904 inputs, 129 classes, a layer of 520).  No ReLU where a layer of 24 takes in 500: a unit within an
# fp32 rounding of zero (one in 10^6) is on in one order of additions and off in another, a 24th of that sample's signal.
@pytest.mark.parametrize("dims,act,bias,M,b", [
    ((896, 256, 40, 2), W.ACT_RELU, True, 16, 129), ((8, 8, 128), W.ACT_GELU, True, 16, 131), ((200, 136, 264 - 8, 16, 17), W.ACT_GELU, True, 16, 257),
    ((72, 40, 33), W.ACT_NONE, False, 24, 321), ((264, 64, 10), W.ACT_RELU, True, 32, 513), ((784, 264, 10), W.ACT_GELU, True, 24, 145),
    ((136, 512, 24, 512, 100), W.ACT_GELU, True, 24, 177), ((40, 336, 128), W.ACT_NONE, True, 24, 192), ((328, 48, 504, 5), W.ACT_GELU, False, 24, 321),
    ((904, 40, 5), W.ACT_RELU, True, 16, 160), ((40, 24, 129), W.ACT_GELU, True, 16, 160), ((40, 520, 24, 6), W.ACT_GELU, True, 24, 177)])
def test_blocks_of_rows_through_all_layers(dims, act, bias, M, b):
    A = _A()
    w = W.Workload("rows", dims, act, bias, W.PREC_BF16, N=512, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.02, test=W.TEST_IP,
                   theta=0.9, data="teacher_mlp", seed=59)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    rep = A.Replicas.from_workload(w, X, y, x0)
    orc = O.Replicas(O.Net(w.dims, w.act, bias), x0, X, y, M, opt=w.opt, mixed=True, want_ip=True, gram_max_b=256)
    try:
        for h in range(2):
            idx = W.step_indices(w, h, 0, b)
            seen = idx.copy()
            seen[:, -1], seen[0, 0] = 2 * w.N, -3
            rep.local_step(seen, w.lr)
            orc.local_step(np.clip(seen, 0, w.N - 1), w.lr)
            res = rep.inner_product_test(w.theta)
            for m in range(M):
                s = orc.stats[m]
                for got, want in ((res[m].sum_sq, s["S1"]), (res[m].gbar_sq, s["S2"]), (res[m].loss_sum, s["loss_sum"])):
                    assert abs(got - want) <= 2e-3 * abs(want), (h, m, got, want)
                n, _ = rep.get_per_sample(m, b)
                np.testing.assert_allclose(n, s["n"], rtol=2e-2, atol=2e-3 * s["n"].max())
                grad = rep.get_grad(m).astype(np.float64)
                assert np.linalg.norm(grad - orc.grads[m]) <= 2e-3 * np.linalg.norm(orc.grads[m]), (h, m)
                p = rep.get_params(m).astype(np.float64)
                assert np.abs(p - orc.x[m]).max() <= 1e-3 * np.abs(orc.x[m]).max(), (h, m)
                orc.x[m] = p
        assert rep.guard_intact()
    finally:
        rep.close()


# The same launches in replayed steps (bit for bit the direct ones, sizes in turns), in the micro-batches of a larger step, and under inner
# products from Gram matrices (up to b = 256) and from the batch gradient; tolerances as accumulated steps have them, twice that for squares.
@pytest.mark.parametrize("dims,act,bias,sizes,micro,total", [((136, 72, 40, 10), W.ACT_GELU, True, (330, 150), 150, 449),
                                                             ((264, 312, 10), W.ACT_NONE, False, (330, 224), 224, 448)])
def test_blocks_of_rows_replayed_and_in_micro_batches(dims, act, bias, sizes, micro, total):
    import ctypes as C
    import torch
    A = _A()
    M, cap = 16, max(sizes)
    w = W.Workload("rows", dims, act, bias, W.PREC_BF16, N=1024, M=M, H=1, rounds=1, b0=cap, b_cap=cap, opt=W.OPT_SHB, lr=0.02, momentum=0.9,
                   test=W.TEST_IP, theta=0.9, data="teacher_mlp", seed=79)
    X, y = W.make_dataset(w)
    x0 = W.make_x0(w)
    orc = O.Replicas(O.Net(w.dims, w.act, bias), x0, X, y, M, opt=w.opt, momentum=w.momentum, mixed=True, want_ip=True, gram_max_b=256)

    def check(r, b, stored):
        res = r.inner_product_test(w.theta)
        for m in range(M):
            s, (n, q) = orc.stats[m], r.get_per_sample(m, stored, want_q=True)
            np.testing.assert_allclose(n, s["n"][:stored], rtol=2e-2, atol=2e-3 * s["n"].max())
            np.testing.assert_allclose(q, s["q"][:stored], rtol=2e-2, atol=2e-3 * np.abs(s["q"]).max())
            for k, got, want in ((1, res[m].sum_sq, s["S1"]), (1, res[m].gbar_sq, s["S2"]), (1, res[m].sum_q, s["S4"]), (2, res[m].sum_q2, s["S3"]),
                                 (1, res[m].loss_sum, s["loss_sum"])):
                assert abs(got - want) <= k * 2e-3 * abs(want), (b, m, got, want)
            grad = r.get_grad(m).astype(np.float64)
            assert np.linalg.norm(grad - orc.grads[m]) <= 2e-3 * np.linalg.norm(orc.grads[m]), (b, m)

    with torch.cuda.stream(torch.cuda.Stream()):
        ref, rep = (A.Replicas.from_workload(w, X, y, x0) for _ in range(2))
        try:
            rows = rep._lib["_ZN4absk14mlp_rows_blockEiPKiiix"]
            assert all(rows(len(dims) - 1, (C.c_int * len(dims))(*dims), b, M, C.c_longlong(w.N)) for b in (*sizes, micro, total % micro or micro))
            for h, b in enumerate(sizes * 4):
                idx = W.step_indices(w, h, 0, b)
                (t1, _), (t2, _) = ref.upload_indices(idx), rep.upload_indices(idx)
                ref.local_step_dev(t1, b, w.lr)
                rep.local_step_graphed_dev(t2, b, w.lr)
                if h < 2:
                    orc.local_step(idx, w.lr)
                    check(ref, b, b)
                for g1, g2 in zip(ref.inner_product_test(w.theta), rep.inner_product_test(w.theta)):
                    assert (g1.sum_sq, g1.gbar_sq, g1.sum_q, g1.sum_q2, g1.loss_sum) == (g2.sum_sq, g2.gbar_sq, g2.sum_q, g2.sum_q2, g2.loss_sum), h
                assert all(np.array_equal(ref.get_params(m), rep.get_params(m)) for m in range(M)), h
            assert rep.graph_count() == 2
            for m in range(M):
                orc.x[m] = rep.get_params(m).astype(np.float64)
            idx = W.step_indices(w, 9, 0, total)
            rep.local_step_accumulated(idx, micro, w.lr)
            orc.local_step(idx, w.lr)
            check(rep, total, cap // micro * micro)          # (whole micro-batches that fit the cap are stored)
            assert ref.guard_intact() and rep.guard_intact()
        finally:
            ref.close()
            rep.close()


# Weight gradients of long batches in slices of 256 x 256 tiles, all layers in one launch: two and four slices, the last one shorter and its
# last k-tile cut, widths that leave most of a tile empty; the sums and the step as in every other form.
@pytest.mark.parametrize("dims,M,b,opt", [((784, 512, 10), 12, 4001, W.OPT_ADAMW), ((784, 256, 256, 10), 8, 4090, W.OPT_SHB),
                                          ((776, 504, 264, 2), 8, 3900, W.OPT_SGD)])
def test_weight_gradients_in_slices_of_large_tiles(dims, M, b, opt):
    A = _A()
    w = W.Workload("slices", dims, W.ACT_RELU, True, W.PREC_BF16, N=512, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=opt, lr=0.02, momentum=0.9,
                   test=W.TEST_NORM, data="teacher_mlp", seed=61)
    X, y = W.make_dataset(w)
    rep = A.Replicas.from_workload(w, X, y, W.make_x0(w))
    try:
        rep.profile_enable(True)
        rep.local_step(W.step_indices(w, 0, 0, b), w.lr)
        assert [n for n in rep.profile_read() if n.startswith("gemm_wgrad_")] == ["gemm_wgrad_256x256_L0"]
    finally:
        rep.close()
    test_weight_gradient_launches_of_long_batches(dims, M, b, opt, 0)


# Slices in more than one round of CUs, which are slower than the other forms though the model prices them a little lower
@pytest.mark.parametrize("dims,M,b", [((400, 136, 176, 256, 152, 12), 26, 1362), ((1496, 240, 472, 768, 192, 23), 15, 1716)])
def test_weight_gradients_in_one_round_of_slices_only(dims, M, b):
    A = _A()
    w = W.Workload("rounds", dims, W.ACT_RELU, True, W.PREC_BF16, N=512, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.02,
                   test=W.TEST_NORM, data="teacher_mlp", seed=61)
    X, y = W.make_dataset(w)
    rep = A.Replicas.from_workload(w, X, y, W.make_x0(w))
    try:
        rep.profile_enable(True)
        rep.local_step(W.step_indices(w, 0, 0, b), w.lr)
        assert "gemm_wgrad_256x256_L0" not in rep.profile_read()
    finally:
        rep.close()


# A launch that is the work of several classes is timed once, and its time goes to them by their bytes
@pytest.mark.parametrize("dims,prec,M,b,n", [((256, 10), W.PREC_F32, 4, 64, 2), ((784, 512, 512, 10), W.PREC_BF16, 2, 32, 5), ((784, 512, 512, 10), W.PREC_BF16, 8, 501, 5),
                                             ((784, 256, 256, 10), W.PREC_BF16, 16, 600, 6)])
def test_profile_shares_the_time_of_a_launch_by_bytes(dims, prec, M, b, n):
    A = _A()
    w = W.Workload("shares", dims, W.ACT_RELU, True, prec, N=1024, M=M, H=1, rounds=1, b0=b, b_cap=b, opt=W.OPT_SGD, lr=0.02, test=W.TEST_NORM,
                   data="teacher_mlp", seed=73)
    X, y = W.make_dataset(w)
    rep = A.Replicas.from_workload(w, X, y, W.make_x0(w))
    try:
        rep.profile_enable(True)
        for h in range(3):
            rep.local_step(W.step_indices(w, h, 0, b), w.lr)
        shared = {k: v for k, v in rep.profile_read().items() if k == "gather_rows" or k.startswith(("gemm_fwd_", "gemm_logits_", "gemm_bwd_")) or prec == W.PREC_F32}
        assert len(shared) == n and all(v["calls"] == 3 and v["total_ms"] > 0 for v in shared.values())
        rate = [v["total_ms"] / v["bytes"] for v in shared.values()]
        assert max(rate) <= min(rate) * (1 + 1e-9)
    finally:
        rep.close()
