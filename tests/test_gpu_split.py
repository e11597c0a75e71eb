"""Contractions on bf16 triples: the step, the queries and the exchange (up to 256
neurons in 2D, 208 in 3D) against the FP64 oracle at the edges of
their tiles: one and two row blocks, an even and an odd number of them (the last K block
holds 16 neurons), the last and the first width of a range, ragged point tiles, both activations."""
import numpy as np
import pytest

import workloads as wl
from parity import assert_close, channel_tolerances, oracle_loss_grad, rel_report

torch = pytest.importorskip("torch")

CASES = [(2, 1, 2, "tanh", 1), (2, 16, 3, "sin", 16), (3, 17, 3, "tanh", 17), (2, 32, 2, "sin", 33),
         (3, 33, 4, "sin", 40), (2, 48, 3, "tanh", 97), (3, 80, 2, "tanh", 15), (2, 112, 3, "tanh", 100),
         (3, 112, 3, "sin", 50), (2, 127, 2, "sin", 64), (3, 128, 3, "tanh", 65), (2, 128, 16, "tanh", 31)]
WIDE = [(2, 129, 2, "tanh", 100), (2, 256, 3, "sin", 97), (3, 144, 2, "tanh", 129), (3, 208, 3, "sin", 130)]


def test_triples_hold_every_fp32():
    """Round-to-nearest bf16 of x, of the remainder, and what is left: the three
    sum to x exactly (the split the kernels make of every operand)."""
    rng = np.random.default_rng(0)
    x = np.concatenate([rng.standard_normal(1 << 16) * 10.0 ** rng.uniform(-25, 25, 1 << 16),
                        1.0 + np.arange(1 << 16) * 2.0 ** -23]).astype(np.float32)

    def bf16(v):
        u = v.view(np.uint32).astype(np.uint64)
        return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)

    h = bf16(x)
    m = bf16(x - h)
    lo = bf16((x - h) - m)
    assert np.array_equal((h.astype(np.float64) + m + lo).astype(np.float32), x)
    assert np.array_equal((x - h) - m, lo)


@pytest.mark.gpu
@pytest.mark.parametrize("dim,W,H,act,npde", CASES + WIDE)
def test_split_kernels_against_oracle(orc, dim, W, H, act, npde):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_15883_amd as P
    print(f"split dim={dim} W={W} H={H} act={act} n={npde}", flush=True)
    orc.set_activation(act)
    try:
        pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=npde, n_obs=5 + npde, n_gh=7, n_anc=1, seed=3 * W + H)
        pb.activation = act
        # rounding of a chain of H contractions over W terms and back, twice differentiated
        tol = 16 * H * np.sqrt(W + 16) * 2.0 ** -24 * 4
        ctx = P.context_from_problem(pb, device="cuda")
        try:
            loss, g = ctx.step(1, update=False, want_grad=True)
            torch.cuda.synchronize()
            Lr, gr = oracle_loss_grad(orc, pb)
            for name, a, b in (("loss", loss.cpu().numpy()[0], Lr), ("grad", g.cpu().numpy()[0], gr)):
                assert rel_report(a, b)[1] <= tol, (name, rel_report(a, b), tol)
            x = pb.subs[0].pde_x
            xt = torch.from_numpy(np.ascontiguousarray(x)).cuda()
            ref = orc.channels(dim, W, H, pb.subs[0].theta, x)
            ch = ctx.query(xt, sub=0, what="channels").cpu().numpy().reshape(len(x), 2 * dim + 2, dim + 1)
            for c, t in enumerate(channel_tolerances(dim)):
                assert_close(ch[:, c], ref[:, c], t, f"channel {c}")
            assert_close(ctx.query(xt, sub=0, what="value").cpu().numpy(), ref[:, 0], 1e-5, "value")
        finally:
            ctx.close()
    finally:
        orc.set_activation("tanh")


@pytest.mark.gpu
@pytest.mark.parametrize("dim,W,H,act,waves", [(3, 96, 3, "tanh", 4), (2, 80, 2, "sin", 4), (3, 65, 2, "sin", 4),
                                               (2, 96, 2, "tanh", 4), (2, 97, 2, "tanh", 7)])
def test_two_workgroups_per_compute_unit(orc, dim, W, H, act, waves):
    """Five or six row blocks and more tiles than compute units: workgroups of four
    waves, one or two of which own two row blocks and hand on the dW of the second;
    seven row blocks: one workgroup of seven waves."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_15883_amd as P
    print(f"halves dim={dim} W={W} H={H} act={act}", flush=True)
    orc.set_activation(act)
    try:
        pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=16 * 300 + 3, n_obs=70, n_gh=7, n_anc=1, seed=W)
        pb.activation = act
        tol = 16 * H * np.sqrt(W + 16) * 2.0 ** -24 * 4
        Lr, gr = oracle_loss_grad(orc, pb)
        for per_cu, threads in ((0, 64 * waves), (1, 64 * ((W + 15) // 16))):
            ctx = P.context_from_problem(pb, device="cuda", blocks_per_cu=per_cu)
            try:
                assert ctx.launch_info()["threads"] == threads
                loss, g = ctx.step(1, update=False, want_grad=True)
                for name, a, b in (("loss", loss.cpu().numpy()[0], Lr), ("grad", g.cpu().numpy()[0], gr)):
                    assert rel_report(a, b)[1] <= tol, (name, per_cu, rel_report(a, b), tol)
            finally:
                ctx.close()
    finally:
        orc.set_activation("tanh")


@pytest.mark.gpu
@pytest.mark.parametrize("dim,W,H,act", [(2, 16, 2, "tanh"), (2, 80, 3, "sin"), (3, 112, 3, "tanh"), (2, 128, 2, "sin"),
                                         (3, 144, 2, "tanh")])
@pytest.mark.parametrize("n", [4097, 8191, 16401, 32769])
def test_value_queries_by_size(orc, dim, W, H, act, n):
    """One tile per compute unit and more: the value kernels of small tiles, of half
    the registers, and of full tiles."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_15883_amd as P
    print(f"values dim={dim} W={W} n={n}", flush=True)
    orc.set_activation(act)
    try:
        pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=n, n_obs=5, n_gh=0, n_anc=1, seed=W)
        pb.activation = act
        x = np.ascontiguousarray(pb.subs[0].pde_x)
        ctx = P.context_from_problem(pb, device="cuda")
        try:
            got = ctx.query(torch.from_numpy(x).cuda(), sub=0, what="value").cpu().numpy()
        finally:
            ctx.close()
        assert_close(got, orc.channels(dim, W, H, pb.subs[0].theta, x)[:, 0], 1e-5, "value")
    finally:
        orc.set_activation("tanh")


@pytest.mark.gpu
@pytest.mark.parametrize("dim,W,H,act,clip", [(2, 50, 3, "tanh", 0.0), (3, 17, 2, "sin", 1e-3), (2, 112, 1, "tanh", 0.0),
                                              (2, 150, 2, "sin", 0.5), (3, 200, 2, "tanh", 0.0), (3, 240, 2, "tanh", 1.0)])
def test_adam_leaves_the_weight_copies_current(dim, W, H, act, clip):
    """The update writes the parameters and the kernels' copies of them together:
    a query after it equals one after the copies are rebuilt from theta, bitwise."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_15883_amd as P
    print(f"copies dim={dim} W={W} H={H} clip={clip}", flush=True)
    pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=40, n_obs=9, n_gh=5, n_anc=2, seed=W)
    pb.activation, pb.clip_norm = act, clip
    x = torch.from_numpy(np.ascontiguousarray(pb.subs[0].pde_x)).cuda()
    ctx = P.context_from_problem(pb, device="cuda", graph=clip == 0.0)
    try:
        before = ctx.query(x, sub=0, what="channels").clone()
        ctx.step(1)
        after = ctx.query(x, sub=0, what="channels").clone()
        ctx.refresh()
        assert torch.equal(after, ctx.query(x, sub=0, what="channels"))
        assert not torch.equal(before, after)
    finally:
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("dim,W", [(2, 16), (3, 30), (2, 40), (3, 100), (2, 150)])
def test_weights_up_to_the_largest_fp32(orc, dim, W):
    """Finite weights above the largest bf16 (3.39e38), whose neurons saturate: values,
    a step on value points and the copies it leaves behind stay finite."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_15883_amd as P
    print(f"large weights dim={dim} W={W}", flush=True)
    H, top = 3, float(np.finfo(np.float32).max)
    pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=300, n_obs=40, n_gh=0, n_anc=0, seed=W)
    s = pb.subs[0]
    x, s.pde_x = np.ascontiguousarray(s.pde_x), s.pde_x[:0]
    D = dim + 1
    w2 = W * D + W                            # W_2, then b_2, then W_3
    s.theta[w2] = top
    s.theta[w2 + (W - 1) * W + 2] = -top
    s.theta[w2 + W * W + W + W + 1] = 3.3961e38
    ref = orc.channels(dim, W, H, s.theta, x)[:, 0]
    pb.lr = 0.0
    ctx = P.context_from_problem(pb, device="cuda")
    try:
        xt = torch.from_numpy(x).cuda()
        assert_close(ctx.query(xt, sub=0, what="value").cpu().numpy(), ref, 1e-5, "value")
        loss, g = ctx.step(1, want_grad=True)
        Lr, gr = oracle_loss_grad(orc, pb)
        assert rel_report(loss.cpu().numpy()[0], Lr)[1] <= 1e-5
        assert bool(torch.isfinite(g).all())
        assert_close(ctx.query(xt, sub=0, what="value").cpu().numpy(), ref, 1e-5, "value after the update")
    finally:
        ctx.close()
