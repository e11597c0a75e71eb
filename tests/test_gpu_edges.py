"""Edges of the launch shapes and of the workspace: many subdomains of a small
network, the smallest and the largest networks of a query kernel, the 32-point tile."""
import numpy as np
import pytest

import workloads as wl
from parity import assert_close, channel_tolerances, oracle_loss_grad, rel_report
from test_split_scheme import BOUND_GRAD

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pkg():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_15883_amd as P
    P.lib()
    return P


@pytest.mark.parametrize("dim,W,n_sub", [(2, 16, 600), (3, 5, 1100)])
def test_range_counters_of_many_subdomains(pkg, monkeypatch, dim, W, n_sub):
    """One hidden layer of one row block has fewer weight copies than there are
    subdomains: the plain launches' range counters, one per subdomain, are all set
    before use, whatever the caller's workspace held."""
    print(f"counters dim={dim} W={W} n_sub={n_sub}", flush=True)
    one = [wl.tiny(dim=dim, width=W, depth=1, n_pde=5 + s % 13, n_obs=3, n_gh=2, n_anc=1, seed=s) for s in range(n_sub)]
    pb = one[0]
    pb.subs = [p.subs[0] for p in one]
    empty = torch.empty

    def filled(*a, **k):   # a workspace full of large positive integers
        t = empty(*a, **k)
        return t.fill_(0x7f) if t.dtype == torch.uint8 else t

    monkeypatch.setattr(torch, "empty", filled)
    ctx = pkg.context_from_problem(pb, device="cuda")
    monkeypatch.undo()
    try:
        for _ in range(2):
            lp, gp = [t.cpu().numpy().astype(np.float64) for t in ctx.step(1, update=False, want_grad=True, per_subdomain=True)]
            lg, gg = [t.cpu().numpy().astype(np.float64) for t in ctx.step(1, update=False, want_grad=True)]
            # the same few terms, added in another grouping
            assert rel_report(lp, lg)[1] <= 64 * 2.0 ** -24 and rel_report(gp, gg)[1] <= 64 * 2.0 ** -24
            for s in (0, n_sub // 2, n_sub - 1):
                assert rel_report(gp[s], gg[s])[1] <= 64 * 2.0 ** -24, s
    finally:
        ctx.close()


@pytest.mark.parametrize("dim,W,act", [(2, 3, "tanh"), (2, 16, "sin"), (3, 16, "tanh"), (2, 17, "tanh"), (3, 24, "sin"),
                                       (2, 32, "sin"), (3, 32, "tanh"), (2, 33, "tanh"), (3, 48, "tanh"), (2, 64, "tanh")])
def test_small_networks_in_every_tile(pkg, orc, dim, W, act):
    """Networks of one to four row blocks: sizes on both sides of every change of the
    query's tile (16 points, the same in half the registers, full, full in one wave).
    A point's result is bitwise the same in all of them, and the oracle's."""
    H = 3
    print(f"tiles dim={dim} W={W} act={act}", flush=True)
    pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=530_001, seed=W)
    pb.activation = act
    x = np.ascontiguousarray(pb.subs[0].pde_x)
    pb.subs[0].pde_x = x[:50]
    xt = torch.from_numpy(x).cuda()
    orc.set_activation(act)
    ctx = pkg.context_from_problem(pb, device="cuda")
    try:
        ref = orc.channels(dim, W, H, pb.subs[0].theta, x[:600])
        whats = {"value": (1, 100, 4097, 17_000, 60_000, 140_000, 320_000), "residual": (16, 3001, 60_000)}
        if dim == 2:
            whats["uvpw"] = (1, 450, 13_000, 30_000, 45_001, 120_000)
        for what, sizes in whats.items():
            full = ctx.query(xt, sub=0, what=what)
            assert bool(torch.isfinite(full).all()), what
            for n in sizes:
                assert torch.equal(ctx.query(xt[:n].contiguous(), sub=0, what=what), full[:n]), (what, n)
            if what != "residual":
                assert_close(full[:600, :dim + 1].cpu().numpy(), ref[:, 0], 1e-5, what)
        ch = ctx.query(xt[:600].contiguous(), sub=0, what="channels").cpu().numpy().reshape(600, 2 * dim + 2, dim + 1)
        for c, t in enumerate(channel_tolerances(dim)):
            assert_close(ch[:, c], ref[:, c], t, f"channel {c}")
        assert torch.equal(ctx.query(xt[:60_000].contiguous(), sub=0, what="channels")[:600].cpu(),
                           torch.from_numpy(ch.reshape(600, -1)))
    finally:
        ctx.close()
        orc.set_activation("tanh")


@pytest.mark.parametrize("dim,W,H,act,ranges", [(2, 32, 4, "tanh", 8), (2, 40, 3, "sin", 4), (3, 64, 3, "tanh", 8)])
def test_gradient_of_many_slabs(pkg, orc, dim, W, H, act, ranges):
    """Several thousand gradient slabs: their sum adds no error to theirs.  A slab's own
    is that of a chain of 24 to 32 accumulations of growing partial sums (0.3 * 2^-23 of
    each, added as independent errors: 1.2e-7) and of the values it is made of
    (0.5e-7 and more); a sum of thousands in 32 bits adds 3e-7."""
    print(f"slabs dim={dim} W={W} H={H} act={act}", flush=True)
    pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=120_000, n_obs=200, n_gh=50, n_anc=1, seed=W)
    pb.activation = act
    orc.set_activation(act)
    ctx = pkg.context_from_problem(pb, device="cuda", ranges_per_wg=ranges)
    try:
        assert ctx.launch_info()["n_segments"] >= 2000
        loss, g = ctx.step(1, update=False, want_grad=True)
        Lr, gr = oracle_loss_grad(orc, pb)
        assert rel_report(loss.cpu().numpy()[0], Lr)[1] <= 2e-7
        assert rel_report(g.cpu().numpy()[0], gr)[1] <= 2e-7, rel_report(g.cpu().numpy()[0], gr)
    finally:
        ctx.close()
        orc.set_activation("tanh")


@pytest.mark.parametrize("dim,W", [(2, 65), (2, 100), (3, 128), (2, 150), (3, 240)])
def test_a_refused_32_point_tile_names_its_limit(pkg, dim, W):
    pb = wl.tiny(dim=dim, width=W, depth=2, n_pde=40, seed=W)
    with pytest.raises(pkg.PinnError, match="only 16-point tiles above 64 neurons") as e:
        pkg.context_from_problem(pb, device="cuda", tile_points=32)
    assert e.value.status == pkg.abi.PINN_E_UNSUPPORTED
    pkg.context_from_problem(wl.tiny(dim=dim, width=64, depth=2, n_pde=40, seed=W), device="cuda", tile_points=32).close()


@pytest.mark.parametrize("dim,W,act", [(2, 80, "sin"), (2, 100, "tanh"), (3, 112, "tanh"), (3, 128, "sin")])
def test_values_are_the_same_in_every_tile(pkg, dim, W, act):
    """Five to eight row blocks: small tiles, those of half the registers and full ones."""
    print(f"values dim={dim} W={W} act={act}", flush=True)
    pb = wl.tiny(dim=dim, width=W, depth=3, n_pde=60_001, seed=W)
    pb.activation = act
    x = torch.from_numpy(np.ascontiguousarray(pb.subs[0].pde_x)).cuda()
    pb.subs[0].pde_x = pb.subs[0].pde_x[:50]
    ctx = pkg.context_from_problem(pb, device="cuda")
    try:
        full = ctx.query(x, sub=0, what="value")
        for n in (100, 4096, 4097, 9000, 20_000, 32_768):
            assert torch.equal(ctx.query(x[:n].contiguous(), sub=0, what="value"), full[:n]), n
    finally:
        ctx.close()


@pytest.mark.parametrize("dim,W,H,act,npde", [(2, 16, 2, "tanh", 31), (2, 33, 3, "sin", 1000), (3, 17, 3, "tanh", 65),
                                              (3, 48, 2, "sin", 33), (2, 50, 4, "tanh", 2000), (2, 64, 3, "tanh", 40_003),
                                              (3, 64, 2, "tanh", 20_000)])
def test_32_point_tiles_against_oracle(pkg, orc, dim, W, H, act, npde):
    print(f"32-point dim={dim} W={W} H={H} act={act} n={npde}", flush=True)
    pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=npde, n_obs=5 + npde // 9, n_gh=23, n_anc=2, seed=W + H)
    pb.activation = act
    orc.set_activation(act)
    ctx = pkg.context_from_problem(pb, device="cuda", tile_points=32, guard_bytes=4096)
    try:
        assert ctx.launch_info()["tile_points"] == 32
        Lr, gr = oracle_loss_grad(orc, pb)
        for kw in ({}, {"per_subdomain": True}):
            loss, g = ctx.step(1, update=False, want_grad=True, **kw)
            assert rel_report(loss.cpu().numpy()[0], Lr)[1] <= BOUND_GRAD
            assert rel_report(g.cpu().numpy()[0], gr)[1] <= BOUND_GRAD, rel_report(g.cpu().numpy()[0], gr)
        ctx.step(1)
        torch.cuda.synchronize()
        assert ctx.check_guards() == 0
    finally:
        ctx.close()
        orc.set_activation("tanh")


@pytest.mark.parametrize("dim,W,act,npde", [(3, 96, "tanh", 5000), (2, 80, "sin", 5000), (2, 65, "tanh", 7001),
                                            (3, 144, "tanh", 5000), (2, 208, "sin", 5000), (2, 32, "tanh", 9000)])
def test_workgroups_of_four_waves_write_in_their_regions(pkg, dim, W, act, npde):
    """Two workgroups of four waves per compute unit, some with two row blocks and
    a dW block of another wave; two row blocks per wave of eight; several small
    workgroups per compute unit: no byte outside a region of the workspace."""
    print(f"guards dim={dim} W={W} act={act}", flush=True)
    pb = wl.tiny(dim=dim, width=W, depth=3, n_pde=npde, n_obs=150, n_gh=30, n_anc=2, seed=W)
    pb.activation = act
    ctx = pkg.context_from_problem(pb, device="cuda", guard_bytes=4096)
    try:
        if 64 < W <= 96:
            assert ctx.launch_info()["threads"] == 256
        ctx.step(1, update=False, want_grad=True)
        ctx.step(1)
        ctx.step(2, time_kernel=True)
        ctx.kernel_time()
        ctx.step(3, update=False, want_grad=True, per_subdomain=True)
        x = torch.from_numpy(np.ascontiguousarray(pb.subs[0].pde_x)).cuda()
        for what in ("value", "residual", "channels"):
            for n in (1, 500, npde):
                ctx.query(x[:n].contiguous(), sub=0, what=what)
        torch.cuda.synchronize()
        assert ctx.check_guards() == 0
    finally:
        ctx.close()
