"""Edges of the launch shapes and of the workspace: many subdomains of a small
network, the smallest and the largest networks of a query kernel, the 32-point tile."""
import numpy as np
import pytest

import workloads as wl
from parity import rel_report

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
