"""The contractions hold fp32 precision: gradients and outputs
against the FP64 oracle within bounds between what the kernels' arithmetic gives
(1 to 2e-7 of the norm: fp32 accumulations and activations) and what is left without any one of
the six products, or one part, of the bf16 triples (test_split_scheme.py: more than 5e-7 of a
gradient, 1e-6 of the outputs), for every way in which waves share the row blocks."""
import numpy as np
import pytest

import workloads as wl
from parity import oracle_loss_grad, rel_report
from test_split_scheme import BOUND_GRAD, BOUND_VALUE

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# dim, width, depth, activation, points: one and two row blocks, an even and an odd number,
# four waves with two workgroups per compute unit, two row blocks per wave
CASES = [(2, 16, 3, "tanh", 3000), (2, 32, 2, "tanh", 3000), (3, 48, 3, "sin", 2000), (2, 64, 3, "tanh", 6000),
         (3, 96, 3, "tanh", 5000), (2, 80, 3, "sin", 5000), (2, 112, 3, "tanh", 2000), (3, 128, 3, "tanh", 2000),
         (2, 150, 3, "sin", 2000), (3, 208, 2, "tanh", 1000), (2, 256, 2, "tanh", 1000), (3, 240, 2, "tanh", 1000)]


@pytest.mark.parametrize("dim,W,H,act,npde", CASES)
def test_fp32_precision_of_steps_and_queries(orc, dim, W, H, act, npde):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_15883_amd as P
    print(f"precision dim={dim} W={W} H={H} act={act}", flush=True)
    pb = wl.tiny(dim=dim, width=W, depth=H, n_pde=npde, n_obs=npde // 4, n_gh=40, n_anc=2, seed=5 * W + H)
    pb.activation = act
    orc.set_activation(act)
    ctx = P.context_from_problem(pb, device="cuda")
    try:
        x = np.ascontiguousarray(pb.subs[0].pde_x)
        xt = torch.from_numpy(x).cuda()
        # twice: the second pass is on the copies that the update wrote
        for t in (1, 2):
            theta = ctx.subs[0].theta.cpu().numpy().copy()
            Lr, gr = oracle_loss_grad(orc, pb, theta=theta)
            ref = orc.channels(dim, W, H, theta, x)
            off = {"value": rel_report(ctx.query(xt, sub=0, what="value").cpu().numpy(), ref[:, 0])[1],
                   "small": rel_report(ctx.query(xt[:300].contiguous(), sub=0, what="value").cpu().numpy(), ref[:300, 0])[1]}
            ch = ctx.query(xt, sub=0, what="channels").cpu().numpy().reshape(npde, 2 * dim + 2, dim + 1)
            off["channel 0"] = rel_report(ch[:, 0], ref[:, 0])[1]
            loss, g = ctx.step(t, want_grad=True)
            off_grad = rel_report(g.cpu().numpy()[0], gr)[1]
            print(t, f"grad {off_grad:.2e}", " ".join(f"{k} {v:.2e}" for k, v in off.items()), flush=True)
            assert off_grad <= BOUND_GRAD
            assert rel_report(loss.cpu().numpy()[0], Lr)[1] <= BOUND_GRAD
            assert max(off.values()) <= BOUND_VALUE, off
    finally:
        ctx.close()
        orc.set_activation("tanh")
