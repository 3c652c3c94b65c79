"""GPU: the two-kernel tick -- kernels and dispatch branches at the sizes
where they can go wrong, against the oracle."""

import numpy as np
import pytest

import oracle
import spff_inputs as si
from gpu_common import device, cfg_for, planes_to_tensor, tensor_to_planes, rel_l2
from oracle import spectral as osp
from paper_2203_16467_amd import spff

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,B", [(128, 128, 1), (256, 2048, 1), (512, 64, 3), (1024, 256, 3), (2048, 128, 1),
                                     (64, 1024, 5)])
def test_fp64_register_kernels_match_oracle_and_lds_kernels(nx, ny, B):
    """FP64 problems take the register kernels where the grid has them
    (rows of 128..1024, columns of 128..2048 points); a plan of the LDS kind
    asks for the LDS kernels.  Both give the operators to FP64 rounding."""
    import torch
    print(f"fp64 {B} x {nx}x{ny}", flush=True)
    cfg = cfg_for(nx, ny, "fp64")
    E = torch.ones((B, ny, nx), dtype=torch.float64, device=device())
    p = spff.Problem(E, cfg)
    x = np.random.default_rng(nx + ny).standard_normal((B, 3, ny, nx))
    xt = torch.from_numpy(x).to(device())
    got = [p.apply_operator(op, xt if op != spff.OP_NEG_LAPLACIAN else xt[:, 0]).cpu().numpy()
           for op in (spff.OP_PROJECT, spff.OP_NEG_LAPLACIAN, spff.OP_DISPLACEMENT)]
    for b in range(B):
        assert rel_l2(got[0][b], tensor_to_planes(osp.project(planes_to_tensor(x[b])))) < 1e-12
        assert rel_l2(got[1][b], -osp.laplacian(x[b, 0])) < 1e-12
    last = len(p.plan_buckets()) - 1
    plan = p.get_plan(last)
    assert plan["row_kind"] == spff.FFT_LDS and plan["col_kind"] == spff.FFT_LDS
    p.set_plan(last, plan)
    for op, g in zip((spff.OP_PROJECT, spff.OP_NEG_LAPLACIAN, spff.OP_DISPLACEMENT), got):
        again = p.apply_operator(op, xt if op != spff.OP_NEG_LAPLACIAN else xt[:, 0]).cpu().numpy()
        assert rel_l2(again, g) < 1e-12
    p.close()


@pytest.mark.parametrize("K,graph", [(1, 0), (2, 0), (3, 1), (32, 0), (32, 1)])
def test_blocks_in_flight_give_the_problems_alone(K, graph):
    """Blocks of ticks are enqueued ahead of the host's checks; problems of a
    batch finish at different times, so that the bucket (launch size) shrinks
    while blocks are in flight.  With the plan fixed, every problem's steps
    are bit for bit those of the problem alone, at any block length."""
    import torch
    n, B = 64, 5
    E = np.stack([si.young_modulus(n, 3.0, 0.05 + 0.06 * b, 90 + b) for b in range(B)])
    ramp = si.uniaxial_ramp(12, 0.2, 2.0)[4:7]
    kw = dict(at=2, plan_rows=2, plan_cols=2)
    p = spff.Problem(torch.from_numpy(E).to(device()), cfg_for(n, use_graph=graph, ticks_per_sync=K, **kw))
    _, stats = p.run_sequence(ramp)
    f = p.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
    ticks = [sum(s["ticks"] for s in row) for row in stats]
    assert len(set(ticks)) > 1  # they do not finish together
    for b in range(B):
        q = spff.Problem(torch.from_numpy(E[b]).to(device()), cfg_for(n, **kw))
        alone = [q.load_step(e)[1][0] for e in ramp]
        g = q.get_fields(spff.FIELD_PHI | spff.FIELD_EPS_STAR)
        for k in f:
            assert torch.equal(f[k][b], g[k][0]), (b, k)
        for s, a in zip(stats[b], alone):
            assert all(s[k] == a[k] for k in ("cg_iters", "bccg_iters", "am_iters", "ticks", "F_e", "F_f"))
        q.close()
    p.close()
