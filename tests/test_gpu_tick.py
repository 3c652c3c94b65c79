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
