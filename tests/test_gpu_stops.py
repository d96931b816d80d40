"""Solves stopped by maxiter: the flag that ends a rhs is set by the very launch
whose other workgroups and waves still read it (the beta step, alone or fused
with the p update), so what a stopped solve returns must not depend on who read
it when.  Every stopped column is bit for bit the same eager and from a graph,
alone and in a batch, run after run.

8^3x16 has 32 |r|^2 partials a rhs (summed by each wave), 16^4 has 256 (summed by
the workgroup); 1, 4, 5, 6 and 11 iterations stop in every kind of iteration
(with and without the reliable-update slot, first and later windows).
"""
import pytest
import torch

from paper_2503_16994_amd import inputs, lqcd

pytestmark = pytest.mark.gpu

PM = lqcd.PM_F64 | lqcd.PM_F32 | lqcd.PM_BF16


@pytest.mark.parametrize("inner", [lqcd.F64, lqcd.F32, lqcd.BF16], ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("L", [(8, 8, 8, 16), (16, 16, 16, 16)], ids=lambda L: "x".join(map(str, L)))
def test_solves_stopped_by_maxiter_are_reproducible(L, inner):
    print(f"\n[gpu case] maxiter stop {L} inner {inner}", flush=True)
    lat = lqcd.Lattice(L, lqcd.BC_PERIODIC, (1, 1, 1, -1))
    g = lqcd.GaugeField(lat, torch.from_numpy(inputs.gauge_field(L, 0.2, seed=5)), PM | lqcd.PM_TWO_ROW)
    gen = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn((3, *reversed(L), 4, 3), generator=gen, dtype=torch.complex128, device="cuda")
    one, many = lqcd.Workspace(lat, PM, 1), lqcd.Workspace(lat, PM, 3)
    stream = torch.cuda.Stream()
    for maxiter in (1, 4, 5, 6, 11):
        kw = dict(tol=1e-12, inner_prec=inner, maxiter=maxiter, raise_on_noconv=False)
        first = lqcd.solve(g, x, 0.13, 1.7, ws=many, **kw)
        assert first.status == lqcd.ENOCONV
        # a pending reliable update is still done, up to the end of its window of five
        assert all(maxiter <= i["iters"] < maxiter + 5 for i in first.info)
        for _ in range(3):
            again = lqcd.solve(g, x, 0.13, 1.7, ws=many, use_graph=True, stream=stream, **kw)
            torch.cuda.synchronize()
            assert torch.equal(again.psi, first.psi), maxiter
        alone = lqcd.solve(g, x[1:2], 0.13, 1.7, ws=one, **kw)
        assert alone.info[0]["iters"] == first.info[1]["iters"] and torch.equal(alone.psi[0], first.psi[1]), maxiter
