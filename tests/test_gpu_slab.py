"""GPU parity of the operator kernels at the edges of their tiles and chunks: degrees 3, 5 and 6 and
the Gauss-Legendre nodes on meshes of partial tiles, one element layer to several chunks, against the
FP64 oracle at the bars of the operator (1e-12 in FP64, 2e-5 in FP32) and the V-cycle (1e-9); and the
independence of a right-hand side's result from the batch, which sets the chunk length, bit for bit.
"""
import numpy as np
import pytest

from oracle import layout, mg
from workloads import configs

from _cases import gpu_sample

pytestmark = pytest.mark.gpu

# E, p, node family: partial tiles on both axes, one layer, several chunks, the 4x4 tile of degree 3
# (from 1000 elements), the bricks of degree 7
CASES = [((5, 3, 1), 3, "gll"), ((10, 10, 14), 3, "gll"), ((8, 5, 5), 5, "gll"), ((1, 3, 2), 5, "gll"),
         ((3, 3, 5), 6, "gll"), ((7, 8, 6), 3, "gl"), ((3, 2, 5), 5, "gl"), ((5, 1, 4), 4, "gl"), ((2, 3, 4), 7, "gl")]


def _t(a, dtype=np.float64):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a, dtype=dtype)).cuda()


@pytest.mark.parametrize("E,p,family", CASES, ids=["E%dx%dx%d-p%d-%s" % (*c[0], c[1], c[2]) for c in CASES])
def test_operator_and_vcycle_match_oracle(gpu_lib, E, p, family):
    lo, hi = (-1.0, 0.0, -2.0), (1.5, 2.0, 1.0)
    ctx = gpu_lib.Context([(E, p, lo, hi)], node_family=family)
    H = mg.Hierarchy(E, p, lo, hi, family=family)
    rng = np.random.default_rng(5)
    for level, L in enumerate(H.levels):
        u = rng.standard_normal((2,) + L.shape)
        uem = np.stack([layout.to_element_major(u[r], L.E, L.n) for r in range(2)])
        ref = np.stack([layout.to_element_major(L.A(u[r]), L.E, L.n) for r in range(2)])
        for dtype, bar in ((np.float64, 1e-12), (np.float32, 2e-5)):
            y = ctx.operator_apply(_t(uem, dtype), level=level).cpu().numpy().reshape(2, -1)
            assert np.abs(y - ref).max() <= bar * np.abs(ref).max(), (level, dtype)
    L0 = H.levels[0]
    r = rng.standard_normal(L0.shape)
    z = ctx.vcycle(_t(layout.to_element_major(r, L0.E, L0.n))).cpu().numpy()
    ref = layout.to_element_major(H.vcycle(r), L0.E, L0.n)
    assert np.abs(z - ref).max() <= 1e-9 * np.abs(ref).max()
    ctx.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32_pc", "bf16f_pc"])
def test_chunk_length_does_not_change_a_solution(gpu_lib, precision):
    """One right-hand side of an 8^3 mesh runs in chunks of one layer, 48 of them in chunks of four."""
    wl = configs.scaled(8, 4, 3, seed=17)
    m = wl.meshes[0]
    ctx = gpu_lib.Context([(m.E, m.p, m.lo, m.hi)], precision=precision, lanes=1)
    rho, g = zip(*[gpu_sample(ctx, 0, d) for d in wl.batch.densities])
    rho, g = np.concatenate(rho).reshape(3, -1), np.concatenate(g).reshape(3, -1)
    big, sb = ctx.solve_batch(_t(np.tile(rho, (16, 1))), _t(np.tile(g, (16, 1))))
    big = big.cpu().numpy().reshape(48, -1)
    for k in range(3):
        one, so = ctx.solve_batch(_t(rho[k]), _t(g[k]))
        assert so[0]["iters"] == sb[k]["iters"] == sb[45 + k]["iters"]
        assert np.array_equal(one.cpu().numpy().reshape(-1), big[k]) and np.array_equal(big[k], big[45 + k])
    ctx.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32_pc"])
@pytest.mark.parametrize("E,p,family", [(8, 3, "gll"), (10, 3, "gll"), (8, 5, "gll"), (7, 6, "gll"), (8, 2, "gl"), (8, 3, "gl"),
                                        (8, 4, "gl"), (6, 5, "gl"), (6, 6, "gl"), (5, 7, "gll")])
def test_chunk_length_does_not_change_a_solution_of_other_degrees(gpu_lib, E, p, family, precision):
    """The kernels of the other degrees and of Gauss-Legendre nodes (10^3: the 4x4 tile of degree 3;
    degree 7: the bricks)."""
    wl = configs.scaled(E, p, 2, seed=17)
    m = wl.meshes[0]
    ctx = gpu_lib.Context([(m.E, m.p, m.lo, m.hi)], precision=precision, lanes=1, node_family=family)
    rho, g = zip(*[gpu_sample(ctx, 0, d) for d in wl.batch.densities])
    rho, g = np.concatenate(rho).reshape(2, -1), np.concatenate(g).reshape(2, -1)
    big, sb = ctx.solve_batch(_t(np.tile(rho, (20, 1))), _t(np.tile(g, (20, 1))))
    big = big.cpu().numpy().reshape(40, -1)
    for k in range(2):
        one, so = ctx.solve_batch(_t(rho[k]), _t(g[k]))
        assert so[0]["iters"] == sb[k]["iters"] == sb[38 + k]["iters"]
        assert np.array_equal(one.cpu().numpy().reshape(-1), big[k]) and np.array_equal(big[k], big[38 + k])
    ctx.close()


def test_alternating_calls_of_one_and_several_meshes_keep_their_graphs(gpu_lib):
    """Calls of one mesh and of three, in turn, with one right-hand side a mesh: the chunk target, and
    with it the captured iterations, changes from call to call.  A call after one of the other kind takes no
    longer than after one of its own (solves of two iterations, where a capture takes nearly as long), and
    solves bit for bit alike."""
    import time

    import torch
    wl = configs.scaled(4, 3, 1, seed=17)
    m = wl.meshes[0]
    ctx = gpu_lib.Context([(m.E, m.p, m.lo, m.hi)] * 3, lanes=1, rtol=0.3)
    rho, g = gpu_sample(ctx, 0, wl.batch.densities[0])
    one = (_t(rho), _t(g), [0])
    three = (_t(np.tile(rho, 3)), _t(np.tile(g, 3)), [0, 1, 2])

    def run(args):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        v, st = ctx.solve_batch(args[0], args[1], mesh_ids=args[2])
        torch.cuda.synchronize()
        return time.perf_counter() - t0, v

    for args in (one, three, one, three):
        run(args)
    alone, turn = [], []
    for _ in range(40):
        turn.append(run(one))
        alone.append(run(one))
        run(three)
    assert all(torch.equal(v, alone[0][1]) for _, v in alone + turn)
    a, t = (float(np.median([x for x, _ in r])) for r in (alone, turn))
    print("after its own kind %.3f ms, after the other %.3f ms" % (1e3 * a, 1e3 * t))
    assert t <= 1.4 * a
    ctx.close()
