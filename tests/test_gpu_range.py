"""Rates near the ends of the exponent range: what the gather and wide kernels
take as a product of exponentials of single species must hold wherever the
rates themselves are finite, against the oracle under ``oracle.gates``."""
import numpy as np
import pytest

import oracle
from oracle.gates import check_jac, check_source
from paper_1809_01029_amd import synth

pytestmark = pytest.mark.gpu

R, W_N2 = 8314.462618, 28.014


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def api(torch_cuda):
    from paper_1809_01029_amd import api as a
    return a


def isomers(g1000, reactions, directory, name):
    """Species of one composition with H/RT - S/R = g1000[k] at 1000 K (cp = 3.5
    R, no temperature dependence), the bath gas last."""
    ns = len(g1000)
    a = np.zeros((ns, 7))
    a[:, 0] = 3.5
    a[:, 5] = 1000.0 * (np.asarray(g1000) - 3.5 + 3.5 * np.log(1000.0))
    comp = np.tile([0, 0, 0, 2], (ns, 1))
    m = synth.Mechanism(names=[f"S{k}" for k in range(ns - 1)] + ["BATH"], W=np.full(ns, W_N2), comp=comp,
                        tmid=np.full(ns, 1000.0), a_lo=a, a_hi=a.copy(), reactions=reactions)
    return m, synth.write_mechanism(m, str(directory / (name + ".pjm")))


def isomer_states(ns, n, T, seed=0):
    rng = np.random.default_rng(seed)
    P = 1.0e5 * (1.0 + rng.random(n))
    y = rng.random((n, ns))
    moles = (P / (R * T))[:, None] * y / y.sum(1, keepdims=True)
    return np.concatenate([np.asarray(T)[:, None], np.ones((n, 1)), moles[:, :-1]], axis=1), P


@pytest.mark.parametrize("shape", [(64, 2), (64, 4), (1, 2), (2, 2), (4, 1)])
def test_irreversible_reaction_beside_an_overflowing_equilibrium(torch_cuda, api, tmp_path, shape):
    """k_f = e^400 is finite and so is its rate; the equilibrium constant it would
    have if it were reversible, e^400, times k_f is not."""
    torch = torch_cuda
    rx = [synth.Reaction("ELEM", False, [(0, 1), (1, 1)], [(2, 1), (3, 1)], 400.0, 0.0, 0.0),
          synth.Reaction("ELEM", True, [(2, 1)], [(3, 1)], 10.0, 0.0, 100.0)]
    m, path = isomers([-150.0, -150.0, 50.0, 50.0, -20.0], rx, tmp_path, "irr")
    n = 70
    x, p = isomer_states(5, n, np.linspace(990.0, 1010.0, n))
    o = oracle.Oracle(path)
    f_o, f_b = o.source(x, p, "conp", bound=True)
    J_o, J_b = o.jacobian(x, p, "conp", bound=True)
    assert np.isfinite(f_o).all() and np.isfinite(J_o).all() and np.abs(f_o).max() > 1e160
    xs, ps = torch.from_numpy(x).cuda(), torch.from_numpy(p).cuda()
    mech = api.load_mechanism(path)
    mech.set_launch(*shape)
    check_source(api.eval_source(mech, xs, ps, "conp", "C").cpu().numpy(), f_o, f_b, f"source terms {shape}")
    J = api.sparse_to_dense(mech, api.eval_jacobian_sparse(mech, xs, ps, "conp", "C").cpu().numpy(), "C")
    check_jac(J, J_o, J_b, f"sparse Jacobian {shape}")


SHAPES = [(64, 2), (64, 8), (1, 2), (1, 4), (2, 2), (2, 4), (4, 1)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("form", ["conp", "conv"])
@pytest.mark.parametrize("low,high", [
    # three molecules a side whose exponentials together underflow (e^-1005) or
    # overflow (e^+990), none alone; the reactions are near equilibrium
    (-340.0, 334.0),
    # two together, or one alone, out of range
    (-420.0, 380.0), (-760.0, 740.0),
    # beside the bounds of the product: three are e^-645 and e^+630, e^-210 ...
    (-217.0, 214.0), (-70.0, 60.0),
])
def test_equilibria_at_the_ends_of_the_range(torch_cuda, api, tmp_path, low, high, form, shape):
    torch = torch_cuda
    E = lambda a, b, lnA, b_, th, **kw: synth.Reaction(kw.pop("type", "ELEM"), True, a, b, lnA, b_, th, **kw)  # noqa: E731
    rx = [E([(0, 2), (1, 1)], [(2, 2), (3, 1)], 3.0, 0.0, 1500.0), E([(4, 1), (5, 2)], [(6, 1), (7, 2)], 4.0, 0.3, 2000.0),
          E([(0, 1), (4, 1)], [(2, 1), (6, 1)], 8.0, 0.0, 500.0),
          E([(1, 1)], [(3, 1)], 6.0, 0.0, 500.0, type="THREEBODY", eff=[(2, 3.0), (8, 0.5)]),
          E([(5, 1)], [(7, 1)], 9.0, 0.0, 700.0, type="LINDEMANN", low=(12.0, 0.0, 300.0)),
          # k_f itself below the range, e^-900; far from equilibrium, but no rate of note
          E([(4, 1)], [(6, 1)], 5.0, 0.0, 905.0e3)]
    m, path = isomers([low, low + 3, low + 5, low + 4, high, high - 4, high - 6, high - 5, -20.0], rx, tmp_path, "ends")
    n = 70
    T = np.linspace(985.0, 1015.0, n)
    x, p = isomer_states(9, n, T)
    if form == "conv":
        x[:, 1], p = p.copy(), np.ones(n)
    o = oracle.Oracle(path)
    f_o, f_b = o.source(x, p, form, bound=True)
    J_o, J_b = o.jacobian(x, p, form, bound=True)
    assert np.isfinite(f_o).all() and np.isfinite(J_o).all()
    xs, ps = torch.from_numpy(x).cuda(), torch.from_numpy(p).cuda()
    mech = api.load_mechanism(path)
    mech.set_launch(*shape)
    check_source(api.eval_source(mech, xs, ps, form, "C").cpu().numpy(), f_o, f_b, f"source terms {shape}")
    J = api.sparse_to_dense(mech, api.eval_jacobian_sparse(mech, xs, ps, form, "C").cpu().numpy(), "C")
    check_jac(J, J_o, J_b, f"sparse Jacobian {shape}")
    if shape[0] <= 4:
        v = np.random.default_rng(1).standard_normal(x.shape)
        j_o, _, j_b, _ = o.adjoint(x, p, v, form, bound=True)
        j, _ = api.eval_adjoint(mech, xs, ps, torch.from_numpy(v).cuda(), form, "C")
        check_jac(j.cpu().numpy(), j_o, j_b, f"J^T v {shape}")


@pytest.mark.parametrize("shape", [(0, 0)] + SHAPES)
@pytest.mark.parametrize("name,n", [("ns13", 131), ("ns53", 131), ("ns111x", 131)])
@pytest.mark.parametrize("odd", ["cold", "absent", "nan"])
def test_results_do_not_depend_on_the_neighbours(torch_cuda, api, name, n, odd, shape, mech_dir):
    """Every third state replaced by one that takes other paths (60 K, where every
    equilibrium is out of range; half the species absent; no number): the others
    keep their bits."""
    from conftest import workload_file
    torch = torch_cuda
    m, path = workload_file(name, mech_dir)
    x, p = synth.pack_state(synth.make_states(m, n, 3), "conp", "C")
    y = x.copy()
    rows = np.arange(1, n, 3)
    if odd == "cold":
        y[rows, 0] = 60.0
    elif odd == "absent":
        y[rows, 2:] *= np.random.default_rng(1).random((len(rows), m.n_species - 1)) < 0.5
    else:
        y[rows, 0] = np.nan
    keep = torch.from_numpy(np.setdiff1d(np.arange(n), rows)).cuda()
    mech = api.load_mechanism(path)
    mech.set_launch(*shape)
    if shape[0] == 4:
        assert mech.kernel("sparse", "C", n)[0] == "scatter"
    ps, v = torch.from_numpy(p).cuda(), torch.from_numpy(np.random.default_rng(2).standard_normal(x.shape)).cuda()
    got = []
    for z in (x, y):
        zs = torch.from_numpy(z).cuda()
        got.append([api.eval_source(mech, zs, ps, "conp", "C")[keep], api.eval_jacobian_sparse(mech, zs, ps, "conp", "C")[keep],
                    api.eval_adjoint(mech, zs, ps, v, "conp", "C", with_grad=False)[0][keep]])
    one_wave = shape[1] == 1
    for what, a, b in zip(("source", "sparse", "adjoint"), *got):
        # (several waves of the scatter kernels add in any order)
        if one_wave or mech.kernel(what, "C", n)[0] != "scatter":
            assert torch.equal(a, b), what


@pytest.mark.parametrize("shapes", [((1, 4), (2, 4), (64, 4))])
@pytest.mark.parametrize("name,n", [("ns53", 600), ("ns111", 200)])
@pytest.mark.parametrize("T_range", [(600.0, 2200.0), (300.0, 700.0)])
def test_rounding_is_no_larger_than_the_scatter_kernels(torch_cuda, api, name, n, T_range, shapes, mech_dir):
    """Errors against the oracle in long double, over the running error bound of
    each value: their root mean square and 99th percentile against the scatter
    kernels' of the same states.  Both are sums over tens of thousands of
    values, to 3 % of each other (a further rounding of ln k_f: 6 % and 11 %)."""
    from conftest import workload_file
    torch = torch_cuda
    m, path = workload_file(name, mech_dir)
    x, p = synth.pack_state(synth.make_states(m, n, 17, T_range=T_range), "conp", "C")
    o = oracle.Oracle(path)
    k = n // 8
    f_l, (_, f_b) = o.source_ld(x, p), o.source(x, p, "conp", bound=True)
    J_l, (_, J_b) = o.jacobian_ld(x[:k], p[:k]), o.jacobian(x[:k], p[:k], "conp", bound=True)
    xs, ps = torch.from_numpy(x).cuda(), torch.from_numpy(p).cuda()
    mech = api.load_mechanism(path)
    on = mech.pattern_dense()
    on[:2] = False

    def errors(shape):
        mech.set_launch(*shape)
        f = api.eval_source(mech, xs, ps, "conp", "C").cpu().numpy()
        J = api.sparse_to_dense(mech, api.eval_jacobian_sparse(mech, xs[:k], ps[:k], "conp", "C").cpu().numpy(), "C")
        got = []
        for a, l, b in ((f, f_l, f_b), (J[:, on], J_l[:, on], J_b[:, on])):
            r = (np.abs(a - l) / np.maximum(b, 1e-300))[b > 0]
            got += [np.sqrt((r * r).mean()), np.quantile(r, 0.99)]
        return np.array(got)
    ref = errors((4, 1))
    for shape in shapes:
        e = errors(shape)
        print(name, T_range, shape, e / ref, flush=True)
        assert (e <= 1.03 * ref).all(), (shape, e / ref)
