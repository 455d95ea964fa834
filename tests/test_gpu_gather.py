"""The gather kernels against the oracle at the edges of their dispatch: every
shape they take (one or two states, an odd last group, a wave with no block of
reactions), both forms and layouts, the approximate and column-ordered
outputs, temperatures low enough that the reverse rates leave the product of
exponentials for the exponential of the sum, absent species, and Arrhenius
parameters of the mechanism and of the call.  Gates as in ``oracle.gates``."""
import numpy as np
import pytest

import oracle
from oracle.gates import check_jac, check_source
from paper_1809_01029_amd import synth
from conftest import tiny_file, workload_file

pytestmark = pytest.mark.gpu


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


def states(m, n, form, seed, edge):
    st = synth.make_states(m, n, seed)
    x, p = synth.pack_state(st, form, "C")
    if edge == "cold":
        x[:, 0] = np.linspace(90.0, 260.0, n)       # H/RT - S/R of stable molecules below -165
    elif edge == "absent":
        x[:, 2:] *= np.random.default_rng(seed).random((n, m.n_species - 1)) < 0.5
    return x, p


@pytest.mark.parametrize("shape", [(0, 0), (1, 2), (1, 4), (1, 8), (2, 2), (2, 4), (2, 8), (2, 6)])
@pytest.mark.parametrize("form,layout", [("conp", "C"), ("conv", "F")])
@pytest.mark.parametrize("case", [("tiny", 1, ""), ("tiny", 5, "cold"), ("tiny", 33, "absent"), ("ns13", 3, "absent"),
                                  ("ns53", 9, ""), ("ns53", 5, "cold"), ("ns111", 3, "absent")])
def test_gather_parity(torch_cuda, api, case, form, layout, shape, mech_dir):
    torch = torch_cuda
    name, n, edge = case
    m, path = tiny_file(3, mech_dir, bath_reactions=1, bath_efficiency=True) if name == "tiny" else workload_file(name, mech_dir)
    x, p = states(m, n, form, 5, edge)
    o = oracle.Oracle(path)
    f_o, f_s = o.source(x, p, form, bound=True)
    print("case", name, n, edge, form, layout, shape, flush=True)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a if layout == "C" else a.T)).cuda()  # noqa: E731
    host = lambda a: a.cpu().numpy() if layout == "C" else a.cpu().numpy().T  # noqa: E731
    xs, ps = dev(x), torch.from_numpy(p.copy()).cuda()
    for opts in (0, api.OPT_CCS, api.OPT_APPROX_JACOBIAN):
        mech = api.load_mechanism(path, opts)
        mech.set_launch(*shape)
        approx = opts == api.OPT_APPROX_JACOBIAN
        J_o, J_s = o.jacobian(x, p, form, bound=True, approx=approx)
        check_source(host(api.eval_source(mech, xs, ps, form, layout)), f_o, f_s, "source")
        d = torch.empty_like(xs)
        j = api.eval_jacobian_sparse(mech, xs, ps, form, layout, dstate=d)
        again = api.eval_jacobian_sparse(mech, xs, ps, form, layout)
        check_source(host(d), f_o, f_s, "fused source")
        vals = j.cpu().numpy() if layout == "C" else j.cpu().numpy().T
        J = np.zeros_like(J_o)
        if opts == api.OPT_CCS:
            J[:, mech.row_idx, np.repeat(np.arange(mech.N), np.diff(mech.col_ptr))] = vals
        else:
            J[:, np.repeat(np.arange(mech.N), np.diff(mech.row_ptr)), mech.col_idx] = vals
        # (of the coldest states the oracle's own intermediates overflow)
        ok = np.isfinite(J_o).all(axis=(1, 2)) & np.isfinite(J_s).all(axis=(1, 2))
        assert ok.any()
        check_jac(J[ok], J_o[ok], J_s[ok], "sparse")
        if not opts:
            jd = api.dense_as_sij(api.eval_jacobian_dense(mech, xs, ps, form, layout), layout).cpu().numpy()
            check_jac(jd[ok], J_o[ok], J_s[ok], "dense")
            assert np.all(jd[:, ~mech.pattern_dense()] == 0.0)
        if shape[0] and m.n_reactions <= 320 * (shape[1] // shape[0]):
            # theirs: no addition depends on the order of the waves
            assert torch.equal(j, again)


@pytest.mark.parametrize("n", [1024, 1025, 2048, 2049, 4097])
@pytest.mark.parametrize("op", ["source", "sparse", "dense"])
@pytest.mark.parametrize("layout", ["C", "F"])
def test_automatic_route_agrees(torch_cuda, api, n, op, layout, mech_dir):
    """Either side of the automatic choice's lines: the same values as at four
    states on one wave (the scatter kernels).  Either
    carries some hundred roundings (1.1e-16 each, 60 times that where a Gibbs
    energy of 60 RT is exponentiated) of terms up to the state's largest value: values
    agree to 1e-12 of that."""
    torch = torch_cuda
    for name in ("tiny", "ns13", "ns53"):
        m, path = tiny_file(3, mech_dir) if name == "tiny" else workload_file(name, mech_dir)
        x, p = synth.pack_state(synth.make_states(m, n, 11), "conp", layout)
        xs, ps = torch.from_numpy(np.ascontiguousarray(x)).cuda(), torch.from_numpy(p.copy()).cuda()
        got = []
        for shape in ((0, 0), (4, 1)):
            mech = api.load_mechanism(path)
            mech.set_launch(*shape)
            f = {"source": api.eval_source, "sparse": api.eval_jacobian_sparse, "dense": api.eval_jacobian_dense}[op]
            y = f(mech, xs, ps, "conp", layout)
            y = y if op != "dense" else api.dense_as_sij(y, layout).reshape(n, -1)
            got.append(y.t() if op != "dense" and layout == "F" else y)
        a, b = got
        scale = b.abs().amax(dim=1, keepdim=True)
        print(name, n, op, layout, float(((a - b).abs() / scale).max()), flush=True)
        assert bool(((a - b).abs() <= 1e-12 * scale).all())


def test_arrhenius_of_the_mechanism_and_the_call(torch_cuda, api, mech_dir):
    torch = torch_cuda
    m, path = workload_file("ns53", mech_dir)
    x, p = synth.pack_state(synth.make_states(m, 37, 3), "conp", "C")
    xs, ps = torch.from_numpy(x).cuda(), torch.from_numpy(p).cuda()
    mech = api.load_mechanism(path)
    lnA, b, th = mech.arrhenius()
    rng = np.random.default_rng(0)
    lnA, b, th = lnA + rng.standard_normal(lnA.shape), b * 0.9, th * 1.1
    mech.set_arrhenius(lnA, b, th)
    got = []
    for shape in ((1, 4), (2, 4), (4, 1)):
        mech.set_launch(*shape)
        got.append((api.eval_source(mech, xs, ps, "conp", "C"), api.eval_jacobian_sparse(mech, xs, ps, "conp", "C")))
    for g in got[:2]:
        for a, c in zip(g, got[2]):
            assert bool(((a - c).abs() <= 1e-12 * c.abs().amax(dim=1, keepdim=True)).all())


@pytest.mark.parametrize("shape", [(1, 2), (1, 3), (1, 4), (1, 8)])
@pytest.mark.parametrize("form,layout", [("conp", "C"), ("conv", "F")])
@pytest.mark.parametrize("case", [("tiny", 1, ""), ("tiny", 5, "absent"), ("ns13", 3, ""), ("ns53", 9, ""),
                                  ("ns53", 7, "absent"), ("ns111", 5, ""), ("ns111x", 3, "")])
def test_gather_adjoint(torch_cuda, api, case, form, layout, shape, mech_dir):
    """J^T v and the parameter sums, with the mechanism's and the call's
    Arrhenius parameters, exact and approximate, with and without the sums.
    The gates of the Jacobian; where species are absent or a column is a small
    difference of large sums, the oracle's running error bound widens them."""
    torch = torch_cuda
    name, n, edge = case
    m, path = tiny_file(3, mech_dir, bath_reactions=1, bath_efficiency=True) if name == "tiny" else workload_file(name, mech_dir)
    x, p = states(m, n, form, 7, edge)
    v = np.random.default_rng(3).standard_normal(x.shape)
    o = oracle.Oracle(path)
    print("case", name, n, edge, form, layout, shape, flush=True)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a if layout == "C" else a.T)).cuda()  # noqa: E731
    host = lambda a: a.cpu().numpy() if layout == "C" else a.cpu().numpy().T  # noqa: E731
    xs, vs, ps = dev(x), dev(v), torch.from_numpy(p.copy()).cuda()
    j_o, g_o, j_s, g_s = o.adjoint(x, p, v, form, bound=True)
    mech = api.load_mechanism(path)
    mech.set_launch(*shape)
    for arr in (None, torch.as_tensor(np.stack(mech.arrhenius())).cuda()):
        j, g = api.eval_adjoint(mech, xs, ps, vs, form, layout, arrhenius=arr)
        check_jac(host(j), j_o, j_s, "J^T v")
        check_jac(g.cpu().numpy(), g_o, g_s, "parameter derivatives")
    j2, g2 = api.eval_adjoint(mech, xs, ps, vs, form, layout, with_grad=False)
    assert g2 is None and torch.equal(j, j2)
    # the approximate Jacobian's product
    mech = api.load_mechanism(path, api.OPT_APPROX_JACOBIAN)
    mech.set_launch(*shape)
    j, _ = api.eval_adjoint(mech, xs, ps, vs, form, layout)
    J, S = o.jacobian(x, p, form, bound=True, approx=True)
    jo = np.einsum("sij,si->sj", J, v)
    # bound: every entry's own, and the rounding of the sum of N products
    so = np.einsum("sij,si->sj", S, np.abs(v)) + J.shape[1] * 2.3e-16 * np.einsum("sij,si->sj", np.abs(J), np.abs(v))
    check_jac(host(j), jo, so, "approximate J^T v")


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("mode,layout", [("source", "C"), ("source", "F"), ("sparse", "C"), ("sparse", "F")])
@pytest.mark.parametrize("sizes", [(1, 0, 3), (1025, 1024, 1023), (1025, 1024, 1024)])
def test_batch_automatic_strategy(torch_cuda, api, sizes, mode, layout, graph, mech_dir):
    """A batch with no strategy set, either side of its choice's line, against
    the persistent launch: 1e-12 of a state's largest value, as above."""
    torch = torch_cuda
    b = api.Batch()
    segs = []
    for name, n in zip(("ns13", "ns53", "tiny"), sizes):
        m, path = tiny_file(3, mech_dir) if name == "tiny" else workload_file(name, mech_dir)
        x, p = synth.pack_state(synth.make_states(m, n, 2), "conp", layout)
        mech = api.load_mechanism(path)
        x, p = torch.from_numpy(np.ascontiguousarray(x)).cuda(), torch.from_numpy(p.copy()).cuda()
        out = torch.zeros((n, mech.nnz) if layout == "C" else (mech.nnz, n), dtype=torch.float64, device="cuda")
        segs.append((out, torch.zeros_like(x)))
        b.add(mech, x, p, layout, out=out, dstate=segs[-1][1])
    got = []
    for k in range(3):
        if k == 2:
            b.set_strategy(mode, False)
        b.eval(mode, "conp", layout, graph=graph)
        torch.cuda.synchronize()
        got.append([[t.clone() if layout == "C" else t.t().clone() for t in sg] for sg in segs])
    for first, again, ref in zip(*got):
        for f, a, r in zip(first, again, ref):
            if r.shape[0]:
                scale = r.abs().amax(dim=1, keepdim=True)
                assert bool(((f - r).abs() <= 1e-12 * scale).all()) and bool(((a - r).abs() <= 1e-12 * scale).all())
