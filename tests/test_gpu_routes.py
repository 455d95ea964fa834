"""Which kernels a call runs, on both sides of every line of the automatic
choice, and the results of both: the route is asserted, so that a case cannot
slip to the other side of its line, and sampled states (the first, the last and
some between) are compared with the oracle under ``oracle.gates``."""
import os

import numpy as np
import pytest

import oracle
from oracle.gates import check_jac, check_source
from paper_1809_01029_amd import synth
from conftest import workload_file

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


def sample(n, k=6):
    return np.unique(np.concatenate([[0, n - 1], np.linspace(0, n - 1, k).astype(int)]))


class Segment:
    def __init__(self, torch, api, mech_dir, name, n, mode, layout, seed, dstate=False, grad=None):
        self.m, self.path = workload_file(name, mech_dir)
        self.x, self.p = synth.pack_state(synth.make_states(self.m, n, seed), "conp", "C")
        self.layout, self.n = layout, n
        self.mech = api.load_mechanism(self.path)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a if layout == "C" else a.T)).cuda()  # noqa: E731
        self.xs, self.ps = dev(self.x), torch.from_numpy(self.p.copy()).cuda()
        self.kw = {}
        if mode == "sparse":
            self.kw["out"] = torch.zeros((n, self.mech.nnz) if layout == "C" else (self.mech.nnz, n), dtype=torch.float64,
                                         device="cuda")
        if mode == "adjoint":
            self.v = np.random.default_rng(seed).standard_normal(self.x.shape)
            self.kw.update(out=torch.zeros_like(self.xs), v=dev(self.v),
                           grad=torch.full((3, self.m.n_reactions), 7.0, dtype=torch.float64, device="cuda")
                           if grad is None else grad)
        if mode != "adjoint" or dstate:
            self.kw["dstate"] = torch.zeros_like(self.xs)

    def states_of(self, t, idx):
        return (t[idx] if self.layout == "C" else t[:, idx].t()).cpu().numpy()

    def check(self, torch, api, mode, what):
        if not self.n:
            return
        idx = sample(self.n)
        ti = torch.from_numpy(idx).cuda()
        o = oracle.Oracle(self.path)
        x, p = self.x[idx], self.p[idx]
        if "dstate" in self.kw:
            f_o, f_b = o.source(x, p, "conp", bound=True)
            check_source(self.states_of(self.kw["dstate"], ti), f_o, f_b, what + " source terms")
        if mode == "sparse":
            J_o, J_b = o.jacobian(x, p, "conp", bound=True)
            check_jac(api.sparse_to_dense(self.mech, self.states_of(self.kw["out"], ti), "C"), J_o, J_b, what + " Jacobian")
        if mode == "adjoint":
            j_o, _, j_b, _ = o.adjoint(x, p, self.v[idx], "conp", bound=True)
            check_jac(self.states_of(self.kw["out"], ti), j_o, j_b, what + " J^T v")


# (13, 53 and 111 species: 1, 6 and 13 blocks of 64 reactions; four a segment
# or more on average let the automatic choice launch per segment)
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("mode,layout,sizes,fused,want", [
    ("source", "C", (1, 0, 3), False, "per_segment"),
    ("source", "F", (1025, 9000, 130), False, "per_segment"),
    ("sparse", "C", (700, 3000, 500), False, "per_segment"),
    ("sparse", "F", (1000, 1572, 500), False, "per_segment"),
    ("sparse", "F", (1000, 1573, 500), False, "persistent"),
    ("sparse", "F", (30000, 2067, 700), False, "persistent"),
    ("sparse", "F", (30000, 2068, 700), False, "per_segment"),
    ("adjoint", "C", (30000, 2000, 767), False, "persistent"),
    ("adjoint", "C", (30000, 2000, 768), False, "per_segment"),
    ("adjoint", "F", (0, 30001, 3001), False, "per_segment"),
    ("adjoint", "C", (1, 2, 3), True, "persistent"),
    # (with source terms every segment's kernels are the persistent launch's)
    ("adjoint", "C", (3000, 30000, 2000), True, "persistent"),
    ("adjoint", "F", (3000, 30000, 2000), True, "persistent"),
])
def test_batch_automatic_route(torch_cuda, api, mode, layout, sizes, fused, want, graph, mech_dir):
    torch = torch_cuda
    b = api.Batch()
    segs = [Segment(torch, api, mech_dir, name, n, mode, layout, 2 + k, dstate=fused)
            for k, (name, n) in enumerate(zip(("ns13", "ns53", "ns111"), sizes))]
    for sg in segs:
        b.add(sg.mech, sg.xs, sg.ps, layout, **sg.kw)
    assert b.route(mode, layout) == want and not b.strategy(mode)
    for again in range(2):
        b.eval(mode, "conp", layout, graph=graph)
        torch.cuda.synchronize()
        for k, sg in enumerate(segs):
            sg.check(torch, api, mode, f"{mode} {layout} {sizes} graph={graph} run {again} segment {k}")
    if mode == "adjoint":
        # the parameter sums of the persistent launch: sums of n terms in another order
        sums = [sg.kw["grad"].clone() for sg in segs]
        b.set_strategy(mode, False)
        assert b.route(mode, layout) == "persistent"
        b.eval(mode, "conp", layout)
        torch.cuda.synchronize()
        for g, sg in zip(sums, segs):
            scale = sg.kw["grad"].abs().amax(dim=1, keepdim=True)
            assert bool(((g - sg.kw["grad"]).abs() <= 1e-11 * scale).all())


def test_batch_segments_that_share_their_parameter_sums(torch_cuda, api, mech_dir):
    """Two segments with one buffer: the sums of both, which a launch of its own
    would clear."""
    torch = torch_cuda
    one = Segment(torch, api, mech_dir, "ns111", 20000, "adjoint", "C", 5)
    two = Segment(torch, api, mech_dir, "ns111", 20000, "adjoint", "C", 6, grad=one.kw["grad"])
    b = api.Batch()
    for sg in (one, two):
        b.add(sg.mech, sg.xs, sg.ps, "C", **sg.kw)
    assert b.route("adjoint", "C") == "persistent"
    b.eval("adjoint", "conp", "C")
    want = sum(api.eval_adjoint(sg.mech, sg.xs, sg.ps, sg.kw["v"], "conp", "C")[1] for sg in (one, two))
    torch.cuda.synchronize()
    scale = want.abs().amax(dim=1, keepdim=True)
    assert bool(((one.kw["grad"] - want).abs() <= 1e-11 * scale).all())
    for sg in (one, two):
        sg.check(torch, api, "adjoint", "shared sums")


@pytest.mark.parametrize("layout", ["C", "F"])
@pytest.mark.parametrize("name,n", [("ns13", 8193), ("ns13", 40000), ("ns53", 8193), ("ns53", 16385), ("ns53", 40001)])
def test_automatic_source_terms_are_reproducible(torch_cuda, api, name, n, layout, mech_dir):
    """The automatic choice for source terms adds in a fixed order: ten runs give
    the same bits, and so do two at every set shape of the wide kernel."""
    torch = torch_cuda
    sg = Segment(torch, api, mech_dir, name, n, "source", layout, 9)
    first = api.eval_source(sg.mech, sg.xs, sg.ps, "conp", layout)
    for _ in range(9):
        assert torch.equal(api.eval_source(sg.mech, sg.xs, sg.ps, "conp", layout), first)
    sg.kw["dstate"] = first
    sg.check(torch, api, "source", f"{name} {n} {layout}")
    for w in (2, 3, 4, 8):
        sg.mech.set_launch(64, w)
        if sg.mech.kernel("source", layout, n)[0] == "wide":
            a, b = (api.eval_source(sg.mech, sg.xs, sg.ps, "conp", layout) for _ in range(2))
            assert torch.equal(a, b)


def described(name, mech_dir):
    """(mechanism, path): a workload, or genN, N species with 6.5 N reactions."""
    if not name.startswith("gen"):
        return workload_file(name, mech_dir)
    ns = int(name[3:])
    m = synth.make_mechanism(ns, 13 * ns // 2, ns)
    return m, synth.write_mechanism(m, os.path.join(str(mech_dir), name + ".pjm"))


@pytest.mark.parametrize("name,shape,mode,layout,n,want", [
    # set shapes (states, waves): reactions a wave takes, 360 species = 34 blocks of 64
    ("ns360", (2, 2), "source", "C", 6410, ("scatter", 2, 2)),
    ("ns360", (1, 3), "source", "C", 6410, ("gather", 1, 3)),
    ("ns360", (1, 2), "adjoint", "C", 6410, ("scatter", 1, 2)),
    ("ns360", (1, 4), "adjoint", "C", 6410, ("gather", 1, 4)),

    # source terms: few states; more than two wide workgroups a compute unit; the
    # last round of 256 x 64 states at least 80 % full; scatter grids of a multiple of 8
    ("gen20", None, "source", "C", 4096, ("gather", 2, 2)),
    ("gen20", None, "source", "C", 4097, ("scatter", 4, 1)),
    ("ns53", None, "source", "C", 13000, ("gather", 2, 2)),
    ("ns53", None, "source", "C", 13001, ("wide", 64, 8)),
    ("ns53", None, "source", "C", 16384, ("wide", 64, 8)),
    ("ns53", None, "source", "C", 16385, ("gather", 2, 2)),
    ("ns53", None, "source", "F", 26214, ("gather", 2, 2)),
    ("ns53", None, "source", "F", 26215, ("wide", 64, 4)),
    ("ns53", None, "source", "C", 49153, ("wide", 64, 4)),
    ("gen32", None, "source", "C", 12000, ("scatter", 4, 1)),
    ("gen32", None, "source", "C", 12001, ("wide", 64, 8)),
    ("ns111", None, "source", "C", 20000, ("gather", 2, 4)),

    # adjoints: few states; from where the workgroups' additions weigh less
    ("ns13", None, "adjoint", "C", 128, ("gather", 1, 4)),
    ("ns13", None, "adjoint", "C", 129, ("scatter", 4, 1)),
    ("ns53", None, "adjoint", "C", 256, ("gather", 1, 4)),
    ("ns53", None, "adjoint", "F", 3072, ("gather", 1, 4)),
    ("ns53", None, "adjoint", "F", 16383, ("gather", 1, 4)),
    ("ns53", None, "adjoint", "F", 16384, ("gather", 1, 2)),
    ("ns360", None, "adjoint", "C", 383, ("scatter", 2, 8)),
    ("ns360", None, "adjoint", "C", 384, ("gather", 1, 8)),

    # Jacobians: waves by reactions; rows a multiple of 4 kB apart
    ("gen60", None, "dense", "C", 3000, ("gather", 1, 4)),
    ("ns53", None, "sparse", "F", 16383, ("gather", 2, 4)),
    ("ns53", None, "sparse", "F", 16384, ("scatter", 8, 8)),
    ("gen60", None, "sparse", "F", 3001, ("gather", 2, 8)),
    ("ns111", None, "dense", "F", 8192, ("scatter", 4, 8)),
    ("ns111", None, "dense", "F", 8193, ("gather", 2, 8)),

    # layout F: 8 states only in launches that fill the chip, and not where 4 run
    # on one wave (whose additions have a fixed order) and 8 don't
    ("ns13", None, "sparse", "F", 16383, ("scatter", 4, 1)),
    ("ns13", None, "sparse", "F", 16384, ("scatter", 8, 1)),
    ("gen20", None, "sparse", "F", 40000, ("scatter", 4, 1)),
    ("gen20", None, "dense", "F", 40000, ("scatter", 4, 1)),

    # one state a workgroup, dense: 7 waves where the rows meet in the same channels
    ("ns360", None, "dense", "F", 1024, ("scatter", 1, 7)),
    ("ns360", None, "dense", "F", 1025, ("scatter", 1, 8)),
])
def test_kernel_choice(torch_cuda, api, name, shape, mode, layout, n, want, mech_dir):
    """Both sides of a line: the route, and the results of the path that it takes."""
    torch = torch_cuda
    m, path = described(name, mech_dir)
    mech = api.load_mechanism(path)
    if shape:
        mech.set_launch(*shape)
    assert mech.kernel(mode, layout, n) == want
    x, p = synth.pack_state(synth.make_states(m, n, 4), "conp", "C")
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a if layout == "C" else a.T)).cuda()  # noqa: E731
    xs, ps = dev(x), torch.from_numpy(p.copy()).cuda()
    idx = sample(n)
    ti = torch.from_numpy(idx).cuda()
    pick = lambda t: (t[ti] if layout == "C" else t[..., ti].movedim(-1, 0)).cpu().numpy()  # noqa: E731
    o = oracle.Oracle(path)
    what = f"{name} {mode} {layout} {n}"
    if mode == "source":
        f_o, f_b = o.source(x[idx], p[idx], "conp", bound=True)
        check_source(pick(api.eval_source(mech, xs, ps, "conp", layout)), f_o, f_b, what)
    elif mode == "adjoint":
        v = np.random.default_rng(4).standard_normal(x.shape)
        j_o, _, j_b, _ = o.adjoint(x[idx], p[idx], v[idx], "conp", bound=True)
        check_jac(pick(api.eval_adjoint(mech, xs, ps, dev(v), "conp", layout)[0]), j_o, j_b, what)
    else:
        J_o, J_b = o.jacobian(x[idx], p[idx], "conp", bound=True)
        if mode == "sparse":
            J = api.sparse_to_dense(mech, pick(api.eval_jacobian_sparse(mech, xs, ps, "conp", layout)), "C")
        else:
            J = api.dense_as_sij(api.eval_jacobian_dense(mech, xs, ps, "conp", layout), layout)[ti].cpu().numpy()
        check_jac(J, J_o, J_b, what)


# (13 species, sparse, layout F: shapes of 8 and more states of the scatter kernels win)
@pytest.mark.parametrize("name,mode,n", [("ns13", "sparse", 32768), ("ns13", "dense", 32768), ("ns53", "sparse", 3000),
                                         ("ns53", "source", 40000)])
@pytest.mark.parametrize("layout,other", [("F", "C"), ("C", "F")])
def test_tuned_shape_stands_for_its_layout(torch_cuda, api, name, mode, n, layout, other, mech_dir):
    """A tuned shape is the one of calls in its layout, whichever kernels won; the
    other layout keeps the automatic choice (the wide kernel stages either)."""
    torch = torch_cuda
    sg = Segment(torch, api, mech_dir, name, n, mode, layout, 12)
    auto = sg.mech.kernel(mode, other, n)
    S, W, _ = api.autotune(sg.mech, sg.xs, sg.ps, "conp", layout, mode=mode, reps=3)
    own = sg.mech.kernel(mode, layout, n)
    assert own[1:] == (S, W) and sg.mech.launch_shape(api.MODES[mode]) == (S, W)
    assert sg.mech.kernel(mode, other, n) == (own if own[0] == "wide" else auto)
