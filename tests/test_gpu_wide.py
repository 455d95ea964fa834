"""The wide source-term kernel (a lane per state) against the oracle at the edges
of its groups of 64 states, waves and batches of four reactions: fewer
reactions than waves, further reaction types, temperatures at which the reverse
rates take the exponential of the sum or the range of the exponential ends,
absent species, Arrhenius parameters of the call, A = 0.  Gates as in
``oracle.gates``."""
import numpy as np
import pytest

import oracle
from oracle.gates import check_source
from paper_1809_01029_amd import synth
from conftest import TYPES_SEEDS, tiny_file, types_file, workload_file

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


@pytest.mark.parametrize("waves", [2, 3, 4, 8])
@pytest.mark.parametrize("form,layout", [("conp", "C"), ("conv", "F"), ("conp", "F"), ("conv", "C")])
@pytest.mark.parametrize("case", [("tiny", 1, ""), ("tiny", 130, "cold"), ("types", 65, ""), ("types", 64, "cold"),
                                  ("ns13", 63, "absent"), ("ns53", 129, ""), ("ns53", 65, "cold")])
def test_wide_parity(torch_cuda, api, case, form, layout, waves, mech_dir):
    torch = torch_cuda
    name, n, edge = case
    m, path = (tiny_file(3, mech_dir, bath_reactions=1, bath_efficiency=True) if name == "tiny"
               else types_file(TYPES_SEEDS[0], mech_dir, bath=True) if name == "types" else workload_file(name, mech_dir))
    x, p = synth.pack_state(synth.make_states(m, n, 5), form, "C")
    if edge == "cold":
        x[:, 0] = np.linspace(170.0, 330.0, n)
    elif edge == "absent":
        x[:, 2:] *= np.random.default_rng(1).random((n, m.n_species - 1)) < 0.5
    f_o, f_s = oracle.Oracle(path).source(x, p, form, bound=True)
    ok = np.isfinite(f_o).all(axis=1) & np.isfinite(f_s).all(axis=1)
    assert ok.any()
    print("case", name, n, edge, form, layout, waves, flush=True)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a if layout == "C" else a.T)).cuda()  # noqa: E731
    xs, ps = dev(x), torch.from_numpy(p.copy()).cuda()
    mech = api.load_mechanism(path)
    mech.set_launch(64, waves)
    assert mech.launch_shape(0) == (64, waves)
    for arr in (None, torch.as_tensor(np.stack(mech.arrhenius())).cuda()):
        f = api.eval_source(mech, xs, ps, form, layout, arrhenius=arr).cpu().numpy()
        check_source((f if layout == "C" else f.T)[ok], f_o[ok], f_s[ok], "source terms")
    # reactions switched off by A = 0 (ln A = -inf): as the scatter kernels have
    # it, nothing of an elementary or third-body reaction (k0 / k_inf of a falloff
    # reaction is no number then)
    off = torch.as_tensor(np.stack(mech.arrhenius())).cuda()
    off[0] = float("-inf")
    f = api.eval_source(mech, xs, ps, form, layout, arrhenius=off)
    mech.set_launch(4, 1)
    g = api.eval_source(mech, xs, ps, form, layout, arrhenius=off)
    assert torch.equal(f.isnan(), g.isnan()) and bool((f.nan_to_num() == 0).all())
