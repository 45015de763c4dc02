"""Parameter records of a batch, made for all lattices at once, are those of a
Params object and the library's coupled rates per lattice, byte for byte."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

from paper_1802_02369_amd import autograd, lbm  # noqa: E402


@pytest.mark.parametrize("n", [1, 2, 1000])
@pytest.mark.parametrize("consts", [None, dict(gamma=1.67, prandtl=0.7, c0=0.4,
                                               lam=1.3, source_on=0)])
def test_records_match_params(n, consts):
    c = autograd._consts(consts)
    g = torch.Generator().manual_seed(n)
    s_e = 0.05 + 1.9 * torch.rand(n, generator=g, dtype=torch.float64)
    s_eps = 0.5 + torch.rand(n, generator=g, dtype=torch.float64)
    records, dpsi = autograd._records(s_e, s_eps, c)
    assert records.itemsize == ctypes.sizeof(lbm.CParams)
    for i in range(n):
        s_psi, _, d = lbm.coupled_rates(float(s_e[i]), c["gamma"], c["prandtl"])
        p = lbm.Params(s_e=float(s_e[i]), s_psi=s_psi, s_eps=float(s_eps[i]), **c)
        assert records[i].tobytes() == bytes(p.c())
        assert dpsi[i] == d


@pytest.mark.parametrize("bad", [0.0, 2.0, -1.0, float("nan"), float("inf")])
def test_records_refuse_what_the_library_refuses(bad):
    s_e = torch.tensor([1.5, bad, 1.2], dtype=torch.float64)
    with pytest.raises(lbm.LBMError, match="s_e must lie in"):
        autograd._records(s_e, torch.ones(3), autograd._consts(None))


@pytest.mark.parametrize("name", ["s_e", "s_psi", "s_eps"])
def test_records_refuse_rates_among_the_constants(name):
    """The rates have arguments of their own: a constant of their name is
    refused, as lbm.Params refuses it beside them."""
    c = autograd._consts({name: 1.2})
    with pytest.raises(TypeError, match="multiple values"):
        autograd._records(torch.tensor([1.5]), torch.tensor([1.5]), c)


@pytest.mark.parametrize("which", [0, 1])
def test_records_refuse_complex_rates(which):
    rates = [torch.tensor([1.5]), torch.tensor([1.5])]
    rates[which] = rates[which].to(torch.complex128)
    with pytest.raises(TypeError):
        autograd._records(*rates, autograd._consts(None))


def test_records_take_constants_as_tensors():
    """A constant may be anything lbm.Params takes, a tensor of one element
    among them, with its value as it is."""
    c = autograd._consts({"gamma": torch.tensor(1.375, dtype=torch.float32)})
    s_e = torch.tensor([1.1, 1.7], dtype=torch.float64)
    records, dpsi = autograd._records(s_e, torch.ones(2), c)
    for i in range(2):
        s_psi, _, d = lbm.coupled_rates(float(s_e[i]), 1.375, 1.0)
        assert records["s_psi"][i] == s_psi and dpsi[i] == d
