"""Which kernels the steps of a large Hubbard cluster take follows its state and its
Hamiltonian, and the adjoint follows the forward pass it belongs to.

The smallest chain whose steps may take one triangle of the pair matrix (33 sites,
33^4 > 2^20 elements) stands for the size; results of the same kernels are compared
bit for bit.
"""
import numpy as np
import pytest
import torch

from workloads import chain_hopping, random_g2, random_gless, rng, square_hopping

pytestmark = pytest.mark.gpu

NS = 33


def _system(r, ns=NS):
    h = chain_hopping(ns)
    h0 = np.stack([h + np.diag(r.uniform(-0.5, 0.5, ns)), 0.8 * h]).astype(complex)
    return h0, np.stack([random_gless(ns, r), random_gless(ns, r)])


def _complex_hopping(h0):
    """The same hopping with a phase on one bond."""
    h = h0.copy()
    h[:, 0, 1] *= 1j
    h[:, 1, 0] *= -1j
    return h


def _states(r):
    sym = random_g2(NS, r, scale=0.05, exchange=False)
    bad = sym.copy()
    bad[3, 4, 5, 6] += 1e-3
    return sym, bad


def _equal(a, b):
    same = [bool(np.array_equal(u, v)) for u, v in zip(a[:2], b[:2])]
    assert same == [True, True]


def test_state_set_under_complex_hoppings(lib):
    """Real hoppings, complex ones, a state without the pair symmetry set under these,
    real ones again: the steps evaluate every element, as the slice kernel does."""
    from paper_2002_12717_amd import binding as B
    r = rng(601)
    h0, g1 = _system(r)
    sym, bad = _states(r)
    out = []
    for flags in (0, B.HUB_SLICE_KERNEL):
        p = B.Propagator(B.HUBBARD, B.SOA, NS, h0, g1, U=1.1, G2_0=sym, flags=flags)
        p.set_h0(_complex_hopping(h0))
        p.set_state(g1, bad)
        p.set_h0(h0)
        p.step(0.01, 3)
        out.append(p.get_state())
        p.close()
    _equal(*out)


def test_hoppings_become_real(lib):
    """A context made with complex hoppings that becomes real takes the triangle for a
    symmetric state, as one made with the real ones."""
    from paper_2002_12717_amd import binding as B
    r = rng(602)
    h0, g1 = _system(r)
    sym, _ = _states(r)
    p = B.Propagator(B.HUBBARD, B.SOA, NS, _complex_hopping(h0), g1, U=1.1, G2_0=sym)
    p.set_h0(h0)
    q = B.Propagator(B.HUBBARD, B.SOA, NS, h0, g1, U=1.1, G2_0=sym)
    s = B.Propagator(B.HUBBARD, B.SOA, NS, h0, g1, U=1.1, G2_0=sym, flags=B.HUB_SLICE_KERNEL)
    for x in (p, q, s):
        x.step(0.01, 3)
    a, b, c = p.get_state(), q.get_state(), s.get_state()
    for x in (p, q, s):
        x.close()
    _equal(a, b)
    apart = not np.array_equal(b[1], c[1])   # the two kernels round differently, so equality tells them apart
    assert apart


def _gradient(p, a, b):
    loss, gc, gu = p.adjoint(a, b, 3)
    return [loss, gu, gc]


@pytest.mark.parametrize("first", ["bad", "sym"])
def test_state_set_between_forward_and_adjoint(lib, first):
    """A state of the other symmetry set between the forward pass and the adjoint: the
    segments are recomputed by the kernels of the forward pass, and the steps after
    the adjoint, which restores the final state, take those that this state calls
    for, also where a graph of the other kernels was captured in between."""
    from paper_2002_12717_amd import binding as B
    r = rng(603)
    h0, g1 = _system(r)
    sym, bad = _states(r)
    a, b = r.uniform(-1, 1, NS), r.uniform(-1, 1, NS)
    x, c, tc = np.arange(NS) - 16.0, 0.1 * r.standard_normal(3), 0.02 * np.arange(3)
    start, other = (bad, sym) if first == "bad" else (sym, bad)
    out = []
    for between in (True, False):
        stream = torch.cuda.Stream()
        p = B.Propagator(B.HUBBARD, B.SOA, NS, h0, g1, U=1.1, stream=stream.cuda_stream)
        p.set_drive(x, c, tc, 0.02)
        p.set_state(g1, start)
        p.forward_checkpointed(0.01, 5, 2)
        if between:
            p.set_state(g1, other)
        res = _gradient(p, a, b)
        p.set_drive(x, [], [], 0.02)
        if between:
            p.set_state(g1, other)
            p.prepare_graph(0.01)
            p.set_drive(x, c, tc, 0.02)
            res += _gradient(p, a, b)
            p.set_drive(x, [], [], 0.02)
        else:
            res += res
        p.step(0.01, 8)
        out.append((res, p.get_state()[:2]))
        p.close()
    same = [bool(np.array_equal(u, v)) for u, v in zip(out[0][0], out[1][0])]
    assert all(same)
    _equal(out[0][1], out[1][1])


@pytest.mark.parametrize("ns,interval", [(NS, 0), (NS, 2), (4, 2)])
def test_adjoint_after_a_forward_pass_that_failed(lib, ns, interval):
    """A forward pass that diverged leaves nothing to differentiate: the adjoint
    answers ESTATE, also where the buffers of an earlier gradient serve again, and a
    later forward pass restores it."""
    from paper_2002_12717_amd import binding as B
    r = rng(604)
    h0, g1 = _system(r, ns)
    a, b = r.uniform(-1, 1, ns), r.uniform(-1, 1, ns)
    p = B.Propagator(B.HUBBARD, B.SOA, ns, h0, g1, U=1.1)
    far = g1.copy()
    far[0, 0, 0] = 2j                          # an occupation of 2
    out = []
    for _ in range(2):
        p.set_state(g1)
        p.forward_checkpointed(0.01, 5, interval)
        out.append(p.adjoint(a, b, 0)[::2])
        p.set_state(far)
        with pytest.raises(B.G1G2Error) as e:
            p.forward_checkpointed(0.01, 5, interval)
        assert e.value.status == B.EDIVERGED
        with pytest.raises(B.G1G2Error) as e:
            p.adjoint(a, b, 0)
        assert e.value.status == B.ESTATE
    p.close()
    assert out[0] == out[1]


@pytest.mark.parametrize("size", [2.0 ** -46, 2.0 ** -51])
def test_slightly_asymmetric_state_is_evolved_in_full(lib, size):
    """An asymmetry of G2, however small, is part of the state: every element is
    evaluated, bit for bit as by the slice kernel."""
    from paper_2002_12717_amd import binding as B
    r = rng(605)
    h0, g1 = _system(r)
    sym, _ = _states(r)
    g2 = sym.copy()
    g2[3, 4, 5, 6] += size * np.abs(sym).max()
    out = []
    for flags in (0, B.HUB_SLICE_KERNEL):
        p = B.Propagator(B.HUBBARD, B.SOA, NS, h0, g1, U=1.1, flags=flags)
        p.set_state(g1, g2)
        p.step(0.01, 2)
        out.append(p.get_state())
        p.close()
    _equal(*out)


@pytest.mark.parametrize("lx,ly,se", [(33, 1, "soa"), (33, 1, "tpp"), (33, 1, "tph"), (9, 5, "soa"), (5, 5, "gw"),
                                      (9, 5, "dsl")])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_steps_keep_the_symmetry_bit_for_bit(lib, lx, ly, se, prec):
    """A symmetric state stays so to the last bit, so that a context restarted from a
    saved state goes on exactly as the one that saved it."""
    from paper_2002_12717_amd import binding as B
    r = rng(606, lx, ly, len(se))
    ns, nch = lx * ly, 3 if se in ("gw", "dsl") else 1
    h = square_hopping(lx, ly, periodic=False) if ly > 1 else chain_hopping(lx)
    h0 = np.stack([h + np.diag(r.uniform(-0.5, 0.5, ns)), 0.8 * h]).astype(complex)
    g1 = np.stack([random_gless(ns, r), random_gless(ns, r)])
    g2 = np.stack([random_g2(ns, r, scale=0.05, exchange=False) for _ in range(nch)])
    g2 = g2 if nch == 3 else g2[0]
    code = {"soa": B.SOA, "tpp": B.TPP, "tph": B.TPH, "gw": B.GW, "dsl": B.DSL}[se]
    kw = dict(U=1.3, precision=B.FP64 if prec == "fp64" else B.MIXED)
    p = B.Propagator(B.HUBBARD, code, ns, h0, g1, **kw)
    p.set_state(g1, g2)
    p.step(0.01, 7)
    s1, s2, _ = p.get_state()
    m = s2.reshape(nch, ns * ns, ns * ns)
    kept = [bool(np.array_equal(s1, -s1.conj().transpose(0, 2, 1))), bool(np.array_equal(m, m.conj().transpose(0, 2, 1)))]
    assert kept == [True, True]
    q = B.Propagator(B.HUBBARD, code, ns, h0, s1, G2_0=s2, **kw)
    p.step(0.01, 3)
    q.step(0.01, 3)
    a, b = p.get_state(), q.get_state()
    p.close()
    q.close()
    _equal(a, b)


def test_unequal_hoppings_are_evolved_in_full(lib):
    """h0 passes as Hermitian to 1e-12; hoppings h_ij and h_ji that differ within that
    take the slice kernel, which reads both."""
    from paper_2002_12717_amd import binding as B
    r = rng(607)
    h0, g1 = _system(r)
    sym, _ = _states(r)
    h0[0, 3, 4] += 5e-13
    h0[1, 7, 20] = 4e-13                       # h_ji = 0: a neighbour in one direction only
    out = []
    for flags in (0, B.HUB_SLICE_KERNEL):
        p = B.Propagator(B.HUBBARD, B.SOA, NS, h0, g1, U=1.1, G2_0=sym, flags=flags)
        p.step(0.01, 2)
        out.append(p.get_state())
        p.close()
    _equal(*out)


def test_step_path_and_profile_name_the_kernels(lib):
    """step_path answers hub_triangle exactly where steps run over one triangle, and the
    profile counts their stages under a name of their own; a gradient that keeps its
    states runs no stage in its reverse sweep."""
    from paper_2002_12717_amd import binding as B
    r = rng(608)
    h0, g1 = _system(r)
    sym, bad = _states(r)
    p = B.Propagator(B.HUBBARD, B.SOA, NS, h0, g1, U=1.1)
    assert p.step_path() == "hub_triangle"
    prof = p.profile(0.01, 2)
    assert prof["hub_tile"][1] == 8 and "hub_stage" not in prof
    p.set_state(g1, bad)
    assert p.step_path() == "hub_slice"
    prof = p.profile(0.01, 2)
    assert prof["hub_stage"][1] == 8 and "hub_tile" not in prof
    p.set_state(g1, sym)
    assert p.step_path() == "hub_triangle"
    p.set_h0(_complex_hopping(h0))
    assert p.step_path() == "hub_slice"
    p.set_h0(h0)
    assert p.step_path() == "hub_triangle"
    a, b = r.uniform(-1, 1, NS), r.uniform(-1, 1, NS)
    p.forward_checkpointed(0.01, 4)
    assert not {"hub_tile", "hub_stage"} & set(p.profile_adjoint(a, b))
    p.set_state(g1, sym)
    p.forward_checkpointed(0.01, 4, 2)
    assert p.profile_adjoint(a, b)["hub_tile"][1] == 14      # two segments of two steps, the last stage left out
    p.set_state(g1, bad)
    p.forward_checkpointed(0.01, 4)
    assert p.profile_adjoint(a, b)["hub_stage"][1] > 0
    p.close()
    for flags, path in ((B.HUB_SLICE_KERNEL, "hub_slice"), (B.HUB_ROW_KERNEL, "hub_row")):
        q = B.Propagator(B.HUBBARD, B.SOA, NS, h0, g1, U=1.1, flags=flags)
        assert q.step_path() == path
        q.close()
    b4 = B.Batch(B.TPP, [NS, 3], [1.0, 1.0], [h0, _system(r, 3)[0]], [g1, _system(r, 3)[1]])
    assert b4.step_path() == "hub_triangle"
    b4.close()
