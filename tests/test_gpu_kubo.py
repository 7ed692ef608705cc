"""The conductivity traces at the edges of their launch: atoms to either side of the eight XCDs' worth a
workgroup index deals out, members to either side of the 64 whose species one register holds, species that
change from member to member, no member at all, species out of range.  Reference: the same traces in extended
precision on the host."""

import numpy as np
import pytest
import torch

import paper_2311_12134_amd as lsms
from paper_2311_12134_amd.api import Liz

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _inputs(n_atoms, members, n_species, seed):
    rng = np.random.default_rng(seed)
    nl = rng.integers(max(0, members - 2), members + 1, n_atoms)
    nl[0] = members
    ptr = np.concatenate([[0], np.cumsum(nl)]).astype(np.int64)
    atom = rng.integers(0, n_atoms, ptr[-1]).astype(np.int32)
    species = rng.integers(0, n_species, n_atoms).astype(np.int32)

    def cplx(*shape):
        return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)

    return ptr, atom, species, cplx(n_species, 4, 3, 16, 16), [cplx(max(1, ptr[-1]), 16, 16) for _ in range(2)]


def _traces(ptr, atom, species, J, tau, kind):
    """Tr[J0(z2,z1) X1^T Ja(z1,z2) X2] summed over the members: [atom, combo, mu, nu]."""
    J, tau = J.astype(kind), [t.astype(kind) for t in tau]
    out = np.zeros((len(ptr) - 1, 4, 3, 3), dtype=kind)
    for m in range(len(ptr) - 1):
        for c in range(4):
            z1, z2 = c >> 1, c & 1
            for a in range(ptr[m], ptr[m + 1]):
                X1, X2, Ja = tau[z1][a], tau[z2][a], J[species[atom[a]], c]
                for nu in range(3):
                    Z = X1.T @ (Ja[nu] @ X2)
                    for mu in range(3):
                        out[m, c, mu, nu] += (J[species[m], z2 * 2 + z1, mu] * Z.T).sum()
    return out


def _run(ptr, atom, species, J, tau, tensor):
    ctx = lsms.Context(0)
    call = ctx.kubo_sigma_tensor if tensor else ctx.kubo_sigma
    liz = Liz(ptr, atom, np.zeros((len(atom), 3)))
    atom_dev = torch.from_numpy(atom if len(atom) else np.zeros(1, np.int32)).cuda()
    _, _, pa = call(liz, atom_dev, *[torch.from_numpy(t).cuda() for t in tau], torch.from_numpy(species).cuda(),
                    torch.from_numpy(J).cuda(), 100.0, per_atom=True)
    return pa.cpu().numpy()


@pytest.mark.parametrize("n_atoms,members,n_species", [(1, 1, 1), (1, 65, 3), (7, 2, 2), (8, 3, 1), (9, 64, 2),
                                                       (17, 5, 4), (2, 130, 2)])
def test_traces(n_atoms, members, n_species):
    args = _inputs(n_atoms, members, n_species, 31 * n_atoms + members)
    ptr, atom, species, J, tau = args
    want = _traces(*args, np.clongdouble)
    # every term passes at most 16 + 16 members + 16 + 8 additions, each complex product four roundings:
    # twice their sum times u bounds the error against the traces of the moduli
    size = _traces(ptr, atom, species, np.abs(J), [np.abs(t) for t in tau], np.float64)
    bound = 2 * (16 * members + 48) * U * 2 * size
    got = _run(*args, True)
    assert (np.abs(got - want) <= bound).all()
    assert (np.abs(got - want).max() <= 1e-12 * np.abs(want).max())  # what well-scaled traces reach, with room
    diag = _run(*args, False)
    assert (np.abs(diag - want[:, :, range(3), range(3)]) <= bound[:, :, range(3), range(3)]).all()


@pytest.mark.parametrize("wrong", [-1, 2])
def test_species_out_of_range_poison_their_atoms_only(wrong):
    ptr, atom, species, J, tau = _inputs(9, 70, 2, 5)
    atom[:] = np.where(atom == 4, 3, atom)
    atom[ptr[6] + 66] = 4  # atom 4 is its own centre, and a late member of atom 6's zone
    good = _run(ptr, atom, np.where(np.arange(9) == 4, 0, species).astype(np.int32), J, tau, True)
    species[4] = wrong
    got = _run(ptr, atom, species, J, tau, True)
    assert np.isnan(got[[4, 6]]).all()
    keep = [0, 1, 2, 3, 5, 7, 8]
    assert (got[keep] == good[keep]).all()


def test_no_members_give_zero():
    ptr, atom, species, J, tau = _inputs(3, 4, 2, 8)
    ptr = np.array([0, ptr[1], ptr[1], ptr[3]], dtype=np.int64)
    got = _run(ptr, atom, species, J, tau, True)
    assert (got[1] == 0).all() and (got[0] != 0).all()


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_no_members_give_zero_whatever_the_currents(value):
    """A skipped atom's species may have no finite currents: it contributes nothing all the same."""
    ptr, atom, species, J, tau = _inputs(3, 4, 1, 8)
    ptr = np.array([0, ptr[1], ptr[1], ptr[3]], dtype=np.int64)
    J = np.concatenate([J, np.full_like(J, value)])
    atom[atom == 1] = 0
    for tensor in (False, True):
        want = _run(ptr, atom, species, J, tau, tensor)
        species[1] = 1
        got = _run(ptr, atom, species, J, tau, tensor)
        species[1] = 0
        assert (got[1] == 0).all() and np.array_equal(got, want) and np.isfinite(got).all()
