"""Atomic Cholesky decomposition (aCD) on the device (Sec. II.A of the paper).

The aCD basis holds one-centre product densities only, chosen for each unique atom/basis
pair: here the pivots of a pivoted CD (to the same threshold delta) of the one-centre
integrals of one atom's functions alone, shared by all atoms with the same exponents.  The
molecular integral tables are the inner projection of Eq. (int_approx) onto those products,
V ~ V[:, A] V[A, A]^-1 V[A, :], computed as a pivoted CD of the full ERI matrix whose pivots
are restricted to A (every row updated; cds_cholesky_sgauss_subset), run until every product
is used or its residual is below fit_delta (default 1e-12 of the largest one-centre
diagonal: only numerically dependent products are dropped).

Host work is bookkeeping only: grouping functions by centre and mapping an atom's local pair
indices to global ones.  Every decomposition runs in the library's kernels.
"""
from __future__ import annotations

import dataclasses

import numpy as np
import torch

from . import core


def _pair_index(a, b):
    """Pair index of functions a and b (numbers or arrays)."""
    lo, hi = np.minimum(a, b), np.maximum(a, b)
    return hi * (hi + 1) // 2 + lo


def _pair_functions(I):
    """The functions (mu <= nu) of pair I (a number or an array)."""
    I = np.asarray(I, dtype=np.int64)
    b = ((np.sqrt(8.0 * I + 1.0) - 1.0) // 2).astype(np.int64)
    b = np.where(b * (b + 1) // 2 > I, b - 1, b)
    b = np.where((b + 1) * (b + 2) // 2 <= I, b + 1, b)
    return I - b * (b + 1) // 2, b


@dataclasses.dataclass
class ACDResult:
    products: np.ndarray        # global pair indices of the aCD basis (sorted)
    per_atom: int               # products of the first atom
    cd: core.CDResult           # restricted decomposition (the integral tables)
    fit_delta: float


def _atoms(centres: torch.Tensor) -> np.ndarray:
    """Atom number of every function (functions of one centre share it)."""
    return np.unique(centres.detach().cpu().numpy(), axis=0, return_inverse=True)[1].ravel()


def atomic_products(centres: torch.Tensor, alpha: torch.Tensor, delta: float,
                    ctx: core.Context | None = None) -> np.ndarray:
    return _products(_atoms(centres), centres, alpha, delta, ctx)


def _products(cid: np.ndarray, centres: torch.Tensor, alpha: torch.Tensor, delta: float,
              ctx: core.Context | None) -> np.ndarray:
    # the functions of each atom in order; an atom's products (pairs of its own functions) are found
    # once per set of exponents and mapped to all atoms that have it in one array operation (a loop
    # over the products took 1.2 ms for 60 atoms of 4 functions, more than half the GPU's work)
    a_h = alpha.detach().cpu().numpy()
    order = np.argsort(cid, kind="stable")
    atoms = np.split(order, np.flatnonzero(np.diff(cid[order])) + 1)
    same: dict[bytes, list] = {}
    for f in atoms:
        same.setdefault(a_h[f].tobytes(), []).append(f)
    out = []
    for group in same.values():
        idx = torch.as_tensor(group[0], device=centres.device)
        r = core.cholesky(delta, centres=centres[idx].contiguous(), alpha=alpha[idx].contiguous(), ctx=ctx)
        a, b = _pair_functions(r.piv[: r.nvec].cpu().numpy())
        f = np.stack(group)
        out.append(_pair_index(f[:, a], f[:, b]).ravel())
    return np.sort(np.concatenate(out)).astype(np.int64)


def acd(centres: torch.Tensor, alpha: torch.Tensor, delta: float, fit_delta: float | None = None,
        ctx: core.Context | None = None) -> ACDResult:
    cid = _atoms(centres)
    A = _products(cid, centres, alpha, delta, ctx)
    nbf = alpha.shape[0]
    np_ = nbf * (nbf + 1) // 2
    dev = alpha.device
    if fit_delta is None:
        # largest diagonal among the products (the largest ERI diagonal is a one-centre one)
        cols = torch.as_tensor(A, device=dev)
        Vc = core.eri_columns(centres, alpha, cols, ctx=ctx)
        vmax = float(Vc[torch.arange(A.size, device=dev), cols].max())
        fit_delta = 1e-12 * vmax
    allowed = torch.zeros(np_, dtype=torch.uint8, device=dev)
    allowed[torch.as_tensor(A, device=dev)] = 1
    cd = core.cholesky(fit_delta, centres=centres, alpha=alpha, allowed=allowed, max_vec=int(A.size), ctx=ctx)
    per_atom = int(np.count_nonzero(cid[_pair_functions(A)[0]] == cid[0]))
    return ACDResult(A, per_atom, cd, fit_delta)
