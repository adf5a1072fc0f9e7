"""Write eigenvector entries of the bare reduced solver to this folder (needs a GPU).

    python tests/golden/make_reduced_vectors.py

An eigenvector's sign follows the rounding of the reduction, so the values are
the library's own: the first entry of each of the 40 lowest eigenvectors of
seeded pencils, two columns (re, im) per size.  Written by
the library at commit c715c31; rewriting the file changes what the test pins.
"""
from __future__ import annotations

import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(os.path.dirname(HERE)))

OUT = os.path.join(HERE, "reduced_vectors.txt")
SIZES = (60, 200, 256, 257, 384, 512, 513, 700, 1100)
NEV = 40


def pencil(n):
    rng = np.random.default_rng(n)
    a = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    b = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    return (a + a.conj().T) / (2.0 * np.sqrt(n)), np.eye(n) + 0.1 * (b + b.conj().T) / (2.0 * np.sqrt(n))


def first_entries(n):
    """The first entries of the lowest eigenvectors, from the library."""
    import torch
    from paper_0906_2569_amd import pwdft
    h, s = pencil(n)
    ctx = pwdft.Context(0)
    _, c, _ = pwdft.reduced_eigh(ctx, torch.from_numpy(h.T.copy()).cuda(), torch.from_numpy(s.T.copy()).cuda(), NEV)
    c = c.cpu().numpy()[:, 0]
    ctx.close()
    return c


def main():
    cols = []
    for n in SIZES:
        c = first_entries(n)
        cols += [c.real, c.imag]
    np.savetxt(OUT, np.array(cols).T, fmt="%.17g",
               header=f"first entries of the {NEV} lowest eigenvectors, (re, im) per size {SIZES}")


if __name__ == "__main__":
    main()
