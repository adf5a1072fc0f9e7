"""Write the densities of tight default solves to this folder (needs a GPU).

    python tests/golden/make_tight_solve_density.py

The values are the library's own: below a residual tolerance of 1e-8 Ha and
with the default iteration limit a solve returns what its arithmetic's rounding
makes of the trial block, and callers compare runs bit for bit.  The file holds
every 97th grid value (x fastest) of the density of the solved block, weights
2, omega = 1000 bohr^3, for the seeded 8-atom, 16-band cell.  It was written by
the library at commit c715c31; rewriting it changes what the test pins.
"""
from __future__ import annotations

import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.dirname(os.path.dirname(HERE)))

OUT = os.path.join(HERE, "tight_solve_density.txt")
SEEDS = (2, 18)
STEP = 97


def main():
    import torch
    from paper_0906_2569_amd import pwdft, pwgen
    ctx = pwdft.Context(0)
    cols = []
    for seed in SEEDS:
        p = pwgen.make_cell(10.0, 15.0, 8, 16, seed, nr=(30, 30, 30))
        plan = pwdft.Plan(ctx, p, nb_max=16, ndim_max=4, density=1)
        x = torch.from_numpy(p.psi0).cuda()
        plan.davidson(x, opts=pwdft.default_opts(ndim=4, tol_resid=1e-10))
        cols.append(plan.density(x, np.full(16, 2.0), 1000.0).cpu().numpy().ravel()[::STEP])
    np.savetxt(OUT, np.array(cols).T, fmt="%.17g",
               header=f"density of tight default solves, every {STEP}th grid value; one column per seed {SEEDS}")


if __name__ == "__main__":
    main()
