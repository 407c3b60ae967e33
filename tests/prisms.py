"""Hexagonal prisms: an orthogonal mesh of cells with 8 neighbours."""
import numpy as np

from paper_1207_1571_amd import meshgen as mg
from paper_1207_1571_amd import workloads as wl


def hex_prisms(nx, ny, nz):
    """nx x ny hexagons (rows shifted by half a cell) in nz layers; patches
    'wall' and 'lid' (the sides of the last row).  Orthogonal: every face is
    normal to the line of centres; up to 8 neighbours per cell."""
    h = 1.0
    a = h / np.sqrt(3.0)           # side of a hexagon with distance h between opposite sides
    area = 1.5 * np.sqrt(3.0) * a * a
    idx = lambda i, j, k: (k * ny + j) * nx + i
    C = np.empty((nx * ny * nz, 3))
    own, nei, S, Cf, bo, bS, bCf = [], [], [], [], [], [], []
    for k in range(nz):
        for j in range(ny):
            for i in range(nx):
                c = idx(i, j, k)
                C[c] = (i * h + 0.5 * h * (j & 1), j * 1.5 * a, k * h)
                for d in range(6):
                    t = np.pi / 3.0 * d
                    n = np.array([np.cos(t), np.sin(t), 0.0])
                    q = {0: (i + 1, j), 3: (i - 1, j), 1: (i + (j & 1), j + 1), 2: (i - 1 + (j & 1), j + 1),
                         4: (i - 1 + (j & 1), j - 1), 5: (i + (j & 1), j - 1)}[d]
                    cf = C[c] + 0.5 * h * n
                    if 0 <= q[0] < nx and 0 <= q[1] < ny:
                        e = idx(q[0], q[1], k)
                        if e > c:
                            own.append(c)
                            nei.append(e)
                            S.append(a * h * n)
                            Cf.append(cf)
                    else:
                        bo.append((1 if q[1] >= ny else 0, c))
                        bS.append(a * h * n)
                        bCf.append(cf)
                for s in (-1, 1):
                    n = np.array([0.0, 0.0, float(s)])
                    cf = C[c] + 0.5 * h * n
                    if 0 <= k + s < nz:
                        if s > 0:
                            own.append(c)
                            nei.append(idx(i, j, k + 1))
                            S.append(area * n)
                            Cf.append(cf)
                    else:
                        bo.append((0, c))
                        bS.append(area * n)
                        bCf.append(cf)
    order = sorted(range(len(bo)), key=lambda b: (bo[b][0], bo[b][1]))
    n0 = sum(1 for b in bo if b[0] == 0)
    Fi = len(own)
    own += [bo[b][1] for b in order]
    return mg.Mesh(owner=np.array(own, np.int32), neighbour=np.array(nei, np.int32),
                   Sf=np.array(S + [bS[b] for b in order]), Cf=np.array(Cf + [bCf[b] for b in order]), C=C,
                   V=np.full(nx * ny * nz, area * h), patch_names=["wall", "lid"],
                   patch_start=np.array([Fi, Fi + n0], np.int32), patch_size=np.array([n0, len(bo) - n0], np.int32),
                   shape=(nx, ny, nz), lex_of_cell=np.arange(nx * ny * nz))


def case(shape, precision=wl.FP64, tol=1e-9, **kw):
    m = hex_prisms(*shape)
    bcs = [wl.PatchBC(wl.FIXED, wl.ZERO_GRAD), wl.PatchBC(wl.FIXED, wl.ZERO_GRAD, (1.0, 0.0, 0.0))]
    return wl.CaseSpec(name="prisms", mesh=m, bcs=bcs, nu=0.1, dt=0.05, precision=precision, p_ctl=wl.SolverCtl(tol),
                       u_ctl=wl.SolverCtl(tol), **kw)
