"""Helpers shared by the GPU parity tests: run the HIP path through the C ABI
and the oracle on the same canonical inputs, and compare.

Tolerances are derived from the arithmetic (float32 unit roundoff
u = 2^-24) and written where they are used:

* sorted state, cell ranges, neighbour sets, counts, status: bit-exact;
* derivatives: per particle and component, |f_gpu - f_oracle| <= 1e-5 S,
  where S is the oracle's sum of the magnitudes of the pair terms (the
  condition scale of the sum; a plain relative error would measure the
  cancellation of the still-water balance, not the implementation);
* integrator: one rounding per operand of y + tau f on top of the
  derivative tolerance: |dy| <= 4 u (|y| + tau |f|) + tau 1e-5 S.
"""
from __future__ import annotations

import sys

import numpy as np
import torch

from oracle import oracle as O
from workloads import scenes as S

U32 = 2.0 ** -24
FORCE_TOL = 1e-5
SENT = np.iinfo(np.int64).max


def log(msg: str):
    print(msg, flush=True)
    sys.stdout.flush()


def make_sim(sc, max_neibs=128, capacity=None, **kw):
    from paper_2207_11328_amd.sim import Simulation
    return Simulation(sc.grid, sc.params, sc.cell, sc.pos, sc.vel, sc.info, max_neibs=max_neibs,
                      capacity=capacity, **kw)


def gpu_lists_padded(sim):
    """GPU split lists -> (fluid idx [n,max] sorted, boundary idx sorted,
    fluid codes, boundary codes) with SENT padding; codes follow the index sort."""
    nb, cnt = sim.lists_host()
    n = sim.n
    M = sim.max_neibs
    E = nb[:, :n].T.astype(np.int64)  # [n, M]
    nf = (cnt & 0xFFFF).astype(np.int64)
    nbd = (cnt >> 16).astype(np.int64)
    col = np.arange(M)[None, :]
    fmask = col < nf[:, None]
    bmask = col >= (M - nbd)[:, None]
    idx = E & ((1 << 26) - 1)
    code = E >> 26
    fi = np.where(fmask, idx, SENT)
    bi = np.where(bmask, idx, SENT)
    fo = np.argsort(fi, axis=1, kind="stable")
    bo = np.argsort(bi, axis=1, kind="stable")
    fi = np.take_along_axis(fi, fo, 1)
    bi = np.take_along_axis(bi, bo, 1)
    fc = np.take_along_axis(np.where(fmask, code, -1), fo, 1)
    bc = np.take_along_axis(np.where(bmask, code, -1), bo, 1)
    return fi, bi, fc, bc, nf, nbd


def gpu_lists_rows(sim, rows):
    """As gpu_lists_padded, for the particles `rows` only (gathered on the
    device from the tiled list, so very large lists are never copied whole)."""
    M = sim.max_neibs
    r = torch.as_tensor(np.asarray(rows, np.int64), device=sim.device)
    k = torch.arange(M, device=sim.device, dtype=torch.int64)
    idx = (r // 64)[:, None] * (64 * M) + k[None, :] * 64 + (r % 64)[:, None]
    E = sim.neibs[idx].cpu().numpy().view(np.uint32).astype(np.int64)  # [m, M]
    cnt = sim.neib_count[r].cpu().numpy().view(np.uint32)
    nf = (cnt & 0xFFFF).astype(np.int64)
    nbd = (cnt >> 16).astype(np.int64)
    col = np.arange(M)[None, :]
    fmask = col < nf[:, None]
    bmask = col >= (M - nbd)[:, None]
    idxv = E & ((1 << 26) - 1)
    code = E >> 26
    fi = np.where(fmask, idxv, SENT)
    bi = np.where(bmask, idxv, SENT)
    fo = np.argsort(fi, axis=1, kind="stable")
    bo = np.argsort(bi, axis=1, kind="stable")
    return (np.take_along_axis(fi, fo, 1), np.take_along_axis(bi, bo, 1),
            np.take_along_axis(np.where(fmask, code, -1), fo, 1), np.take_along_axis(np.where(bmask, code, -1), bo, 1))


def oracle_lists_padded(lists, max_neibs):
    n = lists.nf.shape[0]
    col = np.arange(max_neibs)[None, :]
    fi = np.where(col < lists.nf[:, None], lists.fl.astype(np.int64), SENT)
    bi = np.where(col < lists.nb[:, None], lists.bl.astype(np.int64), SENT)
    return np.sort(fi, axis=1), np.sort(bi, axis=1)


def expected_codes(grid, cell, idx_sorted):
    """Cell-difference codes (k_d + 1 per axis, 2 bits each) for padded
    neighbour index rows of a sorted state."""
    nx, ny, nz = (int(v) for v in grid.ncell)
    lc = cell.astype(np.int64) - int(grid.cell_base)
    c = np.stack([lc % nx, (lc // nx) % ny, lc // (nx * ny)], axis=1)
    valid = idx_sorted != SENT
    j = np.where(valid, idx_sorted, 0)
    code = np.zeros(idx_sorted.shape, dtype=np.int64)
    for d, nd in enumerate((nx, ny, nz)):
        k = c[:, d][:, None] - c[:, d][j]
        if (grid.periodic >> d) & 1:
            k = np.where(k > 1, k - nd, k)
            k = np.where(k < -1, k + nd, k)
        code |= (k & 3) << (2 * d)
    return np.where(valid, code, -1)


def compare_build(sc, sim, max_neibs=128, rows=None):
    """Bit-exact comparison of a GPU build with the oracle's float32 build.
    rows: optional subset of particle indices for the list comparison."""
    ob = O.build_f32(sc.grid, sc.params, sc.cell, sc.pos, sc.vel, sc.info, max_neibs)
    gs = sim.state_host()
    n = sc.n
    assert np.array_equal(gs["info"], ob["info"]), "sort order"
    assert np.array_equal(gs["cell"], ob["cell"]), "cells"
    assert np.array_equal(gs["pos"].view(np.uint32), ob["pos"].view(np.uint32)), "re-binned offsets"
    assert np.array_equal(gs["vel"].view(np.uint32), np.ascontiguousarray(ob["vel"]).view(np.uint32)), "vel"
    nc = sc.grid.n_cells
    assert np.array_equal(sim.cell_start[:nc].cpu().numpy(), ob["start"]), "cell_start"
    assert np.array_equal(sim.cell_end[:nc].cpu().numpy(), ob["end"]), "cell_end"
    st = sim.status_host()
    assert st["n_active"] == ob["n_active"] and st["dropped"] == ob["dropped"], (st, ob["n_active"])
    assert st["overflow"] == ob["lists"].overflow, (st, ob["lists"].overflow)
    fi, bi, fc, bc, nf, nbd = gpu_lists_padded(sim)
    ofi, obi = oracle_lists_padded(ob["lists"], max_neibs)
    if rows is not None:
        fi, bi, fc, bc, ofi, obi = fi[rows], bi[rows], fc[rows], bc[rows], ofi[rows], obi[rows]
        cells = ob["cell"]
    else:
        cells = ob["cell"]
    assert np.array_equal(fi, ofi), "fluid neighbour sets"
    assert np.array_equal(bi, obi), "boundary neighbour sets"
    if st["overflow"] == 0:
        sel = rows if rows is not None else slice(None)
        ec_f = expected_codes_rows(sc.grid, cells, fi, sel)
        ec_b = expected_codes_rows(sc.grid, cells, bi, sel)
        assert np.array_equal(fc, ec_f), "fluid cell codes"
        assert np.array_equal(bc, ec_b), "boundary cell codes"
    return ob


def expected_codes_rows(grid, cell, idx_rows, sel):
    nx, ny, nz = (int(v) for v in grid.ncell)
    lc = cell.astype(np.int64) - int(grid.cell_base)
    c = np.stack([lc % nx, (lc // nx) % ny, lc // (nx * ny)], axis=1)
    ci = c[sel]
    valid = idx_rows != SENT
    j = np.where(valid, idx_rows, 0)
    code = np.zeros(idx_rows.shape, dtype=np.int64)
    for d, nd in enumerate((nx, ny, nz)):
        k = ci[:, d][:, None] - c[:, d][j]
        if (grid.periodic >> d) & 1:
            k = np.where(k > 1, k - nd, k)
            k = np.where(k < -1, k + nd, k)
        code |= (k & 3) << (2 * d)
    return np.where(valid, code, -1)


def oracle_forces_of(sc, ob, state_pos=None, state_vel=None, alpha=None):
    pos = ob["pos"] if state_pos is None else state_pos
    vel = ob["vel"] if state_vel is None else state_vel
    st = O.State.lift(ob["cell"], pos, vel, ob["info"])
    return st, O.forces(sc.grid, sc.params, st, ob["lists"], alpha)


EDGE_REL = 2e-6


def support_edge_rows(sc, ob, rel=EDGE_REL, rows=None, lists=None):
    """Mask of the particles with a listed neighbour at |r - 2h| <= rel 2h.
    A kernel whose F does not vanish at the edge of its support (the
    truncated Gaussian) gives such a pair a finite weight, and the float32
    interaction decision of the GPU and the FP64 one of the oracle may then
    differ, both being correct to rounding: these particles are left out of
    the element-wise comparison for that kernel.  The window, 2e-6 of 2h,
    covers the float32 separation error of the brick form (a few ulp of the
    2.5 cell sizes of a brick-relative offset, about 5e-7 of 2h) with a
    factor of four.  rows/lists: a subset of particles and their row-indexed
    lists (otherwise all, from ob)."""
    L = ob["lists"] if lists is None else lists
    cell_all = ob["cell"].astype(np.int64) - int(sc.grid.cell_base)
    off_all = ob["pos"][:, :3].astype(np.float64)
    sel = slice(None) if rows is None else np.asarray(rows)
    cell, off = cell_all[sel], off_all[sel]
    nx, ny, nz = (int(v) for v in sc.grid.ncell)
    c = np.stack([cell % nx, (cell // nx) % ny, cell // (nx * ny)], axis=1)
    cs = [float(v) for v in sc.grid.cell_size]
    two_h = 2.0 * O.f32(sc.params.h)
    ca = np.stack([cell_all % nx, (cell_all // nx) % ny, cell_all // (nx * ny)], axis=1)
    mask = np.zeros(cell.shape[0], bool)
    for idx, cnt in ((L.fl, L.nf), (L.bl, L.nb)):
        valid = np.arange(idx.shape[1])[None, :] < cnt[:, None]
        j = np.where(valid, idx, 0)
        r2 = np.zeros(idx.shape)
        for d, nd in enumerate((nx, ny, nz)):
            k = c[:, d][:, None] - ca[:, d][j]
            if (sc.grid.periodic >> d) & 1:
                k = np.where(k > 1, k - nd, k)
                k = np.where(k < -1, k + nd, k)
            x = k * cs[d] + (off[:, d][:, None] - off_all[:, d][j])
            r2 += x * x
        mask |= np.any(valid & (np.abs(np.sqrt(r2) - two_h) <= rel * two_h), axis=1)
    return mask


# float32 rounding of a separation component in the derivative kernels: the
# brick form subtracts two brick-relative coordinates of up to 3.5 cell
# sizes, each rounded to half an ulp (at most 2^-22 cs): 2^-21 cs in all
SEP_ULPS = 2.0 ** -21
# relative rounding of r^2, its square root and q = r / h: about 4 u, doubled
EPS_R = 5e-7


def edge_allowance(sc, ob):
    """Wendland kernel, golden rule, artificial viscosity: the first-order
    effect on each pair term of the float32 rounding of the separation
    (dx = 2^-21 cs per component, absolute) and of r (EPS_R, relative):
      * a component x_d of a pair term moves by |coef| dx, which is large
        against |coef x_d| when the pair is nearly perpendicular to axis d;
      * the kernel factor F ~ (2 - q)^3 moves by 3 dr / (2h - r) of itself,
        which grows without bound at the support edge.
    A particle with many pairs hides both in 1e-5 S; a sparse particle whose
    few pairs are such cannot meet it in any float32 evaluation.  Returns
    (allowance of a [n, 3], of Drho/Dt [n]), summed over the particle's
    interacting pairs."""
    p = sc.params
    L = ob["lists"]
    st = O.State.lift(ob["cell"], ob["pos"], ob["vel"], ob["info"])
    n = st.n
    h = O.f32(p.h)
    dx = SEP_ULPS * float(np.max(sc.grid.cell_size))
    x_all = O.positions(sc.grid, st)
    period = sc.grid.ncell * sc.grid.cell_size.astype(np.float64)
    per = np.array([(sc.grid.periodic >> d) & 1 for d in range(3)], bool)
    rho0, c0, gam = O.f32(p.rho0), O.f32(p.c0), O.f32(p.gamma)
    B = rho0 * c0 * c0 / gam
    P = B * ((st.rho / rho0) ** gam - 1.0)
    c = c0 * (st.rho / rho0) ** ((gam - 1.0) / 2.0)
    aa = np.zeros((n, 3))
    ad = np.zeros(n)
    for i in range(n):
        for j in list(L.fluid(i)) + list(L.boundary(i)):
            x = x_all[i] - x_all[j]
            x = np.where(per, x - period * np.round(x / period), x)
            r = float(np.sqrt((x * x).sum()))
            if r >= 2.0 * h:
                continue
            F = abs(O.wendland_F(r, h))
            dr = np.sqrt(3.0) * dx + EPS_R * r
            kappa = 3.0 * dr / (2.0 * h - r)          # relative change of F
            u = st.vel[i] - st.vel[j]
            au = np.abs(u)
            uxa = float(np.abs(u * x).sum())
            m = st.mass[j]
            ad[i] += m * F * (kappa * uxa + float(au.sum()) * dx)
            dd = r * r + O.f32(p.eps_visc) * h * h
            visc_k = O.f32(p.alpha) * h * 0.5 * (c[i] + c[j]) / (0.5 * (st.rho[i] + st.rho[j]) * dd)
            pi_ab = visc_k * uxa if float((u * x).sum()) < 0.0 else 0.0
            dpi = visc_k * float(au.sum()) * dx if float((u * x).sum()) < 0.0 else 0.0
            pres = abs(P[i]) / st.rho[i] ** 2 + abs(P[j]) / st.rho[j] ** 2
            coef = m * (pres + pi_ab) * F
            aa[i] += coef * (kappa * np.abs(x) + dx) + m * F * dpi * np.abs(x)
    return aa, ad


def adjoint_edge_allowance(sc, ob, abar, dbar):
    """edge_allowance for the adjoint (Wendland kernel, golden rule, artificial
    viscosity): what the float32 rounding of the separation (dx per component)
    and of r (dr) can do to each term, to first order.  Every term is a product
    of factors; with all of them in absolute value the sum over the pairs is
    evaluated twice, at |x| and at |x| + dx with F and F'/r larger by the
    relative change that dr makes (3 dr / (2h - r) and 2 dr / (2h - r) + dr / r),
    r^2 + eps h^2 smaller by 2 r dr, and the viscosity of the pairs whose u.x is
    within its own rounding of zero in the second sum only.  Returns the
    differences for dL/do [n, 3], dL/du [n, 3], dL/drho [n]."""
    p = sc.params
    L = ob["lists"]
    st = O.State.lift(ob["cell"], ob["pos"], ob["vel"], ob["info"])
    n, h = st.n, O.f32(p.h)
    period = sc.grid.ncell * sc.grid.cell_size.astype(np.float64)
    per = np.array([(sc.grid.periodic >> d) & 1 for d in range(3)], bool)
    ii, jj = [], []
    for idx, cnt in ((L.fl, L.nf), (L.bl, L.nb)):
        m = np.arange(idx.shape[1])[None, :] < cnt[:, None]
        ii.append(np.nonzero(m)[0])
        jj.append(idx[m])
    i, j = np.concatenate(ii).astype(np.int64), np.concatenate(jj).astype(np.int64)
    x_all = O.positions(sc.grid, st)
    x = x_all[i] - x_all[j]
    x = np.where(per, x - period * np.round(x / period), x)
    r = np.sqrt((x * x).sum(1))
    keep = r < 2.0 * h
    i, j, x, r = i[keep], j[keep], x[keep], r[keep]
    rho0, c0, eps = O.f32(p.rho0), O.f32(p.c0), O.f32(p.eps_visc) * h * h
    B = rho0 * c0 * c0 / 7.0
    b = st.rho / rho0
    P, c = B * (b ** 7 - 1.0), c0 * b ** 3
    pr, dpr = np.abs(P) / st.rho ** 2, np.abs(c * c / st.rho ** 2 - 2.0 * P / st.rho ** 3)
    dc = 3.0 * c / st.rho
    rs, cs = st.rho[i] + st.rho[j], c[i] + c[j]
    ah = O.f32(p.alpha) * h
    u = np.abs(st.vel[i] - st.vel[j])
    w = ((st.vel[i] - st.vel[j]) * x).sum(1)
    mi, mj = st.mass[i], st.mass[j]
    da = np.abs(mj[:, None] * abar[i]) + np.abs(mi[:, None] * abar[j])
    sd = np.abs(mj * dbar[i]) + np.abs(mi * dbar[j])
    coef = 105.0 / (128.0 * np.pi * h ** 5)
    t = 1.0 - r / (2.0 * h)
    F, Fr = 8.0 * coef * t ** 3, 12.0 * coef * t * t / (h * r)
    dx = SEP_ULPS * float(np.max(sc.grid.cell_size))
    dr = np.sqrt(3.0) * dx + EPS_R * r
    dw = u.sum(1) * dx

    def sums(X, F, Fr, dd, act):
        W, DA = (u * X).sum(1), (da * X).sum(1)
        K = np.where(act, ah * cs / (rs * dd), 0.0)
        S_ = pr[i] + pr[j] + K * W
        o = (S_ * F)[:, None] * da + (DA * S_ * Fr + sd * W * Fr + 2.0 * DA * F * K * W / dd)[:, None] * X \
            + (DA * F * K + sd * F)[:, None] * u
        v = (F * K * DA + sd * F)[:, None] * X
        q = F * DA * (dpr[i] + np.where(act, ah * W / dd * (dc[i] + cs / rs) / rs, 0.0))
        add = lambda y: np.bincount(i, y, n)
        return (np.stack([add(o[:, d]) for d in range(3)], 1), np.stack([add(v[:, d]) for d in range(3)], 1), add(q))

    ax, dd = np.abs(x), r * r + eps
    edge = dr / (2.0 * h - r)
    low = sums(ax, F, Fr, dd, w < -dw)
    high = sums(ax + dx, F * (1.0 + 3.0 * edge), Fr * (1.0 + 2.0 * edge + dr / r), dd - 2.0 * r * dr, w < dw)
    return tuple(b_ - a_ for a_, b_ in zip(low, high))


def check_forces(gpu_f, acc, drho, s_acc, s_drho, tol=FORCE_TOL, label="", exclude=None, allowance=None):
    """Returns the max normalised errors (acc, drho); asserts <= tol.
    exclude: optional mask of particles left out (see support_edge_rows).
    allowance: optional (a [n, 3], Drho [n]) added to the error before the
    normalisation is compared (see edge_allowance)."""
    if exclude is not None:
        keep = ~np.asarray(exclude, bool)
        gpu_f, acc, drho, s_acc, s_drho = gpu_f[keep], acc[keep], drho[keep], s_acc[keep], s_drho[keep]
        if allowance is not None:
            allowance = (allowance[0][keep], allowance[1][keep])
    ga = gpu_f[:, :3].astype(np.float64)
    gd = gpu_f[:, 3].astype(np.float64)
    ea = np.abs(ga - acc)
    ed = np.abs(gd - drho)
    if allowance is not None:
        ea = np.maximum(ea - allowance[0], 0.0)
        ed = np.maximum(ed - allowance[1], 0.0)
    za = s_acc == 0
    zd = s_drho == 0
    assert np.all(ga[za] == 0.0), label + ": nonzero acceleration with no interaction"
    assert np.all(gd[zd] == 0.0), label + ": nonzero density rate with no interaction"
    na = np.where(za, 0.0, ea / np.where(za, 1.0, s_acc))
    nd = np.where(zd, 0.0, ed / np.where(zd, 1.0, s_drho))
    worst_a, worst_d = float(na.max(initial=0.0)), float(nd.max(initial=0.0))
    log("%s forces: max |da|/S = %.3e, max |dDrho|/S = %.3e" % (label, worst_a, worst_d))
    assert worst_a <= tol, (label, worst_a, np.unravel_index(np.argmax(na), na.shape))
    assert worst_d <= tol, (label, worst_d, int(np.argmax(nd)))
    return worst_a, worst_d


def torch_sync():
    torch.cuda.synchronize()


def expected_brick_lists(sim, grid, brick=None):
    """Brick-local lists implied by the GPU's own j-lists and cell ranges,
    from the layout the header documents: entry k of particle i is the
    neighbour's position in the staging order of i's brick (the
    (BX+2)(BY+2)(BZ+2) cells of the brick and its halo, x fastest, then z,
    then y, periodic axes wrapped, cells
    past a closed axis empty; particles of a cell in sorted order), entries
    in scan order (neighbour cells z, y, x from -1 to +1, then sorted index),
    fluid and boundary interleaved.  Returns
    ([n, M] int64 with -1 past each list, n_total [n])."""
    if brick is None:
        brick = sim.brick_shape
    BX, BY, BZ = brick
    n, M = sim.n, sim.max_neibs
    nb, cnt = sim.lists_host()
    E = nb[:, :n].T.astype(np.int64)
    cnt = cnt.astype(np.int64)
    nf, nbd = cnt & 0xFFFF, cnt >> 16
    cell = sim.cell[:n].cpu().numpy().astype(np.int64) - int(grid.cell_base)
    cs_ = sim.cell_start[: grid.n_cells].cpu().numpy().astype(np.int64)
    ce_ = sim.cell_end[: grid.n_cells].cpu().numpy().astype(np.int64)
    nx, ny, nz = (int(v) for v in grid.ncell)
    per = [(int(grid.periodic) >> d) & 1 for d in range(3)]
    SX, SY, SZ = BX + 2, BY + 2, BZ + 2
    out = np.full((n, M), -1, np.int64)
    bases = {}

    def staging(bx, by, bz):
        key = (bx, by, bz)
        if key not in bases:
            st = np.zeros(SX * SY * SZ, np.int64)
            ct = np.zeros(SX * SY * SZ, np.int64)
            for t in range(SX * SY * SZ):
                g = [bx * BX - 1 + t % SX, by * BY - 1 + t // (SX * SZ), bz * BZ - 1 + (t // SX) % SZ]
                ok = True
                for d, nd in enumerate((nx, ny, nz)):
                    if per[d]:
                        g[d] %= nd
                    elif not 0 <= g[d] < nd:
                        ok = False
                if ok:
                    lin = g[0] + nx * (g[1] + ny * g[2])
                    st[t], ct[t] = cs_[lin], ce_[lin] - cs_[lin]
            base = np.concatenate([[0], np.cumsum(ct)[:-1]])
            bases[key] = (base - st, int(ct.sum()))
        return bases[key]

    totals = np.zeros(n, np.int64)
    for i in range(n):
        c = cell[i]
        if c < 0:
            continue
        cx, cy, cz = c % nx, (c // nx) % ny, c // (nx * ny)
        delta, tot = staging(cx // BX, cy // BY, cz // BZ)
        totals[i] = tot
        tc = (cx % BX + 1) + SX * ((cz % BZ + 1) + SZ * (cy % BY + 1))
        order = list(range(nf[i])) + [M - 1 - b for b in range(nbd[i])]
        e = E[i, order]
        j = e & ((1 << 26) - 1)
        k = [((e >> (26 + 2 * d)) & 3) for d in range(3)]
        k = [np.where(v >= 2, v - 4, v) for v in k]
        # scan order: neighbour cell offset d = -k, z outermost, then index
        o = np.lexsort((j, -k[0], -k[1], -k[2]))
        j, k = j[o], [v[o] for v in k]
        t = tc - k[0] - SX * (k[2] + SZ * k[1])
        out[i, : len(order)] = np.minimum(j + delta[t], 0xFFFF)
    return out, totals


def gpu_brick_lists(sim):
    """GPU brick-local lists as [n, M] int64 (tile and group layout undone),
    -1 past each list."""
    n, M = sim.n, sim.max_neibs
    G = -(-M // 8)
    E = -(-sim.capacity // 64) * 64 * 8 * G   # the lists; the table of bricks with a pair follows
    t = sim.neibs_brick[:E].view(-1, G, 64, 8).cpu().numpy().view(np.uint16)  # [tile, group, lane, 8]
    L = t.transpose(0, 2, 1, 3).reshape(-1, G * 8)[:n, :M].astype(np.int64)
    cnt = sim.neib_count[:n].cpu().numpy().view(np.uint32).astype(np.int64)
    tot = (cnt & 0xFFFF) + (cnt >> 16)
    return np.where(np.arange(M)[None, :] < tot[:, None], L, -1)
