"""The work that a user of this solver has it do, as cases that can be timed and compared.

A program around the solver assembles the stiffness matrix of a cracked body, builds a
handle, and then applies operators, solves for load cases, solves many bodies together,
or alternates value updates, forward and adjoint solves.  `prepare` makes such a
program's inputs on the GPU, `run` is its call.

The bodies are hex8 meshes of the unit cube with ne elements per axis, clamped at the
bottom and loaded by seeded tractions on the top face, with a planar edge crack or a bent
penny crack (Heaviside and branch enrichment), element moduli exp(sigma g) with seeded
normal g, and rigid-body deflation vectors per subdomain, enriched ones included: the
shapes, sizes and distributions of this repository's own workloads.  A case's mesh,
pattern and Z are fixed by its sizes; the seed gives the moduli and the loads.

Solves run to a relative residual of 1e-12, the tight tolerance the repository's own
gradient and accuracy checks use: at 1e-8 the returned vector is itself only known to a
few 1e-7, so two summation orders would return vectors that cannot be compared closely.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2111_09294_amd as dpcg

DEVICE = "cuda"
TOL = 1e-12
MAX_BATCH = 32

_CORNER = np.array([[0, 0, 0], [1, 0, 0], [1, 1, 0], [0, 1, 0], [0, 0, 1], [1, 0, 1], [1, 1, 1], [0, 1, 1]])
_LAM, _MU = 0.3 / (1.3 * 0.4), 0.5 / 1.3     # Lame constants for E = 1, nu = 0.3


# ------------------------------------------------------------------------------- cases
def listed():
    return [
        # one preconditioner application on the smallest body: a program that runs its own
        # outer iteration, where latency and launches are all there is
        dict(name="precond_10", kind="precond", ne=10, crack="edge", sigma=0.5),
        # one product with K at the largest size, the dominant step of every iteration
        dict(name="product_80", kind="product", ne=80, crack="penny", sigma=0.5, stored="fp64"),
        # another load case on a handle that is kept: the smallest body, and an ordinary one
        dict(name="solve_10", kind="solve", ne=10, crack="edge", sigma=0.5, precision="fp64"),
        dict(name="solve_40", kind="solve", ne=40, crack="penny", sigma=0.5, precision="fp64"),
        # the mixed-precision solve, where K no longer fits the last-level cache; odd size
        dict(name="mixed_61", kind="solve", ne=61, crack="penny", sigma=0.5, precision="mixed"),
        # a new body: set up, solved once and released, as each step of a propagation run is
        dict(name="step_23", kind="step", ne=23, crack="penny", sigma=0.5, blocks="nodal"),
        # the headline workload: 1.66M unknowns, set up and solved
        dict(name="step_80", kind="step", ne=80, crack="penny", sigma=0.0, blocks="nodal"),
        # subdomain-sized block-Jacobi blocks, the paper's own variant
        dict(name="subdomains_21", kind="step", ne=21, crack="penny", sigma=0.5, blocks="subdomain"),
        # independent bodies of uneven sizes solved together
        dict(name="many_20x9", kind="many", ne=20, systems=9, step=2, crack="penny", sigma=0.5),
        # load cases together: a full batch, and the few load cases of an ordinary analysis
        dict(name="loads_40x32", kind="loads", ne=40, crack="penny", sigma=0.5, nrhs=32),
        dict(name="loads_21x6", kind="loads", ne=21, crack="penny", sigma=0.5, nrhs=6),
        # one step of an inverse problem: new moduli, forward and adjoint solve, gradient
        dict(name="inverse_30", kind="inverse", ne=30, crack="penny", sigma=0.5),
    ]


def draw(rng):
    """One more case: a kind of call, and sizes spread over its range by their logarithm."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["precond", "product", "solve", "solve", "step", "step", "loads", "inverse", "many"])
    c = dict(kind=kind, crack=rng.choice(["edge", "penny", "penny"]), sigma=round(max(0.0, rng.uniform(-0.1, 0.6)), 3))
    if kind == "precond":
        c["ne"] = size(8, 30)
    elif kind == "product":
        c.update(ne=size(10, 80), stored=rng.choice(["fp64", "fp32"]))
    elif kind == "solve":
        c.update(ne=size(8, 64), precision=rng.choice(["fp64", "fp64", "mixed"]))
    elif kind == "step":
        c["blocks"] = rng.choice(["nodal", "nodal", "subdomain"])
        c["ne"] = size(8, 64) if c["blocks"] == "nodal" else size(8, 21)
    elif kind == "loads":
        c.update(ne=size(8, 40), nrhs=rng.randint(2, MAX_BATCH))
    elif kind == "inverse":
        c["ne"] = size(8, 36)
    else:
        c.update(ne=size(10, 30), systems=rng.randint(3, 12), step=rng.randint(1, 3))
    return c


def _sizes(case):
    """Mesh sizes of a case: one, or those of the bodies solved together."""
    if case["kind"] != "many":
        return [case["ne"]]
    return [max(8, case["ne"] + case["step"] * (i % 7 - 3)) for i in range(case["systems"])]


# ---------------------------------------------------------------------------- geometry
def _gauss(npt):
    x, w = np.polynomial.legendre.leggauss(npt)
    X = np.stack(np.meshgrid(x, x, x, indexing="ij"), -1).reshape(-1, 3)
    return X, np.einsum("i,j,k->ijk", w, w, w).reshape(-1)


def _shape(xi):
    s = 2.0 * _CORNER - 1.0
    f = 1.0 + xi[:, None, :] * s[None]
    dN = np.stack([s[None, :, 0] * f[..., 1] * f[..., 2], s[None, :, 1] * f[..., 0] * f[..., 2],
                   s[None, :, 2] * f[..., 0] * f[..., 1]], -1) / 8.0
    return f.prod(-1) / 8.0, dN


class _Crack:
    """Planar edge crack x = 0.5, z < 0.45, or a penny crack of radius 0.25 bent into
    z = 0.5 + 0.3 rho^2; coordinates are tensors (..., 3)."""

    def __init__(self, kind):
        self.edge = kind == "edge"
        self.c, self.R = 0.3, 0.25
        self.zf, self.s = 0.5 + self.c * self.R ** 2, 2 * self.c * self.R

    def _polar(self, X):
        dx, dy = X[..., 0] - 0.5, X[..., 1] - 0.5
        return dx, dy, torch.sqrt(dx * dx + dy * dy)

    def level(self, X):
        if self.edge:
            return X[..., 0] - 0.5
        rho = self._polar(X)[2]
        return X[..., 2] - 0.5 - self.c * rho * rho

    def faces(self, X):
        return X[..., 2] < 0.45 if self.edge else self._polar(X)[2] < self.R

    def tip(self, X):
        """Distances (phi, psi) from the crack's surface and its front, with gradients."""
        if self.edge:
            g = torch.zeros_like(X)
            h = torch.zeros_like(X)
            g[..., 0], h[..., 2] = 1.0, 1.0
            return X[..., 0] - 0.5, X[..., 2] - 0.45, g, h
        dx, dy, rho = self._polar(X)
        c, one = self.c, torch.ones_like(dx)
        g = self.level(X)
        a = torch.sqrt(1.0 + 4 * c * c * rho * rho)
        ga = torch.stack([4 * c * c * dx, 4 * c * c * dy, 0 * one], -1) / a[..., None]
        gphi = torch.stack([-2 * c * dx, -2 * c * dy, one], -1) / a[..., None] - (g / (a * a))[..., None] * ga
        nrm = math.sqrt(1.0 + self.s ** 2)
        rs = torch.where(rho > 0, rho, one)
        gpsi = torch.stack([dx / rs, dy / rs, self.s * one], -1) / nrm
        return g / a, ((rho - self.R) + self.s * (X[..., 2] - self.zf)) / nrm, gphi, gpsi

    def front(self, h):
        if self.edge:
            y = np.linspace(0.0, 1.0, int(16 / h) + 2)
            return np.stack([np.full_like(y, 0.5), y, np.full_like(y, 0.45)], -1)
        t = np.linspace(0.0, 2 * math.pi, int(2 * math.pi * self.R * 16 / h) + 2, endpoint=False)
        return np.stack([0.5 + self.R * np.cos(t), 0.5 + self.R * np.sin(t), np.full_like(t, self.zf)], -1)


def _branch(phi, psi, gphi, gpsi):
    """The four crack-tip functions of (r, theta) and their gradients."""
    r, th = torch.sqrt(phi * phi + psi * psi), torch.atan2(phi, psi)
    sr, s2, c2, st, ct = torch.sqrt(r), torch.sin(th / 2), torch.cos(th / 2), torch.sin(th), torch.cos(th)
    F = torch.stack([sr * s2, sr * c2, sr * s2 * st, sr * c2 * st], -1)
    rs = torch.where(r > 0, r, torch.ones_like(r))
    dr = torch.stack([s2, c2, s2 * st, c2 * st], -1) / (2.0 * torch.sqrt(rs))[..., None]
    dt = torch.stack([c2 / 2, -s2 / 2, c2 / 2 * st + s2 * ct, -s2 / 2 * st + c2 * ct], -1) * sr[..., None]
    gr = (phi[..., None] * gphi + psi[..., None] * gpsi) / rs[..., None]
    gt = (psi[..., None] * gphi - phi[..., None] * gpsi) / (rs * rs)[..., None]
    return F, dr[..., None] * gr[..., None, :] + dt[..., None] * gt[..., None, :]


def _stiffness(G, w):
    """(e, 3m, 3m) matrices of m scalar functions per element with gradients G (e, g, m, 3)."""
    e, g, m, _ = G.shape
    A = (G * torch.sqrt(w)[None, :, None, None]).reshape(e, g, 3 * m)
    M = torch.bmm(A.transpose(1, 2).contiguous(), A).reshape(e, m, 3, m, 3)
    tr = M.diagonal(dim1=2, dim2=4).sum(-1)
    K = _LAM * M + _MU * M.transpose(2, 4)
    K = K + _MU * tr[:, :, None, :, None] * torch.eye(3, dtype=M.dtype, device=M.device)[None, None, :, None, :]
    return (0.5 * (K + K.permute(0, 3, 4, 1, 2))).reshape(e, 3 * m, 3 * m)


class _Body:
    """Everything of a body that its mesh fixes: the pattern of K, Z, the block partition
    and the element matrices at unit modulus.  Slots of a node: displacement, Heaviside,
    four branch functions."""

    def __init__(self, ne, crack, blocks):
        t = lambda a: torch.as_tensor(a, device=DEVICE)  # noqa: E731
        self.ne, self.n1, h = ne, ne + 1, 1.0 / ne
        n1, nn, nel = ne + 1, (ne + 1) ** 3, ne ** 3
        i = np.arange(nn)
        ijk = np.stack([i % n1, i // n1 % n1, i // n1 ** 2], -1)
        e = np.arange(nel)
        eijk = np.stack([e % ne, e // ne % ne, e // ne ** 2], -1)
        lin = np.array([1, n1, n1 * n1])
        self.conn = eijk @ lin
        self.conn = self.conn[:, None] + (_CORNER @ lin)[None]
        X, free = ijk * h, ijk[:, 2] > 0
        cr = _Crack(crack)
        self._enrich(cr, t, X, eijk, free, h)

        nsd = max(2, int(round(ne / 10)))
        sub = np.clip(-(-ijk * nsd // ne) - 1, 0, nsd - 1) @ np.array([1, nsd, nsd * nsd])
        nodes = np.nonzero(free)[0]
        if blocks == "subdomain":      # unknowns numbered subdomain by subdomain
            nodes = nodes[np.argsort(sub[nodes], kind="stable")]
        ngrp = np.where(free, 1 + self.H + 4 * self.T, 0)
        start = np.zeros(nn, np.int64)
        start[nodes] = np.cumsum(ngrp[nodes]) - ngrp[nodes]
        self.start, self.ngrp, self.nodes = start, ngrp, nodes
        self.ntrip = int(ngrp.sum())
        self.n = 3 * self.ntrip
        sizes = 3 * ngrp[nodes] if blocks == "nodal" else 3 * np.bincount(sub[nodes], weights=ngrp[nodes])
        sizes = sizes[sizes > 0].astype(np.int64)
        self.bj_values = int((sizes ** 2).sum())
        self.block_ptr = t(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32))

        self._pattern(t, ijk, free)
        self._element_matrices(cr, t, X, eijk, h)
        self._deflation(t, X, sub)
        top = np.nonzero((ijk[:, 2] == ne) & free)[0]
        edge = lambda v: np.where((v == 0) | (v == ne), 0.5, 1.0)  # noqa: E731
        self.top = t(3 * start[top])
        self.area = t(edge(ijk[top, 0]) * edge(ijk[top, 1]) * h * h)

    def _enrich(self, cr, t, X, eijk, free, h):
        """Node sets: H (support cut by the crack) and T (near its front), as 0 / 1."""
        ne, nn = self.ne, len(X)
        P = cr.front(h)
        near = np.zeros(ne ** 3, bool)
        for d in np.array(np.meshgrid([-1, 1], [-1, 1], [-1, 1])).reshape(3, -1).T:
            q = np.floor((P + 1e-9 * d) / h).astype(np.int64)
            q = q[((q >= 0) & (q < ne)).all(1)]
            near[q @ np.array([1, ne, ne * ne])] = True
        xi, wq = _gauss(8)
        centre = t((eijk + 0.5) * h)
        level = cr.level(centre)
        above = (level >= 0).double()
        band = torch.nonzero(level.abs() < 2 * h)[:, 0]
        for ids in band.split(8192):
            pts = t(eijk * h)[ids][:, None, :] + t((xi + 1) * (h / 2))[None]
            above[ids] = ((cr.level(pts) >= 0).double() * t(wq / wq.sum())[None]).sum(1)
        above = above.cpu().numpy()
        pos, cnt, tip = np.zeros(nn), np.zeros(nn), np.zeros(nn, bool)
        for a in range(8):      # a corner's nodes are distinct over the elements
            pos[self.conn[:, a]] += above
            cnt[self.conn[:, a]] += 1
            tip[self.conn[:, a]] |= near
        phi, psi, _, _ = cr.tip(t(X))
        r = torch.sqrt(phi * phi + psi * psi).cpu().numpy()
        frac = pos / cnt
        self.sign = np.where(cr.level(t(X)).cpu().numpy() >= 0, 1.0, -1.0)
        self.H = ((np.minimum(frac, 1 - frac) >= 1e-3) & ~tip & cr.faces(t(X)).cpu().numpy() & free).astype(np.int64)
        self.T = ((tip | (r <= max(0.05, 1.2 * h) * (1 + 1e-9))) & free).astype(np.int64)

    def _pattern(self, t, ijk, free):
        """Block and scalar pattern of K: every pair of functions of neighbouring nodes."""
        n1, nodes = self.n1, self.nodes
        node_of = np.repeat(nodes, self.ngrp[nodes])                 # per triplet
        pos = np.arange(self.ntrip) - self.start[node_of]
        slot = np.where((pos > 0) & (self.H[node_of] == 0), pos + 1, pos)
        off = np.stack(np.meshgrid([-1, 0, 1], [-1, 0, 1], [-1, 0, 1], indexing="ij")[::-1], -1).reshape(27, 3)
        q = t(ijk)[t(node_of)][:, None, :] + t(off)[None]
        ok = ((q >= 0) & (q < n1)).all(-1)
        nb = torch.where(ok, (q * t(np.array([1, n1, n1 * n1]))).sum(-1), 0)
        ok &= t(free)[nb]
        cnt = torch.where(ok, t(self.ngrp)[nb], 0).reshape(-1)
        first = (torch.cumsum(cnt, 0) - cnt).reshape(-1, 27)
        cell = torch.repeat_interleave(torch.arange(len(cnt), device=cnt.device), cnt)
        tt = torch.arange(len(cell), device=cnt.device) - first.reshape(-1)[cell]
        row, o = cell // 27, cell % 27
        J = nb.reshape(-1)[cell]
        col = t(self.start)[J] + tt
        mirror = first[col, 26 - o] + t(pos)[row]
        # where each block's value stands: the 27-point stencil of a node, or the dense
        # table of a node of an enriched element
        enr = ((self.H + self.T) > 0)[self.conn].any(1)
        self.enr = np.nonzero(enr)[0]
        near = np.zeros(len(ijk), bool)
        near[self.conn[self.enr].reshape(-1)] = True
        self.nenr = int(near.sum())
        self.enr_id = np.where(near, np.cumsum(near) - 1, 0)
        I, s = t(node_of)[row], t(slot)[row]
        s2 = t(slot)[col]
        plain = (s == 0) & (s2 == 0)
        self.src_plain = torch.nonzero(plain)[:, 0]
        self.src_enr = torch.nonzero(~plain)[:, 0]
        self.at_plain = (I * 27 + o)[self.src_plain]
        self.at_enr = (((t(self.enr_id)[I] * 27 + o) * 6 + s) * 6 + s2)[self.src_enr]
        deg = cnt.reshape(-1, 27).sum(1)
        bptr = torch.cat([deg.new_zeros(1), torch.cumsum(deg, 0)])
        self.nnzb = len(col)
        # renumbered bodies: columns in increasing order (first and mirror follow)
        order = torch.argsort(row * self.ntrip + col)
        place = torch.empty_like(order)
        place[order] = torch.arange(len(order), device=order.device)
        self.src_plain, self.src_enr = place[self.src_plain], place[self.src_enr]
        row, col, self.mirror = row[order], col[order], place[mirror[order]]
        self.rowptr = torch.cat([deg.new_zeros(1), torch.cumsum(3 * torch.repeat_interleave(deg, 3), 0)])
        self.nnz = 9 * self.nnzb
        inrow = 3 * (torch.arange(self.nnzb, device=row.device) - bptr[row])
        self.at = (self.rowptr[3 * row][:, None] + torch.arange(3, device=row.device) * 3 * deg[row][:, None]
                   + inrow[:, None])                                  # (nnzb, 3): scalar row starts
        self.col = torch.empty(self.nnz, dtype=torch.int32, device=row.device)
        for j in range(3):
            self.col[self.at + j] = (3 * col + j).int()[:, None].expand(-1, 3)

    def _element_matrices(self, cr, t, X, eijk, h):
        xi, wq = _gauss(2)
        G = t(_shape(xi)[1] * (2 / h))[None]
        self.k0 = _stiffness(G, t(wq * (h / 2) ** 3))[0]              # (24, 24)
        xi, wq = _gauss(8)
        N, dN = (t(v) for v in _shape(xi))
        gN, w = dN * (2 / h), t(wq * (h / 2) ** 3)
        out = []
        for ids in np.array_split(self.enr, max(1, len(self.enr) // 512)):
            if not len(ids):
                continue
            nd = self.conn[ids]
            P = t(eijk[ids] * h)[:, None, :] + t((xi + 1) * (h / 2))[None]
            Hg = torch.where(cr.level(P) >= 0, 1.0, -1.0)
            F, gF = _branch(*cr.tip(P))
            Fn, _ = _branch(*cr.tip(t(X[nd])))
            G = torch.zeros(len(ids), len(xi), 8, 6, 3, dtype=torch.float64, device=DEVICE)
            G[:, :, :, 0] = gN[None]
            G[:, :, :, 1] = gN[None] * ((Hg[:, :, None] - t(self.sign[nd])[:, None, :]) * t(self.H[nd])[:, None])[..., None]
            sh = (F[:, :, None, :] - Fn[:, None, :, :]) * t(self.T[nd])[:, None, :, None]
            gFa = gF[:, :, None] * t(self.T[nd])[:, None, :, None, None]
            G[:, :, :, 2:] = gN[None, :, :, None] * sh[..., None] + N[None, :, :, None, None] * gFa
            K = _stiffness(G.reshape(len(ids), len(xi), 48, 3), w).reshape(-1, 8, 6, 3, 8, 6, 3)
            K[:, :, 0, :, :, 0, :] = self.k0.reshape(8, 3, 8, 3)
            out.append(K)
        self.kenr = torch.cat(out) if out else torch.zeros(0, 8, 6, 3, 8, 6, 3, dtype=torch.float64, device=DEVICE)

    def _deflation(self, t, X, sub):
        """Z: per subdomain rigid-body modes, their Heaviside-signed form, and one set per
        branch function; a mode that depends on those before it is left out."""
        order = self.nodes[np.argsort(sub[self.nodes], kind="stable")]
        s = np.unique(sub[order], return_inverse=True)[1]
        begin = np.searchsorted(s, np.arange(s[-1] + 1))
        c = np.add.reduceat(X[order], begin) / np.bincount(s)[:, None]
        x, y, z = (X[order] - c[s]).T
        W = np.zeros((len(order), 3, 6))
        W[:, [0, 1, 2], [0, 1, 2]] = 1.0
        W[:, 1, 3], W[:, 2, 3], W[:, 0, 4], W[:, 2, 4], W[:, 0, 5], W[:, 1, 5] = -z, y, z, -x, -y, x
        g = np.einsum("mci,mcj->mij", W, W)
        H, T, sg = self.H[order], self.T[order], self.sign[order]
        gram = lambda v: np.add.reduceat(v[:, None, None] * g, begin)  # noqa: E731
        gs, gh = gram(np.ones(len(order))), gram(1.0 * H)
        gx = gram(sg)
        both = np.block([[gs, gx], [gx, gs + gh]])
        keep = _independent(both)
        keep[:, 6:] &= np.add.reduceat(H, begin)[:, None] > 0
        keep_t = _independent(gram(1.0 * T))
        keep = np.concatenate([keep] + [keep_t] * 4, 1)                # (subdomains, 36)
        number = np.cumsum(keep.reshape(-1)).reshape(keep.shape) - 1
        self.k = int(keep.sum())
        rows, cols, vals = [], [], []

        def add(sel, trip, group, v):
            m, cc, i = np.nonzero((v != 0) & keep[s[sel]][:, None, 6 * group:6 * group + 6])
            rows.append(3 * trip[m] + cc)
            cols.append(number[s[sel]][m, 6 * group + i])
            vals.append(v[m, cc, i])

        allm, hm, tm = np.arange(len(order)), np.nonzero(H)[0], np.nonzero(T)[0]
        st = self.start[order]
        add(allm, st, 0, W)
        add(allm, st, 1, W * sg[:, None, None])
        add(hm, st[hm] + 1, 1, W[hm])
        for b in range(4):
            add(tm, st[tm] + 1 + H[tm] + b, 2 + b, W[tm])
        rows, cols, vals = (np.concatenate(v) for v in (rows, cols, vals))
        o = np.argsort(rows * np.int64(self.k) + cols)
        self.z_ptr = t(np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=self.n))]).astype(np.int64))
        self.z_col, self.z_val = t(cols[o].astype(np.int32)), t(vals[o])

    # ------------------------------------------------------------------ values of a seed
    def moduli(self, sigma, gen):
        return torch.exp(sigma * torch.randn(self.ne ** 3, generator=gen, dtype=torch.float64)).to(DEVICE)

    def values(self, E):
        """K's CSR values for the element moduli E; exactly symmetric."""
        V = torch.empty(self.nnzb, 3, 3, dtype=torch.float64, device=DEVICE)
        S = torch.zeros(self.n1 ** 3, 27, 3, 3, dtype=torch.float64, device=DEVICE)
        D = torch.zeros(self.nenr, 27, 6, 6, 3, 3, dtype=torch.float64, device=DEVICE)
        k0 = self.k0.reshape(8, 3, 8, 3)
        conn = torch.as_tensor(self.conn, device=DEVICE)
        eid = torch.as_tensor(self.enr_id, device=DEVICE)[conn[torch.as_tensor(self.enr, device=DEVICE)]]
        Ee = E[torch.as_tensor(self.enr, device=DEVICE)]
        for a in range(8):
            for b in range(8):
                o = int((_CORNER[b] - _CORNER[a] + 1) @ np.array([1, 3, 9]))
                S[conn[:, a], o] += E[:, None, None] * k0[a, :, b, :][None]
                D[eid[:, a], o] += Ee[:, None, None, None, None] * self.kenr[:, a, :, :, b].permute(0, 1, 3, 2, 4)
        V[self.src_plain] = S.reshape(-1, 3, 3)[self.at_plain]
        V[self.src_enr] = D.reshape(-1, 3, 3)[self.at_enr]
        V = 0.5 * (V + V[self.mirror].transpose(1, 2))
        out = torch.empty(self.nnz, dtype=torch.float64, device=DEVICE)
        for j in range(3):
            out[self.at + j] = V[:, :, j]
        return out

    def loads(self, nrhs, gen):
        """Tractions on the top face: i.i.d. normal components times the tributary area."""
        F = torch.zeros(self.n, nrhs, dtype=torch.float64, device=DEVICE)
        v = torch.randn(len(self.area), 3, nrhs, generator=gen, dtype=torch.float64).to(DEVICE)
        for c in range(3):
            F[self.top + c] = self.area[:, None] * v[:, c]
        return F

    def solver(self, vals):
        return dpcg.Solver(self.n, self.rowptr, self.col, vals, self.k, self.z_ptr, self.z_col, self.z_val,
                           self.block_ptr)

    @functools.cached_property
    def element_data(self):
        """(elem_ptr, elem_dof, kmat_off, kmat, plain elements): unit-modulus matrices."""
        nel = self.ne ** 3
        trip = np.where(self.ngrp[self.conn] > 0, self.start[self.conn], -1)
        dofs = list(np.where(trip[:, :, None] >= 0, 3 * trip[:, :, None] + np.arange(3), -1).reshape(nel, 24))
        off, mats, end = np.zeros(nel, np.int64), [self.k0.reshape(-1)], 576
        slots = np.stack([np.ones_like(self.H), self.H] + [self.T] * 4, 1).astype(bool)
        for i, e in enumerate(self.enr):
            nd = self.conn[e]
            has = slots[nd] | (np.arange(6) == 0)[None]
            rank = np.cumsum(has, 1) - 1
            tr = np.where(self.ngrp[nd][:, None] > 0, self.start[nd][:, None] + rank, -1)[has]
            dofs[e] = np.where(tr[:, None] >= 0, 3 * tr[:, None] + np.arange(3), -1).reshape(-1)
            sel = torch.as_tensor(np.nonzero(np.repeat(has.reshape(-1), 3))[0], device=DEVICE)
            mats.append(self.kenr[i].reshape(144, 144)[sel][:, sel].reshape(-1))
            off[e] = end
            end += len(sel) ** 2
        ptr = np.concatenate([[0], np.cumsum([len(d) for d in dofs])]).astype(np.int64)
        return ptr, np.concatenate(dofs).astype(np.int32), off, torch.cat(mats)


def _independent(G):
    """Columns kept by in-order Cholesky of the Gram matrices G (s, m, m)."""
    s, m, _ = G.shape
    L, keep = np.zeros_like(G), np.zeros((s, m), bool)
    for j in range(m):
        v = G[:, :, j] - np.einsum("sik,sk->si", L, L[:, j])
        keep[:, j] = v[:, j] > 1e-10 * G[:, j, j]
        d = np.sqrt(np.where(keep[:, j], v[:, j], 1.0))
        L[:, :, j] = np.where(keep[:, j, None], v / d[:, None], 0.0)
        L[:, :j, j] = 0.0
    return keep


@functools.lru_cache(maxsize=16)
def _body(ne, crack, blocks):
    return _Body(ne, crack, blocks)


def _bodies(case):
    return [_body(ne, case["crack"], case.get("blocks", "nodal")) for ne in _sizes(case)]


# ------------------------------------------------------------------------ the interface
def _inputs(case, seed):
    """(body, CSR values, right-hand sides) of each body of the case, and its generator."""
    gen = torch.Generator().manual_seed(int(seed))
    out = []
    for b in _bodies(case):
        vals = b.values(b.moduli(case["sigma"], gen))
        if case["kind"] in ("precond", "product"):
            F = torch.randn(b.n, 1, generator=gen, dtype=torch.float64).to(DEVICE)
        else:
            F = b.loads(case.get("nrhs", 1), gen)
        out.append((b, vals, F if case["kind"] == "loads" else F[:, 0].contiguous()))
    return out, gen


def prepare(case, seed):
    made, gen = _inputs(case, seed)
    state = dict(kind=case["kind"], case=case, made=made)
    if case["kind"] != "step":
        state["solvers"] = [b.solver(v) for b, v, _ in made]
    if case["kind"] == "inverse":
        b = made[0][0]
        ptr, dof, off, kmat = b.element_data
        state["elements"] = dpcg.Elements(ptr, dof, off, kmat, device=DEVICE)
        state["moduli"] = b.moduli(case["sigma"], gen)
        state["vals"] = b.values(state["moduli"])
        state["loss"] = _loss_gradient(b)
    return state


def _loss_gradient(b):
    """Gradient of the loss of the inverse problem: the sum of the vertical displacements
    of the mesh's plain nodes, each weighted by its height."""
    g = torch.zeros(b.n, dtype=torch.float64, device=DEVICE)
    height = torch.as_tensor(b.nodes // b.n1 ** 2 / b.ne, dtype=torch.float64, device=DEVICE)
    g[torch.as_tensor(3 * b.start[b.nodes] + 2, device=DEVICE)] = height / len(b.nodes)
    return g


def run(state):
    kind, case = state["kind"], state["case"]
    b, vals, f = state["made"][0]
    if kind == "step":
        with b.solver(vals) as s:
            return s.solve(f, tol=TOL)[0]
    s = state["solvers"][0]
    if kind == "precond":
        return s.precond(f)
    if kind == "product":
        return s.spmv(f) if case["stored"] == "fp64" else s.spmv_fp32(f)
    if kind == "solve":
        return s.solve(f, tol=TOL, precision=case["precision"])[0]
    if kind == "loads":
        return s.solve_batch(f, tol=TOL)[0]
    if kind == "many":
        return dpcg.solve_many(state["solvers"], [m[2] for m in state["made"]], tol=TOL)[0]
    s.update_values(b.rowptr, b.col, state["vals"])
    u = s.solve(f, tol=TOL)[0]
    lam = s.solve_adjoint(state["loss"], tol=TOL)[0]
    return dict(u=u, adjoint=lam, gradient=s.element_gradient(state["elements"], u, lam))


def _iterations(case, ne):
    """Iterations of a solve to TOL, fitted to measured counts (for the estimate of work)."""
    return (75.0 + 2.9 * ne) * (0.6 if case.get("blocks") == "subdomain" else 1.0)


def work(case):
    """Every operator once per application, K and the inverses by one triangle (they are
    symmetric), and the vectors of the recurrence read and written once."""
    bytes_, flops = 0.0, 0.0
    for b in _bodies(case):
        blocks = (b.nnzb + b.ntrip) / 2
        kb, kf = 76.0 * blocks, 18.0 * b.nnzb
        mb, mf = 4.0 * b.bj_values, 2.0 * b.bj_values
        nz = len(b.z_val)
        pb, pf = mb + 12.0 * nz + 4.0 * b.k ** 2, mf + 4.0 * nz + 2.0 * b.k ** 2
        vec = 8.0 * b.n
        if case["kind"] == "product":
            half = case["stored"] == "fp32"
            bytes_, flops = bytes_ + (40.0 * blocks if half else kb) + 2 * vec, flops + kf
            continue
        if case["kind"] == "precond":
            bytes_, flops = bytes_ + pb + 2 * vec, flops + pf
            continue
        cols = case.get("nrhs", 1) * (2 if case["kind"] == "inverse" else 1)
        passes = 2 if case["kind"] == "inverse" else 1
        if case["kind"] == "solve" and case["precision"] == "mixed":
            kb = 40.0 * blocks
        its = _iterations(case, b.ne)
        bytes_ += its * (passes * (kb + pb) + cols * 8 * vec)
        flops += its * cols * (kf + pf + 12.0 * b.n)
        if case["kind"] in ("step", "inverse"):      # reading K, and inverting the coarse matrix
            bytes_ += 12.0 * b.nnz
            flops += 1.0 * b.k ** 3
    return {"bytes": bytes_, "flops": flops}


# ------------------------------------------------------------- what 64-bit torch gives
def _csr(b, vals):
    return torch.sparse_csr_tensor(b.rowptr, b.col.long(), vals, size=(b.n, b.n))


def _block_inverses(b, vals):
    """[(DoFs (m, s), inverses (m, s, s))] of the nodal blocks, grouped by size."""
    K = _csr(b, vals)
    out = []
    for size in (3, 6, 15, 18):
        first = torch.as_tensor(3 * b.start[b.nodes[3 * b.ngrp[b.nodes] == size]], device=DEVICE)
        if not len(first):
            continue
        dofs = first[:, None] + torch.arange(size, device=DEVICE)
        A = torch.zeros(len(first), size, size, dtype=torch.float64, device=DEVICE)
        for r in range(size):
            # each row's entries inside its own block are consecutive columns
            lo, hi = K.crow_indices()[dofs[:, r]], K.crow_indices()[dofs[:, r] + 1]
            a = lo.clone()
            z = hi.clone()
            while bool((a < z).any()):
                mid = (a + z) // 2
                less = b.col[mid.clamp(max=b.nnz - 1)].long() < first
                a, z = torch.where((a < z) & less, mid + 1, a), torch.where((a < z) & ~less, mid, z)
            A[:, r] = vals[a[:, None] + torch.arange(size, device=DEVICE)]
        out.append((dofs, torch.linalg.inv(A)))
    return out


def _block_apply(inverses, r):
    y = torch.empty_like(r)
    for dofs, inv in inverses:
        y[dofs.reshape(-1)] = torch.matmul(inv, r[dofs.reshape(-1)].reshape(len(dofs), -1, r.shape[1])).reshape(-1, r.shape[1])
    return y


def _solve(b, vals, F):
    """K^-1 F (n x m) by conjugate gradients with nodal blocks, restarted on the true residual."""
    K, inv = _csr(b, vals), _block_inverses(b, vals)
    u = torch.zeros_like(F)
    norm = F.norm(dim=0)
    for _ in range(4):
        r = F - K @ u
        if bool((r.norm(dim=0) <= 2e-14 * norm).all()):
            break
        x, p, z = torch.zeros_like(r), None, _block_apply(inv, r)
        rho = (r * z).sum(0)
        goal = 1e-13 * norm
        for i in range(20000):
            p = z if p is None else z + beta * p
            q = K @ p
            alpha = rho / (p * q).sum(0).clamp(min=1e-300)
            x, r = x + alpha * p, r - alpha * q
            if i % 50 == 49 and bool((r.norm(dim=0) <= goal).all()):
                break
            z = _block_apply(inv, r)
            new = (r * z).sum(0)
            beta, rho = new / rho.clamp(min=1e-300), new
        u = u + x
    return u


def exact(case, seed):
    made, gen = _inputs(case, seed)
    kind = case["kind"]
    b, vals, f = made[0]
    if kind == "product":
        v = vals if case["stored"] == "fp64" else vals.float().double()
        return _csr(b, v) @ f
    if kind == "precond":
        y = _block_apply(_block_inverses(b, vals), f[:, None])
        Zs = torch.sparse_csr_tensor(b.z_ptr, b.z_col.long(), b.z_val, size=(b.n, b.k))
        Z = Zs.to_dense()
        K = _csr(b, vals)
        KZ = torch.cat([K @ c.contiguous() for c in Z.split(256, 1)], 1)
        E = Z.t() @ KZ
        E = 0.5 * (E + E.t())
        scale = E.diagonal().rsqrt()
        L = torch.linalg.cholesky((scale[:, None] * E * scale).cpu())
        g = (Z.t() @ (f[:, None] - K @ y)).cpu() * scale.cpu()[:, None]
        d = torch.cholesky_solve(g, L).to(DEVICE) * scale[:, None]
        return (y + Z @ d)[:, 0]
    if case["ne"] > 64:
        return None      # a plain solve of this size takes too long
    if kind == "loads":
        return _solve(b, vals, f)
    if kind == "many":
        return [_solve(bb, v, ff[:, None])[:, 0] for bb, v, ff in made]
    if kind == "inverse":
        E = b.moduli(case["sigma"], gen)
        vals = b.values(E)
        u = _solve(b, vals, torch.stack([f, _loss_gradient(b)], 1))
        return dict(u=u[:, 0].contiguous(), adjoint=u[:, 1].contiguous(), gradient=_gradient(b, u[:, 0], u[:, 1]))
    return _solve(b, vals, f[:, None])[:, 0]


def _gradient(b, u, lam):
    """-lam_e^T K_e u_e of every element."""
    pad = lambda v: torch.cat([v, v.new_zeros(1)])  # noqa: E731
    ptr, dof, off, kmat = b.element_data
    d = torch.as_tensor(dof.astype(np.int64), device=DEVICE)
    ue, le = pad(u)[d], pad(lam)[d]            # DoF -1 reads the zero at the end
    g = torch.empty(b.ne ** 3, dtype=torch.float64, device=DEVICE)
    plain = np.ones(b.ne ** 3, bool)
    plain[b.enr] = False
    ids = torch.as_tensor(np.nonzero(plain)[0], device=DEVICE)
    at = torch.as_tensor(ptr[:-1][plain], device=DEVICE)[:, None] + torch.arange(24, device=DEVICE)
    g[ids] = -((ue[at] @ b.k0) * le[at]).sum(1)
    for e in b.enr:
        s, m = slice(ptr[e], ptr[e + 1]), int(ptr[e + 1] - ptr[e])
        g[e] = -(le[s] @ (kmat[off[e]:off[e] + m * m].reshape(m, m) @ ue[s]))
    return g
