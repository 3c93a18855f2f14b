"""Index emulation of the marching two-step kernel (csrc/march.h) on the CPU:
every thread's offsets as the kernel computes them, on tagged values.

For every tile, plane and pass it checks that all offsets lie inside the
population plane, the slab and the phi ring, that each ring value read is the
perturbation of the wanted cell, that an interior cell takes each direction's
value from the cell it streams from, that lanes without a cell store nothing,
and that every slot of the second array is written exactly once per launch.
"""
import numpy as np
import pytest

D3Q19 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1),
         (0, 1, 1), (0, 1, -1)]
D3Q19 += [tuple(-a for a in v) for v in D3Q19[1:]]
D3Q27 = D3Q19[:10] + [(1, 1, 1), (1, 1, -1), (1, -1, 1), (1, -1, -1)]
D3Q27 += [tuple(-a for a in v) for v in D3Q27[1:]]
RING = 4


def passes(nx, rows, nt):
    """(ipt, hpt, ppt) of march_tile."""
    return tuple(-(-nx * r // nt) for r in (rows, rows + 2, rows + 4))


def check(nx, ny, nz, rows, planes, lat, nt, shape=None):
    ipt, hpt, ppt = shape or passes(nx, rows, nt)
    Q, nxy = len(lat), nx * ny
    moving = [i for i, c in enumerate(lat) if c[0] or c[1]]
    slot_of = {i: n for n, i in enumerate(moving)}
    SP = ipt * nt
    fnyb, nzb = -(-ny // rows), -(-nz // planes)
    tid = np.arange(nt)
    wbase = tid & ~63
    written = np.zeros((Q, nz * nxy), dtype=int)

    def wrap(v, n):
        return np.where(v < 0, v + n, np.where(v >= n, v - n, v))

    def code(i, cell):  # a post-collision value of direction i
        return cell * Q + i

    for b in range(fnyb * nzb):
        bz, yb = divmod(b, fnyb)
        y0 = yb * rows
        TY = min(rows, ny - y0)
        NI, RC, PC = nx * TY, nx * (TY + 2), nx * (TY + 4)
        z0, z1 = bz * planes, min(bz * planes + planes, nz)
        off, sp, xm, xp, rr = [], [], [], [], []
        for h in range(hpt):
            idx = np.minimum(tid + h * nt, RC - 1)
            e = idx - NI
            r = np.where(idx < NI, idx // nx, np.where(e < nx, -1, TY))
            x = np.where(idx < NI, idx % nx, np.where(e < nx, e, e - nx))
            assert (0 <= x).all() and (x < nx).all()
            y = wrap(y0 + r, ny)
            off.append(y * nx + x)
            assert (0 <= off[h]).all() and (off[h] < nxy).all()
            sp.append(r * nx + x)
            xm.append(np.where(x == 0, nx - 1, -1))
            xp.append(np.where(x + 1 == nx, 1 - nx, 1))
            rr.append(r)
        assert RC <= hpt * nt and NI <= ipt * nt and PC <= ppt * nt
        sr, so = [], []
        for k in range(ipt):
            own = tid + k * nt < NI
            sr.append(np.where(own, sp[k], 0))
            y, x = off[k] // nx, off[k] % nx
            ys = [np.where(y == 0, ny - 1, y - 1), y, np.where(y + 1 == ny, 0, y + 1)]
            so.append([np.where(own, v * nx + x, -10 ** 9) for v in ys])
        pidx = [np.minimum(tid + j * nt, PC - 1) for j in range(ppt)]
        po = [((y0 + i // nx - 2) % ny) * nx + i % nx for i in pidx]

        ring = np.full(RING * PC, -1)
        slab = np.full((len(moving), SP), -1)

        def store_pert(plane, slot):
            for i, o in zip(pidx, po):
                assert (0 <= i).all() and (i < PC).all()
                ring[slot * PC + i] = plane * nxy + o

        def at(byte):
            assert (0 <= byte).all() and (byte < RING * PC).all()
            return ring[byte]

        def stencil(h, s0, s5, z, mask, e6=None, sm=None):
            """The perturbation of the seven cells around pass h's cells."""
            centre = sp[h] + 2 * nx
            k, x, y = s0 * PC + centre, off[h] % nx, off[h] // nx
            want = lambda X, Y, Z: (Z % nz) * nxy + (Y % ny) * nx + X % nx  # noqa: E731
            got = [at(k), at(k + xp[h]), at(k + xm[h]), at(k + nx), at(k - nx), at(s5 * PC + centre)]
            ref = [want(x, y, z), want(x + 1, y, z), want(x - 1, y, z), want(x, y + 1, z),
                   want(x, y - 1, z), want(x, y, z + 1)]
            got.append(at(sm * PC + centre) if e6 is None else e6)
            ref.append(want(x, y, z - 1))
            for g, w in zip(got, ref):
                assert (g == w)[mask].all()
            return got[0]

        pz = (z0 - 1) % nz
        nxt = lambda v: 0 if v + 1 == nz else v + 1  # noqa: E731
        prv = lambda v: nz - 1 if v == 0 else v - 1  # noqa: E731
        store_pert(prv(pz), 0)
        store_pert(pz, 1)
        store_pert(nxt(pz), 2)
        pending = nxt(nxt(pz))
        slot = 1
        up_prev, up_next, mid, zc = {}, {}, {}, [None] * ipt
        for p in range(z0 - 1, z1 + 1):
            full = p > z0
            s0, sp1, sp2, sm1 = (slot, (slot + 1) & 3, (slot + 2) & 3, (slot + 3) & 3)
            pz1 = nxt(pz)
            store_pert(pending, sp2)
            slab[:] = -1
            col = {}
            for h in range(hpt):
                on = wbase + h * nt < RC
                if not on.any():
                    continue
                stencil(h, s0, sp1, pz, on, sm=sm1)
                cell = pz * nxy + off[h]
                for i, c in enumerate(lat):
                    val = code(i, cell)
                    if i not in slot_of:
                        if h < ipt:
                            col[h, i] = val
                        continue
                    dx = xp[h] if c[0] == 1 else xm[h] if c[0] == -1 else 0
                    ok = on & (rr[h] + c[1] >= 0) & (rr[h] + c[1] < TY)
                    d = (sp[h] + c[1] * nx + dx)[ok]
                    assert (0 <= d).all() and (d < NI).all()
                    prev = slab[slot_of[i], d]
                    assert ((prev == -1) | (prev == val[ok])).all()  # repeats: the same value
                    slab[slot_of[i], d] = val[ok]
            pending = nxt(nxt(pz1))
            z = prv(pz)
            for k in range(ipt):
                own = tid + k * nt < NI
                t = {}
                for i, c in enumerate(lat):
                    if i in slot_of:
                        assert (0 <= sr[k]).all() and (sr[k] < SP).all()
                        t[i] = slab[slot_of[i], sr[k]]
                    else:
                        t[i] = col.get((k, i), np.full(nt, -1))
                x, y = off[k] % nx, off[k] // nx
                if full:
                    stencil(k, sm1, s0, z, own, e6=zc[k])
                    zc[k] = at(sm1 * PC + sp[k] + 2 * nx)
                    zs = [prv(z), z, pz]
                    for i, c in enumerate(lat):
                        w = up_prev[k, i] if c[2] == 1 else mid[k, i] if c[2] == 0 else t[i]
                        src = ((z - c[2]) % nz) * nxy + ((y - c[1]) % ny) * nx + (x - c[0]) % nx
                        assert (w == code(i, src))[own].all()
                        o = so[k][c[1] + 1] + (xp[k] if c[0] == 1 else xm[k] if c[0] == -1 else 0)
                        assert ((o >= 0) == own).all() and (o < nxy).all()
                        dest = zs[c[2] + 1] * nxy + o[own]
                        ref = ((z + c[2]) % nz) * nxy + ((y + c[1]) % ny) * nx + (x + c[0]) % nx
                        assert (dest == ref[own]).all()
                        np.add.at(written[i], dest, 1)
                else:
                    zc[k] = at(sm1 * PC + sp[k] + 2 * nx)
                for i, c in enumerate(lat):  # what waits for the next planes
                    if c[2] == 1:
                        up_prev[k, i] = up_next.get((k, i))
                        up_next[k, i] = t[i]
                    elif c[2] == 0:
                        mid[k, i] = t[i]
            pz, slot = pz1, (slot + 1) & 3
    assert (written == 1).all()


CASES = [(64, 8, 6, 4, 3, 512), (64, 9, 4, 4, 8, 512), (33, 17, 5, 5, 2, 512), (7, 5, 3, 2, 1, 512),
         (1, 1, 1, 1, 1, 512), (1, 2, 2, 1, 1, 512), (153, 7, 5, 3, 2, 512), (80, 13, 4, 6, 3, 512),
         (32, 32, 3, 22, 2, 768), (96, 13, 4, 6, 2, 768), (48, 20, 3, 14, 1, 768),
         (256, 8, 4, 4, 3, 1024), (192, 11, 3, 5, 2, 1024), (256, 4, 5, 2, 4, 512),
         (341, 5, 3, 3, 2, 1024), (150, 9, 4, 4, 2, 768), (170, 4, 3, 1, 2, 512)]


@pytest.mark.parametrize("lat", [D3Q19, D3Q27], ids=["D3Q19", "D3Q27"])
@pytest.mark.parametrize("case", CASES)
def test_march_tile_indexing(case, lat):
    check(*case[:5], lat, case[5])


def test_march_tile_indexing_in_a_batch():
    """A batch's members share the passes of the largest member's tile."""
    for nx, ny, nz, rows, planes in ((80, 7, 4, 6, 2), (33, 40, 3, 13, 2), (5, 6, 4, 6, 3)):
        check(nx, ny, nz, rows, planes, D3Q19, 512, shape=(1, 2, 4))


def test_march_tile_indexing_random():
    rng = np.random.default_rng(11)
    for _ in range(25):
        nx, ny, nz = (int(rng.integers(1, n)) for n in (200, 24, 8))
        nt = int(rng.choice([512, 768, 1024]))
        rows = int(rng.integers(1, max(2, min(ny, 2 * nt // nx - 2) + 1)))
        if nx * (rows + 2) > 3 * nt or rows > ny:
            continue
        check(nx, ny, nz, rows, int(rng.integers(1, nz + 1)), D3Q19, nt)
