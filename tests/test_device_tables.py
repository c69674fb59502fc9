"""CPU tests of the tables the kernels read (built per plan on the host, not
reachable through the C ABI): tests/c/device_tables.cpp writes them out and
they are checked here against the mechanism and the places the kernels have
in LDS.  That program is built with the standard library's bounds checks, so
an index out of range while a mechanism compiles ends it."""
import os
import subprocess

import numpy as np
import pytest

import paper_2311_14941_amd as sc
from synth.mechgen import make_mechanism

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2311_14941_amd", "csrc")

# species, reactions, pool fraction, seed, lanes of one cell
MECHS = {"14 x 16": (14, 56, 0.15, 401, 16), "30 x 32": (30, 150, 0.3, 402, 32), "24": (24, 120, 0.5, 400, 64),
         "62": (62, 900, 0.6, 1, 64), "63": (63, 400, 0.15, 400, 64), "126": (126, 2500, 0.5, 4, 64),
         "127": (127, 762, 0.15, 400, 64)}


def mechanism(key):
    ns, nr, pf, seed, lanes = MECHS.get(key) or key
    return make_mechanism(ns, nr, nr // 10, nr // 20, ["C", "H", "O", "N"], seed=seed, pool_frac=pf), lanes


@pytest.fixture(scope="module")
def tables(tmp_path_factory):
    d = tmp_path_factory.mktemp("device_tables")
    exe = str(d / "device_tables")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D_GLIBCXX_ASSERTIONS", f"-I{CSRC}", os.path.join(HERE, "c", "device_tables.cpp"),
                    os.path.join(CSRC, "mech.cpp"), os.path.join(CSRC, "sparse.cpp"), "-o", exe], check=True)

    def get(key):
        mech, lanes = mechanism(key)
        path = str(d / "mech.txt")
        with open(path, "w") as f:
            f.write(mech.to_text())
        r = subprocess.run([exe, path, str(lanes)], capture_output=True)
        assert r.returncode == 0, (r.returncode, r.stderr[-500:])
        out, b, at = {}, r.stdout, 0
        while at < len(b):
            nl = b.index(b"\n", at)
            name, kind, count = b[at:nl].decode().split()
            a = np.frombuffer(b, dtype=kind, count=int(count), offset=nl + 1)
            out[name] = a
            at = nl + 1 + a.nbytes
        return mech, lanes, out
    return get


def records(x, lanes):
    """A table's records by execution position: side slots (pair numbers),
    coefficients, enhanced species (pair numbers), reaction."""
    passes = int(x["counts"][0])
    w = x["rec"].reshape(passes, 3, lanes, 4).transpose(0, 2, 1, 3).reshape(passes * lanes, 12)
    slot = np.stack([(w[:, 6 + i // 2] >> (16 * (i % 2))) & 0xFFFF for i in range(6)], 1) / 16
    nu = np.stack([(w[:, 9] >> (2 * i)) & 3 for i in range(6)], 1)
    enh = np.stack([(w[:, 10] >> (8 * i)) & 0xFF for i in range(4)], 1)
    return slot, nu, enh, w[:, 11]


def family(t, name):
    return {k[len(name) + 1:]: v for k, v in t.items() if k.startswith(name + ".")}


@pytest.mark.parametrize("key", list(MECHS))
def test_slots_name_places_the_kernels_have(tables, key):
    """Every slot of every record names a pair the kernels have: a used one
    its species', an unused one a place that is no species' (the
    temperature's).  The sparse kernels hold a cell's lanes times its slots per
    lane of them, the dense ones a wave's."""
    mech, lanes, t = tables(key)
    N, R, n = (int(v) for v in t["size"][:3])
    held = {"sparse": lanes * (1 if n <= 64 else 2), "dense": 64}
    pos = {"sparse": t["pos"], "dense": np.arange(N + 1)}
    for fam in held:
        x = family(t, fam)
        if not x:
            assert fam == "dense" and N > 63
            continue
        slot, nu, enh, orig = records(x, lanes if fam == "sparse" else 64)
        assert slot.max() < held[fam] and enh.max() < held[fam]
        assert np.all(slot[nu == 0] >= N) and np.all(slot[nu > 0] < N)
        assert sorted(orig[:R]) == list(range(R)) and np.all(nu[R:] == 0)
        for q in range(R):
            r = mech.reactions[orig[q]]
            for i, side in enumerate((r.reac, r.prod)):
                got = {int(s): int(v) for s, v in zip(slot[q, 3 * i:3 * i + 3], nu[q, 3 * i:3 * i + 3]) if v}
                want = {}
                for s, v in side:
                    k = int(pos[fam][s])
                    want[k] = want.get(k, 0) + v
                assert got == want, (fam, q)
            used = {int(pos[fam][k]) for k, a in r.eff.items() if a != 1.0}
            assert {int(e) for e in enh[q] if e < N} == used, (fam, q)


@pytest.mark.parametrize("key", ["24", "63", "126", "127"])
def test_row_masks_of_the_columns(key):
    """"cmask" has a bit for every row of a column, the 129th (of 127
    species) in a third word."""
    sc.ensure_built()
    m = sc.Mechanism(mechanism(key)[0].to_text())
    n = m.N + 2
    words = 3 if n > 128 else 2
    mask = m.sparse_array("cmask").reshape(n, words)
    want = np.zeros((n, words), dtype=np.uint64)
    for i, j in zip(m.sparse_array("erow"), m.sparse_array("ecol")):
        want[j, i // 64] |= np.uint64(1) << np.uint64(i % 64)
    assert np.array_equal(mask, want)


@pytest.mark.parametrize("key", list(MECHS))
def test_regions_keep_the_pairs_aligned(tables, key):
    """A cell's region in LDS holds its places, entries, the zero and the
    trash slots; regions lie one behind the other, so the size is a multiple
    of the 16 bytes the pairs are read in (also where the number of entries is
    even, as with 24 and 126 species)."""
    _, lanes, t = tables(key)
    n, nnz = int(t["size"][2]), int(t["size"][3])
    size, e0 = (int(v) for v in t["region"])
    vectors = lanes * (1 if n <= 64 else 2)
    assert size % 2 == 0 and e0 * vectors % 2 == 0
    assert e0 * vectors + nnz + 1 + 16 <= size < e0 * vectors + nnz + 1 + 16 + 32
    if lanes < 64:
        assert size % 32 == 16


def test_waves_without_a_cell_leave_or_are_waited_for(tables):
    """One slot per lane: a wave waits for the last cell while there is another
    wave (it works alone, of several), and leaves otherwise, also as the only
    wave of its workgroup.  Two slots: the workgroup leaves together."""
    for vpl, w, waves, leaves in tables("24")[2]["leaves"].reshape(-1, 4):
        assert leaves == (vpl == 2 or not (w == 1 and waves > 1)), (vpl, w, waves)


# species (mechanisms of every range of LDS regions): waves a workgroup for few
# cells and for many
CREWS = {53: (4, 4), 57: (4, 1), 62: (4, 1), 63: (2, 1), 65: (2, 1), 80: (2, 1), 90: (2, 2), 96: (2, 2), 126: (2, 2)}


@pytest.mark.parametrize("ns", list(CREWS))
def test_waves_of_a_workgroup_by_the_cells_in_flight(tables, ns):
    """Many cells: no choice of waves a workgroup keeps more cells on a CU than
    the one taken; few: the most waves.  53 species hold two workgroups of four
    waves, 57 to 62 one, three of two or seven of one; two slots per lane two
    crews or more single waves up to 52 KB a cell."""
    t = tables((ns, 6 * ns, 0.15, 400, 64))[2]
    one = int(t["size"][2]) <= 64
    groups, choice = t["crews"][:3], t["crews"][3:]
    cells = groups * (1 << np.arange(3) if one else 1)
    for k in range(3):
        if groups[k]:  # what is taken to be resident is, in pieces of 1,280 bytes
            size = 128 + 8 * int(t["region"][0]) * (1 << k if one else 1)
            assert groups[k] // 256 * -(-size // 1280) * 1280 <= 160 * 1024
    few, many = CREWS[ns]
    assert choice[0] == few and choice[-1] == many
    for n, w in zip(64 << np.arange(choice.size), choice):
        flight = np.minimum(n, cells)
        assert flight[int(w).bit_length() - 1] == flight.max(), (n, w)


@pytest.mark.parametrize("key", ["14 x 16", "30 x 32", "24", "63", "126"])
def test_component_entries(tables, key):
    """What each state component writes when the matrix is formed: its own
    entries, and trash entries (behind the zero slot) where it has none, so
    that every lane writes as many."""
    _, lanes, t = tables(key)
    N, _, n, nnz, _ = (int(v) for v in t["size"])
    entry = -np.ones((n, n), dtype=int)
    entry[t["erow"], t["ecol"]] = np.arange(nnz)
    comp = t["comp"].reshape(-1, 8).astype(int)
    T, S, k = N, N + 1, np.arange(N)
    assert comp.shape[0] == lanes * (1 if n <= 64 else 2)
    for q, e in enumerate((entry[k, k], entry[k, T], entry[k, S], entry[T, k], entry[S, k])):
        assert np.array_equal(comp[:N, q], e)
    assert comp[N, 0] == entry[T, T] and comp[N, 1] == entry[S, S]
    rest = np.concatenate([comp[N, 2:].ravel(), comp[N + 1:].ravel()])
    assert np.all((rest > nnz) & (rest <= nnz + 16))


def _entries(t):
    n, nnz = int(t["size"][2]), int(t["size"][3])
    entry = -np.ones((n, n), dtype=int)
    entry[t["erow"], t["ecol"]] = np.arange(nnz)
    return n, nnz, entry


def _numbers(a, n):
    """Entry numbers of an operand table: byte offsets up to 64 positions."""
    a = a.astype(int)
    if n > 64:
        return a
    assert np.all(a % 8 == 0)
    return a // 8


@pytest.mark.parametrize("key", list(MECHS))
@pytest.mark.parametrize("fam", ["sparse", "dense"])
def test_entries_of_the_reactions(tables, key, fam):
    """Every derivative of every reaction is added to its row's and column's
    entry where both are in use, and to a trash entry otherwise."""
    mech, lanes, t = tables(key)
    x = family(t, fam)
    if not x:
        return
    N, R, n, nnz, npad = (int(v) for v in t["size"])
    lanes = lanes if fam == "sparse" else 64
    slot, nu, enh, orig = records(x, lanes)
    passes, n_tb, _ = (int(v) for v in x["counts"])
    unpack = lambda a, w: a.reshape(-1, w, lanes, 8).transpose(0, 2, 1, 3).reshape(-1, 8 * w)
    ix, ixe = unpack(x["ix"], 6), unpack(x["ixe"], 4)
    if fam == "sparse":
        entry = _entries(t)[2]
        place = lambda r, c: entry[r, c]
        ix, ixe = _numbers(ix, n), _numbers(ixe, n)
        trash = lambda e: (e > nnz) & (e <= nnz + 16)
    else:
        place = lambda r, c: r * (npad + 1) + c
        ix, ixe = ix.astype(int) // 8, ixe.astype(int) // 8
        trash = lambda e: e % (npad + 1) == npad  # the column behind the matrix
    kinds = [mech.reactions[orig[q]].kind for q in range(R)]
    assert sum(k != "plain" for k in kinds) == n_tb and all(k != "plain" for k in kinds[:n_tb])
    for q in range(passes * lanes):
        rows = [int(slot[q, r]) if nu[q, r] else -1 for r in range(6)] + [N if q < R else -1]
        cols = [int(slot[q, s]) if nu[q, s] else -1 for s in range(6)]
        used = [int(e) if e < N and q < n_tb else -1 for e in enh[q]]
        for r in range(7):
            at = [(ix[q, 7 * r + s] if r < 6 else ix[q, 42 + s], cols[s]) for s in range(6)]
            if r < 6:
                at.append((ix[q, 7 * r + 6], N if q < R else -1))
            if q < n_tb:
                at += [(ixe[q, 4 * r + e], used[e]) for e in range(4)]
            for e, c in at:
                if rows[r] >= 0 and c >= 0:
                    assert e == place(rows[r], c) >= 0, (q, r, c)
                else:
                    assert trash(e), (q, r, c, e)


@pytest.mark.parametrize("key", ["14 x 16", "30 x 32"])
def test_rows_of_several_cells_per_wave(tables, key):
    """A lane's row of the matrix, column by column, the zero slot outside."""
    _, lanes, t = tables(key)
    n, nnz, entry = _entries(t)
    row = _numbers(t["row"], n).reshape(lanes, lanes)
    want = np.full((lanes, lanes), nnz)
    want[:n, :n] = np.where(entry >= 0, entry, nnz)
    assert np.array_equal(row, want)


def _lu_from_tables(t, E):
    """The kernels' elimination in blocks of 16 pivots, replayed from the
    operand tables alone; returns 1/u_kk."""
    n = int(t["size"][2])
    nb = (n + 15) // 16
    c, g = np.arange(64) % 16, np.arange(64) // 16
    words, at = _numbers(t["blk"], n), 0

    def take(count, per):
        nonlocal at
        w = words[at:at + count * 64 * per].reshape(count, 64, per)
        at += w.size
        return w

    dinv = np.zeros(n)
    for b in range(nb):
        r, k0 = nb - 1 - b, 16 * b
        diag = take(2, 8).transpose(1, 0, 2).reshape(64, 16)
        upper = take(2, 8).transpose(1, 0, 2).reshape(64, 16)
        ul, ab, ci = take(r, 8), take(r, 8), take(r * r, 4)
        D, u, x = E[diag], E[ul[:, :, :4]], E[ul[:, :, 4:]]
        di = np.zeros(64)
        for k in range(min(16, n - k0)):
            lead = 16 * g + k  # lane k of each row of lanes
            inv = 1.0 / D[lead, k]
            l = np.where(c > k, D[:, k] * inv, 0.0)
            di = np.where(c == k, inv, di)
            D[:, k + 1:] -= D[lead, k + 1:] * l[:, None]
            D[:, k] = np.where(c > k, l, D[:, k])
            u -= u[:, lead] * l[None, :, None]
        D *= np.where(np.arange(16)[None, :] > c[:, None], di[:, None], 1.0)
        E[diag] = D
        dinv[k0:k0 + 16] = di[:16][:n - k0]
        E[ul[:, :, :4]] = u * di[None, :, None]
        U = E[upper]
        for k in range(15):
            x -= x[:, 16 * g + k] * U[None, :, k, None]
        E[ul[:, :, 4:]] = x
        for q1 in range(r):
            for q2 in range(r):
                A, B = E[ab[q1][:, :4]], E[ab[q2][:, 4:]]
                e = ci[q1 * r + q2]
                C = np.zeros((16, 16))
                for i in range(4):
                    C[4 * i + g, c] = E[e[:, i]]
                for s in range(4):
                    As, Bs = np.zeros((16, 4)), np.zeros((4, 16))
                    As[c, g], Bs[g, c] = A[:, s], B[:, s]
                    C -= As @ Bs
                for i in range(4):
                    E[e[:, i]] = C[4 * i + g, c]
        E[ul[:, :, 4:]] = x * di[None, :, None]
        assert E[int(t["size"][3])] == 0.0  # the zero slot
    assert at == words.size
    return dinv


@pytest.mark.parametrize("key", [(14, 56, 0.15, 401, 64), "24", (55, 330, 0.15, 400, 64), "62", "63", (110, 700, 0.15, 110, 64),
                                 "126"], ids=["16", "26", "57", "64", "65", "112", "128"])
def test_blocked_elimination_and_sweeps_solve_like_numpy(tables, key):
    """The factorisation and the two sweeps of one cell per wave from their
    operand tables alone, for n = 16 to 128 positions: equal to
    numpy.linalg.solve on random diagonally dominant matrices of the pattern."""
    _, _, t = tables(key)
    n, nnz, entry = _entries(t)
    slots = 1 if n <= 64 else 2
    rng = np.random.default_rng(n)
    A = np.where(entry >= 0, rng.normal(size=(n, n)), 0.0)
    A[np.arange(n), np.arange(n)] = n + rng.uniform(1, 2, n)
    E = np.zeros(nnz + 17)
    E[entry[entry >= 0]] = A[entry >= 0]
    dinv = _lu_from_tables(t, E)
    row = lambda a: E[_numbers(a, n).reshape(64 * slots, 64 * slots)]
    low, up = row(t["low"]), row(t["up"])
    b = rng.normal(size=n)
    z = np.concatenate([b, np.zeros(64 * slots - n)])
    for k in range(n):
        z -= low[:, k] * z[k]
    z[:n] *= dinv
    for k in range(n - 1, -1, -1):
        z -= up[:, k] * z[k]
    assert not z[n:].any()
    x = np.linalg.solve(A, b)
    assert np.allclose(z[:n], x, rtol=1e-12, atol=1e-12 * np.abs(x).max())
