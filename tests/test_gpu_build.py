"""GPU weight build (stencils, owners, shape vectors) against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_common import TOL_W, annulus_case, dense_strip, say, tgv_case, weight_bounds

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _build(c, dx, K, m, mode, precision=0):
    from paper_2306_01525_amd import Params, Plan
    p = Params(dx=dx, K=K, degree=m, tau=0.8, stencil_mode=mode, precision=precision)
    return Plan.build(c.x, c.y, c.period, p, node_type=c.node_type)


CASES = [
    # (label, cloud factory, dx factor, K, m, mode)
    ("tgv40-K12-m2-own", lambda: tgv_case(40, 12, 2, 1)[0], 1.0, 12, 2, 1),
    ("tgv40-K25-m2-paper", lambda: tgv_case(40, 25, 2, 0)[0], 1.0, 25, 2, 0),
    ("tgv37x41-K30-m4-paper", lambda: tgv_case(37, 30, 4, 0, ny=41, length_y=7.0)[0], 1.0, 30, 4, 0),
    ("tgv23-K20-m3-own", lambda: tgv_case(23, 20, 3, 1, seed=7)[0], 0.7, 20, 3, 1),
    ("annulus-h0.1-K15-m2-paper", lambda: annulus_case(0.1), None, 15, 2, 0),
    ("tgv30-K47-m4-own", lambda: tgv_case(30, 47, 4, 1, seed=3)[0], 1.0, 47, 4, 1),
    ("tgv32-K40-m3-paper", lambda: tgv_case(32, 40, 3, 0, seed=5)[0], 1.0, 40, 3, 0),
    ("lattice16-K12-m2-paper", lambda: tgv_case(16, 12, 2, 0, jitter=0.0, length=16.0)[0], 1.0, 12, 2, 0),
]


@pytest.mark.parametrize("label,make,dxf,K,m,mode", CASES, ids=[c[0] for c in CASES])
def test_build_matches_oracle(label, make, dxf, K, m, mode):
    c = make()
    dx = 0.1 if dxf is None else dxf * c.h
    say("case", label, "n", c.n)
    plan = _build(c, dx, K, m, mode)
    nbr_g = plan.export("nbr")
    own_g = plan.export("owner")
    W_g = plan.export("W")
    perm = plan.export("perm")
    assert sorted(perm.tolist()) == list(range(c.n))
    nbr_o = oracle.knn(c.x, c.y, c.period, K)
    own_o = oracle.owners(c.x, c.y, c.period, dx, mode)
    np.testing.assert_array_equal(nbr_g, nbr_o)
    np.testing.assert_array_equal(own_g, own_o)
    W_o = oracle.weights(c.x, c.y, c.period, dx, K, m, nbr_o, own_o)
    err = np.abs(W_g[:, 1:, :] - W_o[:, 1:, :]).max()
    say("  max |W_gpu - W_oracle| =", err)
    assert err < TOL_W
    # k = 0 is the identity on both sides
    np.testing.assert_allclose(W_o[:, 0, 0], 1.0, atol=1e-10)
    plan.close()


# K and degree whose K + M unknowns (33 to 48) take the 48-unknown matrix-core
# solver: every remainder of K + M modulo 4 (the last panel of four pivot
# columns only partly used) and both ends of the range.
MFMA_RANGE = [(18, 4, 0), (24, 3, 1), (30, 2, 0), (24, 4, 1), (32, 3, 0), (32, 4, 1),
              (33, 4, 0), (38, 3, 1)]


@pytest.mark.parametrize("K,m,mode", MFMA_RANGE,
                         ids=["K%d-m%d-n%d" % (K, m, K + (m + 1) * (m + 2) // 2)
                              for K, m, _ in MFMA_RANGE])
def test_48_unknown_solver_over_its_range(K, m, mode):
    c, _, _ = tgv_case(20, K, m, mode, seed=11)
    plan = _build(c, c.h, K, m, mode)
    nbr_o = oracle.knn(c.x, c.y, c.period, K)
    own_o = oracle.owners(c.x, c.y, c.period, c.h, mode)
    np.testing.assert_array_equal(plan.export("nbr"), nbr_o)
    np.testing.assert_array_equal(plan.export("owner"), own_o)
    W_o = oracle.weights(c.x, c.y, c.period, c.h, K, m, nbr_o, own_o)
    err = np.abs(plan.export("W")[:, 1:, :] - W_o[:, 1:, :]).max()
    say("K %d degree %d (%d unknowns), mode %d: max |W_gpu - W_oracle| = %.2e"
        % (K, m, K + oracle.poly_count(m), mode, err))
    assert err < TOL_W
    assert plan.device_error() == 0
    plan.close()


def test_build_with_crowded_owners_matches_oracle():
    """Weights on the dense-strip cloud, where nodes beside the strip own
    more than 16 departure points: the 48-unknown matrix-core solver solves
    them in groups of 16 (K 30, degree 4, paper rule)."""
    from paper_2306_01525_amd import Params, Plan
    x, y, period, h = dense_strip()
    K, m = 30, 4
    p = Params(dx=h, K=K, degree=m, tau=0.8, stencil_mode=0)
    plan = Plan.build(x, y, period, p)
    nbr_o = oracle.knn(x, y, period, K)
    own_o = oracle.owners(x, y, period, h, 0)
    counts = np.bincount(own_o[:, 1:].ravel(), minlength=x.shape[0])
    say("largest number of departure points of one owner:", counts.max())
    assert counts.max() > 16
    np.testing.assert_array_equal(plan.export("nbr"), nbr_o)
    np.testing.assert_array_equal(plan.export("owner"), own_o)
    W_o = oracle.weights(x, y, period, h, K, m, nbr_o, own_o)
    d = np.abs(plan.export("W") - W_o).max(axis=2)[:, 1:]            # [n][8]
    # the stencils at the strip's edges are lopsided and their systems far
    # worse conditioned than on the lattices: each (node, direction) is held
    # to the backward-error bound of its owner's system
    from types import SimpleNamespace
    c = SimpleNamespace(x=x, y=y, period=period, n=x.shape[0])
    b = weight_bounds(c, nbr_o, own_o, W_o, K, m)[:, 1:]
    worst = np.unravel_index(np.argmax(d / b), d.shape)
    say("max |W_gpu - W_oracle| = %.2e; worst against its bound: %.2e of %.2e (owner of %d points)"
        % (d.max(), d[worst], b[worst], counts[own_o[worst[0], worst[1] + 1]]))
    assert (d <= np.maximum(b, TOL_W)).all()
    assert plan.device_error() == 0
    plan.close()


def test_build_rejects_bad_parameters():
    from paper_2306_01525_amd import MLBMError, Params, Plan
    c, _, _ = tgv_case(10, 12, 2, 0)
    for kw in (dict(K=5, degree=2), dict(K=12, degree=1), dict(K=8, degree=3),
               dict(K=12, degree=2, tau=0.5)):
        p = Params(dx=c.h, tau=kw.pop("tau", 0.8), **kw)
        with pytest.raises(MLBMError):
            Plan.build(c.x, c.y, c.period, p)


@pytest.mark.parametrize("K,m", [(12, 2), (30, 4), (48, 4)])
def test_singular_stencil_is_reported(K, m):
    """Nodes on a straight line make every local system singular (the
    monomials of degree >= 2 are not unisolvent), for each solver shape: two
    systems per wavefront (24 unknowns) and one (48 and 64)."""
    from paper_2306_01525_amd import MLBMError, Params, Plan
    n = 61
    x = np.linspace(0.0, 1.0, n)
    y = 2.0 * x + 0.5
    p = Params(dx=0.01, K=K, degree=m, tau=0.8, stencil_mode=1)
    with pytest.raises(MLBMError) as ei:
        Plan.build(x, y, (0.0, 0.0), p)
    assert ei.value.status == -2


@pytest.mark.parametrize("mode", [0, 1])
def test_duplicate_node_is_reported_singular(mode):
    """Two nodes at the same place: every stencil that holds both has two
    equal rows (and columns) in its local system, which is singular; the
    build reports it (the lower-index twin owns the departure points near it
    in the paper's rule, and every node owns its own in the other)."""
    from paper_2306_01525_amd import MLBMError, Params, Plan
    c, _, _ = tgv_case(20, 20, 3, mode, seed=13)
    x, y = c.x.copy(), c.y.copy()
    x[150], y[150] = x[77], y[77]
    with pytest.raises(MLBMError) as ei:
        Plan.build(x, y, c.period, Params(dx=c.h, K=20, degree=3, tau=0.8, stencil_mode=mode))
    assert ei.value.status == -2


@pytest.mark.parametrize("mode", [0, 1])
def test_tile_tables_are_consistent(mode):
    """Gather tables of the FP32 step, checked on the CPU before any step
    uses them: halo lists sorted, unique and in range; local owners and
    local stencils map back to the global owners and stencils."""
    c, _, _ = tgv_case(64, 30, 4, mode, seed=9)
    plan = _build(c, c.h, 30, 4, mode)
    perm = plan.export("perm")
    iperm = np.empty_like(perm)
    iperm[perm] = np.arange(c.n)
    nbr_u = plan.export("nbr")            # user order, user indices
    own_u = plan.export("owner")
    # internal order, internal indices
    nbr_i = iperm[nbr_u[perm]]
    own_i = iperm[own_u[perm]]
    td = plan.export("tdesc")
    hl = plan.export("hlist")
    words = plan.export("nbrL")
    # three 10-bit halo positions per word -> [ntiles][ocap][K]
    nl = np.stack([(words >> (10 * s_)) & 1023 for s_ in range(3)], axis=-1)
    nl = nl.reshape(words.shape[0], words.shape[1], -1)[:, :, :30]
    ol = plan.export("ownerL") if mode == 0 else None
    T = int(plan.info.tile_nodes)
    say("mode", mode, "tiles", td.shape[0], "max nh", td[:, 1].max(), "max no", td[:, 0].max())
    assert (td[:, 1] > 0).all()
    for t in range(td.shape[0]):
        no, nh = td[t]
        base, cnt = t * T, min(T, c.n - t * T)
        H = hl[t, :nh]
        assert (H >= 0).all() and (H < c.n).all()
        assert (np.diff(H) > 0).all()
        if mode == 0:
            O = np.unique(own_i[base:base + cnt, 1:])
        else:
            O = np.arange(base, base + cnt)
        assert O.size == no
        np.testing.assert_array_equal(H[nl[t, :no, :]], nbr_i[O])
        if mode == 0:
            np.testing.assert_array_equal(O[ol[:, base:base + cnt].T], own_i[base:base + cnt, 1:])
    plan.close()


def _hilbert(x, y, order):
    x, y, d = x.copy(), y.copy(), np.zeros_like(x)
    for b in reversed(range(order)):
        rx, ry = x >> b & 1, y >> b & 1
        d += (3 * rx ^ ry) << 2 * b
        flip = (ry == 0) & (rx == 1)
        x, y = np.where(flip, (1 << order) - 1 - x, x), np.where(flip, (1 << order) - 1 - y, y)
        x, y = np.where(ry == 0, y, x), np.where(ry == 0, x, y)
    return d


@pytest.mark.parametrize("nx,ny,crowd", [(8, 8, 0), (101, 101, 0), (128, 64, 0), (64, 256, 0),
                                         (32, 256, 0), (400, 16, 0), (500, 7, 0), (70, 70, 1)])
def test_internal_order_is_the_stable_order_of_the_cells(nx, ny, crowd):
    """The build's node order, whether the Hilbert keys are counted (up to four
    keys a node) or sorted (longer domains): by key, then by user index, as a
    stable sort on the CPU gives it. `crowd`: half of the nodes in a few cells."""
    from paper_2306_01525_amd import Params, Plan
    c, _, _ = tgv_case(nx, 12, 2, 1, seed=3, ny=ny, length=float(nx), length_y=float(ny))
    x, y = c.x.copy(), c.y.copy()
    if crowd:
        rng = np.random.default_rng(8)
        i = rng.permutation(c.n)[:c.n // 2]
        x[i], y[i] = 1.0 + 0.05 * x[i], 2.0 + 0.05 * y[i]
    plan = Plan.build(x, y, c.period, Params(dx=c.h, K=12, degree=2, tau=0.8, stencil_mode=1))
    perm = plan.export("perm")
    plan.close()
    Lx, Ly = c.period
    cells = max(1.0, c.n / 2.0)
    g = []
    for v in (np.sqrt(cells * (Lx / Ly)), np.sqrt(cells / (Lx / Ly))):
        p2 = 1
        while p2 * 2 <= v * np.sqrt(2.0):
            p2 *= 2
        g.append(p2)
    order = int(max(g)).bit_length() - 1
    cx = np.clip(np.floor(x / (Lx / g[0])).astype(np.int64), 0, g[0] - 1)
    cy = np.clip(np.floor(y / (Ly / g[1])).astype(np.int64), 0, g[1] - 1)
    key = _hilbert(cx, cy, order)
    say("%d nodes, %d x %d cells, %.2f keys a node, fullest cell %d" % (
        c.n, g[0], g[1], 4.0 ** order / c.n, np.unique(key, return_counts=True)[1].max()))
    np.testing.assert_array_equal(perm, np.argsort(key, kind="stable"))


@pytest.mark.parametrize("mode,no,nh", [(1, 256, 13), (1, 256, 1024), (1, 256, 1025),
                                        (1, 256, 3072), (0, 1, 12), (0, 512, 1024),
                                        (0, 513, 700), (0, 2048, 700)])
def test_tile_tables_of_scattered_stencils(mode, no, nh):
    """The gather tables where no two owners or members are near one another in
    the node order, at the sizes around the tables' capacities (512 owners, 1,024
    members: beyond them the tile is marked for the global path), against numpy's
    sorted unique sets. Whole numbers: equal."""
    from paper_2306_01525_amd import Params, Plan
    K, T = 12, 256
    n = 3072 * 40 + 13                       # members 40 apart: a word of 32 holds one
    rng = np.random.default_rng(nh)
    pool = rng.permutation(np.arange(3072) * 40 + 7)[:nh]
    opool = rng.permutation(np.arange(2048) * 60 + 11)[:no]
    nbr = np.empty((n, K), dtype=np.int32)
    if mode == 0:
        nbr[:] = pool[0]
        nbr[opool] = pool[(np.arange(no)[:, None] * K + np.arange(K)) % nh]
        at = (np.arange(n) % T)[:, None] + T * np.arange(-1, 8)[None, :]
        owner = opool[at % no]               # a tile's 2,048 candidates go round the pool
        owner[:, 0] = np.arange(n)
    else:
        nbr[:] = pool[((np.arange(n) % T)[:, None] * K + np.arange(K)) % nh]
        owner = np.repeat(np.arange(n)[:, None], 9, axis=1)
    owner = owner.astype(np.int32)
    x = np.arange(n, dtype=np.float64)
    plan = Plan.from_arrays(x, x, nbr, owner, np.zeros((n, 9, K)),
                            Params(dx=1.0, K=K, degree=2, tau=0.8, stencil_mode=mode))
    td, hl, words = plan.export("tdesc"), plan.export("hlist"), plan.export("nbrL")
    nl = np.stack([(words >> (10 * s_)) & 1023 for s_ in range(3)], axis=-1)
    nl = nl.reshape(words.shape[0], words.shape[1], -1)[:, :, :K]
    ol = plan.export("ownerL") if mode == 0 else None
    plan.close()
    fit = 0
    for t in list(range(0, td.shape[0], 97)) + [td.shape[0] - 1]:
        base, cnt = t * T, min(T, n - t * T)
        O = np.unique(owner[base:base + cnt, 1:])
        H = np.unique(nbr[O])
        assert td[t, 0] == O.size
        if O.size > 512 or H.size > 1024:
            assert td[t, 1] == 0
            continue
        fit += 1
        assert td[t, 1] == H.size
        np.testing.assert_array_equal(hl[t, :H.size], H)
        np.testing.assert_array_equal(H[nl[t, :O.size]], nbr[O])
        if mode == 0:
            np.testing.assert_array_equal(O[ol[:, base:base + cnt].T], owner[base:base + cnt, 1:])
    say("mode", mode, "owners", no, "members", nh, "tiles with tables", fit)
    assert fit >= 1     # the last tile holds 13 nodes and always fits


def _uncompact(units, hd, lw, n, fill):
    """Row heads compacted per group of 64 nodes ([units][8]: group g from
    unit 64 g lw, slot e a block of the group's nodes with hd > e in node
    order, entries 0-3 of the block's units before entries 4-7) back to
    [8][lw][n], with `fill` where a node has no unit."""
    n64 = (n + 63) // 64 * 64
    G = n64 // 64
    H = np.zeros(n64, dtype=np.int64)
    H[:n] = hd
    act = np.arange(lw)[:, None, None] < H.reshape(G, 64)[None]   # [lw][G][64]
    cnt = act.sum(axis=2)
    start = np.cumsum(cnt, axis=0) - cnt                          # units of earlier slots
    u0 = (np.arange(G) * 64 * lw)[None, :] + start                 # [lw][G] first unit
    rank = np.cumsum(act, axis=2) - 1
    e, g, l_ = np.nonzero(act)
    flat = units.reshape(-1)
    k = np.arange(8)[:, None]
    at = 8 * u0[e, g][None] + 4 * ((k // 4) * cnt[e, g][None] + rank[e, g, l_][None]) + k % 4
    out = np.full((8, lw, n64), fill, dtype=units.dtype)
    out[:, e, g * 64 + l_] = flat[at]
    return out[:, :, :n]


@pytest.mark.parametrize("mode,precision,K,m", [(0, 0, 30, 4), (1, 1, 30, 4), (1, 0, 48, 4),
                                                (0, 0, 12, 2)])
def test_adjoint_tables_are_consistent(mode, precision, K, m):
    """Transposed stencil operator and the gather tables of the adjoint step,
    checked on the CPU before any adjoint step uses them: row lengths and row
    heads match the transpose of the forward stencils (rows sorted by arriving
    node), inverse halo lists are sorted, unique and in range, and the local
    columns map back to the row heads. The fill stages 128-node tiles up to
    K = 30 in FP32 and 64-node tiles for FP64 or larger K."""
    from paper_2306_01525_amd import Params, Plan
    c, _, _ = tgv_case(61, K, m, mode, seed=9)   # 3,721 nodes: a partial last group of 64
    p = Params(dx=c.h, K=K, degree=m, tau=0.8, stencil_mode=mode, precision=precision,
               with_adjoint=1)
    plan = Plan.build(c.x, c.y, c.period, p)
    n = c.n
    perm = plan.export("perm")
    iperm = np.empty_like(perm)
    iperm[perm] = np.arange(n)
    nbr_i = iperm[plan.export("nbr")[perm]]
    own_i = iperm[plan.export("owner")[perm]]
    ptr = plan.export("tr_ptr")
    lw = K + 4
    hd = np.minimum(np.diff(ptr).reshape(8, n), lw).max(axis=0)
    ecol = _uncompact(plan.export("ell_col"), hd, lw, n, -1)            # [8][slot][n]
    td = plan.export("tdescT")
    il = plan.export("ilist")
    words = _uncompact(plan.export("elocal"), (hd + 2) // 3, (lw + 2) // 3, n, 0)
    # every slot of a node's head is there, padded with its own index
    pad = (np.arange(lw)[None, :, None] >= np.diff(ptr).reshape(8, 1, n)) \
        & (np.arange(lw)[None, :, None] < hd[None, None, :])
    assert (ecol[pad] == np.broadcast_to(np.arange(n), ecol.shape)[pad]).all()
    el = np.stack([(words >> (10 * s_)) & 1023 for s_ in range(3)], axis=2)
    el = el.reshape(8, -1, n)[:, :lw, :]              # [8][lw][n] (slot-major)
    assert (el[:, :, :][np.arange(lw)[None, :, None] >= np.diff(ptr).reshape(8, 1, n)] == 0).all()
    assert ptr[0] == 0 and ptr[-1] == 8 * K * n and (np.diff(ptr) >= 0).all()
    lens = np.diff(ptr).reshape(8, n)
    arrive = np.repeat(np.arange(n), K)
    for k in range(1, 9):
        S = nbr_i[own_i[:, k]] if mode == 0 else nbr_i
        src = S.ravel()
        np.testing.assert_array_equal(lens[k - 1], np.bincount(src, minlength=n))
        order = np.lexsort((arrive, src))
        rows_src, rows_arr = src[order], arrive[order]
        start = np.concatenate([[0], np.cumsum(lens[k - 1])[:-1]])
        slot = np.arange(src.size) - start[rows_src]
        head = slot < lw
        np.testing.assert_array_equal(ecol[k - 1][slot[head], rows_src[head]], rows_arr[head])
    T = int(plan.info.tile_nodes)
    say("mode", mode, "precision", precision, "tiles", td.size, "max |I_t|", td.max(),
        "global tiles", int((td == 0).sum()))
    assert (td > 0).all()
    assert td.max() <= 1024
    for t in range(td.size):
        ni = td[t]
        I = il[t, :ni]
        assert (I >= 0).all() and (I < n).all() and (np.diff(I) > 0).all()
        ms = np.arange(t * T, min(n, (t + 1) * T))
        for k in range(8):
            hl = np.minimum(lens[k, ms], lw)
            mask = np.arange(lw)[:, None] < hl[None, :]
            np.testing.assert_array_equal(I[el[k][:, ms][mask]], ecol[k][:, ms][mask])
    plan.close()


def test_fp32_weights_only_plan_steps_like_the_full_plan():
    """A plan built with fp32_weights_only holds no FP64 shape vectors: its
    buffer is smaller by 64 K bytes per node; its steps (one cloud, a batch,
    the static-workspace build) and its gradient are bitwise those of the full
    plan; the calls that need the FP64 vectors refuse."""
    from paper_2306_01525_amd import MLBMError, Params, Plan
    from paper_2306_01525_amd.autograd import rollout_loss
    from synth import jittered_lattice, tgv_initial_velocity
    c, ux, uy = tgv_case(48, 30, 4, 0, seed=4)
    ux, uy = tgv_initial_velocity(c.x, c.y, c.period[0], 0.01)

    def prm(lean, K=30, m=4, **kw):
        return Params(dx=c.h, K=K, degree=m, tau=0.8, stencil_mode=0,
                      fp32_weights_only=int(lean), **kw)

    full = Plan.build(c.x, c.y, c.period, prm(False))
    lean = Plan.build(c.x, c.y, c.period, prm(True))
    stat = Plan.build(c.x, c.y, c.period, prm(True), static_workspace=True)
    saved = full._buf.numel() - lean._buf.numel()
    say("plan bytes per node: full %.0f, fp32_weights_only %.0f"
        % (full._buf.numel() / c.n, lean._buf.numel() / c.n))
    assert saved >= 64 * 30 * c.n
    g_full = full.step(full.init(ux, uy), full.new_state(), 20)
    for q in (lean, stat):
        assert torch.equal(q.step(q.init(ux, uy), q.new_state(), 20), g_full)
        assert q.device_error() == 0
    for call in (lambda: lean.export("W"), lambda: lean.interpolate(np.zeros(c.n))):
        with pytest.raises(MLBMError) as ei:
            call()
        assert ei.value.status == -5
    for q in (full, lean, stat):
        q.close()
    # built, initialised and stepped inside one captured graph, replayed twice
    s = torch.cuda.Stream()
    gp, _, _, res = Plan.build_graph([(c.x, c.y, c.period, None)], [prm(True)], ux, uy, 20, s)
    for _ in range(2):
        gp.graph_launch(s)
        s.synchronize()
        assert torch.equal(res.reshape(-1), g_full.reshape(-1))
    assert gp.device_error() == 0
    gp.close()

    # a batch of two clouds
    c2 = jittered_lattice(30, seed=8)
    u2x, u2y = tgv_initial_velocity(c2.x, c2.y, c2.period[0], 0.01)
    clouds = [(c.x, c.y, c.period, None), (c2.x, c2.y, c2.period, None)]
    bx, by = np.concatenate([ux, u2x]), np.concatenate([uy, u2y])
    states = []
    for lean_flag in (False, True):
        b = Plan.build_batch(clouds, [prm(lean_flag), prm(lean_flag, K=20, m=3)])
        states.append(b.step(b.init(bx, by), b.new_state(), 10))
        b.close()
    assert torch.equal(states[0], states[1])

    # the gradient of a short checkpointed rollout
    tx, ty = (torch.tensor(a, device="cuda") for a in (ux, uy))
    grads = []
    for lean_flag in (False, True):
        q = Plan.build(c.x, c.y, c.period, prm(lean_flag, with_adjoint=1))
        u0x = torch.tensor(ux, device="cuda", requires_grad=True)
        u0y = torch.tensor(uy, device="cuda", requires_grad=True)
        tau = torch.tensor(0.8, dtype=torch.float64, device="cuda", requires_grad=True)
        J = rollout_loss(q, u0x, u0y, tau, 6, 0.5 * tx, 0.5 * ty, 3)
        J.backward()
        grads.append((J.detach(), u0x.grad, u0y.grad, tau.grad))
        q.close()
    for a, b in zip(*grads):
        assert torch.equal(a, b)


# Sizes of the null-space solver (K up to 32, 31 at degree 4): members beyond the
# polynomials at the edges of its compiled sizes (0, 8, 12, 16, 20, 24 and 28),
# and the first stencils past it
SOLVER_CASES = [(6, 2), (7, 2), (14, 2), (15, 2), (18, 2), (19, 2), (22, 2), (23, 2), (26, 2),
                (27, 2), (32, 2), (33, 2), (10, 3), (18, 3), (19, 3), (26, 3), (27, 3), (31, 3),
                (32, 3), (33, 3), (16, 4), (23, 4), (24, 4), (27, 4), (28, 4), (31, 4), (32, 4)]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("K,m", SOLVER_CASES)
def test_weights_at_the_edges_of_the_solver_sizes(K, m, mode):
    """Shape vectors against the oracle's within the conditioning bound, on a
    cloud whose last wavefront is partial."""
    from paper_2306_01525_amd import Params, Plan
    c, _, _ = tgv_case(13, K, m, mode, seed=29, ny=11, length_y=2 * np.pi * 11 / 13, jitter=0.2)
    nbr, own, W = oracle.build_plan(c, c.h, K, m, mode)
    wb = weight_bounds(c, nbr, own, W, K, m)
    plan = Plan.build(c.x, c.y, c.period,
                      Params(dx=c.h, K=K, degree=m, tau=0.8, stencil_mode=mode, precision=1))
    np.testing.assert_array_equal(plan.export("nbr"), nbr)
    dW = np.abs(plan.export("W")[:, 1:, :] - W[:, 1:, :]).max(axis=2)
    say("K %d degree %d mode %d: n %d, most points of a node %d, max |dW| %.2e, of its bound %.2e"
        % (K, m, mode, c.n, np.bincount(own[:, 1:].ravel()).max(), dW.max(),
           (dW / wb[:, 1:]).max()))
    assert (dW <= wb[:, 1:]).all()
    assert plan.device_error() == 0
    plan.close()


@pytest.mark.parametrize("K,m", [(12, 2), (20, 3), (30, 4)])
@pytest.mark.parametrize("gap", [1e-2, 1e-4])
def test_weights_of_a_node_pair_close_together(gap, K, m):
    """Two nodes a hundredth and a ten-thousandth of a spacing apart: the
    latter's systems (condition numbers near 1e9 and beyond) are solved again
    by the general elimination. Both within the conditioning bound."""
    from paper_2306_01525_amd import Params, Plan
    c, _, _ = tgv_case(20, K, m, 0, seed=3)
    c.x[101], c.y[101] = c.x[57] + gap * c.h, c.y[57] + 0.3 * gap * c.h
    nbr, own, W = oracle.build_plan(c, c.h, K, m, 0)
    wb = weight_bounds(c, nbr, own, W, K, m)
    plan = Plan.build(c.x, c.y, c.period,
                      Params(dx=c.h, K=K, degree=m, tau=0.8, stencil_mode=0, precision=1))
    dW = np.abs(plan.export("W")[:, 1:, :] - W[:, 1:, :]).max(axis=2)
    say("gap %.0e K %d degree %d: max |dW| %.2e, of its bound %.2e"
        % (gap, K, m, dW.max(), (dW / wb[:, 1:]).max()))
    assert (dW <= wb[:, 1:]).all()
    plan.close()


def _search_clouds():
    """(label, x, y, period, dx): exact lattices (many equal distances), clouds
    smaller than the search block, an open strip, uniform random nodes, and a
    lattice with 130 nodes inside a billionth of a spacing (no radius lists
    them in part, for the nodes around it)."""
    r = np.random.Generator(np.random.PCG64(41))
    out = []
    for nx, ny in ((24, 24), (9, 7)):
        c = tgv_case(nx, 12, 2, 1, jitter=0.0, ny=ny, length=float(nx), length_y=float(ny))[0]
        out.append(("lattice%dx%d" % (nx, ny), c.x, c.y, c.period, 1.0))
    out.append(("open-strip", r.uniform(0, 60, 300), r.uniform(0, 3, 300), (0.0, 0.0), 0.5))
    out.append(("random", r.uniform(0, 30, 1100), r.uniform(0, 36, 1100), (30.0, 36.0), 1.0))
    c = tgv_case(20, 12, 2, 1, seed=5, length=20.0)[0]
    a, d = r.uniform(0, 2 * np.pi, 130), 1e-9 * r.uniform(0.1, 1, 130)
    out.append(("crowd", np.concatenate([c.x, 10.3 + d * np.cos(a)]),
                np.concatenate([c.y, 9.7 + d * np.sin(a)]), c.period, 1.0))
    return out


@pytest.mark.parametrize("K", [6, 16, 17, 32, 33, 48])
@pytest.mark.parametrize("which", range(5))
def test_stencil_search_is_exact(which, K):
    """Stencils and owners bit-exact against the oracle's, K at the edges of
    the search's list sizes. The plan is captured, so that a singular local
    system (the crowd's neighbours have them) does not end the build."""
    from paper_2306_01525_amd import Params, Plan
    label, x, y, period, dx = _search_clouds()[which]
    m = 4 if K > 32 else 3 if K > 16 else 2
    say("cloud", label, "n", x.shape[0], "K", K)
    st = torch.cuda.Stream()
    z = np.zeros(x.shape[0])
    plan, _, _, _ = Plan.build_graph([(x, y, period, None)],
                                     [Params(dx=dx, K=K, degree=m, tau=0.8)], z, z, 0, st)
    plan.graph_launch(st)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(plan.export("nbr"), oracle.knn(x, y, period, K))
    np.testing.assert_array_equal(plan.export("owner"), oracle.owners(x, y, period, dx, 0))
    plan.close()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("nx,ny,K", [(5, 5, 6), (13, 5, 7), (43, 3, 11), (16, 8, 12), (17, 15, 29)])
def test_interpolation_at_ragged_sizes(nx, ny, K, mode):
    """The interpolation operator against its definition on the plan's own
    stencils and weights; slots left over from groups of six, partial
    workgroups. Both sum K products in FP64: off by at most K 2^-53 of the sum
    of their magnitudes, twice."""
    from paper_2306_01525_amd import Params, Plan
    c, _, _ = tgv_case(nx, K, 2, mode, seed=31, ny=ny, length_y=2 * np.pi * ny / nx, jitter=0.2)
    dx = min(c.h, 0.4 * min(c.period))
    plan = Plan.build(c.x, c.y, c.period,
                      Params(dx=dx, K=K, degree=2, tau=0.8, stencil_mode=mode, precision=1))
    f = np.random.Generator(np.random.PCG64(7)).standard_normal(c.n)
    got = plan.interpolate(f).cpu().numpy()
    nbr, own, W = (plan.export(a) for a in ("nbr", "owner", "W"))
    for k in range(1, 9):
        terms = W[:, k] * f[nbr[own[:, k]]]
        assert (np.abs(got[k - 1] - terms.sum(1)) <= 2 * K * 2.0 ** -53 * np.abs(terms).sum(1)).all()
    plan.close()


@pytest.mark.parametrize("n,frac,width,K,m,precision", [(2000, 0.97, 0.02, 12, 2, 1),
                                                        (2000, 0.9, 0.05, 20, 3, 1),
                                                        (1500, 0.9, 0.05, 30, 4, 0)])
def test_transposed_rows_of_uneven_clouds(n, frac, width, K, m, precision):
    """Row lengths from none to several hundred (a dense strip whose edge nodes own
    many departure points), around the 16, 32, 48 and 64 entries that the last
    pass ranks at a time and beyond, where one lane sorts: row lengths and heads
    equal the transpose of the forward stencils, sorted by arriving node, and a
    reversed step equals the one on rows that the host put in order. All exact."""
    from paper_2306_01525_amd import Params, Plan
    x, y, period, h = dense_strip(n, frac, width)
    p = Params(dx=h, K=K, degree=m, tau=0.8, stencil_mode=0, precision=precision, with_adjoint=1)
    plan = Plan.build(x, y, period, p)
    perm = plan.export("perm")
    iperm = np.empty_like(perm)
    iperm[perm] = np.arange(n)
    nbr = iperm[plan.export("nbr")[perm]]
    own = iperm[plan.export("owner")[perm]]
    ptr, ecol = plan.export("tr_ptr"), plan.export("ell_col")
    # the rows' weights and tails: a reversed step, bit for bit that of an import
    # of the same weights, whose rows the host puts in order
    back = Plan.from_arrays(x[perm], y[perm], nbr, own, plan.export("W")[perm], p)
    f = plan.init_f(0.02 * np.sin(x) * np.cos(y), -0.02 * np.cos(x) * np.sin(y))
    lam = torch.linspace(-1.0, 1.0, f.numel(), device="cuda").reshape(f.shape).to(f.dtype)
    out = []
    for q in (plan, back):
        dtau = torch.zeros(1, dtype=torch.float64, device="cuda")
        out.append((q.step_adjoint(f, lam, torch.empty_like(f), dtau), dtau))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    back.close()
    plan.close()
    lens, lw = np.diff(ptr).reshape(8, n), K + 4
    say("n %d K %d: rows of up to %d entries, %d above 64, %d empty" % (
        n, K, lens.max(), (lens > 64).sum(), (lens == 0).sum()))
    assert lens.max() > 64 and lens.min() == 0
    hd = np.minimum(lens, lw).max(axis=0)
    head = _uncompact(ecol, hd, lw, n, -1)
    for k in range(1, 9):
        src, arr = nbr[own[:, k]].ravel(), np.repeat(np.arange(n), K)
        np.testing.assert_array_equal(lens[k - 1], np.bincount(src, minlength=n))
        order = np.lexsort((arr, src))
        src, arr = src[order], arr[order]
        slot = np.arange(src.size) - (np.cumsum(lens[k - 1]) - lens[k - 1])[src]
        want = np.full((lw, n), -1)
        want[:] = np.where(np.arange(lw)[:, None] < hd, np.arange(n), -1)   # padding
        want[slot[slot < lw], src[slot < lw]] = arr[slot < lw]
        np.testing.assert_array_equal(head[k - 1], want)


@pytest.mark.parametrize("K,m,width,seed", [(9, 2, 3.16e-4, 7), (12, 2, 3e-4, 9),
                                            (14, 3, 5.6e-3, 8), (17, 4, 3.4e-2, 9)])
def test_strips_too_thin_for_the_polynomials_are_refused(K, m, width, seed):
    """Nodes of an open strip so thin that some systems' smallest pivot, in the
    elimination of the whole system, lies below the singularity threshold (0.02 to
    0.2 of it), while the polynomials' own pivots are only near its square root:
    refused by the oracle and by the build. Four times as wide, both accept it."""
    from types import SimpleNamespace
    from paper_2306_01525_amd import MLBMError, Params, Plan
    n = 80
    for scale in (1, 4):
        r = np.random.default_rng(seed)
        x = np.linspace(0, 1, n) + r.uniform(-0.3, 0.3, n) / n
        y = scale * width * r.uniform(-1, 1, n) * K / n
        c = SimpleNamespace(x=x, y=y, period=(0.0, 0.0), n=n)
        p = Params(dx=0.01, K=K, degree=m, tau=0.8, stencil_mode=1, precision=1)
        say("K %d degree %d width %.1e" % (K, m, scale * width))
        if scale == 1:
            with pytest.raises(np.linalg.LinAlgError):
                oracle.build_plan(c, 0.01, K, m, 1)
            with pytest.raises(MLBMError) as ei:
                Plan.build(x, y, c.period, p)
            assert ei.value.status == -2
        else:
            oracle.build_plan(c, 0.01, K, m, 1)
            Plan.build(x, y, c.period, p).close()


@pytest.mark.parametrize("n,K,m,precision", [(2500, 12, 2, 1), (2500, 20, 3, 0), (9000, 12, 2, 0)])
def test_transposed_rows_of_clustered_clouds(n, K, m, precision):
    """Four dense clusters in a sparse cloud: departure points leave a cluster for the
    nodes at its edge, whose rows hold hundreds to thousands of entries, several
    blocks of 64. Row lengths against the stencils, and a reversed step, bit for
    bit, that of an import of the same weights, whose rows the host puts in order
    and nothing reorders."""
    from paper_2306_01525_amd import Params, Plan
    r = np.random.default_rng(3)
    at, which = r.uniform(0.2, 0.8, (4, 2)), r.integers(0, 4, n)
    q = at[which] + 0.002 * r.standard_normal((n, 2))
    q[:n // 10] = r.uniform(0, 1, (n // 10, 2))
    x, y, period, h = q[:, 0] % 1, q[:, 1] % 1, (1.0, 1.0), n ** -0.5
    p = Params(dx=h, K=K, degree=m, tau=0.8, stencil_mode=0, precision=precision, with_adjoint=1)
    plan = Plan.build(x, y, period, p)
    perm = plan.export("perm")
    iperm = np.empty_like(perm)
    iperm[perm] = np.arange(n)
    nbr, own = iperm[plan.export("nbr")[perm]], iperm[plan.export("owner")[perm]]
    lens = np.diff(plan.export("tr_ptr")).reshape(8, n)
    for k in range(1, 9):
        np.testing.assert_array_equal(lens[k - 1], np.bincount(nbr[own[:, k]].ravel(), minlength=n))
    say("n %d K %d: rows of up to %d entries, %d above 64, %d above 256" % (
        n, K, lens.max(), (lens > 64).sum(), (lens > 256).sum()))
    assert lens.max() > 256
    back = Plan.from_arrays(x[perm], y[perm], nbr, own, plan.export("W")[perm], p)
    f = plan.init_f(0.02 * np.sin(x) * np.cos(y), -0.02 * np.cos(x) * np.sin(y))
    lam = torch.linspace(-1.0, 1.0, f.numel(), device="cuda").reshape(f.shape).to(f.dtype)
    out = []
    for one in (plan, back):
        dtau = torch.zeros(1, dtype=torch.float64, device="cuda")
        out.append((one.step_adjoint(f, lam, torch.empty_like(f), dtau), dtau))
        one.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("K", [6, 20, 48])
@pytest.mark.parametrize("which", ["strip", "clusters", "outliers"])
def test_stencil_search_around_dense_parts(which, K):
    """Few nodes around dense parts, whose radius has to be found within a thousandth:
    stencils and owners bit-exact against the oracle's. The plan is captured, so
    that a singular local system does not end the build."""
    from paper_2306_01525_amd import Params, Plan
    r = np.random.default_rng(6)
    n, period = 4000, (1.0, 1.0)
    x, y = r.uniform(0, 1, n), r.uniform(0, 1, n)
    if which == "strip":
        x[20:] *= 0.003
    elif which == "clusters":
        at, c = r.uniform(0.2, 0.8, (8, 2)), r.integers(0, 8, n)
        q = at[c] + 1e-3 * r.standard_normal((n, 2))
        x[400:], y[400:] = q[400:].T
    else:
        period = (0.0, 0.0)
        x[:5] += 30.0
        y[3:7] -= 200.0
    m = 4 if K > 32 else 3 if K > 16 else 2
    st, z = torch.cuda.Stream(), np.zeros(n)
    plan, _, _, _ = Plan.build_graph([(x, y, period, None)],
                                     [Params(dx=0.015, K=K, degree=m, tau=0.8)], z, z, 0, st)
    plan.graph_launch(st)
    torch.cuda.synchronize()
    say("cloud", which, "K", K, "searched")
    np.testing.assert_array_equal(plan.export("nbr"), oracle.knn(x, y, period, K))
    np.testing.assert_array_equal(plan.export("owner"), oracle.owners(x, y, period, 0.015, 0))
    plan.close()
