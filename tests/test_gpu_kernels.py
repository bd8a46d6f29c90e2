"""Kernels at the sizes where their tiling can go wrong, on the GPU."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
import scgen
from scgen.rng import signs_from_seed

P = pytest.importorskip("paper_2509_21037_amd")
pytestmark = pytest.mark.gpu


def _plan(subs, **kw):
    import torch
    assert torch.cuda.is_available()
    torch.cuda.init()
    plan = P.Plan(subs, **kw)
    plan.factor()
    plan.assemble()
    return plan


def _columns(s, m, seed):
    """s with m multipliers on random DOFs, some of them repeated, in no order."""
    dof = np.random.default_rng(seed).choice(s.n, size=m, replace=True).astype(np.int32)
    return s.with_columns(dof, signs_from_seed(seed, m))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_dense_F_on_device_at_tile_edges(precision):
    """sc_get_F on the device at the edges of its 64-row quadrants and of the
    stored 128 x 128 tiles, columns in random order: the host copy's values
    bit for bit, nothing else written."""
    import torch
    box = scgen.box_subdomain("heat", (20, 14), 1.0 / 20, seed=3)
    subs = [_columns(box, m, 40 + m) for m in (1, 63, 64, 65, 127, 128, 129, 193, 260)]
    plan = _plan(subs, precision=precision)
    for i, s in enumerate(subs):
        ld = s.m + i % 3
        out = torch.full((ld * s.m + 5,), -3.0, dtype=torch.float64, device="cuda")
        F = plan.get_F_device(i, out=out, ld=ld)
        assert np.array_equal(F.cpu().numpy(), plan.get_F(i)), s.m
        assert bool((out[:ld * s.m].view(s.m, ld)[:, s.m:] == -3.0).all()) and bool((out[ld * s.m:] == -3.0).all())
    plan.destroy()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_dense_F_where_no_kernel_writes(precision):
    """sc_get_F "on the device" into memory that takes a copy and no kernel of
    this GPU: pinned host memory, and device memory off the 8-byte grid."""
    import ctypes

    import torch
    box = scgen.box_subdomain("heat", (20, 14), 1.0 / 20, seed=3)
    subs = [_columns(box, m, 40 + m) for m in (1, 130)]
    plan = _plan(subs, precision=precision)
    for i, s in enumerate(subs):
        ld = s.m + 3
        for kind in ("pinned", "off"):
            raw = torch.zeros(8 * (ld * s.m + 1), dtype=torch.uint8, **(dict(pin_memory=True) if kind == "pinned"
                                                                       else dict(device="cuda")))
            at = 0 if kind == "pinned" else 4
            torch.cuda.synchronize()
            st = P.load().sc_get_F(plan._h, i, ctypes.c_void_p(raw.data_ptr() + at), ld, 1, ctypes.c_void_p(0))
            assert st == P.SC_OK
            F = raw.cpu().numpy()[at:at + 8 * ld * s.m].copy().view(np.float64).reshape(s.m, ld)
            assert np.array_equal(F[:, :s.m].T, plan.get_F(i)) and not F[:, s.m:].any(), (s.m, kind)
    plan.destroy()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("shape", ["one block", "two blocks", "pairs", "no pairs"])
def test_trsm_small_launch_matches_large(precision, shape):
    """One subdomain alone (at most one TRSM workgroup per CU: the chunks come
    from a fifth wavefront) and among 520 others (each wavefront loads its
    share): the same sums in the same order, so the same F bit for bit, for a
    tile of one block (one chunk), of two, of merged pairs and without."""
    s, merge = {"one block": (scgen.box_subdomain("heat", (4, 4), 0.25, 80), False),
                "two blocks": (scgen.box_subdomain("heat", (9, 8), 1.0 / 9, 81), False),
                "pairs": (scgen.box_subdomain("elasticity", (7, 6, 8), 0.125, 82), True),
                "no pairs": (scgen.box_subdomain("elasticity", (6, 6, 7), 1.0 / 7, 83), False)}[shape]
    one = scgen.box_subdomain("heat", (5, 3), 0.2, 84)
    kw = dict(precision=precision, pair_merge=merge, syrk_kind=1)
    alone = _plan([s], **kw)
    batch = _plan([s] + [one] * 520, **kw)
    F = alone.get_F(0)
    assert np.array_equal(F, batch.get_F(0))
    sel = np.sort(np.random.default_rng(85).choice(s.m, size=min(64, s.m), replace=False))
    assert oracle.relF(F[np.ix_(sel, sel)], oracle.schur(s, sel=sel)) <= (1e-12 if precision == "fp64" else 1e-5)
    alone.destroy()
    batch.destroy()


@pytest.mark.parametrize("mode", ["two kernels", "overlapped", "waves", "preprocess"])
@pytest.mark.parametrize("count", [1, 3, 9])
def test_work_lists_of_few_uneven_subdomains(count, mode):
    """Fewer subdomains than XCDs, or one more, of very different sizes: their
    tiles and SYRK items are dealt out over the XCDs, every one of them once
    in each way to assemble (F bit for bit as each subdomain's alone)."""
    edges = [(9, 8, 9), (2, 2, 2), (6, 7, 5), (4, 4, 4), (3, 2, 5), (7, 7, 3), (1, 1, 1), (5, 5, 6), (8, 2, 2)]
    subs = [scgen.box_subdomain("elasticity", e, 0.125, 90 + i) for i, e in enumerate(edges[:count])]
    kw = {"overlapped": dict(assembly="overlap"),
          "waves": dict(arena_cap_bytes=2 * max(s.n * ((s.m + 63) // 64) * 512 for s in subs))}.get(mode, {})
    plan = _plan(subs, syrk_kind=2, **kw)
    if mode == "preprocess":
        plan.preprocess([s.val for s in subs])
    for i, s in enumerate(subs):
        alone = _plan([s], syrk_kind=2)
        assert np.array_equal(plan.get_F(i), alone.get_F(0)), i
        alone.destroy()
    sel = np.arange(0, subs[0].m, 7)
    assert oracle.relF(plan.get_F(0)[np.ix_(sel, sel)], oracle.schur(subs[0], sel=sel)) <= 1e-12
    plan.destroy()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("split", ["uniform", "etree"])
def test_trsm_reads_only_rows_it_wrote(precision, split):
    """The X buffer full of another batch's values (temporary-memory waves
    that reuse it, subdomains of several sizes, stripes that start late): the
    same F bit for bit as with an X of its own, and as the oracle's."""
    subs = [scgen.box_subdomain("elasticity", e, 1.0 / 8, 60 + i)
            for i, e in enumerate([(8, 7, 6), (5, 5, 5), (7, 3, 8), (6, 6, 4)])]
    subs += [scgen.box_subdomain("heat", (12, 11, 9), 1.0 / 12, 70), scgen.simplex_subdomain(2, 40, 71)]
    subs += [_columns(scgen.box_subdomain("heat", (12, 12, 12), 1.0 / 12, 72), 300, 73)]
    kw = dict(precision=precision, block_split=split, panel_width=48)
    ref = _plan(subs, **kw)
    size = 8 if precision == "fp64" else 4
    cap = max(s.n * ((s.m + 63) // 64) * 64 * size for s in subs)
    wav = _plan(subs, arena_cap_bytes=cap, **kw)
    wav.assemble()
    tol = 1e-12 if precision == "fp64" else 1e-5
    for i, s in enumerate(subs):
        F = wav.get_F(i)
        assert np.array_equal(F, ref.get_F(i)), i
        sel = np.sort(np.random.default_rng(i).choice(s.m, size=min(64, s.m), replace=False))
        assert oracle.relF(F[np.ix_(sel, sel)], oracle.schur(s, sel=sel)) <= tol, i
    wav.destroy()
    ref.destroy()


@pytest.mark.parametrize("merge", [True, False])
def test_trsm_slab_of_4_gib(merge):
    """A column tile whose X rows hold 4 GiB and more (64-bit row offsets in
    the TRSM): 8.4 million rows kept down to the first pivot or not, the same
    values where only the last few rows are kept (32-bit offsets)."""
    n = 8_400_000
    s = scgen.laplace_1d(n, dof=np.array([n // 2, 3 * n // 4, 7 * n // 8], dtype=np.int32), seed=4)
    F = []
    for staircase in (True, False):
        plan = _plan([s], staircase=staircase, panel_width=16, pair_merge=merge)
        F.append(plan.get_F(0))
        plan.destroy()
    assert np.isfinite(F[0]).all() and np.abs(F[0]).min() > 0
    assert np.abs(F[1] - F[0]).max() <= 1e-13 * np.abs(F[0]).max()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", [1, 2])
def test_syrk_at_tile_edges(kind, precision):
    """The SYRK (64 x 64 blocks, 128 x 128 tiles) with first pivots at
    every offset of its 16-row steps, last columns and rows at every remainder
    and one to three column tiles: F within the bar of the oracle, exactly
    symmetric, the two kinds the same bit for bit."""
    subs = []
    for i, (e, m) in enumerate([((3, 2), 1), ((9, 7), 17), ((16, 9), 63), ((15, 13), 65), ((11, 18), 127),
                                ((14, 17), 129), ((20, 11), 192), ((19, 19), 193)]):
        subs.append(_columns(scgen.box_subdomain("heat", e, 1.0 / 16, i), m, 80 + i))
    subs += [_columns(scgen.box_subdomain("elasticity", (4, 3, 5), 0.2, 5), 140, 90)]
    plan = _plan(subs, precision=precision, syrk_kind=kind, block_split="etree", panel_width=48)
    other = _plan(subs, precision=precision, syrk_kind=3 - kind, block_split="etree", panel_width=48)
    for i, s in enumerate(subs):
        F = plan.get_F(i)
        assert np.array_equal(F, F.T) and np.array_equal(F, other.get_F(i)), i
        assert oracle.relF(F, oracle.schur(s)) <= (1e-12 if precision == "fp64" else 1e-5), i
    plan.destroy()
    other.destroy()


def _pairs(count, seed, scales=(0, 0, 0)):
    """`count` uncoupled pairs of nodes with the matrices [[a, b], [b, c]] (a, b
    and c of the sizes 2^scales), a multiplier on every node, in the order of
    elimination, and the X of the mixed assembly (rounded to FP32): [x00, x10,
    x11] of every pair, X = (sign0 (x00, x10), sign1 (0, x11))."""
    rng = np.random.default_rng(seed)
    a, b, c = (np.ldexp(rng.uniform(lo, hi, count), k) for (lo, hi), k in zip([(1, 4), (-0.9, 0.9), (1, 4)], scales))
    n = 2 * count
    i = np.arange(n)
    s = SimpleNamespace(n=n, rowptr=2 * np.arange(n + 1), col=np.stack([i - i % 2, i - i % 2 + 1], 1).ravel(),
                        val=np.stack([a, b, b, c], 1).ravel(), dof=i.astype(np.int32),
                        sign=signs_from_seed(seed, n), dofs_per_node=1, perm=i.astype(np.int32))
    order = np.empty(n, dtype=np.int64)
    order[P.host_analyze(s, values=False)["perm"]] = i
    first = np.where(order[0::2] < order[1::2], i[0::2], i[1::2])
    second = first ^ 1
    l00 = np.sqrt(np.where(first % 2 == 0, a, c))
    l10 = b / l00
    l11 = np.sqrt(np.where(first % 2 == 0, c, a) - l10 * l10)
    with np.errstate(over="ignore"):
        x = np.stack([1 / l00, -l10 / l00 / l11, 1 / l11]).astype(np.float32)
    return s, first, second, x


@pytest.mark.parametrize("kind", [1, 2])
def test_mixed_syrk_rounds_like_fp32_products(kind):
    """Mixed F entries that are one product of two X entries: as accurate as
    one FP32 product.  Half an ulp of the result from the last addition; the
    small partial products are at most 2^-7 of it and rounded seven times in
    FP32, each sum but the last two at most 2^-14 (2^-6 + 2^-9 ulp), and the
    one left out is at most 2^-34 (2^-10 ulp): below 17/32 ulp.  The six
    largest partial products alone leave up to 0.95 ulp (one entry in 50 above
    17/32), two planes of bf16 hundreds."""
    s, first, second, x = _pairs(400, 21)
    plan = _plan([s], precision="mixed", syrk_kind=kind)
    F = plan.get_F(0)
    sg = s.sign.astype(np.float64)
    F = sg[:, None] * F * sg[None, :]
    x = x.astype(np.float64)
    for got, want in ((F[second, second], x[2] * x[2]), (F[first, second], x[1] * x[2])):
        ulp = np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
        assert np.abs(got - want).max() > 0
        assert (np.abs(got - want) / ulp).max() <= 17 / 32
    want = x[0] * x[0] + x[1] * x[1]
    assert (np.abs(F[first, first] - want) <= 2.0 ** -22 * want).all()
    plan.destroy()


@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("scales", [(-61, 87, 236), (-91, 72, 236), (126, 126, 126), (140, 140, 140), (-66, -66, -66),
                                    (-70, -70, -70), (-124, -124, -124), (-160, -160, -160), (-254, -254, -254),
                                    (-300, -300, -300)])
def test_mixed_syrk_over_the_fp32_range(scales, kind):
    """X values at the ends of the FP32 range, in one subdomain of a batch: of
    10^9 or 10^13 and 10^-35 in one product, F at the smallest normal number and
    below, X on either side of 2^34 (where the FP32 units take over), F near
    the top, F infinite (with its sign), X infinite: as accurate as one FP32
    product (the bound of the test above, ulps of a subnormal result included).
    The other subdomain's F is what it is alone."""
    s, first, second, x = _pairs(150, 22, scales)
    other = _pairs(150, 23)[0]
    plan, alone = (_plan(b, precision="mixed", syrk_kind=kind) for b in ([s, other], [other]))
    sg = s.sign.astype(np.float64)
    F = sg[:, None] * plan.get_F(0) * sg[None, :]
    x = x.astype(np.float64)
    pairs = [(F[second, second], x[2] * x[2])]
    if np.isfinite(x).all():                     # (an infinity times the zeros of other columns is NaN)
        pairs.append((F[first, second], x[1] * x[2]))
        G = F.copy()                             # uncoupled pairs
        for p, q in ((first, first), (second, second), (first, second), (second, first)):
            G[p, q] = 0
        assert np.abs(G).max() == 0
    for got, want in pairs:
        with np.errstate(over="ignore", invalid="ignore"):
            w32 = want.astype(np.float32)
            ulp = np.spacing(np.abs(w32)).astype(np.float64)
        big = np.isinf(w32)
        assert np.array_equal(got[big], w32[big].astype(np.float64))
        assert (np.abs(got[~big] - want[~big]) <= 17 / 32 * ulp[~big]).all()
    assert np.array_equal(plan.get_F(1), alone.get_F(0))
    plan.destroy()
    alone.destroy()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_syrk_quarters_match_whole_blocks(precision):
    """A launch of few blocks (four workgroups a block) and of many (one), at
    every remainder of the last column tile: the same F bit for bit."""
    subs = [_columns(scgen.box_subdomain("heat", e, 1.0 / 16, 300 + m), m, 310 + m)
            for e, m in [((3, 2), 1), ((16, 9), 31), ((15, 13), 33), ((9, 7), 64), ((11, 18), 97), ((19, 19), 193)]]
    few = _plan(subs, precision=precision, syrk_kind=1)
    many = _plan(subs + [scgen.box_subdomain("heat", (3, 3), 0.3, 9)] * 600, precision=precision, syrk_kind=1)
    for i, s in enumerate(subs):
        assert np.array_equal(few.get_F(i), many.get_F(i)), s.m
    few.destroy()
    many.destroy()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_apply_and_pcpg_at_tile_edges(precision):
    """q = F p through both explicit applies, and one projected CG step count
    of each workgroup width, at m around the stored 128 x 128 tiles: against
    the dense product of the assembled F (FP64 sums of at most 400 terms: 1e-13
    of their size) and against the oracle's CG on that F."""
    import torch
    box = scgen.box_subdomain("heat", (20, 14), 1.0 / 20, seed=3)
    wide = scgen.box_subdomain("elasticity", (6, 7, 8), 1.0 / 8, seed=4)
    for subs in ([_columns(box, m, 140 + m) for m in (1, 127, 128, 129, 256, 257, 400)],
                 [wide, _columns(box, 100, 7)]):
        plan = _plan(subs, precision=precision)
        rng = np.random.default_rng(9)
        p = torch.from_numpy(rng.uniform(-1, 1, plan.dual_total)).cuda()
        q, q2 = torch.zeros_like(p), torch.zeros_like(p)
        plan.apply(p, q)
        plan.apply_noalloc(p, q2)
        assert torch.equal(q, q2)
        for i, s in enumerate(subs):
            o, F = plan.query(i)["dual_offset"], plan.get_F(i)
            x = p[o:o + s.m].cpu().numpy()
            bound = 1e-13 * (np.abs(F) @ np.abs(x))
            assert np.all(np.abs(q[o:o + s.m].cpu().numpy() - F @ x) <= bound), s.m
        plan.destroy()
    subs = [scgen.box_subdomain("elasticity", e, 1.0 / 8, 20 + i) for i, e in enumerate([(6, 7, 8), (7, 7, 7)])]
    for batch in (subs, [scgen.box_subdomain("elasticity", (2, 3, 2), 0.5, 30)]):
        plan = _plan(batch, precision=precision)
        d = torch.from_numpy(np.random.default_rng(8).uniform(-1, 1, plan.dual_total)).cuda()
        lam = torch.zeros_like(d)
        plan.pcpg(d, lam, 4)
        for i, s in enumerate(batch):
            o = plan.query(i)["dual_offset"]
            G = s.sign[:, None] * s.R[s.dof]
            ref = oracle.pcpg(plan.get_F(i), G, d[o:o + s.m].cpu().numpy(), 4)
            ref = ref[0] if isinstance(ref, tuple) else ref
            got = lam[o:o + s.m].cpu().numpy()
            assert np.linalg.norm(got - ref) <= 1e-9 * np.linalg.norm(ref), i
        plan.destroy()


@pytest.mark.parametrize("split", ["uniform", "etree"])
@pytest.mark.parametrize("count", [1, 5])
def test_implicit_apply_split_levels(count, split):
    """The implicit apply where its levels are split over workgroups (blocks of
    more than 512 pruned rows, few per level), where they are not, and with
    repeated DOFs: against the explicit product of the assembled F."""
    import torch
    subs = [scgen.box_subdomain("elasticity", (12, 11, 10), 1.0 / 12, 50 + i, gluing="per_face") for i in range(count)]
    subs += [scgen.box_subdomain("heat", (3, 2), 0.5, 8), _columns(scgen.box_subdomain("heat", (9, 9, 9), 0.1, 9), 70, 3)]
    plan = _plan(subs, block_split=split)
    p = torch.from_numpy(np.random.default_rng(2).uniform(-1, 1, plan.dual_total)).cuda()
    q, ref = torch.zeros_like(p), torch.zeros_like(p)
    plan.apply(p, ref)
    for _ in range(2):
        plan.apply_implicit(p, q)
        for i, s in enumerate(subs):
            o = plan.query(i)["dual_offset"]
            a, b = q[o:o + s.m], ref[o:o + s.m]
            assert float((a - b).norm()) <= 1e-11 * float(b.norm()), i
    plan.destroy()


@pytest.mark.parametrize("count,width,split", [(1100, 16, "etree"), (900, 16, "uniform"), (3, 16, "uniform"),
                                                (1, 16, "etree"), (40, 32, "uniform"), (3, 64, "uniform")])
def test_implicit_apply_chains(count, width, split):
    """Levels of thousands of blocks below a chain of smaller ones, chains alone
    (more workgroups than run at once, one subdomain), subdomains at either
    side of the block count up to which one workgroup does all (13 and 7 blocks):
    against the explicit product, and the same bit for bit on every call and
    after other work in between."""
    import torch
    box = scgen.box_subdomain("heat", (20, 18), 1.0 / 20, 11)
    subs = [_columns(box, 3 + i % 5, 200 + i) for i in range(count)]
    subs += [scgen.box_subdomain("heat", (2, 2), 0.5, 12)]
    plan = _plan(subs, block_split=split, panel_width=width)
    p = torch.from_numpy(np.random.default_rng(13).uniform(-1, 1, plan.dual_total)).cuda()
    q, ref, other = torch.zeros_like(p), torch.zeros_like(p), torch.zeros_like(p)
    plan.apply(p, ref)
    plan.apply_implicit(p, q)
    first = q.clone()
    o = 0
    for i, s in enumerate(subs):
        a, b = q[o:o + s.m], ref[o:o + s.m]
        assert float((a - b).norm()) <= 1e-11 * float(b.norm()), i
        o += s.m
    for _ in range(3):
        plan.apply_implicit(ref, other)
        plan.apply_implicit(p, q)
        assert torch.equal(q, first)
    plan.destroy()


@pytest.mark.parametrize("use_graph", [False, True])
def test_implicit_wait_that_gives_up(use_graph):
    """A wait of the chains that ends at its limit (0 looks: at once, set from
    the host) leaves no number that could be taken for a result: NaN for its
    subdomain, an error from the projected CG; with the limit back the same
    plan is right again."""
    import torch
    subs = [scgen.box_subdomain("elasticity", e, 1.0 / 8, 400 + i) for i, e in enumerate([(8, 7, 6), (5, 6, 5), (7, 7, 7)])]
    subs += [scgen.box_subdomain("heat", (2, 2), 0.5, 410)]
    ref = _plan(subs, block_split="etree")
    p = torch.from_numpy(np.random.default_rng(14).uniform(-1, 1, ref.dual_total)).cuda()
    want, q = torch.zeros_like(p), torch.zeros_like(p)
    ref.apply(p, want)
    plan = _plan(subs, block_split="etree", use_graph=use_graph)
    hybrid = _plan(subs, block_split="etree", select_iters=1)
    assert any(hybrid.selection(i)["implicit"] for i in range(3))

    def check(may_fail):
        o, failed = 0, 0
        for s in subs:
            a, b = q[o:o + s.m], want[o:o + s.m]
            o += s.m
            if may_fail and bool(torch.isnan(a).all()):
                failed += 1
            else:
                assert float((a - b).norm()) <= 1e-11 * float(b.norm())
        assert not may_fail or failed

    for pl, apply in ((plan, plan.apply_implicit), (hybrid, hybrid.apply)):
        for limit in (1 << 24, 0, 1 << 24):
            pl.set_wait_limit(limit)
            for _ in range(2):
                apply(p, q)
                check(limit == 0)
    lam = torch.zeros_like(p)
    hybrid.pcpg(p, lam, 3)
    hybrid.set_wait_limit(0)
    with pytest.raises(P.ScasmError) as e:
        hybrid.pcpg(p, lam, 3)
    assert e.value.status == P.SC_ERR_DEVICE
    hybrid.set_wait_limit(1 << 24)
    again = torch.zeros_like(p)
    hybrid.pcpg(p, again, 3)
    for pl in (ref, plan, hybrid):
        pl.destroy()


@pytest.mark.parametrize("width", [16, 32, 48, 64])
def test_diagonal_inverses_at_block_widths(width):
    """Diagonal blocks of every width up to 64 (chains of 2 .. 140 nodes: the
    last block is the remainder), well and badly scaled: the explicit F and the
    implicit apply, both through the inverses, against the oracle."""
    import torch
    subs = [scgen.laplace_1d(n, dof=np.arange(0, n + 1, max(1, n // 7)), seed=n) for n in (1, 2, 15, 16, 17, 31, 33, 47, 62, 63,
                                                                                   64, 65, 79, 127, 139)]
    plan = _plan(subs, panel_width=width)
    p = torch.from_numpy(np.random.default_rng(6).uniform(-1, 1, plan.dual_total)).cuda()
    q = torch.zeros_like(p)
    plan.apply_implicit(p, q)
    for i, s in enumerate(subs):
        ref = oracle.schur(s)
        assert oracle.relF(plan.get_F(i), ref) <= 1e-12, s.n
        o = plan.query(i)["dual_offset"]
        x = ref @ p[o:o + s.m].cpu().numpy()
        assert np.linalg.norm(q[o:o + s.m].cpu().numpy() - x) <= 1e-12 * np.linalg.norm(x), s.n
    plan.destroy()
