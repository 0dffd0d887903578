"""The planner's choices for products with prefix groups, on the CPU: the
planner is compiled for the host and asked for its plans."""
import json
import os
import subprocess

import numpy as np
import pytest

from paper_1303_7425_amd import build as B
from paper_1303_7425_amd import workloads as W

RINGS = {"modp": 0, "f64": 1, "i64": 2, "modq": 3}
EMPTY, COMBINE, RAW, DENSE, IVAL, BKT, GRP, GRPD, TINY = range(9)


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_report")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "plan_report.cpp")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", B.CSRC, src,
                           os.path.join(B.CSRC, "pm_plan.cpp"), "-o", exe])

    def run(*products, tuned=None):
        got = subprocess.run([exe, "plan"] + ([tuned] if tuned else []), input="\n".join(products), capture_output=True, text=True, check=True).stdout
        return [json.loads(ln) for ln in got.splitlines()]
    run.exe = exe
    return run


def line(f, g, ring, tile_cfg=-1, combine=-1, tiny=0):
    """A product's sizes, ranges and group counts as plan_report reads them."""
    nv, bits = f.layout.nvars, f.layout.bits
    cols = []
    for p in (f, g):
        e = W.unpack(p.keys, nv, bits)
        diff = p.keys[1:] ^ p.keys[:-1]
        cnt = [1 + int(np.count_nonzero(diff >> np.uint64((nv - 1 - v) * bits))) for v in range(nv)]
        cols.append((e.min(0), e.max(0), cnt))
    (fl, fh, fc), (gl, gh, gc) = cols
    per = " ".join(f"{fl[v]} {fh[v]} {gl[v]} {gh[v]} {fc[v]} {gc[v]}" for v in range(nv))
    return f"{nv} {bits} {RINGS[ring]} {len(f)} {len(g)} {tile_cfg} {combine} {tiny} {per}"


def simplex(nvars, n, bits):
    """All monomials of degree at most n, coefficients one."""
    rows = [()]
    for _ in range(nvars):
        rows = [r + (x,) for r in rows for x in range(n - sum(r) + 1)]
    e = np.array(rows)
    return W.Poly(W.Layout(nvars, bits, "modp"), np.sort(W.pack(e, nvars, bits)), np.ones(len(e), np.uint64))


def ragged_box(bits=16):
    """Exponents 0..1000 x 0..4 x 0..14 x 0..14, eight terms per prefix."""
    rng = W.rng_for(3)
    e = [(x, y, z, t) for x in range(1001) for y in range(5) for z, t in rng.integers(0, 15, (8, 2))]
    e += [(0, 0, 0, 0), (1000, 4, 14, 14)]
    keys = np.unique(W.pack(np.array(e), 4, bits))
    return W.Poly(W.Layout(4, bits, "modp"), keys, np.ones(len(keys), np.uint64))


def test_cut_of_a_run_tiles_it_and_fits_the_cells(report):
    got = subprocess.run([report.exe, "runs"], capture_output=True, text=True)
    assert got.returncode == 0, got.stdout


# degree boxes whose runs do not divide into whole bins of cells: with as many
# work items as cells ask for, the widest one had 4147, 4205, 4374 and 4205
@pytest.mark.parametrize("ring", ["modp", "i64", "modq"])
def test_boxes_whose_runs_do_not_divide_evenly(report, ring):
    for p in (simplex(3, 71, 8), ragged_box(), simplex(5, 13, 8), simplex(5, 14, 8), simplex(3, 70, 8), simplex(4, 30, 8)):
        (r,) = report(line(p, p, ring))
        assert r["mode"] == GRPD
        assert -(-r["K"] // r["least"]) * r["S"] <= r["cells"]
        assert r["ibound"] >= r["nbins"] // r["K"] * r["least"]


def test_explicit_sparse_modes_run_what_they_name(report):
    # the sparse family and a dense one without its box form groups that pay;
    # a requested mode is taken all the same
    f, g = W.config3("modp", n=8)
    for ring, auto in (("modp", GRP), ("i64", GRP), ("f64", GRP)):
        got = report(*(line(W.config3("modp", n=12)[0], W.config3("modp", n=12)[1], ring, combine=c) for c in (-1, 3, 2, 0)))
        assert [r["mode"] for r in got] == [auto, BKT, IVAL, RAW]
    got = report(*(line(f, g, "modp", combine=c) for c in (-1, 3, 2, 1, 0)))
    assert [r["mode"] for r in got] == [GRP, BKT, IVAL, COMBINE, RAW]
    small = W.random_sparse(W.rng_for(1), 57, 6, 10, 15, "modp"), W.random_sparse(W.rng_for(2), 61, 6, 10, 15, "modp")
    got = report(*(line(*small, "modp", combine=c, tiny=1) for c in (-1, 3, 0)))
    assert [r["mode"] for r in got] == [TINY, BKT, RAW]
    box = simplex(4, 12, 8)
    got = report(*(line(box, box, "modp", tile_cfg=t) for t in (-1, 0, 2)))
    assert [r["mode"] for r in got] == [GRPD, DENSE, DENSE]


def test_remembered_choices_leave_automatic_paths_alone(report, tmp_path):
    # choices among the explicit settings, as files of before hold them, do not
    # switch the single workgroup or prefix groups off; one that was timed
    # against them does, for its own class; a box's choice is no sparse mode
    sparse = W.config3("modp", n=8)
    small = W.random_sparse(W.rng_for(1), 57, 6, 10, 15, "f64"), W.random_sparse(W.rng_for(2), 61, 6, 10, 15, "f64")
    box, other = simplex(4, 12, 8), (W.random_sparse(W.rng_for(1), 1820, 12, 5, 3, "modp"), W.random_sparse(W.rng_for(2), 1820, 12, 5, 3, "modp"))
    cases = [line(*sparse, "modp"), line(*small, "f64", tiny=1), line(box, box, "modp")]
    log2 = [(len(f) * len(g)).bit_length() - 1 for f, g in (sparse, small, (box, box))]

    def modes(lines, *products):
        path = tmp_path / "tune.txt"
        path.write_text("\n".join(lines) + "\n")
        return [r["mode"] for r in report(*products, tuned=str(path))]

    auto = [GRP, TINY, GRPD]
    old = [f"0 0 {log2[0]} -1 0 1", f"1 0 {log2[1]} -1 0 1", f"0 1 {log2[2]} 1 0 -1"]
    assert modes(["# none"], *cases) == auto
    assert modes(old, *cases) == auto
    assert modes([o + " 1" for o in old], *cases) == [RAW, RAW, DENSE]
    assert modes([f"0 0 {log2[0] + 1} -1 0 1 1", f"0 1 {log2[0]} 1 0 -1 1"], *cases) == auto
    # without groups, the remembered mode is taken; a dense class's is not
    k = (len(other[0]) * len(other[1])).bit_length() - 1
    free = report(line(*other, "modp"))[0]["mode"]
    assert free not in (GRP, GRPD)
    assert modes([f"0 0 {k} -1 1 1"], line(*other, "modp")) == [COMBINE]
    assert modes([f"0 1 {k} -1 1 1"], line(*other, "modp")) == [free]


def lattice(shape, share=1.0, bits=16):
    """All exponent vectors below `shape` (a share of them), coefficients one."""
    e = np.indices(shape).reshape(len(shape), -1).T
    if share < 1:
        keep = W.rng_for(5).uniform(size=len(e)) < share
        keep[0] = keep[-1] = True
        e = e[keep]
    return W.Poly(W.Layout(len(shape), bits, "modp"), np.sort(W.pack(e, len(shape), bits)), np.ones(len(e), np.uint64))


def test_boxes_of_single_terms(report):
    # one term to a prefix: bins of a whole variable where there are enough of
    # them, a thread per term else, and the tile kernel for full lattices
    pairs = {"square": (lattice((100, 100)),) * 2, "tenth": (lattice((300, 300), 0.1),) * 2, "slab": (lattice((10, 1000)),) * 2,
             "line": (lattice((20000,), bits=32),) * 2, "sparse line": (lattice((100000,), 0.1, bits=32),) * 2,
             "few by many": (lattice((1000,), bits=32), lattice((1000000,), bits=32)), "simplex": (simplex(2, 300, 16),) * 2,
             "four variables": (simplex(4, 20, 16),) * 2}
    got = dict(zip(pairs, report(*(line(f, g, "modp") for f, g in pairs.values()))))
    want = {"square": (GRPD, 199, 0), "tenth": (GRPD, 599, 0), "slab": (DENSE, 0, 0), "line": (DENSE, 0, 0),
            "sparse line": (GRPD, 1, 1), "few by many": (GRPD, 1, 0), "simplex": (GRPD, 601, 0), "four variables": (GRPD, 41, 0)}
    assert {k: (r["mode"], r["S"], r["rows"]) for k, r in got.items()} == want


def random_pair(nvars, bits, top, na, nb, ring):
    return tuple(W.random_sparse(W.rng_for(m), m, nvars, bits, top, ring) for m in (na, nb))


def test_f64_products_whose_work_items_cost_more_than_the_sort(report):
    # thousands of non-empty bins of few pairs, a term or two to a block, few
    # waves for wide bins: pair-index sort; blocks of many pairs: prefix groups
    cases = {(5, 12, 30, 16, 300000): RAW, (6, 10, 7, 3000, 3000): RAW, (3, 20, 60, 1000, 20000): RAW, (3, 21, 400, 16, 1000000): RAW,
             (4, 15, 15, 3000, 3000): GRP, (5, 12, 10, 8000, 8000): GRP, (7, 9, 6, 300, 100000): GRP}
    got = report(*(line(*random_pair(*c, "f64"), "f64") for c in cases))
    assert [r["mode"] for r in got] == list(cases.values())
    got = report(*(line(*W.config3("modp", n=n), "f64") for n in (9, 10, 12)))
    assert [r["mode"] for r in got] == [GRP] * 3


def test_sparser_products_beyond_32_bit_keys(report):
    # box of 7^12 cells: a listed work item per key span, most of them nearly
    # empty; the same sizes within 31^6 and 15^8 cells
    cases = {(12, 5, 3, 300, 20000): RAW, (12, 5, 3, 5000, 5000): RAW, (6, 10, 15, 300, 20000): GRP, (8, 7, 7, 5000, 5000): GRP}
    got = report(*(line(*random_pair(*c, "modp"), "modp") for c in cases))
    assert [r["mode"] for r in got] == list(cases.values())


def test_bins_of_more_pairs_than_cells(report):
    # 5^8 exponents: a prefix of four variables (bins of 1372 pairs) instead of
    # three (12346, three rounds of ranks)
    (r,) = report(line(*random_pair(8, 7, 4, 3000, 3000, "modp"), "modp"))
    assert (r["mode"], r["S"]) == (GRP, 6561)


def test_products_of_few_bins(report):
    # three leading exponents each: five non-empty bins, however many pairs;
    # a whole range of them keeps the prefix groups
    def slabs(shape, step):
        e = np.indices(shape).reshape(len(shape), -1).T * np.array(step)
        return W.Poly(W.Layout(2, 16, "modp"), np.sort(W.pack(e, 2, 16)), np.ones(len(e), np.uint64))

    few = slabs((3, 460), (500, 7)), slabs((3, 2870), (500, 1))
    box = slabs((3, 400), (200, 1)), slabs((3, 400), (200, 1))
    many = slabs((60, 23), (25, 7)), slabs((60, 140), (25, 1))
    got = report(line(*few, "modp"), line(*box, "modp"), line(*many, "modp"), line(*few, "f64"), line(*many, "f64"))
    assert [r["mode"] for r in got] == [BKT, DENSE, GRPD, RAW, GRP]


def test_small_blocks_far_apart(report):
    # clusters: blocks of 14 pairs whose prefixes fill a few thousandths of
    # their ranges are listed; blocks of 22 are not
    rng = W.rng_for(3)

    def clusters(count, n, shape, width):
        c = rng.integers(0, shape, (count, 2))
        e = np.concatenate([c[rng.integers(0, count, n)], rng.integers(0, width, n)[:, None]], 1)
        keys = np.unique(W.pack(e, 3, 16))
        return W.Poly(W.Layout(3, 16, "modp"), keys, np.ones(len(keys), np.uint64))

    near = clusters(1000, 2800, (300, 300), 93), clusters(1000, 5600, (300, 300), 93)
    far = clusters(1600, 4000, (480, 700), 60), clusters(1600, 8000, (480, 700), 60)
    got = report(line(*far, "modp"), line(*near, "modp"))
    assert [(r["mode"], r["rows"] != 0) for r in got] == [(GRP, True), (GRP, False)]
