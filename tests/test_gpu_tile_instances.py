"""GPU tests of every compiled resident-tile instance (columns per lane, rows per
block), whichever of them the launcher's cost model picks: its launchers are called
with forced shapes on grids whose widths divide by 4, by 2 and are odd (edge tiles
with vectors, mirrored vectors and lanes that move column by column), under both
rules, with odd, even and deep passes and few and many wavefronts.  Plain passes of
each model and recording passes are bit for bit the one-step kernels'; reverse passes
give the streamed pairs' (lam, mu) bit for bit and sums within 1e-4 of the largest
(regrouped float32 sums, the bar two tilings are held to)."""
import ctypes as ct

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

GRIDS = [(75, 132), (70, 134), (67, 131)]
WAVES = (4, 6, 8, 10, 12, 16)
PLAIN = [(2, rw) for rw in range(1, 7)] + [(4, rw) for rw in range(2, 7)]
ADJ = [(cpl, rw) for cpl in (2, 4) for rw in (2, 3, 4)]
GENE = W.gene(Du=0.1, Dv=0.5)
FIELDS = ("dt", "a", "b", "eps", "c", "k3", "Du", "Dv")
GRAY_SCOTT = dict(dt=0.5, F=0.037, k=0.06, Du=0.2, Dv=0.1)
A = [[0.1, -0.2, 0.1], [0.3, 2.0, 0.3], [0.1, -0.2, 0.1]]  # mirror symmetric
B = [[-1.0] * 3, [-1.0, 8.0, -1.0], [-1.0] * 3]


class Shape(ct.Structure):
    _fields_ = [(k, ct.c_int) for k in ("cpl", "rw", "w", "K")]


class Gene(ct.Structure):
    _fields_ = [(k, ct.c_float) for k in FIELDS]


class Record(ct.Structure):
    _fields_ = [("at", ct.c_void_p), ("every", ct.c_int), ("first", ct.c_bool)]


class Planes(ct.Structure):
    _fields_ = [(k, ct.c_void_p) for k in ("in_l", "in_m", "out_l", "out_m")]


class Geom(ct.Structure):
    _fields_ = [(k, ct.c_int) for k in ("cpl", "depth", "kpad", "wout", "h", "nstrips", "nsegs",
                                        "ntiles", "per_xcd")] + [("paired", ct.c_bool),
                                                                 ("anchored", ct.c_bool)]


def _fn(name, *args, res=ct.c_int):
    from paper_2102_10340_amd import _lib
    f = getattr(_lib.lib, name)
    f.argtypes, f.restype = args, res
    return f


P, I, Q = ct.c_void_p, ct.c_int, ct.c_longlong


def _gene():
    return Gene(*[GENE[k] for k in FIELDS])


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _shapes(cpl, rw, depths, most=16):
    """Shapes of each depth with the fewest wavefronts that leave output rows, and
    with the most."""
    for K in depths:
        few = next(w for w in WAVES if 2 * w * rw - 2 * K > 0)
        for w in {few, most}:
            yield Shape(cpl, rw, w, K)


def _rand(shape, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(shape, generator=gen, device="cuda") * 2 - 1


@pytest.mark.parametrize("model", ["fhn", "gray_scott", "cnn"])
@pytest.mark.parametrize("cpl,rw", PLAIN)
def test_plain_instances_bitwise(cpl, rw, model):
    from paper_2102_10340_amd import Simulation
    if model == "fhn":
        launch = _fn("_ZN2rd11launch_tileEPKfPfiiiRKNS_4GeneERKNS_9TileShapeEP12ihipStream_tPKNS_"
                     "10TileRecordE", P, P, I, I, I, P, P, P, P)
        g, extra = _gene(), (None,)
    else:
        name = "14launch_tile_gs" if model == "gray_scott" else "15launch_tile_cnn"
        launch = _fn(f"_ZN2rd{name}EPKfPfiiiS1_RKNS_9TileShapeEP12ihipStream_t", P, P, I, I, I, P,
                     P, P)
        flat = list(GRAY_SCOTT.values()) if model == "gray_scott" else \
            [0.1] + sum(A, []) + sum(B, []) + [-0.5]
        g, extra = (ct.c_float * 20)(*flat), ()
    for (R, C) in GRIDS:
        for bc, rule in ((0, "periodic"), (1, "zeroflux")):
            x, y = _rand((R, C), R), _rand((R, C), C)
            sim = Simulation.from_state(x, y, GENE, rule, tuned=False) if model == "fhn" else \
                Simulation.gray_scott(x, y, bc=rule, **GRAY_SCOTT) if model == "gray_scott" else \
                Simulation.cnn(x, y, A, B, -0.5, 0.1, rule)
            sim.set_kernel(*((1,) if model == "fhn" else (2, 1, 1, 0)))
            start, want = sim.state().clone(), {}
            for K in range(1, 13):
                sim.step(1)
                want[K] = sim.state().clone()
            sim.close()
            for sh in _shapes(cpl, rw, (1, 5, 6, 12)):
                print(f"case tile {model} {cpl}x{rw} w={sh.w} K={sh.K} {R}x{C} {rule}", flush=True)
                out = torch.full((2, R, C), 7.0, device="cuda")
                assert launch(start.data_ptr(), out.data_ptr(), R, C, bc, ct.byref(g), ct.byref(sh),
                              _stream(), *extra) == 0
                assert torch.equal(out, want[sh.K]), (sh.w, sh.K, R, C, rule)


@pytest.mark.parametrize("cpl,rw", PLAIN)
def test_recording_instances_bitwise(cpl, rw):
    from paper_2102_10340_amd import Simulation
    launch = _fn("_ZN2rd11launch_tileEPKfPfiiiRKNS_4GeneERKNS_9TileShapeEP12ihipStream_tPKNS_"
                 "10TileRecordE", P, P, I, I, I, P, P, P, P)
    g = _gene()
    for (R, C) in GRIDS:
        for bc, rule in ((0, "periodic"), (1, "zeroflux")):
            sim = Simulation(_rand((R, C), R), GENE, rule, tuned=False)
            sim.set_kernel(1)
            want = [sim.state().clone()]
            for _ in range(12):
                sim.step(1)
                want.append(sim.state().clone())
            sim.close()
            for sh in _shapes(cpl, rw, (1, 5, 6, 12)):
                for every, first in ((1, True), (2, False)):
                    print(f"case tile record {cpl}x{rw} w={sh.w} K={sh.K} {R}x{C} {rule} "
                          f"every={every} first={first}", flush=True)
                    n = (sh.K + 1) // 2
                    out = torch.full((2, R, C), 7.0, device="cuda")
                    rec = torch.full((n * every, 2, R, C), 7.0, device="cuda")
                    to = Record(rec.data_ptr(), every, first)
                    assert launch(want[0].data_ptr(), out.data_ptr(), R, C, bc, ct.byref(g),
                                  ct.byref(sh), _stream(), ct.byref(to)) == 0
                    assert torch.equal(out, want[sh.K])
                    for i in range(n * every):
                        kept = i % every == 0 and (i > 0 or first)
                        assert torch.equal(rec[i], want[2 * i // every]) if kept else \
                            torch.all(rec[i] == 7.0), (i, sh.w, sh.K)


@pytest.mark.parametrize("lams", [False, True])
@pytest.mark.parametrize("cpl,rw", ADJ)
def test_reverse_instances_match_streamed(cpl, rw, lams):
    tile = _fn("_ZN2rd19launch_tile_adjointERKNS_9AdjPlanesEPKfixiiiRKNS_4GeneERKNS_9TileShapeEPdbP"
               "12ihipStream_t", P, P, I, Q, I, I, I, P, P, P, ct.c_bool, P)
    pairs = _fn("_ZN2rd19launch_adjoint_pairERKNS_9AdjPlanesEPKfixiiiRKNS_4GeneERKNS_10StreamGeomEPd"
                "bP12ihipStream_t", P, P, I, Q, I, I, I, P, P, P, ct.c_bool, P)
    geometry = _fn("_ZN2rd15stream_geometryEiiiiiPNS_10StreamGeomE", I, I, I, I, I, P,
                   res=ct.c_bool)
    g = _gene()
    for (R, C) in GRIDS:
        for bc, rule in ((0, "periodic"), (1, "zeroflux")):
            states, adj = _rand((3, 2, R, C), R), _rand((2, R, C), C)
            for K in (2, 6):
                geom, want = Geom(), torch.empty_like(adj)
                assert geometry(R, C, 1, K, 0, ct.byref(geom))
                sums = torch.zeros((geom.ntiles, 8), dtype=torch.float64, device="cuda")
                io = Planes(adj[0].data_ptr(), adj[1].data_ptr(), want[0].data_ptr(),
                            want[1].data_ptr())
                assert pairs(ct.byref(io), states.data_ptr(), 1, K, R, C, bc, ct.byref(g),
                             ct.byref(geom), sums.data_ptr(), lams, _stream()) == 0
                want_sums = sums.sum(0).cpu().numpy()
                for sh in _shapes(cpl, rw, (K,), most=8):
                    print(f"case tile reverse {cpl}x{rw} lams={lams} w={sh.w} K={K} {R}x{C} {rule}",
                          flush=True)
                    h, wout = 2 * sh.w * rw - 2 * K, 32 * cpl - 2 * (-(-K // cpl) * cpl)
                    tiles = -(-R // h) * -(-C // wout)
                    out = torch.full_like(adj, 7.0)
                    sums = torch.zeros((tiles * sh.w, 8), dtype=torch.float64, device="cuda")
                    io = Planes(adj[0].data_ptr(), adj[1].data_ptr(), out[0].data_ptr(),
                                out[1].data_ptr())
                    assert tile(ct.byref(io), states.data_ptr(), 1, K, R, C, bc, ct.byref(g),
                                ct.byref(sh), sums.data_ptr(), lams, _stream()) == 0
                    assert torch.equal(out, want), (sh.w, K, R, C, rule)
                    got = sums.sum(0).cpu().numpy()
                    assert np.all(np.abs(got - want_sums) <= 1e-4 * np.abs(want_sums).max())
