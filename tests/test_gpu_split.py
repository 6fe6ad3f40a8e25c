"""Grids with few tiles, whose tiles are shared by several workgroups of the
particle kernel (launch shape 0), against the same run in launch shape 1,
which takes one workgroup per tile: in mixed precision the current does not
depend on the split (FP64 sums of FP32 terms, rounded once per tile), so
fields and particles are equal bit for bit.  Also FP64 against the oracle."""
import numpy as np
import pytest

import synth
from pic_cases import by_id, gpu_run, log, oracle_run, rel_err, stack

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pic():
    from paper_0808_4078_amd import pic as p
    p.lib()
    return p


def _run(pic, wl, tile, shape, reserve=0.0):
    g, sp = pic.workload_descs(wl, precision=pic.PIC_PREC_MIXED, tile=tile, diag_every=1, shape=shape,
                               reserve=reserve, flags=pic.PIC_FLAG_TRACK_IDS)
    return pic.Run(g, sp)


def _same(a, b, ns=2):
    for x, y in zip(a.read_fields(), b.read_fields()):
        assert np.array_equal(x, y)
    for s in range(ns):
        for x, y in zip(by_id(*a.read_particles(s)), by_id(*b.read_particles(s))):
            assert np.array_equal(x, y)


# one tile; tile counts that are and are not multiples of the 8 XCDs; parts
# with few or no particles; every tile edge; re-layouts (a reserve of 64 slots)
@pytest.mark.parametrize("n,tile,ppc,reserve", [
    ((16, 16), 16, 40, 0.0), ((8, 8), 8, 9, 0.0), ((24, 24), 8, 33, 0.0), ((32, 32), 32, 5, 0.0),
    ((64, 48), 16, 16, 0.001), ((72, 200), 8, 11, 0.001), ((16, 8, 24), 8, 8, 0.001)])
def test_split_equals_unsplit(pic, n, tile, ppc, reserve):
    log(f"case split {n} tile {tile} ppc {ppc} reserve {reserve}")
    wl = synth.beam_plasma(n, ppc=ppc, u_th_beam=0.5, u_th_plasma=0.2, nu=0.2)
    a, b = _run(pic, wl, tile, 0, reserve), _run(pic, wl, tile, 1, reserve)
    for k in (1, 29):
        a.step(k)
        b.step(k)
        _same(a, b)
    ha, hb = a.history(), b.history()
    assert [h["collisions"] for h in ha] == [h["collisions"] for h in hb]
    assert all(np.array_equal(x["n_particles"], y["n_particles"]) for x, y in zip(ha, hb))
    assert max(abs(x["kinetic"] - y["kinetic"]).max() / abs(y["kinetic"]).max() for x, y in zip(ha, hb)) < 1e-13
    if reserve:
        assert a.diagnostics()["rebins"] > 0
    a.close()
    b.close()


def test_split_run_in_and_out_of_a_batch(pic):
    """A batch steps its members with one workgroup per tile: steps alone,
    in a batch and alone again go on from the same state."""
    log("case split in and out of a batch")
    wl = synth.beam_plasma((64, 64), ppc=16, u_th_beam=0.3, nu=0.1)
    a, b = _run(pic, wl, 16, 0), _run(pic, wl, 16, 1)
    a.step(5)
    batch = pic.Batch([a])
    batch.step(5)
    batch.close()
    a.step(5)
    b.step(15)
    _same(a, b)
    a.close()
    b.close()


@pytest.mark.parametrize("n,tile,ppc", [((48, 48), 16, 12), ((32, 32), 32, 7), ((8, 16, 8), 8, 9)])
def test_split_fp64_against_the_oracle(pic, n, tile, ppc):
    """20 steps, the FP64 bar of the edge cases (1e-9; differences are the
    order of FP64 sums, about 1e-13)."""
    log(f"case split fp64 {n} tile {tile} ppc {ppc}")
    wl = synth.beam_plasma(n, ppc=ppc, u_th_beam=0.4, u_th_plasma=0.1, nu=0.1)
    parts = synth.load(wl)
    orc = oracle_run(wl, parts)
    orc.step(20)
    g = gpu_run(wl, parts, pic.PIC_PREC_FP64, tile=tile)
    g.step(20)
    E, B, _ = g.read_fields()
    err = rel_err(stack(E, B), stack(orc.f.E, orc.f.B))
    log(f"  fields {err:.2e}")
    g.close()
    assert err < 1e-9


@pytest.mark.parametrize("n,tile", [((48, 32), 16), ((16, 8, 16), 8)])
def test_counts_of_steps_in_one_call(pic, n, tile):
    """Calls of one to eleven steps (replays of four steps and of one) against
    as many steps launched kernel by kernel: the same bits."""
    log(f"case steps per call {n}")
    wl = synth.beam_plasma(n, ppc=8, u_th_beam=0.3, nu=0.1)
    a = _run(pic, wl, tile, 0)
    g, sp = pic.workload_descs(wl, precision=pic.PIC_PREC_MIXED, tile=tile, diag_every=1,
                               flags=pic.PIC_FLAG_TRACK_IDS | pic.PIC_FLAG_NO_GRAPH)
    b = pic.Run(g, sp)
    done = 0
    for k in (1, 3, 4, 5, 8, 11):
        a.step(k)
        b.step(k)
        done += k
        _same(a, b)
        ia, ib = a.info(), b.info()
        assert ia["graph_launches"] == ib["direct_steps"] == ia["steps_enqueued"] == done
        assert a.diagnostics()["step"] == b.diagnostics()["step"]
    a.close()
    b.close()


@pytest.mark.parametrize("n,batch", [((1024, 2048), False), ((1032, 2048), False), ((1024, 2048), True),
                                     ((1032, 2048), True)])
def test_field_passes_of_large_grids(pic, n, batch):
    """Both sides of the grid size (2^21 cells) up to which the field passes are
    fused, alone and as an ensemble: 3 steps against the oracle, FP64 to 1e-9."""
    log(f"case field passes {n} batch {batch}")
    wl = synth.beam_plasma(n, ppc=1, u_th_beam=0.4, u_th_plasma=0.1, nu=0.1)
    parts = synth.load(wl)
    orc = oracle_run(wl, parts)
    orc.step(3)
    g = gpu_run(wl, parts, pic.PIC_PREC_FP64, tile=8)
    if batch:
        b = pic.Batch([g])
        b.step(3)
        b.close()
    else:
        g.step(3)
    E, B, _ = g.read_fields()
    err = rel_err(stack(E, B), stack(orc.f.E, orc.f.B))
    log(f"  fields {err:.2e}")
    assert err < 1e-9
    g.close()
