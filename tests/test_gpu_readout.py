"""Read-out of the particles: packed on the device, in parts where the free
particle set is smaller than the FP64 result, copied in pieces."""
import numpy as np
import pytest

import synth
from pic_cases import by_id, log

pytestmark = pytest.mark.gpu


# few and many particles (a part of the store, one piece and several); rows
# that fill the caller's arrays and rows that do not (fewer particles loaded
# than the store's nominal count); both precisions; a store without spare room
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n,ppc,drop", [((8, 8), 1, 0), ((64, 48), 33, 0), ((64, 48), 33, 1000), ((16, 8, 24), 40, 7)])
def test_particles_come_back_as_loaded(n, ppc, drop, prec):
    """x to the rounding of the stored position (FP64 one ulp of the box,
    mixed 2^-24 of a cell), u to that of the stored momentum, ids exactly."""
    from paper_0808_4078_amd import pic
    log(f"case read-out {n} ppc {ppc} drop {drop} {prec}")
    wl = synth.beam_plasma(n, ppc=ppc, u_th_beam=0.3)
    parts = synth.load(wl)
    g, sp = pic.workload_descs(wl, precision=pic.PIC_PREC_FP64 if prec == "fp64" else pic.PIC_PREC_MIXED,
                               reserve=0.001, flags=pic.PIC_FLAG_HOST_LOAD | pic.PIC_FLAG_TRACK_IDS)
    r = pic.Run(g, sp)
    for s, p in enumerate(parts):
        m = p.id.size - drop
        r.load_particles(s, p.x[:, :m], p.u[:, :m], p.id[:m])
    L = np.array(wl.n)[:, None] * np.array(wl.d)[:, None]
    for s, p in enumerate(parts):
        m = p.id.size - drop
        x, u, ids = by_id(*r.read_particles(s))
        assert np.array_equal(ids, p.id[:m])
        dx = np.abs(x - p.x[:, :m])
        dx = np.minimum(dx, L - dx)
        assert np.all(dx <= (4e-16 * L if prec == "fp64" else 2.0 ** -24 * wl.d[0] + 4e-16 * L))
        assert np.all(np.abs(u - p.u[:, :m]) <= (0 if prec == "fp64" else 2.0 ** -24) * np.abs(p.u[:, :m]))
    r.step(1)
    for s, p in enumerate(parts):
        assert np.array_equal(np.sort(r.read_particles(s)[2]), p.id[:p.id.size - drop])
    r.close()
