"""Rounding of one FP64 push.  The reciprocal square roots and the reciprocal
of the rotation come from the hardware's estimates (about 24 bits) and one
correction; these bars lie 2^27 below what an uncorrected estimate would give."""
import numpy as np
import pytest

from pic_cases import by_id, log

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _push(x, u, B=None):
    from paper_0808_4078_amd import pic
    g, sp = pic.make_descs(2, (8, 8), (0.2, 0.2), 0.1, [dict(density=1.0, ppc=64)], precision=pic.PIC_PREC_FP64,
                           flags=pic.PIC_FLAG_HOST_LOAD | pic.PIC_FLAG_TRACK_IDS | pic.PIC_FLAG_FREEZE_FIELDS)
    r = pic.Run(g, sp)
    r.load_particles(0, x, u, np.arange(x.shape[1], dtype=np.uint32))
    if B is not None:
        full = np.zeros(r.field_shape)
        full[:] = np.asarray(B)[:, None, None, None]
        r.write_fields(None, full)
    r.step(1)
    out = by_id(*r.read_particles(0))
    r.close()
    return out


def test_velocity_of_free_particles():
    """From x = 0, u up to 1e6: x = dt u / gamma to 10 roundings (argument 2,
    reciprocal root 2, the products and the read-out 4, and 2 to spare)."""
    log("case fp64 free particles")
    rng = np.random.default_rng(11)
    u = np.abs(rng.normal(size=(3, 4096)))
    u *= 10.0 ** rng.uniform(-6, 6, 4096) / np.linalg.norm(u, axis=0)
    u[:, 0] = 0.0
    x, u1, _ = _push(np.zeros((2, 4096)), u)
    assert np.array_equal(u1, u)
    ul = u.astype(np.longdouble)
    ref = np.longdouble(0.1) * ul[:2] / np.sqrt(1 + (ul ** 2).sum(axis=0))
    err = np.abs(x - ref) / np.where(ref > 0, ref, 1)
    log(f"  worst {float(err.max()) / U:.2f} roundings")
    assert err.max() <= 10 * U


def test_rotation_keeps_the_momentum():
    """Uniform B, rotations by up to about 110 degrees: |u| kept to 16
    roundings (reciprocal 4, twice; the cross products 8)."""
    log("case fp64 rotation")
    rng = np.random.default_rng(12)
    u = rng.normal(size=(3, 4096)) * 10.0 ** rng.uniform(-3, 1, 4096)
    x = rng.uniform(0, 1.6, (2, 4096))
    _, u1, _ = _push(x, u, B=(9.0, -17.0, 21.0))
    a, b = (np.sqrt((v.astype(np.longdouble) ** 2).sum(axis=0)) for v in (u, u1))
    err = np.abs(b / a - 1)
    turn = np.degrees(np.arccos(np.clip((u * u1).sum(axis=0) / (np.linalg.norm(u, axis=0) * np.linalg.norm(u1, axis=0)),
                                        -1, 1)))
    log(f"  worst {float(err.max()) / U:.2f} roundings, turns up to {turn.max():.0f} degrees")
    assert turn.max() > 90
    assert err.max() <= 16 * U
