"""16-bit fixed-point storage (MCLBM_I16) on the GPU, through the C ABI: a
population of lattice l, direction i is stored as an integer v with
f = f_ref + v h / 32767, f_ref and h shared by the directions of a class (equal
|c_x|, |c_y|, |c_z|); the ranges are fitted to the initial state and fitted again
(with the state re-encoded) when a value passes 3/4 of its range, checked after
steps 1, 2, 4 and every multiple of 8. The collision is the FP32 one of the
16-bit floating-point storage. The paper fixes no storage precision: these tests hold
the format to the 1e-3 field-error bar against the FP64 oracle, and check the
range bookkeeping (checks that depend only on the step count, checkpoints, a
value that leaves its range)."""
import numpy as np
import pytest

from gpu_common import FIELDS, _CLS, _TUBE, _HDR, absolute_populations, decode_checkpoint, field_errors
from paper_2004_11286_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mc():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_11286_amd import mclbm

    return mclbm


def _crop():
    """A 32 x 64 x 16 crop of the shear layer (two interfaces of thickness 4, bands
    at +-0.1, H2/N2 mole fractions 0.9 and 0.1)."""
    return W.shear_layer(nx=32, ny=64, nz=16)


def test_initial_tables_hold_the_state(mc):
    """After initialisation every stored integer lies within half of its class's
    range (the range is twice the spread of the initial values); decoding the
    checkpoint gives the local equilibria to a fraction of a storage unit."""
    params, f = _crop()
    s = mc.Sim(params, mc.MCLBM_I16)
    s.init_fields(**f)
    hdr, vals = decode_checkpoint(s.save())
    m = s.read_moments()
    s.close()
    L = vals.shape[0]
    v = vals.reshape(L, 27, -1).astype(np.int64)
    for l in range(L):
        for k in range(8):
            top = int(np.abs(v[l][_CLS == k]).max())
            assert top <= 16400, (l, k, top)
    errs = {k: float(np.abs(m[k] - f[k]).max() / np.abs(f[k]).max()) for k in ("X", "u", "p", "T")}
    print("i16 init read-back", errs)
    for k in errs:
        assert errs[k] < 5e-4, (k, errs[k])


def test_shear_layer_crop_against_the_oracle(mc, oracle_mod):
    """The crop for 300 steps against the FP64 oracle: every field within the 1e-3
    bar (velocity against its maximum), the masses and the energy kept to 1e-4."""
    params, f = _crop()
    o = oracle_mod.OracleSim(params)
    o.init_fields(**f)
    o.step(300)
    om = o.read_moments()
    s = mc.Sim(params, mc.MCLBM_I16)
    s.init_fields(**f)
    c0 = s.conservation()
    s.step(300)
    g = s.read_moments()
    c1 = s.conservation()
    refits = s.range_refits()
    s.close()
    errs = field_errors(g, om)
    M = params["M"]
    print("i16 shear crop 300", errs, "refits", refits, "drift",
          np.abs(c1[:M + 1] / c0[:M + 1] - 1).max(), abs(c1[M + 4] / c0[M + 4] - 1))
    for k in FIELDS:
        assert errs[k] < 1e-3, (k, errs[k])
    np.testing.assert_allclose(c1[:M + 1], c0[:M + 1], rtol=1e-4)
    np.testing.assert_allclose(c1[M + 4], c0[M + 4], rtol=1e-4)


def test_split_calls_and_checkpoints_are_bitwise(mc):
    """100 steps of the crop in one call, in calls of 7, 50 and 43 steps, and from
    a checkpoint taken at step 57 (between two range checks) give the same state bit
    for bit: the checks fall on step counts fixed in advance and the checkpoint
    keeps the range flags."""
    params, f = _crop()

    def run(splits, save_at=None):
        s = mc.Sim(params, mc.MCLBM_I16)
        s.init_fields(**f)
        mid = None
        for n in splits:
            s.step(n)
            if s.step_count == save_at:
                mid = bytearray(s.save())
        out = bytes(s.save())
        refits = s.range_refits()
        s.close()
        return out, mid, refits

    a, _, ra = run([100])
    b, mid, rb = run([7, 50, 43], save_at=57)
    s = mc.Sim(params, mc.MCLBM_I16)
    s.load(mid)
    s.step(43)
    c = bytes(s.save())
    s.close()
    print("i16 refits in 100 steps", ra, rb)
    assert a == b
    assert a == c


def test_batch_tubes_evolve_as_alone_over_range_checks(mc):
    """A batch of five ragged ternary tubes over 100 steps (15 range checks)
    matches single contexts of the same tubes bit for bit: each tube's tables are
    fitted and refitted from its own state only."""
    tubes = W.tube_ensemble(ntubes=5, ny=4, nz=4, lmin=8, lmax=40, seed=21)
    b = mc.Batch([p for p, _ in tubes], mc.MCLBM_I16)
    b.init_fields([f for _, f in tubes])
    b.step(100)
    g = b.read_moments()
    b.close()
    for t, (params, f) in enumerate(tubes):
        s = mc.Sim(params, mc.MCLBM_I16)
        s.init_fields(**f)
        s.step(100)
        r = s.read_moments()
        s.close()
        for k in FIELDS:
            np.testing.assert_array_equal(g[t][k], r[k], err_msg=f"tube {t} {k}")


def test_value_out_of_range_is_an_error(mc):
    """Forced from the host: a checkpoint whose fixed-point factors were scaled so
    that a storage unit is a thousandth of what it was is loaded. The next
    collisions produce values far outside the ranges, the stores clamp, and
    mclbm_step reports MCLBM_ESTATE at the next range check; the context can be
    initialised and stepped again."""
    params, f = W.ternary_tube(nx=32, ny=4, nz=4)
    s = mc.Sim(params, mc.MCLBM_I16)
    s.init_fields(**f)
    s.step(5)
    buf = bytearray(s.save())
    tube = np.frombuffer(buf, dtype=_TUBE, count=1, offset=_HDR.itemsize).copy()
    tube["inv_qs"] /= 1000.0
    tube["qs"] *= 1000.0
    buf[_HDR.itemsize:_HDR.itemsize + _TUBE.itemsize] = tube.tobytes()
    s.load(buf)
    with pytest.raises(mc.MclbmError) as e:
        s.step(40)
    assert e.value.code == mc.MCLBM_ESTATE and "range" in str(e.value)
    s.init_fields(**f)
    s.step(40)
    assert np.isfinite(s.conservation()).all()
    s.close()


@pytest.mark.parametrize("nx,ny,nz", [(16, 16, 16), (16, 16, 17), (37, 53, 26)])   # 16, 17 and 200 blocks
def test_initial_ranges_see_the_last_node(mc, nx, ny, nz):
    """The range measurement takes 16 blocks to a workgroup: the grid's extreme value
    sits at its last node, and no stored value may pass half of its range."""
    params, f = W.shear_layer(nx=nx, ny=ny, nz=nz)
    f["p"] = np.array(f["p"])
    f["p"].reshape(-1)[-1] *= 1.2
    s = mc.Sim(params, mc.MCLBM_I16)
    s.init_fields(**f)
    _, vals = decode_checkpoint(s.save())
    p = s.read_moments()["p"].reshape(-1)
    s.close()
    v = vals.reshape(vals.shape[0], 27, -1).astype(np.int64)
    for l in range(v.shape[0]):
        for k in range(8):
            assert np.abs(v[l][_CLS == k]).max() <= 16400, (l, k)
    ref = f["p"].reshape(-1)[-1]
    assert abs(p[-1] - ref) < 5e-4 * ref


# blocks: 511 and 512 (one and two to a workgroup), 537 (two, a ragged last one), 4112 (sixteen, one left over)
@pytest.mark.parametrize("nx,ny,nz", [(16, 16, 511), (16, 16, 512), (37, 53, 70), (64, 64, 257)])
def test_initial_ranges_over_shared_workgroups(mc, nx, ny, nz):
    """The range measurement gives a workgroup one block to sixteen, by the number of blocks: the extreme
    pressure sits at the first node of the last block, and no stored value may pass half of its range."""
    params, f = W.shear_layer(nx=nx, ny=ny, nz=nz)
    n = nx * ny * nz
    at = (n - 1) // 256 * 256
    f["p"] = np.array(f["p"])
    f["p"].reshape(-1)[at] *= 1.2
    s = mc.Sim(params, mc.MCLBM_I16)
    s.init_fields(**f)
    _, vals = decode_checkpoint(s.save())
    p = s.read_moments()["p"].reshape(-1)
    s.close()
    v = vals.reshape(vals.shape[0], 27, -1)
    for l in range(v.shape[0]):
        for k in range(8):
            assert np.abs(v[l][_CLS == k].astype(np.int32)).max() <= 16400, (l, k)
    ref = f["p"].reshape(-1)[at]
    assert abs(p[at] - ref) < 5e-4 * ref
