"""How a context runs its stages can be read and set: what a small context
starts with or the autotuner leaves is restored by the three set calls, on the
same context or another of the same boxes, with the same bits."""
import pytest
import torch

from paper_2405_02483_amd import inputs

pytestmark = pytest.mark.gpu


def _read(ctx):
    return ctx.get_launch() + (ctx.get_final_tile(), ctx.get_cells())


def _set(ctx, launch):
    ctx.set_launch(*launch[:2])
    ctx.set_final_tile(launch[2])
    ctx.set_cells(launch[3])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("tuned", [False, True])
def test_a_launch_read_is_a_launch_restored(tuned, dtype):
    from paper_2405_02483_amd.lib import Context
    f, box, prm = inputs.turbulent(n=24, seed=3)
    ctx, other = Context(box, prm, dtype=dtype), Context(box, prm, dtype=dtype)
    fd = ctx.upload([f])
    assert ctx.get_cells() == 1                    # a small context starts with it
    if tuned:
        ctx.autotune(fd, reps=2)
    saved = _read(ctx)
    want = [t.clone() for t in ctx.rhs(fd)]
    ctx.set_launch("16x16", 1)                     # the march, asked for
    assert _read(ctx) == ("16x16", 1, "16x16", 0)
    assert all(torch.equal(a, b) for a, b in zip(want, ctx.rhs(fd)))
    for c in (ctx, other):
        _set(c, saved)
        assert _read(c) == saved
        assert all(torch.equal(a, b) for a, b in zip(want, c.rhs(fd)))
    ctx.set_cells(1)
    ctx.set_final_tile("32x8")
    assert ctx.get_cells() == 0
    ctx.set_cells(1)
    ctx.set_tile("32x8")
    assert ctx.get_cells() == 0
    # the profile shows which passes ran: one thread per cell books no pass P
    for cells, p in ((1, 0), (0, 1)):
        ctx.set_cells(cells)
        ctx.profile(True)
        ctx.rhs(fd)
        assert (ctx.profile_read()["P"][1] > 0) == bool(p)
    ctx.close()
    other.close()


def test_contexts_that_march_only():
    from paper_2405_02483_amd.lib import Context, MhdError, MHD_EINVAL, MHD_EUNSUPPORTED, T_ALL, T_SMAG
    f, box, prm = inputs.turbulent(n=24, seed=3)
    for b, p in ((box, dict(prm, terms=T_ALL | T_SMAG, c_smag=0.1)), (dict(box, nx=128, ny=128, nz=128), prm)):
        ctx = Context(b, p, dtype=torch.float32)
        assert ctx.get_cells() == 0
        with pytest.raises(MhdError) as ei:
            ctx.set_cells(1)
        assert ei.value.code == MHD_EUNSUPPORTED
        ctx.set_cells(0)
        with pytest.raises(MhdError) as ei:
            ctx.set_cells(2)
        assert ei.value.code == MHD_EINVAL
        ctx.close()


def test_null_arguments():
    import ctypes
    from paper_2405_02483_amd import lib
    L = lib.load()
    v = ctypes.c_int32()
    assert L.mhd_set_cells(None, 0) == lib.MHD_EINVAL
    assert L.mhd_get_cells(None, ctypes.byref(v)) == lib.MHD_EINVAL


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_the_tables_follow_each_set_call(dtype):
    """Whatever shapes the passes had before, a shape gives what a new context
    set to it gives: RHS, step, time step and reductions."""
    from paper_2405_02483_amd.lib import Context, TILES
    (f, box, prm), (g, small, _) = inputs.turbulent(n=24, seed=3), inputs.turbulent(n=12, seed=4)
    boxes, fs = [box, small, box], [f, g, f]

    def results(ctx):
        fd = ctx.upload(fs)
        d = ctx.rhs(fd)
        red = ctx.reductions(fd, d)
        out = [t.clone() for t in d]
        ctx.step(fd, 0.0)
        return out + [t.clone() for t in fd], red, ctx.last_dt()

    ctx = Context(boxes, prm, dtype=dtype)
    for tile in TILES:
        for final in TILES:
            new = Context(boxes, prm, dtype=dtype)
            for c in (ctx, new):
                c.set_tile(tile)
                c.set_final_tile(final)
                assert c.get_launch()[0] == tile and c.get_final_tile() == final
            (a, ra, ta), (b, rb, tb) = results(ctx), results(new)
            assert all(torch.equal(x, y) for x, y in zip(a, b)) and ra == rb and ta == tb
            new.close()
    ctx.close()
