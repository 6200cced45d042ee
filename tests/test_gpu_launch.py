"""Launch shapes of the fused query: workgroup size by the number of pixels
and the order of the tiles over the XCDs.  A launch shape only decides which
wave computes a pixel, so every shape gives the same bits."""
import numpy as np
import pytest

from niv_synth import get_workload, make_params, unit_cube_queries

pytestmark = pytest.mark.gpu


def _setup(name, n, prec):
    import torch
    from paper_2602_12949_amd import NIV
    w = get_workload(name)
    m = NIV(w.model_dict())
    params = make_params(m.n_grid_values, m.mat_shapes(), w.param_seed, *w.grid_init)
    pos, nrm = unit_cube_queries(n, 11)
    pos *= np.asarray(w.aabb_max, np.float32)
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    return m, m.prepare(t(params), prec), t(pos), t(nrm), (0.37,) * w.n_extra


# chunks of 64 pixels around the steps of the default shape (256, 512 and
# 1024 chunks: workgroups of 64, 128, 256 and 512 threads) and a count whose
# tiles end inside a strip of the last round
@pytest.mark.parametrize("n", [1, 65, 64 * 256, 64 * 256 + 1, 64 * 512 + 1, 64 * 1024, 64 * 1024 + 1,
                               64 * 8 * (8 * 32 + 33) + 5])
@pytest.mark.parametrize("name,prec", [("room_1080p", "fp16"), ("unit_cube_16k", "fp32"), ("room_1080p_g4", "bf16"),
                                       ("room_1080p_pe32", "fp16")])
def test_launch_shapes_give_the_same_bits(name, prec, n):
    import torch
    m, model, pos, nrm, extra = _setup(name, n, prec)
    E, _, flags = m.query(pos, nrm, model, prec, extra=extra)
    assert torch.isfinite(E).all()
    for shape in ((512, 0, 0), (512, 0, 1), (256, 1, 1), (512, 2, 1)):
        m.set_tune(prec, *shape)
        E2, _, flags2 = m.query(pos, nrm, model, prec, extra=extra)
        assert torch.equal(E, E2) and torch.equal(flags, flags2), shape


@pytest.mark.parametrize("n", [1, 64 * 1024, 64 * 1024 + 1])
def test_wide_field_default_shapes(n):
    import torch
    m, model, pos, nrm, extra = _setup("room_4k_6d", n, "bf16")
    E, _, flags = m.query(pos, nrm, model, "bf16", extra=extra)
    m.set_tune("bf16", 512, 0, 0)
    E2, _, flags2 = m.query(pos, nrm, model, "bf16", extra=extra)
    assert torch.isfinite(E).all() and torch.equal(E, E2) and torch.equal(flags, flags2)


# few tiles: strips shorter than 32, down to one tile (tiles of one chunk at
# these sizes: 8 and 16 tiles, then the ends of the ranges of each length)
@pytest.mark.parametrize("tiles", [8, 16, 64, 127, 128, 255, 256])
def test_short_strips_give_the_same_bits(tiles):
    import torch
    m, model, pos, nrm, extra = _setup("room_1080p", 64 * tiles - 1, "fp16")
    E, _, flags = m.query(pos, nrm, model, "fp16", extra=extra)
    for shape in ((512, 0, 0), (512, 0, 1), (256, 0, 1)):
        m.set_tune("fp16", *shape)
        E2, _, flags2 = m.query(pos, nrm, model, "fp16", extra=extra)
        assert torch.equal(E, E2) and torch.equal(flags, flags2), shape


@pytest.mark.parametrize("n", [64 * 3, 64 * 3 + 1])
def test_wide_field_fp32_small_shapes(n):
    import torch
    m, model, pos, nrm, extra = _setup("room_4k_6d", n, "fp32")
    E, _, flags = m.query(pos, nrm, model, "fp32", extra=extra)
    for shape in ((512, 0, 0), (256, 0, 0)):
        m.set_tune("fp32", *shape)
        E2, _, flags2 = m.query(pos, nrm, model, "fp32", extra=extra)
        assert torch.isfinite(E).all() and torch.equal(E, E2) and torch.equal(flags, flags2), shape
