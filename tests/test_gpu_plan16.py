"""The automatic plans of 16-bit storage on grids of 2^22 cells or more that
are no multiple of any tile: the stored bits and traces equal the naive
kernel's, and the plan fills rounds of the work-groups the GPU holds."""
import numpy as np
import pytest
import torch

from paper_2204_03775_amd import inputs

pytestmark = pytest.mark.gpu


def run(wave, p, dtype, variant, nt):
    prop = wave.Propagator(p.nx, p.ny, p.nz, p.h, p.k32(), src=p.src, rec=p.rec,
                           sponge_width=p.sponge_width, sponge_alpha=p.sponge_alpha, dtype=dtype)
    prop.configure(variant)
    prop.record(nt)
    prop.run(nt, torch.tensor(p.s[:nt], dtype=torch.float32, device="cuda"))
    cur, prev, _ = prop.fields()
    raw = [prop.padded(b).view(torch.int16).cpu().numpy().copy() for b in (cur, prev)]
    out = raw + [prop.traces.cpu().numpy()]
    cfg = prop.config()
    prop.close()
    return out, cfg


# one cell over 2^22, wide and flat, thin in x, and two rounds of small tiles
@pytest.mark.parametrize("shape", [(163, 161, 160), (476, 77, 181), (67, 259, 243), (203, 181, 157)])
@pytest.mark.parametrize("dtype", ["f16", "bf16uv"])
def test_plan_matches_naive_kernel(wave_mod, shape, dtype):
    nx, ny, nz = shape
    p = inputs.random_problem(nx, ny, nz, 6, seed=nx, sponge_width=5, nrec=16)
    print(f"case: {dtype} {shape}", flush=True)
    got, (v, zc, wg) = run(wave_mod, p, dtype, 0, p.nt)
    ref, _ = run(wave_mod, p, dtype, 1, p.nt)
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    name = wave_mod.wave_variant_name(v)
    assert name in ("t64x16_r1", "t128x32_r2")
    cap = torch.cuda.get_device_properties(0).multi_processor_count * (3 if name == "t64x16_r1" else 1)
    assert wg / (-(-wg // cap) * cap) > 0.6


# a z-chunk given with the tile shape left to the library: the shape is chosen
# for that chunk, not for the one the library would have taken
@pytest.mark.parametrize("shape,zc", [((256, 256, 256), 64), ((256, 256, 256), 256), ((512, 512, 256), 256)])
@pytest.mark.parametrize("dtype", ["f16", "bf16uv"])
def test_tile_shape_fits_a_given_chunk(wave_mod, shape, zc, dtype):
    nx, ny, nz = shape
    k = torch.full((1, 1, 1), 2.0, device="cuda").expand(nz, ny, nx)
    prop = wave_mod.Propagator(nx, ny, nz, (10.0, 10.0, 10.0), k, dtype=dtype)
    us = {}
    for variant in (0, "t64x16_r1", "t128x32_r2"):
        prop.configure(variant, zc)
        best = float("inf")
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            prop.run(4)
            e0.record()
            prop.run(20)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1) * 1e3 / 20)
        us[variant] = best
        if variant == 0:
            assert prop.config()[1] == zc
    prop.close()
    print(f"case: {dtype} {shape} chunk {zc}: {us}", flush=True)
    assert us[0] <= 1.2 * min(us.values())
