"""The phantom builder's culling of far voxels and beamlets: geometries at the
edges of its runs (64 rows) and groups of runs (4,096 rows), with one and two
beams, kernels that reach everything or a single voxel, strong attenuation
and coarse tissue.  Sparsity and structure ids bit for bit against the
brute-force oracle, values within one float32 ulp (the exponential's own
rounding)."""
import dataclasses

import numpy as np
import pytest

from gpu_util import banner, f32_ulp_diff
from oracle import phantom
from workloads import PhantomSpec

pytestmark = pytest.mark.gpu

BASE = PhantomSpec(name="base", nx=16, ny=16, nz=8, h=4.0, r_ptv=11.3, r_rectum=4.7, r_bladder=8.1, n_beams=3,
                   beamlet=5.0, sigma=3.0, tau=0.005)


def variant(name, **kw):
    return dataclasses.replace(BASE, name=name, **kw)


SPECS = [
    variant("one_partial_run", nx=5, ny=3, nz=1),
    variant("one_run", nx=4, ny=4, nz=4),
    variant("one_row_past_a_run", nx=13, ny=5, nz=1),
    variant("one_group", nx=16, ny=16, nz=16),
    variant("one_row_past_a_group", nx=17, ny=241, nz=1),
    variant("one_beam", n_beams=1),
    variant("two_beams", n_beams=2, nx=15),
    variant("peaks_only", tau=1.0),
    variant("near_peaks", tau=0.99),
    variant("strong_attenuation", mu=0.3),
    variant("no_attenuation", mu=0.0),
    variant("narrow_kernel", sigma=0.2),
    # every run near every beamlet: 18 groups, more than are listed at a time
    variant("reaches_everything", nx=64, ny=48, nz=24, sigma=200.0, beamlet=10.0),
    variant("coarse", nx=18, ny=14, nz=9, coarse_normal=True),
]


@pytest.mark.parametrize("tiles", [1, 0], ids=["voxel_tiles", "api_order"])
@pytest.mark.parametrize("spec", SPECS, ids=lambda s: s.name)
def test_culled_builder_matches_oracle(spec, tiles):
    from paper_0908_4421_amd.imrt import Context, Dose
    banner(f"culled build {spec.name} tiles={tiles}")
    want = phantom.build_dose_matrix(spec)
    lib = Dose.from_geometry(Context(0, voxel_tiles=tiles), spec)
    assert (lib.nv, lib.nb, lib.nnz) == (want.nv, want.nb, want.nnz)
    ex = lib.export(structures=True)
    assert np.array_equal(ex["struct_id"], want.struct_id)
    assert np.array_equal(ex["row_ptr"], want.csr.indptr) and np.array_equal(ex["col_idx"], want.csr.indices)
    assert np.array_equal(ex["col_ptr"], want.csc.indptr) and np.array_equal(ex["row_idx"], want.csc.indices)
    assert f32_ulp_diff(ex["val"], want.csr.data) <= 1 and f32_ulp_diff(ex["cval"], want.csc.data) <= 1
