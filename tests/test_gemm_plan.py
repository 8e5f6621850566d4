"""The GEMM launch heuristic, asked on the host (CPU only: no compute call is made)."""
import pytest


def _lib():
    import os
    from paper_2401_12522_amd import binding, build
    if not os.path.exists(build.LIB_PATH):
        build.build_library()
    return binding.lib()


@pytest.mark.parametrize("m,n,k", [(106, 6144, 28672), (116, 6144, 23824), (131, 6128, 21416), (256, 2656, 17840), (139, 5984, 22840)])
def test_a_finer_cut_takes_no_shape_away_from_the_static_scratch(m, n, k):
    """Long-k products whose passes of 5 or 8 m-tiles fit the scratch of bita_gemm_noalloc with 5 k splits:
    the 12-tile form would need 8 and does not fit."""
    L = _lib()
    assert L.bita_gemm_noalloc_scratch_bytes(m, n, k) <= L.bita_gemm_noalloc_max_scratch_bytes()
