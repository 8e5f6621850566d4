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


@pytest.mark.parametrize("m,n,k,splits", [(128, 22016, 4096, 1), (144, 22016, 4096, 1), (272, 12288, 4096, 1), (512, 22016, 4096, 1),
                                          (96, 22016, 4096, 1), (170, 4096, 11008, 5), (112, 1024, 4096, 8)])
def test_one_plane_is_planned_for_the_passes_it_runs(m, n, k, splits):
    """A single-plane launch has no tall form: its splits are those of passes of 5 m-tiles (or, for a small
    matrix up to 7 m-tiles, of the 8-tile form), not of a form that only two planes have."""
    import ctypes
    from paper_2401_12522_amd import binding as B
    L = _lib()
    one, two = B.gemm_plan_info(m, n, k, planes=1), B.gemm_plan_info(m, n, k)
    assert one["mt_pass"] == one["tall_tiles"] == 0 and one["splits"] == splits, one
    out4 = (ctypes.c_int32 * 4)()
    assert L.bita_gemm_plan_info(m, n, k, out4) == 0
    assert list(out4) == [two[f] for f in ("splits", "variant", "mt_pass", "ksteps_per_split")]
    frag = 2 * ((k + 31) // 32) * ((m + 15) // 16) * 1024
    for plan in (one, two):
        part = (plan["splits"] * m * n * 4 + 255) // 256 * 256 if plan["splits"] > 1 else 0
        assert L.bita_gemm_noalloc_scratch_bytes(m, n, k) >= part + frag
    assert L.bita_gemm_plan_detail(m, n, k, 3, out4) == -1


@pytest.mark.parametrize("m,n,k", [(150, 32000, 4096), (300, 32000, 5120), (440, 32000, 4096), (512, 27648, 5120), (240, 40960, 2048),
                                   (136, 16384, 17000), (160, 16384, 40000)])
@pytest.mark.parametrize("planes", [1, 2])
def test_passes_of_five_take_the_fewer_rounds(m, n, k, planes):
    """Many rows of 1024 to 2999 tiles: 16 waves per workgroup where 14 would take a round more on the 256 CUs, unless
    that means k splits, which the static scratch would have to hold."""
    from paper_2401_12522_amd import binding as B
    _lib().bita_tune_gemm(-2, -1)               # without the tall forms, which two planes may take instead
    try:
        plan = B.gemm_plan_info(m, n, k, planes)
    finally:
        _lib().bita_tune_gemm(-1, -1)
    passes, tiles = ((m + 15) // 16 + 4) // 5, n // 16
    rounds = {t: -(-(-(-tiles // t) * passes) // 256) for t in (14, 16)}
    splits = 256 // (-(-tiles // 16) * passes)
    assert plan["variant"] == (11 if splits > 1 or rounds[14] * (14 + 5 * planes) <= rounds[16] * (16 + 5 * planes) else 9), plan
    assert plan["mt_pass"] == 0 and plan["splits"] == 1


@pytest.mark.parametrize("m,n,k,variant,mt_pass,tiles,splits", [
    # a fifth or a seventh less than the other form
    (170, 22016, 4096, 12, 6, 12, 1), (84, 27648, 5120, 12, 6, 16, 2), (120, 27648, 5120, 12, 8, 16, 2), (204, 10240, 8192, 12, 7, 16, 3),
    (272, 15360, 5120, 9, 0, 0, 1), (340, 4096, 11008, 9, 0, 0, 3), (216, 10240, 8192, 9, 0, 0, 2),
    # more m-tiles executed than in passes of 5: a tenth less than those asks for, an eighth from 80 k-steps on
    (301, 32000, 8192, 9, 0, 0, 1), (300, 32000, 5120, 9, 0, 0, 1), (460, 40960, 2048, 9, 0, 0, 1), (538, 27648, 5120, 9, 0, 0, 1),
    (547, 26928, 1496, 12, 9, 16, 1), (524, 33312, 3472, 12, 9, 12, 1), (459, 32000, 4096, 12, 8, 16, 1), (457, 57344, 8192, 12, 8, 16, 1),
    (295, 32048, 432, 12, 7, 12, 1), (300, 32000, 736, 12, 7, 12, 1), (300, 32000, 744, 9, 0, 0, 1),
    # as many or fewer: ties go to the tall form
    (211, 19440, 4552, 12, 7, 12, 1), (508, 16720, 2240, 12, 7, 12, 1),
    # 12 tiles that promise a fifth against 16 that promise a seventh: in two passes, in one, in three
    (188, 4720, 11528, 12, 6, 12, 5), (182, 5648, 4968, 12, 6, 12, 4), (107, 12288, 4096, 12, 7, 16, 5), (330, 4720, 3336, 12, 7, 16, 4),
    # a tall form of more k splits than the static scratch holds is left out, unless it promises a fifth by 16 tiles
    (160, 16384, 40000, 11, 0, 0, 1), (136, 16384, 17000, 12, 9, 16, 4)])
def test_tall_passes_where_they_are_faster(m, n, k, variant, mt_pass, tiles, splits):
    from paper_2401_12522_amd import binding as B
    _lib()
    plan = B.gemm_plan_info(m, n, k)
    assert (plan["variant"], plan["mt_pass"], plan["tall_tiles"], plan["splits"]) == (variant, mt_pass, tiles, splits), plan


@pytest.mark.parametrize("m,n,k,mt_pass,splits", [
    # in place of passes of 5, with more k splits too
    (145, 22016, 4096, 10, 2), (160, 22016, 4096, 10, 2), (150, 12288, 4096, 10, 4), (289, 12288, 4096, 10, 2), (150, 20480, 6144, 10, 2),
    (300, 22016, 4096, 10, 1), (340, 22016, 4096, 11, 1), (470, 27648, 5120, 10, 1), (152, 40960, 2048, 10, 1),
    # in place of two passes of 6 m-tiles with as many splits, but not with more
    (161, 40960, 2048, 11, 1), (176, 40960, 2048, 11, 1), (161, 22016, 4096, 6, 1), (166, 22016, 4096, 6, 1), (161, 19440, 4552, 6, 1),
    (176, 19440, 4552, 6, 1), (170, 20480, 6144, 6, 1),
    # left with passes of 5
    (300, 12288, 4096, 0, 1), (300, 7088, 16128, 0, 2)])
def test_passes_of_ten_and_eleven(m, n, k, mt_pass, splits):
    from paper_2401_12522_amd import binding as B
    _lib()
    plan = B.gemm_plan_info(m, n, k)
    assert (plan["mt_pass"], plan["splits"]) == (mt_pass, splits), plan
    assert plan["tall_tiles"] == (12 if mt_pass else 0)
