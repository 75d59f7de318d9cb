"""The C-ABI library loads, exports every symbol include/sf.h declares, and
rejects bad arguments on the host before anything is enqueued (these calls
never reach the device, so they run without a GPU)."""
import ctypes as C
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def sf():
    import paper_2407_06107_amd as sf
    if not os.path.exists(sf.LIB_PATH):
        from paper_2407_06107_amd import build
        build.build()
    sf.lib()
    return sf


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "sf.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sf_[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_exported(sf):
    declared = _declared_symbols()
    assert "sf_raymarch" in declared and "sf_filter2d" in declared
    out = subprocess.run(["nm", "-D", "--defined-only", sf.LIB_PATH], capture_output=True, text=True, check=True).stdout
    exported = set(re.findall(r"\bT (sf_\w+)", out))
    missing = [s for s in declared if s not in exported]
    assert not missing, missing
    for s in declared:
        assert hasattr(sf.lib(), s)
    assert set(sf.EXPORTED) == set(declared)


def test_versions(sf):
    assert sf.sf_abi_version() == 3
    assert sf.sf_rng_version() == 1


STRUCTS = ["sf_sampling", "sf_tex2d", "sf_ggx", "sf_volume", "sf_latent_grid", "sf_mlp", "sf_train_state"]


def test_struct_layouts_match_header(sf, tmp_path):
    """Every ctypes mirror has the size and field offsets that a C compiler
    gives the header's struct."""
    lines = ["#include <stdio.h>", "#include <stddef.h>", '#include "sf.h"', "int main(void) {"]
    for st in STRUCTS:
        lines.append(f'printf("{st} size %zu\\n", sizeof({st}));')
        for name, _ in getattr(sf, st)._fields_:
            lines.append(f'printf("{st} {name} %zu\\n", offsetof({st}, {name}));')
    lines += ["return 0; }"]
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c11", f"-I{os.path.join(ROOT, 'include')}", str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    got = {tuple(l.split()[:2]): int(l.split()[2]) for l in out if l}
    for st in STRUCTS:
        cls = getattr(sf, st)
        assert got[(st, "size")] == C.sizeof(cls), st
        for name, _ in cls._fields_:
            assert got[(st, name)] == getattr(cls, name).offset, (st, name)
    assert C.sizeof(sf.sf_sampling) == 24


def _vol(sf, **kw):
    v = sf.sf_volume(0x1000, 8, 8, 8, sf.SF_R16F, (C.c_float * 3)(0, 0, 0), (C.c_float * 3)(8, 8, 8), None, 0, 0)
    for k, x in kw.items():
        setattr(v, k, x)
    return v


FAKE = C.c_void_p(0x10000)   # a host-side stand-in pointer: never dereferenced, validation fails first


@pytest.mark.parametrize("case, status", [
    ("n_negative", 2), ("n_zero", 0), ("null_rays", 1), ("steps_zero", 2), ("steps_big", 2),
    ("bad_filter", 2), ("bad_mode", 2), ("spp_zero", 2), ("bad_variant", 2), ("null_volume", 1),
    ("bad_format", 3), ("dims_zero", 2), ("scale_zero", 2), ("misaligned_rays", 2), ("n_huge", 2),
    ("bad_brick", 2), ("reserved", 2), ("keys", 3), ("split", 3),
])
@pytest.mark.parametrize("entry", ["sf_raymarch", "sf_raymarch_emission"])
def test_raymarch_validation(sf, case, status, entry):
    L = sf.lib()
    smp = sf.sampling(sf.SF_BSPLINE3, sf.SF_STOCHASTIC, 1)
    vol = _vol(sf)
    n, steps, rays, T = 4, 16, FAKE, FAKE
    if case == "n_negative":
        n = -1
    elif case == "n_zero":
        n = 0
    elif case == "null_rays":
        rays = None
    elif case == "steps_zero":
        steps = 0
    elif case == "steps_big":
        steps = 70000
    elif case == "bad_filter":
        smp.filter = 9
    elif case == "bad_mode":
        smp.mode = 4
    elif case == "spp_zero":
        smp.spp = 0
    elif case == "bad_variant":
        smp.rng_variant = 2
    elif case == "null_volume":
        vol = None
    elif case == "bad_format":
        vol.format = sf.SF_RGBA8_UNORM
    elif case == "dims_zero":
        vol.nx = 0
    elif case == "scale_zero":
        vol.scale[1] = 0.0
    elif case == "misaligned_rays":
        rays = C.c_void_p(0x10004)
    elif case == "n_huge":
        n = 2 ** 31
    elif case == "bad_brick":
        vol.occupancy = 0x20000
        vol.brick_log2 = 9
    elif case == "reserved":
        vol.reserved = 1
    elif case == "keys":
        smp.filter = sf.SF_KEYS3
    elif case == "split":
        smp.mode = sf.SF_SPLIT
    args = (C.byref(vol) if vol is not None else None, rays, n, steps, C.byref(smp))
    if entry == "sf_raymarch_emission":
        args += (C.c_float(0.0),)
    st = getattr(L, entry)(*args, T, None, None)
    assert st == status, sf.sf_last_error()
    if status:
        assert sf.sf_last_error()


@pytest.mark.parametrize("case, status", [
    ("ok_zero", 0), ("null_tex", 1), ("null_base", 1), ("bad_format", 3), ("levels_zero", 2),
    ("levels_too_many", 2), ("bad_wrap", 2), ("bad_mip", 2), ("ggx_missing", 1), ("bad_shade", 2),
    ("ggx_backfacing", 2), ("misaligned_level", 2), ("width_zero", 2), ("keys_ok_zero", 0),
    ("keys_reuse", 3), ("filter_9", 2), ("mitchell_reuse", 3), ("ewa", 3), ("split_gauss", 3), ("split_reuse", 3), ("mode_4", 2), ("gauss_sigma_small", 2), ("gauss_sigma_nan", 2), ("fis_sigma_big", 2),
    ("gauss_reuse", 3), ("fis_bspline_reuse", 3), ("fis_bspline_any_sigma_zero", 0),
])
def test_filter2d_validation(sf, case, status):
    L = sf.lib()
    smp = sf.sampling(sf.SF_BSPLINE3, sf.SF_STOCHASTIC, 4)
    tex = sf.sf_tex2d()
    tex.base, tex.width, tex.height, tex.levels = 0x10000, 64, 64, 1
    tex.format, tex.wrap, tex.mip = sf.SF_RGBA32F, 0, 0
    n, shade, g = 10, sf.SF_SHADE_NONE, None
    texp = C.byref(tex)
    if case == "ok_zero":
        n = 0
    elif case == "null_tex":
        texp = None
    elif case == "null_base":
        tex.base = None
    elif case == "bad_format":
        tex.format = sf.SF_R16F
    elif case == "levels_zero":
        tex.levels = 0
    elif case == "levels_too_many":
        tex.levels = 8      # 64x64 has 7 levels
    elif case == "bad_wrap":
        tex.wrap = 5
    elif case == "bad_mip":
        tex.mip = 3
    elif case == "ggx_missing":
        shade = sf.SF_SHADE_GGX
    elif case == "bad_shade":
        shade = 4
    elif case == "ggx_backfacing":
        shade = sf.SF_SHADE_GGX
        g = sf.ggx(wi=(0.0, 0.3, -1.0))
    elif case == "misaligned_level":
        tex.levels = 2
        tex.level_offset[1] = 8
    elif case == "width_zero":
        tex.width = 0
    elif case == "keys_ok_zero":
        smp = sf.sampling(sf.SF_KEYS3, sf.SF_STOCHASTIC, 4)
        n = 0
    elif case == "keys_reuse":
        smp = sf.sampling(sf.SF_KEYS3, sf.SF_STOCHASTIC, 4, rng_variant=1)
    elif case == "filter_9":
        smp = sf.sampling(9, sf.SF_STOCHASTIC, 4)
    elif case == "ewa":
        smp = sf.sampling(sf.SF_EWA, sf.SF_STOCHASTIC, 4)
    elif case == "mitchell_reuse":
        smp = sf.sampling(sf.SF_MITCHELL, sf.SF_STOCHASTIC, 4, rng_variant=1)
    elif case == "split_gauss":
        smp = sf.sampling(sf.SF_GAUSS_FRS, sf.SF_SPLIT, 4)
    elif case == "split_reuse":
        smp = sf.sampling(sf.SF_LINEAR, sf.SF_SPLIT, 4, rng_variant=1)
    elif case == "mode_4":
        smp = sf.sampling(sf.SF_LINEAR, 4, 4)
    elif case == "gauss_sigma_small":
        smp = sf.sampling(sf.SF_GAUSS_FRS, sf.SF_STOCHASTIC, 4, sigma=0.05)
    elif case == "gauss_sigma_nan":
        smp = sf.sampling(sf.SF_GAUSS_FRS, sf.SF_AFTER_EXACT, 1, sigma=float("nan"))
    elif case == "fis_sigma_big":
        smp = sf.sampling(sf.SF_GAUSS_FIS, sf.SF_STOCHASTIC, 4, sigma=4.5)
    elif case == "gauss_reuse":
        smp = sf.sampling(sf.SF_GAUSS_FIS, sf.SF_STOCHASTIC, 4, rng_variant=1)
    elif case == "fis_bspline_reuse":
        smp = sf.sampling(sf.SF_BSPLINE3_FIS, sf.SF_STOCHASTIC, 4, rng_variant=1)
    elif case == "fis_bspline_any_sigma_zero":
        smp = sf.sampling(sf.SF_BSPLINE3_FIS, sf.SF_STOCHASTIC, 4, sigma=0.0)    # sigma unused
        n = 0
    st = L.sf_filter2d(texp, FAKE, n, C.byref(smp), shade, C.byref(g) if g is not None else None, FAKE, None, None)
    assert st == status, sf.sf_last_error()


@pytest.mark.parametrize("case, status", [
    ("ok_zero", 0), ("null_tex", 1), ("null_q", 1), ("keys", 3), ("gauss_frs", 3), ("fis_det", 3),
    ("reuse", 3), ("aniso_0", 2), ("aniso_65", 2), ("fis_sigma", 2), ("bad_levels", 2), ("bad_shade", 2),
    ("ewa_ok_zero", 0), ("ewa_amax17", 2), ("ewa_partial", 3), ("ewa_aspect", 3), ("ewa_reuse", 3),
    ("ewa_aspect8_partial", 3), ("split_ewa", 3), ("split_fis", 3),
])
def test_filter2d_aniso_validation(sf, case, status):
    L = sf.lib()
    smp = sf.sampling(sf.SF_BSPLINE3, sf.SF_STOCHASTIC, 4)
    tex = sf.sf_tex2d()
    tex.base, tex.width, tex.height, tex.levels = 0x10000, 64, 64, 7
    tex.format, tex.wrap, tex.mip = sf.SF_RGBA32F, 0, 0
    n, amax, shade, texp, q = 10, 64, sf.SF_SHADE_NONE, C.byref(tex), FAKE
    if case == "ok_zero":
        n = 0
    elif case == "null_tex":
        texp = None
    elif case == "null_q":
        q = None
    elif case == "keys":
        smp = sf.sampling(sf.SF_KEYS3, sf.SF_STOCHASTIC, 4)
    elif case == "gauss_frs":
        smp = sf.sampling(sf.SF_GAUSS_FRS, sf.SF_STOCHASTIC, 4)
    elif case == "fis_det":
        smp = sf.sampling(sf.SF_GAUSS_FIS, sf.SF_AFTER_EXACT, 1)
    elif case == "reuse":
        smp = sf.sampling(sf.SF_LINEAR, sf.SF_STOCHASTIC, 4, rng_variant=1)
    elif case == "aniso_0":
        amax = 0
    elif case == "aniso_65":
        amax = 65
    elif case == "fis_sigma":
        smp = sf.sampling(sf.SF_GAUSS_FIS, sf.SF_STOCHASTIC, 4, sigma=0.01)
    elif case == "bad_levels":
        tex.levels = 8
    elif case == "bad_shade":
        shade = 3
    elif case == "split_ewa":
        smp = sf.sampling(sf.SF_EWA, sf.SF_SPLIT, 4)
    elif case == "split_fis":
        smp = sf.sampling(sf.SF_GAUSS_FIS, sf.SF_SPLIT, 4)
    elif case.startswith("ewa"):
        smp = sf.sampling(sf.SF_EWA, sf.SF_STOCHASTIC, 4, rng_variant=1 if case == "ewa_reuse" else 0)
        amax = 16
        if case == "ewa_ok_zero":
            n = 0
        elif case == "ewa_amax17":
            amax = 17
        elif case == "ewa_partial":
            tex.levels = 6
        elif case == "ewa_aspect":
            tex.width, tex.height, tex.levels = 1024, 64, 11           # 16:1
        elif case == "ewa_aspect8_partial":
            tex.width, tex.height, tex.levels = 512, 64, 9            # 8:1 needs 10 levels
    st = L.sf_filter2d_aniso(texp, q, n, C.byref(smp), amax, shade, None, FAKE, None, None)
    assert st == status, sf.sf_last_error()


def test_dct_layout_and_validation(sf):
    L = sf.lib()
    offs = (C.c_int64 * 16)()
    assert sf.sf_dct_layout(4096, 4096, 13, offs) == 5593360            # 16x below the RGBA8 pyramid
    assert [offs[i] % 256 for i in range(13)] == [0] * 13
    assert sf.sf_dct_layout(60, 44, 1) == 8 * 6 * 16
    assert L.sf_dct_layout(0, 4, 1, None) == -1 and L.sf_dct_layout(8, 8, 17, None) == -1
    tex = sf.sf_tex2d()
    tex.base, tex.width, tex.height, tex.levels = 0x10000, 64, 64, 1
    tex.format, tex.wrap, tex.mip = sf.SF_RGBA32F, 0, 0
    rng = C.c_void_p(0x20000)
    assert L.sf_dct_encode(C.byref(tex), FAKE, offs, rng, None) == 2          # not RGBA8
    tex.format = sf.SF_RGBA8_UNORM
    assert L.sf_dct_encode(None, FAKE, offs, rng, None) == 1
    assert L.sf_dct_encode(C.byref(tex), FAKE, offs, C.c_void_p(0x20004), None) == 2   # misaligned ranges
    # a DCT texture needs its ranges
    tex.format = sf.SF_DCT8
    smp = sf.sampling(sf.SF_LINEAR, sf.SF_STOCHASTIC, 1)
    assert L.sf_filter2d(C.byref(tex), FAKE, 4, C.byref(smp), 0, None, FAKE, None, None) == 1
    tex.dct_range = 0x20008
    assert L.sf_filter2d(C.byref(tex), FAKE, 4, C.byref(smp), 0, None, FAKE, None, None) == 2


@pytest.mark.parametrize("case, status", [
    ("ok_zero", 0), ("null_q", 1), ("gauss", 3), ("reuse", 3), ("plane_mode", 2), ("scale0", 2), ("scale_nan", 2),
    ("misaligned_q", 2), ("bad_shade", 2),
])
def test_triplanar_validation(sf, case, status):
    L = sf.lib()
    smp = sf.sampling(sf.SF_LINEAR, sf.SF_STOCHASTIC, 4)
    tex = sf.sf_tex2d()
    tex.base, tex.width, tex.height, tex.levels = 0x10000, 64, 64, 1
    tex.format, tex.wrap, tex.mip = sf.SF_RGBA8_UNORM, 0, 0
    n, q, pm, scale, shade = 10, FAKE, 1, 1.0, 0
    if case == "ok_zero":
        n = 0
    elif case == "null_q":
        q = None
    elif case == "gauss":
        smp = sf.sampling(sf.SF_GAUSS_FIS, sf.SF_STOCHASTIC, 4)
    elif case == "reuse":
        smp = sf.sampling(sf.SF_LINEAR, sf.SF_STOCHASTIC, 4, rng_variant=1)
    elif case == "plane_mode":
        pm = 2
    elif case == "scale0":
        scale = 0.0
    elif case == "scale_nan":
        scale = float("nan")
    elif case == "misaligned_q":
        q = C.c_void_p(0x10008)
    elif case == "bad_shade":
        shade = 2
    st = L.sf_triplanar(C.byref(tex), q, n, C.byref(smp), scale, pm, shade, None, FAKE, None, None)
    assert st == status, sf.sf_last_error()


@pytest.mark.parametrize("case, status", [("negative", 2), ("nan", 2), ("inf", 2), ("too_wide", 2),
                                          ("deterministic", 3), ("n_zero", 0)])
def test_emission_footprint_validation(sf, case, status):
    L = sf.lib()
    smp = sf.sampling(sf.SF_BSPLINE3, sf.SF_STOCHASTIC, 1)
    vol = _vol(sf)                         # scale 8 voxels per unit
    n, fp = 4, 0.1
    if case == "negative":
        fp = -0.1
    elif case == "nan":
        fp = float("nan")
    elif case == "inf":
        fp = float("inf")
    elif case == "too_wide":
        fp = 2.0 ** 20 / 8 * 1.01
    elif case == "deterministic":
        smp = sf.sampling(sf.SF_BSPLINE3, sf.SF_AFTER_EXACT, 1)
    elif case == "n_zero":
        n = 0
    st = L.sf_raymarch_emission(C.byref(vol), FAKE, n, 16, C.byref(smp), C.c_float(fp), FAKE, None, None)
    assert st == status, sf.sf_last_error()


def test_filter3d_validation(sf):
    L = sf.lib()
    smp = sf.sampling(sf.SF_LINEAR, sf.SF_BEFORE, 1)
    vol = _vol(sf)
    assert L.sf_filter3d(C.byref(vol), FAKE, 3, C.byref(smp), 3, 1.0, FAKE, None, None) == 2
    assert L.sf_filter3d(C.byref(vol), FAKE, 3, C.byref(smp), 1, float("nan"), FAKE, None, None) == 2
    assert L.sf_filter3d(C.byref(vol), None, 3, C.byref(smp), 0, 1.0, FAKE, None, None) == 1
    big = _vol(sf, nx=4096, ny=4096, nz=256)     # 8 GiB: beyond one 32-bit-offset buffer
    assert L.sf_filter3d(C.byref(big), FAKE, 3, C.byref(smp), 0, 1.0, FAKE, None, None) == 3
    for f in (sf.SF_KEYS3, sf.SF_GAUSS_FRS, sf.SF_GAUSS_FIS, sf.SF_BSPLINE3_FIS):   # 2-D only
        s2 = sf.sampling(f, sf.SF_STOCHASTIC, 1)
        assert L.sf_filter3d(C.byref(vol), FAKE, 3, C.byref(s2), 0, 1.0, FAKE, None, None) == 3
        assert L.sf_raymarch(C.byref(vol), FAKE, 3, 8, C.byref(s2), FAKE, None, None) == 3


def test_error_stats_validation(sf):
    L = sf.lib()
    need = sf.sf_error_stats_workspace(5000)
    assert need == 5 * 64
    assert sf.sf_error_stats_workspace(10 ** 9) == 1024 * 64
    assert L.sf_error_stats(FAKE, FAKE, 5000, 1, FAKE, FAKE, need - 8, None) == 5
    assert L.sf_error_stats(FAKE, FAKE, 5000, 0, FAKE, FAKE, need, None) == 2
    assert L.sf_error_stats(None, FAKE, 5000, 1, FAKE, FAKE, need, None) == 1
    # the allocation-free variant validates the same way before touching a device
    assert sf.sf_error_stats_noalloc_max_bytes() == 1024 * 64
    assert L.sf_error_stats_noalloc(FAKE, FAKE, 5000, 0, FAKE, None) == 2
    assert L.sf_error_stats_noalloc(FAKE, FAKE, -1, 1, FAKE, None) == 2
    assert L.sf_error_stats_noalloc(FAKE, FAKE, 2 ** 62, 4, FAKE, None) == 2
    assert L.sf_error_stats_noalloc(None, FAKE, 5000, 1, FAKE, None) == 1
    assert L.sf_error_stats_noalloc(FAKE, FAKE, 5000, 1, None, None) == 1


def test_product_path_has_no_fallback(sf, monkeypatch, tmp_path):
    """Without the built library the binding raises instead of computing."""
    monkeypatch.setattr(sf, "LIB_PATH", str(tmp_path / "missing.so"))
    monkeypatch.setattr(sf, "_lib", None)
    with pytest.raises(ImportError):
        sf.lib()


def test_occupancy_words_and_validation(sf):
    # one bit per brick in rows of nbx + 1 and planes of nby + 1 rows, in 32-bit words
    assert sf.sf_occupancy_words(512, 512, 512, 3) == -(-(65 * 65 * 64) // 32)
    assert sf.sf_occupancy_words(10, 9, 8, 2) == 1                     # 4 x 4 x 2 bits
    assert sf.sf_occupancy_words(1, 1, 1, 1) == 1
    assert sf.sf_occupancy_words(4096, 4096, 1024, 1) == 0             # 2049^2 x 512 bits: over 2^30
    assert sf.sf_occupancy_words(4096, 2048, 256, 1) == -(-(2049 * 1025 * 128) // 32)
    assert sf.sf_occupancy_words(8, 8, 8, 0) == 0
    L = sf.lib()
    vol = _vol(sf, brick_log2=2)
    assert L.sf_build_occupancy(C.byref(vol), FAKE, 0, None) == 2         # too few words
    vol.brick_log2 = 7
    assert L.sf_build_occupancy(C.byref(vol), FAKE, 100, None) == 2
    assert L.sf_build_occupancy(None, FAKE, 100, None) == 1


def _latgrid(sf, **kw):
    g = sf.sf_latent_grid(0x10000, 0x20000, 2, (C.c_int32 * 3)(32, 32, 1), 8, sf.SF_LATENT_BF16, 0,
                          (C.c_float * 3)(0, 0, 0), (C.c_float * 3)(1, 1, 1))
    for k, x in kw.items():
        setattr(g, k, x)
    return g


def test_neural_shapes_and_sizes(sf):
    assert sf.sf_mlp_nparams(8, 64, 4) == 4996          # config-4 network
    assert sf.sf_mlp_nparams(16, 64, 1) == 5313         # config-5 network
    # 63 per-wavefront partials + 1 chunk sum (chunks of 64 partials), each nparams + 1 floats
    assert sf.sf_neural_train_workspace(8, 4, 1000) == (63 + 1) * (4996 + 1) * 4
    assert sf.sf_neural_train_workspace(16, 1, 1 << 20) == (2048 + 32) * (5313 + 1) * 4
    assert sf.sf_neural_train_workspace(8, 3, 1000) == 0
    assert C.sizeof(sf.sf_latent_grid) == 8 + 8 + 4 + 12 + 4 * 3 + 24 + 4   # padded to pointer alignment
    assert C.sizeof(sf.sf_mlp) == 8 + 16
    assert C.sizeof(sf.sf_train_state) == 6 * 8 + 8 + 16


@pytest.mark.parametrize("case, status", [
    ("ok_zero", 0), ("null_grid", 1), ("bad_dims", 2), ("bad_channels", 3), ("bad_format", 3),
    ("mlp_shape", 3), ("null_mlp", 1), ("variant", 3), ("grid3d", 3), ("misaligned", 2),
])
def test_neural_decode_validation(sf, case, status):
    L = sf.lib()
    smp = sf.sampling(sf.SF_BSPLINE3, sf.SF_STOCHASTIC, 1)
    g = _latgrid(sf)
    m = sf.sf_mlp(0x30000, 8, 64, 4, 0)
    n, gp, mp = 10, C.byref(g), C.byref(m)
    if case == "ok_zero":
        n = 0
    elif case == "null_grid":
        gp = None
    elif case == "bad_dims":
        g.dims = 4
    elif case == "bad_channels":
        g.channels = 12
    elif case == "bad_format":
        g.format = sf.SF_LATENT_F32
    elif case == "mlp_shape":
        m.out_dim = 3
    elif case == "null_mlp":
        mp = None
    elif case == "variant":
        smp.rng_variant = 1
    elif case == "grid3d":
        g.dims, g.channels = 3, 16
        g.res[2] = 8
    elif case == "misaligned":
        g.latents = 0x10008
    st = L.sf_neural_decode(gp, mp, FAKE, n, C.byref(smp), 0, None, FAKE, None, None)
    assert st == status, sf.sf_last_error()


def test_neural_raymarch_and_train_validation(sf):
    L = sf.lib()
    g = _latgrid(sf, dims=3, channels=16)
    g.res[2] = 8
    m = sf.sf_mlp(0x30000, 16, 64, 1, 0)
    det = sf.sampling(sf.SF_BSPLINE3, sf.SF_AFTER_EXACT, 1)
    assert L.sf_neural_raymarch(C.byref(g), C.byref(m), FAKE, 5, 16, C.byref(det), FAKE, None, None) == 3
    g2 = _latgrid(sf)
    sto = sf.sampling(sf.SF_BSPLINE3, sf.SF_STOCHASTIC, 1)
    m2 = sf.sf_mlp(0x30000, 8, 64, 4, 0)
    assert L.sf_neural_raymarch(C.byref(g2), C.byref(m2), FAKE, 5, 16, C.byref(sto), FAKE, None, None) == 3
    st = sf.sf_train_state(0x1000, 0x2000, 0x3000, 0x4000, 0x5000, 0x6000, 100, 8, 64, 4, 0)
    ws = sf.sf_neural_train_workspace(8, 4, 50)
    args = (FAKE, FAKE, 50, 1, 1e-2, 1e-3, FAKE, None, None, FAKE)
    assert L.sf_neural_train_step(C.byref(st), *args, ws - 4, None) == 5
    assert L.sf_neural_train_step(C.byref(st), FAKE, FAKE, 500, 1, 1e-2, 1e-3, FAKE, None, None, FAKE, 10 ** 9, None) == 2
    assert L.sf_neural_train_step(C.byref(st), FAKE, FAKE, 50, 0, 1e-2, 1e-3, FAKE, None, None, FAKE, ws, None) == 2
    st.compute = 2   # neither SF_TRAIN_BF16 nor SF_TRAIN_FP32
    assert L.sf_neural_train_step(C.byref(st), *args, ws, None) == 2
    st.compute = sf.SF_TRAIN_FP32
    st.hidden = 32
    assert L.sf_neural_train_step(C.byref(st), *args, ws, None) == 3


def test_timed_kernel_code_digest(sf):
    """bench.py keys the measured HBM traffic to the timed kernel's machine
    code: its digest is found in the built library (function bytes and
    kernel descriptor of the gfx950 code object)."""
    import importlib.util
    import os
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    spec = importlib.util.spec_from_file_location("bench_for_test", os.path.join(root, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    d = bench.kernel_code_digest()
    assert d is not None and len(d) == 64 and int(d, 16) >= 0
    assert bench.kernel_code_digest(name=bench.TIMED_KERNEL + "_absent") is None


def test_committed_counters_belong_to_the_timed_kernel(sf):
    """The hardware counters committed under profiles/ were taken on the
    machine code of the kernel bench.py times (same digest), so the bench
    line's roofline and traffic figures are not stale."""
    import importlib.util
    import os
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    spec = importlib.util.spec_from_file_location("bench_for_test2", os.path.join(root, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    c = bench.counters_from_profile(bench.kernel_code_digest())
    assert c.get("valu_insts_per_launch") and c.get("hbm_bytes_per_launch"), c


def test_current_stream_without_torchs_private_call(sf, monkeypatch):
    """A torch that no longer has the private call for the current stream's
    handle: the public one gives it."""
    import types
    import torch
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1234))
    assert sf._stream(None).value == 0x1234
    assert sf._stream(types.SimpleNamespace(cuda_stream=0x5678)).value == 0x5678
