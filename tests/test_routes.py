"""Which kernels a GEMM takes by its sizes (host arithmetic, no GPU): the rules' boundaries, and the routes that the GPU tests
rely on."""
import ctypes as C

import paper_2312_04916_amd as ee
from workload import CONFIGS

from common import ee_config_of

GEMMS = (ee.EE_K_QKV, ee.EE_K_OPROJ, ee.EE_K_SWIGLU, ee.EE_K_DOWN)


def config(d, F, vocab=1056, **tuning):
    hd = 128 if d % 128 == 0 else 64 if d % 64 == 0 else 32
    return ee.make_config(2, d, d // hd, hd, F, vocab, (1,), "bf16", 4096, **tuning)


def route(cfg, kernel, rows, prompt=False):
    return ee.gemm_route(cfg, kernel, rows, prompt)[0]


def test_arguments_are_checked():
    r, L = C.c_int32(), ee.lib()
    bf, f32 = config(1024, 2816), ee_config_of(CONFIGS["C1"].shape, 256)
    call = lambda cfg, *a: L.ee_debug_gemm_route(C.byref(cfg), *a, C.byref(r), None)  # noqa: E731
    assert call(bf, 64, 4, ee.EE_K_QKV, 64, 0) == 0
    assert call(f32, 64, 4, ee.EE_K_QKV, 64, 0) == -1
    assert call(bf, 64, 4, ee.EE_K_ATTN, 64, 0) == -7
    assert call(bf, 64, 4, ee.EE_K_QKV, 65, 0) == -7   # more rows than max_rows
    assert call(bf, 64, 4, ee.EE_K_HEAD, 5, 0) == -7   # more sequences than max_seqs
    assert call(bf, 64, 4, ee.EE_K_HEAD, 4, 1) == -7   # heads of the prompt phase have one route
    assert call(bf, 64, 4, ee.EE_K_QKV, 2048, 1) == 0 and call(bf, 64, 4, ee.EE_K_QKV, 2049, 1) == -7
    assert L.ee_debug_gemm_route(None, 64, 4, ee.EE_K_QKV, 1, 0, C.byref(r), None) == -7


def test_few_rows_are_staged_in_lds():
    """One row always; two or three of up to 36 KB, or of all the LDS where the launch is a single round of workgroups."""
    cfg = config(4096, 11008)
    for k in GEMMS:
        assert route(cfg, k, 1) == ee.EE_ROUTE_STAGED
        assert route(cfg, k, 2) == ee.EE_ROUTE_STAGED
        assert route(cfg, k, 3) == (ee.EE_ROUTE_STAGED if k == ee.EE_K_DOWN else ee.EE_ROUTE_ROWS)
        assert route(cfg, k, 4) == ee.EE_ROUTE_ROWS and route(cfg, k, 32) == ee.EE_ROUTE_ROWS


def test_head_panels_from_33_rows_and_32768_words_on():
    for vocab, n, want in ((32768, 33, ee.EE_ROUTE_PANELS), (32768, 64, ee.EE_ROUTE_PANELS), (32768, 32, ee.EE_ROUTE_ROWS), (32736, 64, ee.EE_ROUTE_ROWS)):
        assert route(config(1024, 2816, vocab), ee.EE_K_HEAD, n) == want


def test_the_documented_default_of_gemm_min_workgroups_equals_zero():
    for value, cut in ((0, True), (512, True), (100000, True), (511, False), (1, False)):
        cfg = config(4096, 11008, 32768, gemm_min_workgroups=value)
        assert route(cfg, ee.EE_K_DOWN, 64) == (ee.EE_ROUTE_CUT if cut else ee.EE_ROUTE_ROWS)
        assert route(cfg, ee.EE_K_HEAD, 64) == (ee.EE_ROUTE_PANELS if cut else ee.EE_ROUTE_ROWS)


def test_scratch_of_the_prompt_phase_is_what_its_cuts_can_use():
    """workspace_bytes against that of the same model without scratch (measured before there was any): nothing more for a
    model whose GEMMs are never cut, and no more than 256 workgroups and 256 result tiles can fill for the widest."""
    for d, F, vocab, max_pos, seqs, without in ((128, 352, 1056, 4096, 4, 11030528), (1024, 2080, 544, 256, 1, 18149376),
                                                (2048, 5504, 50304, 2048, 1, 151994624), (4096, 11008, 50304, 2048, 1, 294174976),
                                                (6656, 17920, 50304, 4096, 4, 472172544)):
        cfg = ee.make_config(2, d, d // (128 if d > 128 else 32), 128 if d > 128 else 32, F, vocab, (1,), "bf16", max_pos)
        sb = C.c_size_t()
        assert ee.lib().ee_model_bytes(C.byref(cfg), 64, seqs, None, C.byref(sb)) == 0
        scratch = sb.value - without
        assert 0 <= scratch <= 512 * 128 * 1024 and (scratch == 0) == (d == 128)
        if d == 1024:
            assert scratch <= 16 << 20


def test_eight_waves_on_short_contractions_only_where_they_were_measured_to_win():
    waves = lambda cfg, k, rows=1: ee.gemm_route(cfg, k, rows)[1]  # noqa: E731
    for d, F in ((1024, 1024), (1280, 1280), (1536, 1536)):  # 32, 40 and 48 k-tiles
        cfg = config(d, F, 2048)
        assert [waves(cfg, k) for k in (*GEMMS, ee.EE_K_HEAD)] == [4] * 5
    assert waves(config(768, 2048), ee.EE_K_DOWN) == waves(config(1024, 2048), ee.EE_K_DOWN, 3) == 8  # 64 k-tiles
    wide = config(2048, 2048)
    assert waves(wide, ee.EE_K_OPROJ) == waves(wide, ee.EE_K_SWIGLU) == 8 and waves(wide, ee.EE_K_QKV) == 4  # 128, 256 | 384 workgroups
    assert waves(config(2048, 2080), ee.EE_K_SWIGLU) == 4
    assert waves(config(4096, 11008), ee.EE_K_QKV) == 8 and waves(config(4096, 11008), ee.EE_K_DOWN) == 16
