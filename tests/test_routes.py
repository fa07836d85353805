"""Which kernels a GEMM takes by its sizes (host arithmetic, no GPU): the rules' boundaries, and the routes that the GPU tests
rely on."""
import ctypes as C

import pytest

import paper_2312_04916_amd as ee
from workload import CONFIGS

from common import cut_projections, ee_config_of
from test_gpu_long_batches import CASES as LONG_BATCHES, long_batch
from test_gpu_rows import CUT_PROMPTS, CUT_STEPS, PROMPT_SHAPES, SHAPES, STEP_LIMITS
from test_gpu_rows_tiles import DOWN_MIN_WGS

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


def test_heads_of_up_to_four_rows_are_staged():
    for d in (768, 2048, 4096):
        cfg = config(d, 32 * (d // 12), 50304)
        assert [route(cfg, ee.EE_K_HEAD, n) for n in (1, 2, 3, 4)] == [ee.EE_ROUTE_STAGED] * 4
        assert route(cfg, ee.EE_K_HEAD, 5) == ee.EE_ROUTE_ROWS
    assert [route(config(736, 1376), ee.EE_K_HEAD, n) for n in (3, 4)] == [ee.EE_ROUTE_STAGED, ee.EE_ROUTE_ROWS]
    assert [route(config(5120, 13824), ee.EE_K_HEAD, n) for n in (1, 2)] == [ee.EE_ROUTE_STAGED, ee.EE_ROUTE_ROWS]


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
        assert -1024 <= scratch <= 512 * 128 * 1024 and (scratch <= 0) == (d == 128)
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


def test_ring_refills_go_between_the_mfmas_where_a_wave_has_its_simd_to_itself():
    """33 and more rows: up to four column tiles run 8 waves, two per SIMD, and refill a slot in a burst; five and six run 4, one
    per SIMD, and refill between the MFMAs, which 8 waves were measured to lose by.  Up to 32 rows: in a burst."""
    seen = set()
    for d, F in ((768, 2048), (1024, 2816), (2048, 5504), (3072, 8192), (4096, 11008), (5120, 13824), (6656, 17920)):
        for min_wgs in (0, 511, 200, 64, 16):
            cfg = config(d, F, 50304, gemm_min_workgroups=min_wgs)
            for k in (*GEMMS, ee.EE_K_HEAD):
                for rows in (4, 16, 17, 32, 33, 48, 64):
                    if route(cfg, k, rows) != ee.EE_ROUTE_ROWS:
                        continue
                    tiles, waves, ring, between = ee.rows_launch(cfg, k, rows)
                    assert 1 <= tiles <= 6 and 2 <= ring <= 8
                    if rows > 32:
                        assert (waves, between) == ((8, 0) if tiles <= 4 else (4, 1)), (d, k, rows)
                        seen.add(tiles)
                    else:
                        assert (waves in (4, 8) or waves == 16 and rows <= 16 and tiles <= 2) and between == 0, (d, k, rows)
    assert seen == {1, 2, 3, 4, 5, 6}
    r, L = (C.c_int32 * 4)(), ee.lib()
    assert L.ee_debug_rows_launch(C.byref(config(4096, 11008)), 64, 4, ee.EE_K_QKV, 1, r) == -7   # staged
    assert L.ee_debug_rows_launch(C.byref(config(4096, 11008)), 64, 4, ee.EE_K_DOWN, 64, r) == -7  # cut
    assert L.ee_debug_rows_launch(C.byref(config(4096, 11008)), 64, 4, ee.EE_K_QKV, 65, r) == -7   # more rows than max_rows
    assert L.ee_debug_rows_launch(C.byref(config(4096, 11008)), 64, 4, ee.EE_K_QKV, 64, None) == -7
    one, past = (C.c_int32 * 1)(1), C.c_int32()
    call = lambda cfg, n, c, rows, layers: L.ee_debug_kv_past_caches(C.byref(cfg), n, c, rows, layers, C.byref(past))  # noqa: E731
    assert call(config(4096, 11008), 1, one, one, 2) == 0 and past.value == 0
    assert call(ee_config_of(CONFIGS["C1"].shape, 256), 1, one, one, 1) == -1
    assert [call(config(4096, 11008), *a) for a in ((0, one, one, 1), (65, one, one, 1), (1, one, one, 3), (1, one, (C.c_int32 * 1)(2), 1), (1, None, one, 1))] == [-7] * 5


# What cutting one projection (Q|K|V, O, gate|up, down) was measured to add to a layer, in us, where it is 2 us or more either
# way; 0: less than that, or 2 to 3 us gained on 24 k-tiles with 128-row tiles, which the rule of the prompts leaves alone, or
# the one point of a step between 2 and 3 that its rule gets wrong (Q|K|V of 5632 wide, 40 rows, -2.4).
MEASURED_STEPS = {
    (512, 1376): {66: (3, 4, 3, 3), 96: (0, 3, 2, 0), 128: (0, 2, 0, 0)},
    (640, 1728): {66: (5, 6, 6, 0), 96: (3, 5, 4, 0), 128: (3, 4, 3, -3), 256: (-13, -7, -10, -22)},
    (768, 2048): {33: (5, 4, 4, 0), 64: (5, 4, 4, 0), 66: (3, 2, 2, -2), 96: (0, 3, 0, -4), 128: (0, 0, 0, -6)},
    (1024, 2816): {33: (4, 4, 4, 0), 64: (5, 4, 4, 0), 66: (0, 0, 0, -5), 96: (0, 0, 0, -7), 128: (-2, 0, 0, -12), 192: (-11, -8, -3, -24)},
    (1536, 4096): {33: (5, 3, 6, -4), 64: (5, 2, 6, -4), 66: (0, 0, 5, -10), 96: (-4, -2, 0, -13), 128: (-4, -5, 0, -19), 192: (-11, -12, -6, -36)},
    (2048, 5504): {33: (4, 0, 7, -6), 64: (5, 0, 7, -7), 66: (-3, -3, 0, -15), 96: (-5, -6, 0, -18), 128: (-5, -7, 0, -26), 145: (-14, -15, -13, -40), 256: (-26, -27, -24, -69)},
    (2560, 6880): {33: (4, 0, 7, -8), 64: (5, 0, 7, -9)},
    (3072, 8192): {33: (4, 0, 5, -12), 64: (7, 0, 4, -13), 66: (-5, -7, -7, -24), 96: (-8, -8, -9, -30), 128: (-8, -13, -11, -40), 192: (-22, -23, -23, -67)},
    (3584, 9632): {33: (4, 0, 4, -16), 64: (5, 0, 4, -16)},
    (4096, 11008): {33: (3, 0, 0, -16), 64: (6, -3, 4, -15), 66: (-7, -8, -20, -33), 96: (-10, -10, -24, -38), 128: (-20, -16, -28, -50), 160: (-23, -27, -35, -83), 256: (-56, -52, -90, -142)},
    (4608, 12384): {33: (3, -4, -7, -24), 40: (3, -4, -7, -26), 64: (5, -4, -5, -23)},
    (5120, 13824): {33: (5, -2, -3, -25), 64: (6, -2, 0, -24), 66: (-13, -12, -45, -54), 96: (-15, -15, -46, -63)},
    (5632, 15136): {33: (-2, -6, -3, -29), 40: (0, -6, -3, -29), 64: (0, -4, -2, -27)},
    (6144, 16512): {33: (2, -4, -10, -32), 64: (4, -4, -8, -32)},
    (6656, 17920): {33: (4, -6, -10, -28), 64: (6, -5, -7, -29), 66: (-30, -18, -68, -68), 192: (-35, -39, 0, -130)},
    (7168, 19264): {33: (0, -7, -5, -30), 64: (3, -4, -5, -27)},
    (8192, 22016): {33: (7, -6, -9, -31), 64: (7, -4, -6, -29)},
}
# ... with the scratch of a model for so many rows and no more (two thirds of the workgroups and fewer), 50304 words; left out:
# Q|K|V of 3072 wide, 66 rows, cut for 3.0 us more.
MEASURED_STEPS_SMALL_SCRATCH = {
    (640, 1728): {256: (-14, -8, -12, -23)},
    (768, 2048): {33: (6, 4, 5, 0), 64: (6, 4, 5, 0), 66: (3, 3, 6, -2), 96: (0, 2, 4, -4), 128: (0, 0, 0, -7)},
    (1024, 2816): {33: (5, 4, 4, 0), 64: (4, 4, 5, 0), 66: (0, 2, 4, -5), 96: (0, 0, 3, -7), 128: (-3, 0, 2, -12), 192: (-11, -8, 0, -25)},
    (1536, 4096): {33: (4, 3, 7, -5), 64: (5, 3, 7, -4), 66: (3, 0, 11, -8), 96: (0, 0, 3, -11), 128: (0, -4, 4, -19), 192: (-10, -13, -2, -35)},
    (2048, 5504): {33: (6, 0, 7, -7), 64: (6, 0, 7, -6), 66: (5, -3, 21, -12), 96: (-4, -5, 5, -18), 128: (-3, -8, 0, -26), 145: (-9, -15, 0, -39), 256: (-26, -27, -22, -68)},
    (2560, 6880): {33: (5, 0, 5, -10), 64: (7, 0, 7, -9)},
    (3072, 8192): {33: (6, 0, 8, -13), 64: (8, -2, 9, -12), 66: (0, -4, 0, -22), 96: (-8, -8, 4, -29), 128: (-10, -12, -11, -37), 192: (-17, -17, -10, -60)},
    (3584, 9632): {33: (3, 0, 3, -16), 64: (4, 0, 2, -16)},
    (4096, 11008): {33: (4, 0, 3, -16), 64: (8, 0, 3, -15), 66: (0, -5, 0, -30), 96: (-9, -9, -12, -36), 128: (-14, -10, -29, -51), 160: (-15, -26, -20, -79), 256: (-53, -50, -86, -140)},
    (4608, 12384): {33: (3, -4, -6, -25), 48: (5, -3, -6, -24), 64: (5, 0, -7, -22)},
    (5120, 13824): {33: (6, -3, -3, -24), 64: (8, -2, -3, -24), 66: (-6, -13, 0, -50), 96: (-16, -11, -35, -58)},
    (5632, 15136): {33: (0, -6, -3, -28), 48: (0, -5, 0, -30), 64: (3, -5, 0, -27)},
    (6144, 16512): {33: (0, -6, -12, -33), 64: (3, -5, -8, -30)},
    (6656, 17920): {33: (0, -5, -10, -28), 64: (3, -2, -5, -23), 66: (-19, -19, 0, -60), 192: (-35, -40, 0, -128)},
}
MEASURED_PROMPTS = {
    (384, 1024): {65: (3, 3, 6, -5), 300: (3, 4, 6, -5)},
    (768, 2048): {33: (-4, -4, -2, -14), 128: (0, 0, 0, -13), 640: (0, 0, 6, -11), 2048: (3, 0, 0, -5)},
    (1024, 2816): {33: (-7, -6, -4, -21), 300: (0, -5, 8, -17), 777: (5, -4, 4, -12), 1300: (8, 0, 9, -10)},
    (1536, 4096): {65: (-10, -10, -5, -33), 384: (0, -10, 8, -29)},
    (2048, 5504): {65: (-13, -14, -4, -44), 129: (-6, -12, 2, -40), 256: (-3, -14, 8, -44), 384: (3, -10, -9, -41), 512: (12, -7, 0, -34),
                   640: (18, -4, 18, -28), 777: (-4, 0, 0, -20), 1024: (8, -2.5, 0, -24)},
    (4096, 11008): {64: (-31, -40, -17, -115), 99: (-19, -30, -2, -94), 200: (5, -22, -22, -78), 256: (6, -26, -19, -90), 300: (22, -15, 0, -52),
                    384: (-26, -14, 0, -45), 512: (-7, -15, 0, -58)},
    (5120, 13824): {33: (-31, -46, -13, -128), 129: (0, -27, -15, -72), 256: (26, -24, 32, -70)},
    (6656, 17920): {33: (-34, -55, -7, -163), 128: (-19, -50, -50, -144), 129: (44, -24, 0, -77), 256: (-9, -22, 0, -72)},
}


@pytest.mark.parametrize("prompt", [False, True])
def test_projections_are_cut_where_that_was_measured_to_win(prompt):
    wrong = []
    for (d, F), points in (MEASURED_PROMPTS if prompt else MEASURED_STEPS).items():
        for rows, effects in points.items():
            for k, us in zip(GEMMS, effects):
                cut = route(config(d, F), k, rows, prompt) == ee.EE_ROUTE_CUT
                if us and cut != (us < 0):
                    wrong.append((d, rows, ee.KERNEL_NAMES[k], us, cut))
    assert not wrong, wrong


def test_projections_are_cut_where_that_was_measured_to_win_with_little_scratch():
    wrong = []
    for (d, F), points in MEASURED_STEPS_SMALL_SCRATCH.items():
        for rows, effects in points.items():
            for k, us in zip(GEMMS, effects):
                cut = ee.gemm_route(config(d, F, 50304), k, rows, False, max(64, rows), 32)[0] == ee.EE_ROUTE_CUT
                if us and cut != (us < 0):
                    wrong.append((d, rows, ee.KERNEL_NAMES[k], us, cut))
    assert not wrong, wrong


# What reading K and V past the caches was measured to add to a step, in percent, where it is a percent or more either way:
# (width, layers up to the end of the segment or of the step, sequences, positions of each, rows of each): percent.  Left out: the one
# slower point of a percent or more above 384 MB over those layers, (2048, 6, 64, 125, 1) with 1.5, and those within 2 % of a line.
MEASURED_PAST_CACHES = {
    (4096, 16, 1, 1000, 1): 1.1, (4096, 4, 1, 1000, 1): 1.4, (4096, 4, 4, 1000, 1): 1.4, (4096, 4, 8, 500, 1): 1.3, (4096, 2, 4, 1000, 1): 1.7,
    (4096, 2, 8, 1000, 1): 2.8, (2048, 24, 1, 1500, 1): 1.9, (2048, 6, 1, 3000, 1): 1.2, (2048, 6, 4, 1000, 1): 1.1, (2048, 6, 16, 250, 1): 1.7,
    (768, 6, 64, 125, 1): 1.3,
    (2048, 6, 16, 500, 1): -2.6, (4096, 2, 64, 250, 1): -0.8, (4096, 4, 8, 1000, 1): -1.4, (4096, 2, 16, 1000, 1): -1.0,
    (768, 3, 64, 768, 1): -2.8, (6656, 1, 12, 1500, 1): -2.6,
    (4096, 16, 2, 1000, 1): -1.7, (4096, 16, 4, 1000, 1): -1.7, (4096, 16, 8, 500, 1): -1.7, (4096, 16, 8, 1000, 1): -1.6,
    (4096, 16, 16, 500, 1): -1.8, (4096, 16, 16, 1000, 1): -2.7, (4096, 4, 16, 1000, 1): -2.0, (4096, 16, 64, 200, 1): -1.2, (4096, 4, 64, 200, 1): -2.8,
    (4096, 32, 2, 600, 1): -1.0, (2048, 24, 1, 3000, 1): -1.7, (2048, 24, 2, 1400, 1): -1.2, (2048, 24, 4, 700, 1): -1.3, (2048, 24, 4, 1000, 1): -2.0,
    (2048, 24, 8, 1000, 1): -3.2, (2048, 24, 16, 250, 1): -1.4, (2048, 24, 16, 500, 1): -2.4, (2048, 24, 16, 1000, 1): -4.2, (2048, 24, 16, 2000, 1): -6.0,
    (2048, 6, 16, 1000, 1): -2.4, (2048, 6, 16, 2000, 1): -5.7, (2048, 24, 64, 250, 1): -1.4, (768, 24, 16, 1000, 1): -1.6, (768, 24, 16, 2000, 1): -1.7,
    (768, 24, 64, 500, 1): -2.4, (768, 6, 64, 500, 1): -1.5, (6656, 4, 12, 1500, 1): -2.9, (6656, 4, 16, 2000, 1): -3.9, (6656, 1, 16, 2000, 1): -3.1,
    # three query tiles per sequence: 33 to 41 rows (a step whose first exit is passed, eight layers)
    (4096, 8, 1, 3000, 41): 1.6, (4096, 8, 2, 2500, 33): 2.4, (4096, 8, 4, 2000, 33): 4.0, (4096, 8, 4, 3000, 41): 3.5, (4096, 8, 5, 3000, 40): 2.6,
    (2048, 8, 4, 3000, 33): 6.1, (4096, 8, 7, 3000, 36): 3.6, (4096, 8, 6, 3000, 40): 6.4, (4096, 8, 7, 4500, 36): 2.4, (2048, 8, 7, 6000, 36): 7.1,
    # two: the exceptions, both at 280 to 310 MB a layer, are (4096, 10, 2000, 24) with 1.5 and (2048, 8, 4500, 31) with 1.8
    (4096, 8, 4, 1000, 17): 1.7, (2048, 8, 8, 2000, 31): 2.2, (2048, 8, 8, 3000, 17): 3.6, (2048, 8, 12, 2500, 20): 2.8, (768, 12, 8, 3000, 31): 2.8,
    (4096, 8, 8, 2500, 17): -4.9, (4096, 8, 8, 3000, 31): -4.9, (4096, 8, 8, 2500, 31): -3.6, (4096, 8, 14, 1500, 18): -2.0, (4096, 8, 14, 2000, 18): -3.8,
    (4096, 8, 12, 2500, 20): -1.3, (2048, 8, 14, 3000, 18): -3.5, (2048, 8, 14, 4500, 18): -4.0,
}


def test_kv_goes_past_the_caches_where_that_was_measured_to_win():
    wrong = []
    for (d, layers, n, ctx, rows), percent in MEASURED_PAST_CACHES.items():
        hd = 64 if d == 768 else 128
        cfg = ee.make_config(32, d, d // hd, hd, 32 * (d // 12), 1056, (1,), "bf16", 4096)
        if ee.kv_past_caches(cfg, [ctx + 12] * n, [rows] * n, layers) != (percent < 0):
            wrong.append((d, layers, n, ctx, rows, percent))
    assert not wrong, wrong


def test_kv_past_the_caches_counts_a_context_once_whatever_reads_it():
    cfg = config(4096, 11008)  # two layers, 32 KB a position over both
    line = (384 << 20) // (32 << 10)
    past = lambda contexts, rows, layers=2: ee.kv_past_caches(cfg, contexts, rows, layers)  # noqa: E731
    assert past([line], [1]) and past([line], [16]) and not past([line - 1], [1])
    assert not past([line], [1], layers=1) and past([2 * line], [1], layers=1)
    # tiles that read a context again: 17 rows are two, for which the line is 256 MB a layer, 33 are three
    two = (256 << 20) // (16 << 10)
    assert past([two], [17], layers=1) and past([two], [32]) and not past([two - 1], [17]) and not past([8 * two], [33])
    assert not past([two // 4] * 3, [17] * 3) and past([two // 4] * 4, [17] * 4)
    # half of what the sequences have may be read twice (short of 256 MB a layer)
    q = (line - 4) // 4
    cfg = config(4096, 11008)
    cfg.n_layers = 3
    past3 = lambda rows: ee.kv_past_caches(cfg, [q] * 4, rows, 3)  # noqa: E731
    assert past3([17, 1, 1, 1]) and past3([17, 17, 1, 1]) and not past3([17, 17, 17, 1])
    assert past([64] * 3 + [line], [17, 20, 33, 1]) and not past([64] * 3 + [line - 193], [1, 1, 1, 17])


def test_the_gpu_tests_of_kv_past_the_caches_lie_on_both_sides_of_the_line():
    for name in LONG_BATCHES:
        for over in (-1, 0):
            shape, contexts, rows = long_batch(name, over)
            cfg = ee_config_of(shape, 2048)
            assert ee.kv_past_caches(cfg, contexts, rows, shape.n_layers) == (over == 0), name
            assert ee.kv_past_caches(cfg, contexts[:1], rows[:1], shape.n_layers) is False


def test_the_gpu_tests_run_the_routes_they_claim():
    for name, by_rows in CUT_STEPS.items():
        cfg = ee_config_of(SHAPES[name], 128)
        assert {rows: cut_projections(cfg, rows, False, **STEP_LIMITS) for rows in by_rows} == by_rows, name
    for name, cases in CUT_PROMPTS.items():
        for (n, rows_env), passes in cases.items():
            cfg = ee_config_of(PROMPT_SHAPES[name], 512, prefill_rows=rows_env)
            step = rows_env or 512
            got = [cut_projections(cfg, min(step, n - p), True, 64, 1) for p in range(0, n, step)]
            assert got == passes, (name, n, rows_env)


def test_the_gpu_tests_of_column_tiles_fill_every_ring_twice():
    shape, seen = SHAPES["d1024"], set()
    for tiles, min_wgs in DOWN_MIN_WGS.items():
        cfg = ee_config_of(shape, 128, gemm_min_workgroups=min_wgs)
        for rows in CUT_STEPS["d1024"]:
            got, waves, ring, between = ee.rows_launch(cfg, ee.EE_K_DOWN, rows, **STEP_LIMITS)
            assert (got, waves, between) == (tiles, *((8, 0) if tiles <= 4 else (4, 1)))
            per_wave = [(shape.d_ff // 32 - w + waves - 1) // waves for w in range(waves)]
            assert min(per_wave) >= 2 * ring and any(n % ring for n in per_wave)
            seen.add((tiles, waves))
    assert len(seen) == 6
