"""Which kernels a problem is given to, on the host: widths that are no multiple of 128, the split counts of the untuned choice,
and that the remembered choice is the one a fresh search finds.  No HIP call is made."""
import ctypes
import threading

import pytest

import paper_2602_11808_amd as dfk

A = 1 << 30     # fake device addresses: every call here ends before the first HIP call, or is a query
MFMA, VALU = dfk.DFK_PATH_MFMA, dfk.DFK_PATH_VALU
TWO, FUSED = dfk.DFK_VARIANT_TWO_KERNEL, dfk.DFK_VARIANT_FUSED


def cands(M, d, ff, dt):
    return [dfk.dfk_get_candidate(M, d, ff, dt, i) for i in range(dfk.dfk_num_candidates(M, d, ff, dt))]


@pytest.mark.parametrize("d", [392, 504, 520, 632, 1000, 2888, 8200, 32760])
@pytest.mark.parametrize("M", [1, 16, 64, 65, 256])
def test_widths_off_128_run_on_the_matrix_cores_in_bf16_only(M, d):
    ff = 1000
    pick, _ = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
    assert (pick.path, pick.variant, pick.kmajor, pick.a2_dtype) == (MFMA, TWO, 1, dfk.DFK_BF16)
    assert {c.kmajor for c in cands(M, d, ff, dfk.DFK_BF16) if c.path == MFMA} == {1}
    for c in cands(M, d, ff, dfk.DFK_BF16):
        assert dfk.dfk_config_valid(c, M, d, ff, dfk.DFK_BF16)
        if c.path == MFMA:      # A_2 would be rounded to half there, which the plain-FMA pair keeps in fp32
            h = dfk.dfk_config_t(**dict(c.as_dict(), a2_dtype=dfk.DFK_FP16))
            assert not dfk.dfk_config_valid(h, M, d, ff, dfk.DFK_FP16)
    for dt in (dfk.DFK_FP16, dfk.DFK_FP32):
        assert all(c.path == VALU for c in cands(M, d, ff, dt))
    # the plain-FMA candidates stay on offer, and so does the single launch among them
    assert any(c.path == VALU and c.variant == FUSED for c in cands(M, d, ff, dfk.DFK_BF16))


@pytest.mark.parametrize("d", [8, 264, 376])
def test_narrow_widths_off_128_stay_on_the_plain_fma_kernels(d):
    assert all(c.path == VALU for c in cands(4, d, 1000, dfk.DFK_BF16))


def test_the_block_and_the_other_layout_refuse_what_they_refused():
    import ctypes
    L = dfk.lib()
    M, d, ff = 4, 2888, 7688
    wsb = dfk.dfk_workspace_bytes(M, d, ff)
    p = [A + (i << 28) for i in range(7)]
    km = next(c for c in cands(M, d, ff, dfk.DFK_BF16) if c.path == MFMA)
    for cfg in (None, ctypes.byref(km)):
        assert L.dfk_mlp_block(p[0], p[1], 1e-5, p[2], p[3], p[4], p[5], M, d, ff, dfk.DFK_BF16, cfg, p[6], wsb, None) == dfk.DFK_ERR_UNSUPPORTED_SHAPE
    n = dfk.dfk_num_candidates_wdt(M, d, ff, dfk.DFK_BF16)
    assert n and all(dfk.dfk_get_candidate_wdt(M, d, ff, dfk.DFK_BF16, i).path == VALU for i in range(n))


def _rows_of_two_blocks(d, ff):
    """Rows of a d_ff split where workgroups of the down kernel own two column blocks."""
    return ff // min(16, 256 // (d // 256))


def _two_from(M, d, c):
    """Rows from which on two blocks win."""
    if c.reduce == dfk.DFK_REDUCE_ATOMIC:
        return 1152 if M > 16 else 896
    blocks = d // 128
    return 4096 if M > 16 and blocks * min(16, 256 // blocks) >= 208 else 1280


@pytest.mark.parametrize("dt", [dfk.DFK_BF16, dfk.DFK_FP16])
def test_split_counts_and_widths_of_the_untuned_choice(dt):
    for M in (1, 4, 16, 32, 33, 64):
        for d in (512, 896, 1024, 2304, 4096, 5120, 8192, 16384):
            for ff in (1536, 9216, 28672):
                pick, _ = dfk.dfk_get_choice(M, d, ff, dt)
                if pick.k2_splits == 0:
                    continue
                if ff <= 12 * d:
                    assert pick.k2_splits <= 16, (M, d, ff, pick)
                assert d // 128 // pick.k2_col_blocks == (2 if d >= 5120 and M <= 32 and _rows_of_two_blocks(d, ff) >= _two_from(M, d, pick) else 1), (M, d, ff, pick)
    for M, d, ff, width in ((32, 8192, 40960, 2), (32, 5120, 40960, 1), (16, 5120, 40960, 2), (32, 11008, 40960, 2), (32, 16384, 53248, 2)):
        pick, _ = dfk.dfk_get_choice(M, d, ff, dt)     # (slices too long for the single launch: the pair, counter reduction)
        assert (pick.variant, pick.kmajor, pick.reduce, d // 128 // pick.k2_col_blocks) == (TWO, 1, dfk.DFK_REDUCE_TICKET, width), pick
    for d in (512, 1024, 2304, 4096):
        assert dfk.dfk_get_choice(200, d, 6144, dt)[0].k2_splits <= (16 if d < 1280 else 12)


@pytest.mark.parametrize("dt", [dfk.DFK_BF16, dfk.DFK_FP16])
@pytest.mark.parametrize("M,d,ff,width", [
    (8, 5888, 5760, 1), (20, 5376, 7680, 1), (27, 5120, 8192, 1),       # short splits: one block
    (16, 5120, 11264, 2), (32, 5120, 11264, 1), (16, 7168, 12544, 2), (32, 7168, 12544, 2), (4, 5120, 27648, 2), (32, 16384, 16384, 2),
    (2, 11008, 11008, 2), (33, 16384, 16384, 1), (4, 4096, 28672, 1)])
def test_column_blocks_of_a_workgroup(M, d, ff, width, dt):
    """Two 128-column blocks where a split keeps enough rows (single launch, atomic reduction)."""
    c, _ = dfk.dfk_get_choice(M, d, ff, dt)
    assert (c.variant, c.kmajor, c.reduce, d // 128 // c.k2_col_blocks) == (FUSED, 4, dfk.DFK_REDUCE_ATOMIC, width), c


@pytest.mark.parametrize("dt", [dfk.DFK_BF16, dfk.DFK_FP16])
@pytest.mark.parametrize("d,ff", [(512, 14336), (512, 28672), (640, 28672), (896, 28672), (1024, 28672), (1280, 28672)])
@pytest.mark.parametrize("M", [2, 16, 17, 64])
def test_a_long_d_ff_over_a_narrow_layer_is_cut_into_more_splits(M, d, ff, dt):
    """16 splits of such a layer are 900 to 1800 rows long and a quarter to a half of the CUs' worth of workgroups: up to 28 % slower than
    more of them (512 x 28672).  No split is longer than the layer is wide (counter reduction; twice that where it adds the blocks of
    more than 16 tokens) or three quarters of that (atomic reduction), and there are never more workgroups of the down kernel than CUs."""
    pick, _ = dfk.dfk_get_choice(M, d, ff, dt)
    rows = d * 3 // 4 if pick.reduce == dfk.DFK_REDUCE_ATOMIC else d * (2 if M > 16 else 1)
    blocks = d // 128
    assert pick.k2_splits == min(256 // blocks, max(16, ff // rows)), pick
    block_pick = next(c for c in cands(M, d, ff, dt) if c.kmajor == 1 and c.variant == TWO and c.k2_col_blocks == blocks)
    assert block_pick.reduce == dfk.DFK_REDUCE_TICKET      # what dfk_mlp_block takes
    assert block_pick.k2_splits == min(256 // blocks, max(16, ff // (d * (2 if M > 16 else 1))))


@pytest.mark.parametrize("dt", [dfk.DFK_BF16, dfk.DFK_FP16])
@pytest.mark.parametrize("M,d,ff,splits", [
    (256, 512, 28672, 56), (256, 128, 28672, 56), (1, 256, 28672, 56), (1, 256, 8192, 16), (100, 1024, 14336, 16), (200, 1024, 14336, 16), (256, 2048, 11264, 16),  # a long d_ff
    (96, 1920, 10496, 16), (128, 1152, 5504, 12), (205, 1152, 5504, 16), (200, 2048, 5504, 12), (200, 1024, 5376, 14),  # no whole steps; few column blocks
    (256, 2304, 9216, 12), (212, 2048, 4096, 8), (231, 2304, 3456, 9), (256, 3072, 8192, 8), (256, 3584, 18944, 8), (85, 2048, 9984, 13),   # whole steps
    (256, 1536, 8960, 14), (256, 2432, 6656, 8),
    (128, 3200, 13312, 10), (68, 4480, 23040, 7), (212, 6912, 20352, 4),            # whole steps would leave too few workgroups
    (239, 2816, 3712, 11), (80, 896, 2816, 11), (200, 1024, 1000, 12), (256, 4096, 14336, 8), (150, 8192, 28672, 4), (256, 32768, 8192, 1), (65, 512, 64, 8)])
def test_split_counts_of_the_256_token_pair(M, d, ff, splits, dt):
    pick, _ = dfk.dfk_get_choice(M, d, ff, dt)
    assert (pick.kmajor, pick.reduce, pick.k2_splits) == (2, dfk.DFK_REDUCE_TICKET, splits)


def test_the_remembered_choice_is_what_a_new_thread_finds():
    """More problems than a thread remembers, asked for twice in different orders, against a thread that starts from nothing."""
    probs = [(M, d, ff, dt) for M in (1, 7, 64, 65, 256) for d in (512, 520, 896, 4096, 5120) for ff in (1536, 14336)
             for dt in (dfk.DFK_BF16, dfk.DFK_FP16, dfk.DFK_FP32)]
    ask = lambda q: [(dfk.dfk_get_choice(*x)[0].as_dict(), dfk.dfk_get_choice_wdt(*x)[0].as_dict()) for x in q]
    first, again = ask(probs), ask(probs[::-1])[::-1]
    got = []
    t = threading.Thread(target=lambda: got.extend(ask(probs)))
    t.start()
    t.join()
    assert first == again == got


@pytest.mark.parametrize("M,d,ff,split", [(16, 4096, 14336, False), (17, 4096, 14336, True), (64, 4096, 14336, True), (65, 12288, 12288, True),
                                          (64, 12288, 12288, False), (48, 8192, 7168, False), (64, 8192, 7168, True), (64, 1024, 2816, False),
                                          (32, 896, 4864, True), (32, 512, 2048, False), (48, 512, 2048, True), (256, 512, 1024, True),
                                          (20, 3072, 7680, False), (32, 3584, 9216, False), (33, 3584, 9216, True), (17, 2304, 9216, True), (32, 4096, 8192, False),
                                          (48, 4096, 8192, False), (64, 4096, 8192, True), (48, 3072, 8192, True), (48, 1536, 4096, False), (64, 1536, 4096, True),
                                          (48, 6144, 8064, True), (32, 6144, 8064, False)])
def test_which_down_kernel_the_transposed_layout_gets(M, d, ff, split):
    for dt in (dfk.DFK_BF16, dfk.DFK_FP16):
        pick, tuned = dfk.dfk_get_choice_wdt(M, d, ff, dt)
        assert not tuned and (pick.path, pick.kmajor) == (MFMA, 5)
        assert pick.k2_col_blocks == (d // 128 if split else 1), pick
        assert dfk.dfk_config_valid(pick, M, d, ff, dt)


@pytest.mark.parametrize("d,ff,kmajor", [(4096, 14336, 1), (4096, 16384, 1), (4096, 16392, 4), (4096, 8184, 4), (2048, 5504, 1), (3072, 8192, 1),
                                         (1024, 5632, 4), (2304, 9216, 4), (5120, 13824, 4), (8192, 28672, 4)])
def test_which_single_launch_one_token_gets(d, ff, kmajor):
    for dt in (dfk.DFK_BF16, dfk.DFK_FP16):
        pick, tuned = dfk.dfk_get_choice(1, d, ff, dt)
        assert not tuned and (pick.variant, pick.path, pick.kmajor, pick.reduce) == (FUSED, MFMA, kmajor, dfk.DFK_REDUCE_ATOMIC), pick


@pytest.mark.parametrize("M,d,ff,splits", [(2, 896, 4864, 16), (3, 768, 3072, 12), (16, 896, 4864, 16), (17, 896, 4864, 12), (16, 896, 4608, 12), (64, 640, 2560, 12),
                                           (16, 512, 6136, 16), (64, 512, 6144, 12), (64, 512, 6152, 16)])
def test_splits_of_the_counter_reduction_on_narrow_layers(M, d, ff, splits):
    pick, tuned = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
    assert not tuned and (pick.variant, pick.kmajor, pick.reduce, pick.k2_splits) == (TWO, 1, dfk.DFK_REDUCE_TICKET, splits), pick


@pytest.mark.parametrize("M,d,ff,depth", [(1, 2304, 9216, 3), (8, 4096, 14336, 2), (16, 1024, 2816, 3), (8, 1024, 2816, 3), (24, 1024, 2816, 3), (16, 2432, 4096, 3),
                                           (1, 3072, 8192, 3), (16, 3456, 8192, 3), (29, 3200, 4352, 3), (1, 3584, 8192, 2), (16, 3584, 18944, 2), (1, 3968, 8192, 2), (4, 8192, 7168, 2)])
def test_ring_of_the_transposed_layout(M, d, ff, depth):
    """Three slots below seven eighths of the CUs' worth of 16-row tiles, at every token count (3200 x 4352 at 29 tokens is 3 % slower
    with two, 3584 x 18944 at 16 4 % with three)."""
    pick, _ = dfk.dfk_get_choice_wdt(M, d, ff, dfk.DFK_BF16)
    assert (pick.kmajor, pick.k2_col_blocks, pick.waves, pick.depth) == (5, 1, 8, depth), pick


@pytest.mark.parametrize("d,ff", [(256, 128), (256, 14336), (384, 640), (512, 128), (1024, 256), (4096, 384)])
@pytest.mark.parametrize("M", [1, 16, 17, 33, 64, 65, 200, 256])
def test_half_inputs_of_the_transposed_layout_keep_a_wide_a2_where_they_had_it(M, d, ff):
    """Without four 128-wide chunks each way the plain-FMA pair is the choice for half inputs, at every token count alike: it keeps A_2 in
    fp32.  The split form rounds it to half, so it is there for a caller who asks, and nobody else."""
    pick, tuned = dfk.dfk_get_choice_wdt(M, d, ff, dfk.DFK_FP16)
    assert not tuned and (pick.path, pick.a2_dtype) == (VALU, dfk.DFK_FP32), pick
    pick, _ = dfk.dfk_get_choice_wdt(M, 512, 512, dfk.DFK_FP16)
    assert pick.path == MFMA, pick


def _pair_of(M, d, ff, dt):
    return next(c for c in cands(M, d, ff, dt) if c.variant == TWO and c.kmajor == 1)


def _is_launch_form_of(c, pair):
    return c.as_dict() == dict(pair.as_dict(), variant=FUSED, kmajor=4, depth=4)


# 48 MB of weights, 100 MB where the width is a multiple of 1024, whatever the token count up to 64; eight wavefronts; not where nearly
# every slice of d_ff has two row tiles
@pytest.mark.parametrize("dt", [dfk.DFK_BF16, dfk.DFK_FP16])
@pytest.mark.parametrize("d,ff,single", [(1536, 5248, True), (1536, 5120, False), (2048, 8192, True), (2048, 8064, False), (1152, 8192, True), (1152, 4096, False),
                                         (896, 28672, False), (2304, 9216, True), (4096, 14336, True), (5120, 40960, True),
                                         (2816, 3328, True), (2816, 3336, False), (3584, 3968, False), (4224, 4096, False), (4224, 4104, True)])
def test_the_form_in_which_a_block_runs_the_pair(d, ff, single, dt):
    for M in (1, 16, 17, 64):
        c, tuned = dfk.dfk_get_choice_block(M, d, ff, dt)
        pair = _pair_of(M, d, ff, dt) if d < 5120 else None       # (wide layers: not the first one listed)
        assert not tuned and dfk.dfk_config_valid(c, M, d, ff, dt)
        assert (c.variant, c.kmajor, c.reduce) == ((FUSED, 4) if single else (TWO, 1)) + (dfk.DFK_REDUCE_TICKET,), c
        if pair is not None:
            assert _is_launch_form_of(c, pair) if single else c.as_dict() == pair.as_dict(), (c, pair)
    c, _ = dfk.dfk_get_choice_block(65, d, ff, dt)
    assert (c.variant, c.kmajor) == (TWO, 2)


@pytest.mark.parametrize("M,d,ff,single", [(1, 2888, 7688, True), (16, 2008, 4008, True), (16, 2008, 3960, False), (17, 2008, 3960, True), (64, 1000, 1008, True),
                                           (64, 1000, 1000, False), (64, 8200, 1000, False), (17, 904, 2400, True), (64, 896 + 64, 2400, True), (64, 888, 2816, False),
                                           (65, 2888, 7688, False)])
def test_the_form_in_which_a_width_off_128_runs_the_pair(M, d, ff, single):
    c, tuned = dfk.dfk_get_choice(M, d, ff, dfk.DFK_BF16)
    pair = _pair_of(M, d, ff, dfk.DFK_BF16)
    assert not tuned and dfk.dfk_config_valid(c, M, d, ff, dfk.DFK_BF16)
    assert _is_launch_form_of(c, pair) if single else c.as_dict() == pair.as_dict(), (c, pair)
    h = dfk.dfk_config_t(**dict(c.as_dict(), a2_dtype=dfk.DFK_FP16))
    assert not dfk.dfk_config_valid(h, M, d, ff, dfk.DFK_FP16)


def test_a_table_does_not_lose_the_single_launch(tmp_path):
    """A tuned pair runs a block in the form that the untuned one would; off 128 that form can be the tuned choice, also through a file, and is
    not taken for an entry of the fused variant."""
    bf = dfk.DFK_BF16
    try:
        M, d, ff = 8, 2304, 9216
        for reduce in (dfk.DFK_REDUCE_TICKET, dfk.DFK_REDUCE_ATOMIC):
            pair = next(c for c in cands(M, d, ff, bf) if c.variant == TWO and c.kmajor == 1 and c.reduce == reduce and c.waves == 8)
            dfk.dfk_set_choice(M, d, ff, bf, pair, 30.0)
            c, tuned = dfk.dfk_get_choice_block(M, d, ff, bf)
            assert tuned and _is_launch_form_of(c, pair), c
        assert dfk.dfk_get_choice(M, d, ff, bf)[0].as_dict() == pair.as_dict()      # the plain call: as set
        M, d, ff = 12, 2888, 7688
        fused = next(c for c in cands(M, d, ff, bf) if c.variant == FUSED)
        one, _ = dfk.dfk_get_choice(M, d, ff, bf)
        pair = _pair_of(M, d, ff, bf)
        for c, us in ((fused, 50.0), (pair, 39.0), (one, 37.0)):
            dfk.dfk_set_choice(M, d, ff, bf, c, us)
        path = str(tmp_path / "table.txt")
        dfk.dfk_save_tuning(path)
        for _ in range(2):
            got, tuned = dfk.dfk_get_choice(M, d, ff, bf)
            assert tuned and got.as_dict() == one.as_dict()
            dfk.dfk_clear_tuning()
            dfk.dfk_load_tuning(path)
        lines = [l.split() for l in open(path) if not l.startswith("#") and l.split()[1] == "2888"]
        assert [(l[4], l[14]) for l in lines] == [(str(fused.variant), str(fused.kmajor)), (str(TWO), "1"), (str(FUSED), "4")], lines
        dfk.dfk_set_choice(M, d, ff, bf, pair, 36.0)
        assert dfk.dfk_get_choice(M, d, ff, bf)[0].as_dict() == pair.as_dict()
    finally:
        dfk.dfk_clear_tuning()


def test_a_block_takes_the_single_launch_by_name():
    import ctypes
    L = dfk.lib()
    M, d, ff = 8, 2304, 9216
    one, _ = dfk.dfk_get_choice_block(M, d, ff, dfk.DFK_BF16)
    p, wsb = [A + (i << 28) for i in range(7)], dfk.dfk_workspace_bytes(M, d, ff)
    call = lambda cfg, d=d: L.dfk_mlp_block(p[0], p[1], 1e-5, p[2], p[3], p[4], p[0] + 16, M, d, ff, dfk.DFK_BF16, ctypes.byref(cfg), p[6], wsb, None)
    assert call(one) == dfk.DFK_ERR_ALIAS                       # accepted as far as that
    local = next(c for c in cands(M, d, ff, dfk.DFK_BF16) if c.variant == FUSED and c.kmajor == 1)
    ok = lambda cfg: L.dfk_mlp_block(p[0], p[1], 1e-5, p[2], p[3], p[4], p[5], M, d, ff, dfk.DFK_BF16, ctypes.byref(cfg), p[6], wsb, None)
    assert ok(local) == dfk.DFK_ERR_UNSUPPORTED_SHAPE
    out = dfk.dfk_config_t()
    q = lambda *a: L.dfk_get_choice_block(*a, ctypes.byref(out), None)
    assert q(8, 2888, 7688, dfk.DFK_BF16, 0) == dfk.DFK_ERR_UNSUPPORTED_SHAPE      # as the call
    assert q(8, 2304, 9216, dfk.DFK_FP32, 0) == dfk.DFK_ERR_UNSUPPORTED_SHAPE
    assert q(0, 2304, 9216, dfk.DFK_BF16, 0) == dfk.DFK_ERR_INVALID_ARG
    assert q(8, 2304, 9216, 7, 0) == dfk.DFK_ERR_INVALID_ARG
    assert q(8, 2304, 9216, dfk.DFK_FP16, 1) == dfk.DFK_OK and out.kmajor == 5
    assert L.dfk_get_choice_block(8, 2304, 9216, dfk.DFK_BF16, 0, None, None) == dfk.DFK_ERR_INVALID_ARG


@pytest.mark.parametrize("M,d,ff,splits", [(8, 512, 4096, 16), (17, 512, 3072, 12), (8, 768, 4224, 12), (33, 896, 7168, 16), (3, 1024, 5632, 12), (3, 1024, 8192, 16), (64, 1024, 8192, 16),
                                           (3, 1536, 12288, 12), (8, 1536, 18176, 16), (64, 2048, 11264, 12), (33, 2048, 16384, 16), (2, 1024, 5632, 16), (8, 1000, 5000, 12), (8, 1000, 8000, 16)])
def test_twelve_splits_where_they_cost_no_wavefront_another_block(M, d, ff, splits):
    """Pair of launches, counter reduction: what a block takes, and a width off 128."""
    c = _pair_of(M, d, ff, dfk.DFK_BF16)
    assert (c.reduce, c.k2_splits) == (dfk.DFK_REDUCE_TICKET, splits), c
    if d % 128 == 0:
        assert dfk.dfk_get_choice_block(M, d, ff, dfk.DFK_BF16)[0].k2_splits == splits


@pytest.mark.parametrize("M,d,ff", [(65, 256, 128), (100, 4096, 14336), (256, 2304, 9216), (256, 1024, 40960)])
def test_candidates_of_the_split_transposed_layout_are_different_launches(M, d, ff):
    """Beyond 64 tokens its kernels take neither waves nor depth from the configuration, so no two candidates differ in those alone."""
    for dt in (dfk.DFK_BF16, dfk.DFK_FP16):
        cs = [dfk.dfk_get_candidate_wdt(M, d, ff, dt, i).as_dict() for i in range(dfk.dfk_num_candidates_wdt(M, d, ff, dt))]
        split = [tuple(v for k, v in c.items() if k not in ("waves", "depth")) for c in cs if c["k2_col_blocks"] > 1]
        assert split and len(set(split)) == len(split)


@pytest.mark.parametrize("d,ff", [(512, 36864), (1024, 32776), (1024, 53248), (4096, 40960), (16384, 53248)])
def test_one_token_of_a_d_ff_that_no_single_launch_takes(d, ff):
    """Beyond 512 slices of 64 rows: the pair of launches, for every small token count alike; up to there the single launch."""
    for dt in (dfk.DFK_BF16, dfk.DFK_FP16):
        for M in (1, 2):
            pick, _ = dfk.dfk_get_choice(M, d, ff, dt)
            assert (pick.variant, pick.kmajor, pick.reduce) == (TWO, 1, dfk.DFK_REDUCE_TICKET), pick
        if d >= 1024:
            assert dfk.dfk_get_choice(1, d, 32768, dt)[0].kmajor == 4


def test_half_off_128_on_the_matrix_cores_is_a_configuration_of_its_own():
    """Path VALU with kmajor = 1: for half inputs off 128 alone, with A_2 in fp32 and the counter reduction; first where it pays."""
    h = dfk.DFK_FP16
    for M, d, ff in ((1, 736, 3472), (3, 2888, 7688), (64, 904, 1000)):
        c, _ = dfk.dfk_get_choice(M, d, ff, h)
        assert (c.path, c.variant, c.kmajor, c.a2_dtype, c.reduce) == (VALU, TWO, 1, dfk.DFK_FP32, dfk.DFK_REDUCE_TICKET), c
        for over in (dict(a2_dtype=h), dict(reduce=dfk.DFK_REDUCE_ATOMIC), dict(variant=FUSED), dict(kmajor=2), dict(kmajor=4), dict(waves=2), dict(path=MFMA)):
            assert not dfk.dfk_config_valid(dfk.dfk_config_t(**dict(c.as_dict(), **over)), M, d, ff, h), over
        for dt in (dfk.DFK_BF16, dfk.DFK_FP32):
            assert not dfk.dfk_config_valid(c, M, d, ff, dt)
        assert not dfk.dfk_config_valid(c, M, (d + 127) // 128 * 128, ff, h)
        plain = next(o for o in cands(M, d, ff, h) if o.variant == TWO and o.kmajor == 0)
        plain = dfk.dfk_config_t(**dict(plain.as_dict(), k2_col_blocks=(d + 127) // 128))
        assert dfk.dfk_config_valid(plain, M, d, ff, h)
        # tokens of a launch: 64 there, 8 of plain FMA, whatever its column blocks (asked of the per-kernel timer, which stops at the scratch)
        us = (ctypes.c_double * 2)()
        timed = lambda cfg, m: dfk.lib().dfk_time_kernels(ctypes.byref(cfg), m, d, ff, h, A, 0, 1, 1, None, us)
        assert (timed(plain, 8), timed(plain, 9)) == (dfk.DFK_ERR_WORKSPACE, dfk.DFK_ERR_UNSUPPORTED_SHAPE)
        assert (timed(c, 64), timed(c, 65)) == (dfk.DFK_ERR_WORKSPACE, dfk.DFK_ERR_UNSUPPORTED_SHAPE)
    for M, d, ff in ((1, 2888, 7688), (2, 8200, 4000), (1, 264, 1000)):
        c, _ = dfk.dfk_get_choice(M, d, ff, h)
        assert (c.path, c.kmajor) == (VALU, 0), c


def test_tables_of_before_that_name_load_as_what_they_named(tmp_path):
    """Version 2 tables say path VALU with a column block per 128 columns for it; the first two shapes have such lines that plain FMA does not take."""
    h = dfk.DFK_FP16
    path = str(tmp_path / "table.txt")
    # M, d_model, d_ff, splits, waves, k2_splits, whether plain FMA takes the configuration too
    for M, d, ff, splits, waves, k2, plain in ((100, 10208, 8376, 256, 8, 3, False), (4, 7632, 25432, 512, 8, 4, False), (16, 736, 3472, 256, 4, 16, True)):
        nblk = (d + 127) // 128
        line = f"{M} {d} {ff} {h} {TWO} {VALU} {splits} {waves} 0 0 {k2} {nblk} {dfk.DFK_FP32} 0 0 25.0\n"
        try:
            open(path, "w").write("# dfk tuning table v2: M d_model d_ff ...\n" + line)
            dfk.dfk_load_tuning(path)
            c, tuned = dfk.dfk_get_choice(M, d, ff, h)
            assert tuned and (c.path, c.kmajor, c.depth, c.k2_splits, c.k2_col_blocks) == (VALU, 1, 3 if waves == 8 else 6, k2, nblk), c
            dfk.dfk_save_tuning(path)
            dfk.dfk_clear_tuning()
            dfk.dfk_load_tuning(path)                                   # as written now: nothing to rename
            assert dfk.dfk_get_choice(M, d, ff, h)[0].as_dict() == c.as_dict()
            dfk.dfk_clear_tuning()
            for head in ("# dfk tuning table v3: M d_model d_ff ...\n", ""):
                open(path, "w").write(head + line)
                if not plain:
                    with pytest.raises(dfk.DfkError):
                        dfk.dfk_load_tuning(path)
                    continue
                dfk.dfk_load_tuning(path)
                assert dfk.dfk_get_choice(M, d, ff, h)[0].kmajor == 0
                dfk.dfk_clear_tuning()
        finally:
            dfk.dfk_clear_tuning()
