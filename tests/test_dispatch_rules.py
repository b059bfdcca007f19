"""The host-side rules that choose a kernel form or size its scratch.  They depend on sizes only: no GPU is needed."""
import ctypes as C

import pytest


@pytest.mark.parametrize("T,d_out,d_in,K2,dense", [
    (300, 22016, 8192, 0, False), (512, 22016, 8192, 128, False), (700, 16384, 8192, 128, False),
    (512, 16384, 8192, 1024, False),
    (512, 4096, 4096, 0, True), (1337, 5120, 5120, 64, True), (2048, 22016, 8192, 0, True), (8192, 4096, 4096, 128, True),
])
def test_forward_dequantizes_first_only_where_it_pays(rules, T, d_out, d_in, K2, dense):
    """22016 x 8192 at 512 tokens: 223 us from the codes, 264 us dequantized first."""
    assert rules.dense_pays(T, d_out, d_in, K2) == dense


@pytest.mark.parametrize("T,d_in,d_out,K2,dense", [
    (1, 22016, 8192, 0, False), (256, 22016, 8192, 0, False), (512, 22016, 8192, 1024, False), (512, 11008, 4096, 0, False),
    (256, 512, 512, 32, True), (512, 4096, 11008, 128, True), (700, 8192, 8192, 0, True), (8192, 8192, 22016, 256, True),
])
def test_backward_dequantizes_first_only_where_it_pays(rules, T, d_in, d_out, K2, dense):
    """dX of 256 tokens, 8192 x 22016: 123 us from the codes, 209 us dequantized first."""
    assert rules.dense_pays_t(T, d_in, d_out, K2) == dense


SHAPES = [(64, 64), (512, 512), (1000, 768), (4096, 4096), (11008, 4096), (4096, 11008), (5120, 13824), (13824, 5120),
          (19200, 768), (22016, 8192), (8192, 22016)]


def _weight(qb, d_out, d_in, grouped=False, block_rows=1, block=64):
    q = qb.CQWeight()
    q.d_out, q.d_in, q.block, q.block_rows = d_out, d_in, block, block_rows
    q.codes = q.scales = 0x1000                          # never dereferenced
    if grouped:
        q.scale_mode, q.scale_group = qb.SCALES_E4M3_GROUPED, 256
        q.scale_codes = q.scale_step = q.scale_mid = 0x1000
    return q


@pytest.mark.parametrize("d_out,d_in", SHAPES)
@pytest.mark.parametrize("kind", ["plain", "grouped", "8x4"])
def test_inference_workspace_serves_smaller_batches(rules, d_out, d_in, kind):
    q = _weight(rules.qb, d_out, d_in, kind == "grouped", *((8, 32) if kind == "8x4" else ()))
    need = [rules.L.qblora_linear_decode_tokens_workspace_bytes(C.byref(q), T) for T in range(0, 300)]
    assert all(a <= b for a, b in zip(need, need[1:]))
    assert need[256] == need[299]


TILES = ["256 x 256", "128 x 256", "256 x 128", "128 x 128", "128 x 192", "192 x 128", "192 x 192"]
TOKENS = sorted({*range(1, 400), *range(400, 3300, 13), 511, 512, 513, 767, 768, 769, 1024, 2047, 2048, 4096, 8192})


@pytest.mark.parametrize("d_out,d_in", SHAPES)
@pytest.mark.parametrize("R,lam,op", [(0, 1, 0), (16, 2, 0), (136, 4, 0), (512, 8, 0), (24, 2, 2)])
def test_layer_workspaces_serve_fewer_tokens(rules, d_out, d_in, R, lam, op):
    """One workspace for the largest batch, then a ragged last one: the slices of a contraction may grow as tokens get
    fewer, the sizes may not."""
    qb, L = rules.qb, rules.L
    d_out = d_out // 64 * 64
    q = _weight(qb, d_out, d_in, grouped=R == 136)
    ad = qb.CAdapter()
    ad.lambda1, ad.lambda2, ad.R, ad.s, ad.scale_op = lam, lam, R, 1.0, op
    if R:
        ad.A = ad.B = 0x1000
    for f in (L.qblora_linear_fwd_workspace_bytes, L.qblora_linear_bwd_workspace_bytes):
        need = [f(C.byref(q), C.byref(ad), T) for T in TOKENS]
        assert need[0] > 0 and all(a <= b for a, b in zip(need, need[1:]))
    for f in (L.qablora_linear_fwd_workspace_bytes, L.qablora_linear_bwd_workspace_bytes):
        need = [f(C.byref(q), lam, lam, T) for T in TOKENS]
        assert need[0] > 0 and all(a <= b for a, b in zip(need, need[1:]))


@pytest.mark.parametrize("N,k1,k2", [(512, 512, 0), (4096, 11008, 128), (4160, 448, 8), (11008, 4096, 1376), (64, 22016, 0)])
def test_partial_sum_rows_are_the_most_of_any_count(rules, N, k1, k2):
    rows = rules.L["_ZN6qblora15dense_part_rowsEliii"]
    rows.argtypes, rows.restype = [C.c_int64, C.c_int, C.c_int, C.c_int], C.c_int64
    most = 0
    for T in range(1, 1500):
        s = rules.dense_plan(T, N, k1, k2, 8).splits
        most = max(most, s * T if s > 1 else 0)
        assert rows(T, N, k1, k2) == most, T


@pytest.mark.parametrize("N,k1,k2", [(512, 512, 0), (4096, 11008, 128), (4160, 448, 8), (11008, 4096, 1376), (64, 22016, 0), (4160, 22720, 24)])
def test_no_contraction_takes_more_slices_than_workspaces_count_on(rules, N, k1, k2):
    """The rows of partial sums of every number of tokens, against what the workspace query reserves for it and for any larger one."""
    rows = rules.L["_ZN6qblora15dense_part_rowsEliii"]
    rows.argtypes, rows.restype = [C.c_int64, C.c_int, C.c_int, C.c_int], C.c_int64
    taken = reserved = 0
    for T in [*range(1, 1500), 2048, 8192]:
        call = rules.dense_call_plan(T, N, k1, k2, 8)
        assert call.splits >= 1 and rules.dense_call_plan(T, N, k1, k2, 1).splits == 1
        taken = max(taken, call.splits * T if call.splits > 1 else 0)
        assert taken <= rows(T, N, k1, k2), T
        assert reserved <= (reserved := rows(T, N, k1, k2))


@pytest.mark.parametrize("T,N,k1,k2,shape", [
    (8192, 22016, 8192, 256, "256 x 256"), (8192, 4096, 4096, 128, "256 x 256"), (2048, 4096, 4096, 128, "128 x 256"),
    (3000, 8192, 3072, 64, "128 x 256"), (1024, 4096, 4096, 512, "128 x 128"), (334, 4224, 8000, 64, "128 x 128"),
    (512, 11008, 4096, 128, "128 x 192"), (260, 14336, 2560, 32, "192 x 128"), (1337, 5120, 5120, 64, "128 x 256"), (1337, 5760, 5760, 64, "192 x 192"),
    (2921, 12416, 13120, 0, "256 x 256"), (2156, 16512, 13952, 64, "256 x 256"), (637, 14528, 8512, 0, "256 x 256"),
])
def test_tiles_of_a_contraction(rules, T, N, k1, k2, shape):
    """512 x 11008 x 4224: 39 us in 128 x 192 tiles, 42 in 128 x 256, 54 in 128 x 128.  2921 x 12416 x 13120 with the pass over the weight:
    875 in 256 x 256, 1013 in 128 x 192, which fetch half as much again from beyond the memory-side cache."""
    assert TILES[rules.dense_call_plan(T, N, k1, k2, 1).shape] == shape


@pytest.mark.parametrize("T,N,k1,k2,shape,slices", [
    (512, 4096, 11008, 128, "128 x 256", 4), (698, 4160, 22720, 0, "256 x 256", 5), (663, 6016, 16960, 64, "192 x 192", 2),
    (775, 10688, 19776, 0, "256 x 256", 1), (154, 896, 14016, 64, "128 x 128", 8),
])
def test_slices_of_a_contraction(rules, T, N, k1, k2, shape, slices):
    """698 x 4160 x 22720: 183 us with the pass over the weight in five slices of 256 x 256, 201 in two of 128 x 256, 244 in 128 x 128."""
    plan = rules.dense_call_plan(T, N, k1, k2, 8)
    assert (TILES[plan.shape], plan.splits) == (shape, slices)


@pytest.mark.parametrize("T,d_out,d_in,R", [(1950, 64, 4672, 32), (4887, 64, 2368, 64), (14, 192, 17152, 8), (200, 64, 3072, 16),
                                            (1337, 5120, 5120, 64)])
def test_backward_needs_no_room_for_a_recomputed_activation(rules, T, d_out, d_in, R):
    """s*U that is recomputed beside dU takes the room of the gradients: sizes that a program keeps stay enough."""
    splits = rules.L["_ZN6qblora11grad_splitsElii"]
    splits.argtypes, splits.restype = [C.c_int64, C.c_int, C.c_int], C.c_int
    rows = {}
    for name, sym in (("dense", "_ZN6qblora15dense_part_rowsEliii"), ("narrow", "_ZN6qblora16skinny_part_rowsElii")):
        rows[name] = rules.L[sym]
        rows[name].argtypes, rows[name].restype = [C.c_int64] + [C.c_int] * (3 if name == "dense" else 2), C.c_int64
    q = _weight(rules.qb, d_out, d_in)
    ad = rules.qb.CAdapter()
    ad.lambda1, ad.lambda2, ad.R, ad.s, ad.A, ad.B = 2, 2, R, 1.0, 0x1000, 0x1000
    part = max(4 * rows["dense"](T, d_in, d_out, R) * d_in, 4 * splits(T, d_in, 1) * d_in * R,
               4 * R * max(rows["narrow"](T, R, d_in), rows["narrow"](T, R, d_out)))
    buffers = [2 * d_out * d_in, 2 * R * d_in, 2 * R * d_out, *[2 * T * R] * 5, part, 4 * splits(T, d_out, 1) * d_out * R]
    need = rules.L.qblora_linear_bwd_workspace_bytes(C.byref(q), C.byref(ad), T)
    assert need == sum((b + 255) // 256 * 256 for b in buffers)


@pytest.mark.parametrize("d_out,d_in,T,table,groups", [
    (22016, 8192, 1, False, 3), (22016, 8192, 2, False, 6), (22016, 4096, 8, False, 3), (22016, 8192, 8, True, 3),
    (22016, 8192, 1, True, 1), (19200, 4096, 1, True, 1), (16384, 1024, 1, True, 4), (13824, 4096, 2, True, 4),
    (19200, 8192, 17, True, 6), (11008, 4096, 48, False, 3), (13824, 8192, 32, False, 4), (4096, 4096, 64, False, 1),
])
def test_row_groups_of_small_batches(rules, d_out, d_in, T, table, groups):
    """19200 x 4096 codebook weights, one token: 12.7 us with one group, 14.4 with the three of packed INT4."""
    f = rules.L["_ZN6qblora13w4_row_groupsEiiib"]
    f.argtypes, f.restype = [C.c_int, C.c_int, C.c_int, C.c_bool], C.c_int
    assert f(d_out, d_in, T, table) == groups


@pytest.mark.parametrize("d_out,d_in,T,table,tiled,rows", [
    (2048, 13824, 32, False, True, False), (4096, 8192, 48, False, True, True), (4096, 9728, 64, False, True, False),
    (8192, 22016, 32, False, True, False), (8192, 13824, 48, False, True, True), (19200, 8192, 17, True, True, False),
    (19200, 8192, 17, True, False, True), (22016, 13824, 16, True, True, True), (11008, 4096, 48, False, True, True),
    (3072, 8192, 49, False, True, False), (13824, 13824, 49, True, True, False), (13824, 8192, 17, True, True, True),
    (22016, 13824, 64, False, True, True), (4096, 13824, 32, True, True, True), (4096, 4096, 65, False, True, False),
])
def test_form_of_up_to_64_tokens(rules, d_out, d_in, T, table, tiled, rows):
    """INT4 2048 x 13824 at 32 tokens, weights from HBM: 19.9 us in whole rows, 16.8 in slices of the input."""
    f = rules.L["_ZN6qblora15w4_rows_appliesEiiibb"]
    f.argtypes, f.restype = [C.c_int, C.c_int, C.c_int, C.c_bool, C.c_bool], C.c_bool
    assert f(d_out, d_in, T, table, tiled) == rows


@pytest.mark.parametrize("d_out,d_in,T,slices", [(8192, 8192, 96, 4), (11008, 13824, 65, 5), (22016, 13824, 97, 2), (11008, 4096, 65, 2)])
def test_slices_of_65_to_128_tokens(rules, d_out, d_in, T, slices):
    """INT4 11008 x 13824 at 65 tokens: 54.3 us in two slices, which one round of workgroups holds, 43.7 in five."""
    call = rules.L["_ZN6qblora18w4_mid_call_splitsEiiib"]
    call.argtypes, call.restype = [C.c_int, C.c_int, C.c_int, C.c_bool], C.c_int
    assert call(d_out, d_in, T, False) == slices


def test_no_call_takes_more_slices_than_its_workspace_counts_on(rules):
    call, most = rules.L["_ZN6qblora18w4_mid_call_splitsEiiib"], rules.L["_ZN6qblora13w4_mid_splitsEiii"]
    call.argtypes, call.restype = [C.c_int, C.c_int, C.c_int, C.c_bool], C.c_int
    most.argtypes, most.restype = [C.c_int] * 3, C.c_int
    for d_out in [8, 64, 1000, 4096, 8192, 11008, 16384, 22016, 50000]:
        for d_in in [64, 192, 1024, 4096, 13824, 22016]:
            for T in [17, 32, 64, 65, 96, 97, 128, 129, 192, 256]:
                for table in (False, True):
                    assert 1 <= call(d_out, d_in, T, table) <= most(d_out, d_in, T)


class MergeDesc(C.Structure):
    """The library's description of one weight's merge (csrc/common.h)."""
    _fields_ = [*[(n, C.c_void_p) for n in ("codes", "scales", "beta", "scale_codes", "scale_step", "scale_mid")],
                ("scale_group", C.c_int), ("codebook", C.c_float * 16), ("d_out", C.c_int), ("d_in", C.c_int),
                ("H", C.c_void_p), ("lam1", C.c_int), ("lam2", C.c_int), ("s", C.c_float),
                *[(n, C.c_void_p) for n in ("codes_out", "alpha_out", "beta_out", "w16_out")],
                ("block_rows", C.c_int), ("block_cols", C.c_int), ("magic", C.c_uint32)]


@pytest.mark.parametrize("kind", ["absmax", "int4", "grouped", "8x8", "8x4"])
def test_merges_that_wait_for_each_other_share_no_launch(rules, kind):
    """No output of one weight may lie in what another reads or writes, up to its last byte: the weights of a launch run side
    by side.  The addresses are made up; nothing is launched where the rule says so."""
    rule, launch = rules.L["_ZN6qblora11independentEPKNS_9MergeDescEi"], rules.L["_ZN6qblora26launch_merge_requant_batchEPKNS_9MergeDescEiP12ihipStream_t"]
    rule.argtypes, rule.restype = [C.c_void_p, C.c_int], C.c_bool
    launch.argtypes, launch.restype = [C.c_void_p, C.c_int, C.c_void_p], C.c_int
    d_out, d_in, lam1, lam2, group = 24, 192, 2, 4, 7
    blocks = d_out * d_in // {"8x4": 32}.get(kind, 64)
    groups = -(-blocks // group)
    sizes = {"codes": d_out * d_in // 2, "scales": 4 * blocks, "beta": 4 * blocks, "scale_codes": blocks, "scale_step": 4 * groups,
             "scale_mid": 4 * groups, "H": 4 * (d_in // lam1) * (d_out // lam2), "codes_out": d_out * d_in // 2,
             "alpha_out": 4 * blocks, "beta_out": 4 * blocks}
    names = [n for n in sizes if not (n.startswith("scale_") and kind != "grouped") and (n, kind) not in
             {("scales", "grouped"), ("beta", "absmax"), ("beta", "grouped")}]

    def pair():
        ds, at = (MergeDesc * 2)(), 1 << 20
        for d in ds:
            for n in names:
                setattr(d, n, at)
                at += -(-sizes[n] // 4) * 4                                    # one right behind the other
            d.scale_group, d.d_out, d.d_in, d.lam1, d.lam2, d.s = group, d_out, d_in, lam1, lam2, 1.0
            d.block_rows, d.block_cols = (8, int(kind[2])) if kind[0] == "8" else (1, 64)
        return ds

    assert rule(pair(), 2)
    ds = pair()
    for n in names[:-3]:
        setattr(ds[1], n, getattr(ds[0], n))                                   # what is only read may be shared
    ds[0].codes_out, ds[0].alpha_out = ds[0].codes, ds[0].scales or ds[0].alpha_out
    ds[1].codes = ds[1].codes_out
    if kind != "grouped":
        ds[1].scales = ds[1].alpha_out
    assert rule(ds, 2)                                                         # each in place
    for x, y in ((0, 1), (1, 0)):
        for out in ("codes_out", "alpha_out", "beta_out"):
            for n in names:
                for at in (0, sizes[n] - 1, 1 - sizes[out]):
                    ds = pair()
                    setattr(ds[x], out, getattr(ds[y], n) + at)
                    assert not rule(ds, 2), (x, out, n, at)
                    assert launch(ds, 2, None) == -3           # QBLORA_ERR_UNSUPPORTED
