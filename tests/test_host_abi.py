"""Host-side logic of the library, through the C ABI, against the oracle and the paper's examples (no GPU)."""
import ctypes as C
import os
import random
import re

import numpy as np
import pytest

from paper_2111_14255_amd import binding as B, api, report
from oracle import schedule as S, fold as ofold, ops as oops
from synth import GraphBuilder, zoo, weights
import code_objects

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
I32 = C.c_int32


def arr(vals):
    return (I32 * max(1, len(vals)))(*vals)


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "mtsched.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(mt_[a-z0-9_]+)\s*\(", hdr)) - {"mt_cost_fn"}
    declared -= {"mt_share_cost_fn"}
    assert declared == set(B.SIGNATURES), declared ^ set(B.SIGNATURES)
    lib = B.load()
    for name in declared:
        assert getattr(lib, name) is not None


def lib_expand(lens, rho, n_stages):
    n = len(lens)
    flat = [v for r in rho for v in r]
    out = (I32 * (n_stages * n * 2))()
    rc = B.load().mt_expand_pointers(n, arr(lens), n_stages, arr(flat), out)
    if rc != 0:
        return rc
    return [[(out[(s * n + i) * 2], out[(s * n + i) * 2 + 1]) for i in range(n)] for s in range(n_stages)]


def test_expand_worked_examples():
    st = lib_expand([10], [[3, 5, 7]], 4)
    assert [list(range(b + 1, e + 1)) for (b, e), in st] == [[1, 2, 3], [4, 5], [6, 7], [8, 9, 10]]
    st = lib_expand([10, 4, 5], [[3, 5], [1, 2], [2, 2]], 3)
    assert st[0] == [(0, 3), (0, 1), (0, 2)] and st[1] == [(3, 5), (1, 2), (2, 2)]


def test_expand_matches_oracle_random():
    rng = random.Random(1)
    for _ in range(300):
        n, p = rng.randint(1, 8), rng.randint(0, 7)
        lens = [rng.randint(1, 150) for _ in range(n)]
        rho = [sorted(rng.randint(0, L) for _ in range(p)) for L in lens]
        assert lib_expand(lens, rho, p + 1) == [list(s) for s in S.expand(lens, rho)]


def test_expand_rejects_invalid():
    assert lib_expand([5], [[3, 2]], 3) == B.MT_ERR_INVALID_SCHEDULE
    assert b"non-decreasing" in B.load().mt_last_error()
    assert lib_expand([5], [[6]], 2) == B.MT_ERR_INVALID_SCHEDULE
    assert lib_expand([5], [[1] * 16], 17) == B.MT_ERR_INVALID_SCHEDULE


def lib_issue(stage, conc, order):
    n = len(stage)
    flat = [v for s in stage for v in s]
    total = sum(e - b for b, e in stage)
    out = (I32 * max(1, 3 * total))()
    cnt = I32()
    rc = B.load().mt_issue_order_of_stage(n, arr(flat), conc, order, out, C.byref(cnt))
    assert rc == 0
    return [(out[3 * k], out[3 * k + 1], out[3 * k + 2]) for k in range(cnt.value)]


def test_issue_order_examples_and_oracle():
    stage = [(0, 3), (0, 1), (0, 2)]
    assert [(s + 1, i + 1) for s, t, i in lib_issue(stage, 3, B.MT_ISSUE_BFS)] == [(1, 1), (2, 1), (3, 1), (1, 2), (3, 2), (1, 3)]
    assert [(s + 1, i + 1) for s, t, i in lib_issue(stage, 3, B.MT_ISSUE_DFS)] == [(1, 1), (1, 2), (1, 3), (2, 1), (3, 1), (3, 2)]
    rng = random.Random(2)
    for _ in range(300):
        n = rng.randint(1, 8)
        stage = []
        for _ in range(n):
            b = rng.randint(0, 20)
            stage.append((b, b + rng.choice([0, 0, 1, 2, 5, 9])))
        conc = rng.randint(1, n + 1)
        for order, name in ((B.MT_ISSUE_BFS, "bfs"), (B.MT_ISSUE_DFS, "dfs")):
            assert lib_issue(stage, conc, order) == S.issue_order(stage, conc, name)


def lib_search(lens, n_stages, rounds, cands, seed, algo, cost, seed_baselines=0):
    n, P = len(lens), n_stages - 1
    opts = B.mt_search_opts(algo, n_stages, rounds, cands, 1, 0, 0, 0, seed_baselines, 0, 0, 0, 0, 0, seed)
    cap = rounds * n * cands + 2
    best = (I32 * max(1, n * P))()
    bc = C.c_double()
    recp = (I32 * max(1, cap * n * P))()
    recc = (C.c_double * cap)()
    nrec = I32()

    def cb(ptr, _user):
        return cost([[ptr[i * P + j] for j in range(P)] for i in range(n)])

    fn = B.mt_cost_fn(cb)
    rc = B.load().mt_search_pointers(n, arr(lens), C.byref(opts), fn, None, best, C.byref(bc), recp, recc, cap, C.byref(nrec))
    assert rc == 0, B.load().mt_last_error()
    rho = [[best[i * P + j] for j in range(P)] for i in range(n)]
    recs = [([[recp[(k * n + i) * P + j] for j in range(P)] for i in range(n)], recc[k]) for k in range(nrec.value)]
    return rho, bc.value, recs


def _cost(target):
    return lambda rho: float(sum((a - b) ** 2 for r, t in zip(rho, target) for a, b in zip(r, t))) + 0.5


def test_coordinate_descent_matches_oracle():
    lens = [23, 21, 54]
    target = [[5, 11, 17], [3, 9, 20], [10, 30, 50]]
    for seed in (1, 7, 123456789):
        rho, c, recs = lib_search(lens, 4, 3, 4, seed, B.MT_SEARCH_COORDINATE, _cost(target))
        orho, oc, orecs = S.coordinate_descent(lens, 3, 3, 4, _cost(target), seed)
        assert recs == [(r, c2) for r, c2 in orecs]
        assert rho == orho and c == oc
        assert len(recs) == 3 * 3 * 4


def test_search_with_baseline_seeds_matches_oracle():
    lens = [23, 21, 54]
    target = [[23, 23, 23], [21, 21, 21], [50, 52, 54]]       # close to "everything in stage 1"
    for algo, fn in ((B.MT_SEARCH_COORDINATE, lambda: S.coordinate_descent(lens, 3, 2, 3, _cost(target), 5, seed_baselines=True)[:3]),
                     (B.MT_SEARCH_RANDOM, lambda: S.random_search(lens, 3, 2 * 3 * 3, _cost(target), 5, seed_baselines=True)[:3])):
        rho, c, recs = lib_search(lens, 4, 2, 3, 5, algo, _cost(target), seed_baselines=1)
        orho, oc, orecs = fn()
        assert recs == orecs and rho == orho and c == oc
        assert recs[0][0] == [[23] * 3, [21] * 3, [54] * 3] and recs[1][0] == S.even_split(lens, 3)


def test_random_search_matches_oracle():
    lens = [9, 12]
    target = [[2, 6], [4, 8]]
    rho, c, recs = lib_search(lens, 3, 10, 5, 99, B.MT_SEARCH_RANDOM, _cost(target))
    orho, oc, orecs, skipped = S.random_search(lens, 2, 10 * 2 * 5, _cost(target), 99)
    assert recs == orecs and rho == orho and c == oc and skipped > 0


def lib_playoff(lens, n_stages, recs, top_k, cost):
    n, P = len(lens), n_stages - 1
    flat = [v for rho, _ in recs for row in rho for v in row]
    costs = (C.c_double * max(1, len(recs)))(*[c for _, c in recs])
    best = (I32 * max(1, n * P))()
    bc = C.c_double()
    nev = I32()
    seen = []

    def cb(ptr, _user):
        rho = [[ptr[i * P + j] for j in range(P)] for i in range(n)]
        seen.append(rho)
        return cost(rho)

    fn = B.mt_cost_fn(cb)
    rc = B.load().mt_playoff_pointers(n, arr(lens), n_stages, arr(flat), costs, len(recs), top_k, fn, None, best, C.byref(bc), C.byref(nev))
    assert rc == 0, B.load().mt_last_error()
    assert nev.value == len(seen)
    return [[best[i * P + j] for j in range(P)] for i in range(n)], bc.value, seen


def test_record_memory_round_trips_through_a_file_and_feeds_the_playoff(tmp_path):
    from paper_2111_14255_amd import api
    lens = [9, 12]
    target = [[2, 6], [4, 8]]
    rho, c, recs = lib_search(lens, 3, 3, 4, 5, B.MT_SEARCH_COORDINATE, _cost(target))
    path = str(tmp_path / "records.json")
    api.save_records(path, lens, 3, recs, note="unit test")
    lens2, n_stages2, recs2 = api.load_records(path)
    assert (lens2, n_stages2, recs2) == (lens, 3, recs)
    # the stored memory is all the play-off needs: same winner as on the live records, and as the oracle's rule
    final = lambda r: _cost(target)(r) + 0.25
    got = lib_playoff(lens2, n_stages2, recs2, 3, final)
    assert got[:2] == lib_playoff(lens, 3, recs, 3, final)[:2] == S.playoff(lens, 2, recs, 3, final)[:2]
    # a file whose matrices do not fit the operator counts is refused
    import json
    doc = json.load(open(path))
    doc["records"][0]["pointers"][0] = [7, 3]
    json.dump(doc, open(path, "w"))
    with pytest.raises(ValueError):
        api.load_records(path)


def test_playoff_matches_oracle_and_can_overturn_the_first_measurement():
    lens = [23, 21, 54]
    target = [[5, 11, 17], [3, 9, 20], [10, 30, 50]]
    _, _, recs = S.coordinate_descent(lens, 3, 2, 4, _cost(target), 11, seed_baselines=True)
    recs = recs + [recs[3]]                                       # a duplicate matrix must be measured once only
    one_stage = [[n] * 3 for n in lens]
    # second measurement: the noisy first one is replaced by a cost that prefers the one-stage matrix, then the third-best record
    order = sorted(range(len(recs)), key=lambda j: (recs[j][1], j))
    third = recs[order[2]][0]
    final = lambda rho: 1.0 if rho == one_stage else 2.0 if rho == third else 3.0 + _cost(target)(rho)
    for top_k in (1, 3, 5):
        rho, c, seen = lib_playoff(lens, 4, recs, top_k, final)
        orho, oc, oscored = S.playoff(lens, 3, recs, top_k, final)
        assert rho == orho and c == oc and seen == [m for m, _ in oscored]
        assert rho == one_stage and c == 1.0 and seen[-1] == one_stage and len(seen) == top_k + 1
    # without the one-stage preference the winner is the best of the second measurements, not of the first
    final2 = lambda rho: 2.0 if rho == third else 3.0 + _cost(target)(rho)
    rho, c, seen = lib_playoff(lens, 4, recs, 3, final2)
    assert (rho, c) == S.playoff(lens, 3, recs, 3, final2)[:2] and rho == third
    # the one-stage matrix is not measured twice when it is already among the leaders; ties go to the earlier candidate
    recs2 = [(one_stage, 0.1)] + recs
    rho, c, seen = lib_playoff(lens, 4, recs2, 2, lambda r: 5.0)
    assert seen.count(one_stage) == 1 and rho == one_stage and len(seen) == 2
    assert (rho, c) == S.playoff(lens, 3, recs2, 2, lambda r: 5.0)[:2]


def test_single_stage_search_is_trivial():
    rho, c, recs = lib_search([4, 5], 1, 1, 2, 5, B.MT_SEARCH_COORDINATE, lambda r: 3.0)
    assert rho == [[], []] and c == 3.0


def test_fold_bn_matches_oracle_bitwise():
    m = zoo.resnet18("f16", 1)
    raw = weights.make_params(m, 5, 0)
    for p in raw[:6]:
        if p is None or p["bn"] is None:
            continue
        w1, b1 = api.fold_bn(p["w"], p["bn"])
        w2, b2 = ofold.fold_bn(p["w"], p["bn"])
        np.testing.assert_array_equal(w1, w2)
        np.testing.assert_array_equal(b1, b2)


def test_storage_casts_match_oracle_rounding():
    v = (np.random.default_rng(3).standard_normal(5000) * np.exp(np.random.default_rng(4).uniform(-20, 12, 5000))).astype(np.float32)
    for dt in ("f16", "bf16"):
        with np.errstate(over="ignore"):
            mine = api.from_storage(api.to_storage(v, dt), dt)
        np.testing.assert_array_equal(mine, oops.round_array(v, dt))


@pytest.mark.parametrize("name", ["tinyA", "tinyB", "tinyC", "tinyD", "resnet18", "resnet50", "vgg16", "mobilenetv2", "alexnet",
                                  "alexnet_published", "inceptionv3"])
def test_shape_inference_matches_model_tables(name):
    spec = zoo.BUILDERS[name]("f16", 2)
    m = api.Model(spec)
    assert m.num_ops() == len(spec.ops)
    flops = 0
    for i, op in enumerate(spec.ops):
        info = m.op_info(i)
        assert (info.in_h, info.in_w, info.in_c) == tuple(op.in_shape)
        assert (info.out_h, info.out_w, info.out_c) == tuple(op.out_shape)
        if op.kind in ("conv", "dwconv", "fc"):        # the MAC-counting kinds; normalisation and add report their own count
            flops += info.flops
        assert info.bytes > 0
    assert flops == 2 * spec.macs()
    assert m.out_features() == spec.out_features
    assert m.arena_bytes() > 0


@pytest.mark.parametrize("c,k", [(64, 320), (512, 512), (512, 2048)])
def test_3x3_layers_on_maps_of_a_few_pixels_have_a_kernel_at_every_batch(c, k):
    """The taps of a 3x3 layer are read from a patch of input pixels in LDS, which holds the rows around a tile in every image
    the tile touches: on maps of a pixel or two those of a batch are more than any patch holds."""
    for h, w in ((1, 1), (1, 2), (2, 1), (2, 2), (1, 3), (3, 1), (1, 7), (7, 1)):
        for n in (1, 2, 31, 65, 300, 800, 1200, 2048, 5000):
            for dtype in ("f16", "f32"):
                g = GraphBuilder("t", dtype, n, h, w, c)
                g.conv(0, k, 3, pad=1)
                m = api.Model(g.done())
                info = m.op_info(0)
                assert info.grid_blocks > 0 and info.split_k >= 1
                assert m.arena_bytes() < (1 << 31)
                m.close()


@pytest.mark.parametrize("dtype,n,hw,c,k,win,form", [
    ("f16", 1, 14, 256, 256, 3, ("ring_16x16", 16, 16, 1, 1, 8, 0)),
    ("f16", 1, 4, 1024, 100, 3, ("tile_64x16", 64, 16, 2, 8, 0, 0)),
    ("f16", 1, 28, 512, 256, 3, ("patch_64x64", 64, 64, 3, 4, 0, 28)),
    ("f16", 1, 9, 100, 40, 3, ("elements_64x16", 64, 16, 1, 2, 0, 0)),
    ("f16", 1, 14, 64, 64, 1, ("igemm_pointwise", 0, 0, 0, 1, 0, 0)),
    ("f16", 1, 200, 64, 64, 1, ("igemm_resident_filters", 0, 0, 0, 1, 0, 0)),
    ("f16", 1, 96, 64, 64, 1, ("tile_64x64", 64, 64, 1, 1, 0, 0)),
    ("f32", 1, 41, 32, 70, 3, ("tile_64x16", 64, 16, 2, 1, 0, 0)),
    ("f32", 1, 57, 16, 24, 3, ("registers_32x16", 32, 16, 0, 1, 0, 0)),
])
def test_op_form_names_the_kernel_and_tells_a_split_from_a_ring(dtype, n, hw, c, k, win, form):
    g = GraphBuilder("t", dtype, n, hw, hw, c)
    g.conv(0, k, win, pad=win // 2)
    m = api.Model(g.done())
    f = m.op_form(0)
    assert (f.name.decode(), f.tile_channels, f.tile_pixels, f.stage_slices, f.split_k, f.ring_waves, f.panel_columns) == form
    assert m.op_info(0).split_k == f.split_k
    tiles = -(-k // max(1, f.tile_channels)) * -(-n * hw * hw // max(1, f.tile_pixels))
    assert f.workspace_bytes == (0 if f.split_k == 1 else tiles * f.split_k * f.tile_channels * f.tile_pixels * 4 + tiles * 4)
    out = B.mt_op_form()
    assert B.load().mt_model_op_form(m.h, 1, C.byref(out)) == B.MT_ERR_INVALID_ARG
    assert B.load().mt_model_op_form(None, 0, C.byref(out)) == B.MT_ERR_INVALID_ARG
    m.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("n,h,w,win,columns", [
    (1, 14, 14, 3, 8),       # 14 rectangles of 2 x 8, 13 tiles of consecutive pixels
    (1, 12, 12, 3, 4),       # 9 of 4 x 4, 12 of 2 x 8
    (1, 8, 8, 3, 4),         # as many of either
    (1, 18, 8, 3, 8),        # 9 of 2 x 8, 10 of 4 x 4, 9
    (1, 22, 40, 3, 8),       # 55 of 2 x 8, 60 of 4 x 4, 55
    (1, 21, 40, 3, 8),       # 55, 53: 4 % more
    (5, 4, 5, 3, 0),         # 10 of either, 7
    (4, 14, 14, 3, 0),       # 56, 49: 14 % more
    (4, 7, 7, 3, 0),         # 16, 13
    (1, 14, 14, 5, 0),
])
def test_rings_take_rectangles_where_they_cover_the_map(n, h, w, win, columns, dtype):
    """3x3 windows on rings: the rectangle of which fewer cover the map, unless they are more than a tenth more tiles than consecutive pixels make."""
    g = GraphBuilder("t", dtype, n, h, w, 128)
    g.conv(0, 40, win, pad=win // 2)
    m = api.Model(g.done())
    assert m.op_form(0).ring_waves
    assert m.op_rectangle(0) == columns
    assert B.load().mt_model_op_rectangle(m.h, 0, None) == B.MT_ERR_INVALID_ARG
    assert B.load().mt_model_op_rectangle(m.h, 1, C.byref(C.c_int32())) == B.MT_ERR_INVALID_ARG
    m.close()


@pytest.mark.parametrize("arch,batch,mib", [("resnet101", 1, 0), ("resnet50", 64, 1.26), ("resnet101", 128, 2.51), ("vgg16", 1, 6.51), ("vgg16", 12, 4.51),
                                            ("vgg16", 128, 12.02), ("inceptionv3", 48, 0.95), ("alexnet", 6, 10.02), ("mobilenetv2", 1, 0)])
def test_what_a_tenant_takes_of_the_fixed_scratch_array(arch, batch, mib):
    """Workspaces of at most a quarter of the array are in it; sets of tenants that used to fit still do."""
    m = api.Model(zoo.BUILDERS[arch]("f16", batch))
    sizes = [m.op_form(i).workspace_bytes for i in range(m.num_ops())]
    m.close()
    assert sum(v for v in sizes if v <= B.MT_STATIC_SCRATCH_BYTES // 4) <= mib * 2 ** 20


def _model(ops, dtype=B.MT_F16, dims=(1, 8, 8, 8)):
    lib = B.load()
    h = C.c_void_p()
    assert lib.mt_model_begin(dtype, *dims, C.byref(h)) == 0
    for d in ops:
        assert lib.mt_model_add_op(h, C.byref(d), None) == 0
    rc = lib.mt_model_end(h)
    lib.mt_model_destroy(h)
    return rc


def _op(kind=B.MT_CONV, src=0, res=-1, dst=1, oc=8, coff=0, ctot=0, r=3, s=3, sh=1, sw=1, ph=1, pw=1, act=0, groups=1):
    return B.mt_op_desc(kind, src, res, dst, oc, coff, ctot, r, s, sh, sw, ph, pw, act, groups, 1e-4, 0.75, 2.0)


def test_model_validation_errors():
    lib = B.load()
    assert _model([_op()]) == 0
    assert _model([_op(src=3)]) == B.MT_ERR_SHAPE_MISMATCH            # input never produced
    assert _model([_op(r=11, s=11, ph=0, pw=0)]) == B.MT_ERR_SHAPE_MISMATCH   # window larger than input
    assert _model([_op(ph=3)]) == B.MT_ERR_SHAPE_MISMATCH              # pad >= window
    assert _model([_op(res=2)]) == B.MT_ERR_SHAPE_MISMATCH             # residual never produced
    assert _model([_op(), _op(src=1, dst=2, oc=4, res=1)]) == 0        # residual wider than the output is allowed
    assert _model([_op(), _op(src=1, dst=2, oc=16, res=1)]) == B.MT_ERR_SHAPE_MISMATCH
    assert _model([_op(coff=4, ctot=8)]) == B.MT_ERR_SHAPE_MISMATCH    # channel range exceeds the tensor
    assert _model([_op(dst=1, ctot=16), _op(dst=1, coff=8, ctot=16, sh=2, sw=2)]) == B.MT_ERR_SHAPE_MISMATCH
    assert _model([_op(kind=B.MT_MAXPOOL, res=0)]) == B.MT_ERR_SHAPE_MISMATCH
    assert _model([]) == B.MT_ERR_SHAPE_MISMATCH
    assert _model([_op(dst=1 << 30)]) == B.MT_ERR_SHAPE_MISMATCH       # tensor id far beyond what one operator can define
    assert _model([_op(groups=3)]) == B.MT_ERR_SHAPE_MISMATCH                      # 8 channels do not split into 3 groups
    assert _model([_op(groups=2)]) == 0
    assert _model([_op(kind=B.MT_MAXPOOL, groups=2)]) == B.MT_ERR_SHAPE_MISMATCH   # groups on a pool
    assert _model([_op(kind=B.MT_LRN, r=4)]) == B.MT_ERR_SHAPE_MISMATCH            # even window
    assert _model([_op(kind=B.MT_LRN, r=5)]) == 0
    assert _model([_op(kind=B.MT_ADD)]) == B.MT_ERR_SHAPE_MISMATCH                 # no second summand
    assert _model([_op(oc=8), _op(kind=B.MT_ADD, src=1, res=0, dst=2)]) == 0
    assert _model([_op(oc=16), _op(kind=B.MT_ADD, src=1, res=0, dst=2)]) == B.MT_ERR_SHAPE_MISMATCH   # 16 + 8 channels
    # 32-bit offsets inside the kernels: a tensor of 2 GiB or more is refused when the model is finalised
    assert _model([_op(oc=64)], dims=(64, 512, 512, 64)) == B.MT_ERR_SHAPE_MISMATCH        # 2 GiB fp16 input and output
    assert "2 GiB" in lib.mt_last_error().decode()
    assert _model([_op(oc=64)], dims=(32, 512, 512, 63)) == 0                              # just below
    h = C.c_void_p()
    assert lib.mt_model_begin(7, 1, 8, 8, 8, C.byref(h)) == B.MT_ERR_INVALID_ARG
    assert lib.mt_model_begin(B.MT_F16, 0, 8, 8, 8, C.byref(h)) == B.MT_ERR_INVALID_ARG
    assert lib.mt_model_end(None) == B.MT_ERR_INVALID_ARG


def test_set_weights_checks_sizes():
    lib = B.load()
    h = C.c_void_p()
    assert lib.mt_model_begin(B.MT_F16, 1, 8, 8, 8, C.byref(h)) == 0
    d = _op()
    assert lib.mt_model_add_op(h, C.byref(d), None) == 0
    w = np.zeros(8 * 3 * 3 * 8, dtype=np.float16)
    assert lib.mt_model_set_weights(h, 0, w.ctypes.data_as(C.c_void_p), w.nbytes, None, 0) == B.MT_ERR_NOT_FINALIZED
    assert lib.mt_model_end(h) == 0
    assert lib.mt_model_set_weights(h, 0, w.ctypes.data_as(C.c_void_p), w.nbytes - 2, None, 0) == B.MT_ERR_SHAPE_MISMATCH
    b = np.zeros(7, dtype=np.float32)
    assert lib.mt_model_set_weights(h, 0, w.ctypes.data_as(C.c_void_p), w.nbytes, b.ctypes.data_as(C.POINTER(C.c_float)), 7) == B.MT_ERR_SHAPE_MISMATCH
    assert lib.mt_model_set_weights(h, 0, w.ctypes.data_as(C.c_void_p), w.nbytes, None, 0) == 0
    assert lib.mt_model_set_weights(h, 1, w.ctypes.data_as(C.c_void_p), w.nbytes, None, 0) == B.MT_ERR_INVALID_ARG
    lib.mt_model_destroy(h)


def test_speedup_definition_matches_printed_tables():
    from bench import speedup
    with open(os.path.join(ROOT, "tests", "golden", "speedups.txt")) as f:
        rows = [l.split() for l in f if l.strip() and not l.startswith("#")]
    assert len(rows) == 12
    for seq, ours, printed in rows:
        assert abs(speedup(float(seq), float(ours)) - float(printed)) < 0.01   # printed to two decimals, some rounded, some truncated


def test_cu_share_descent_matches_oracle():
    target = [64, 160, 32]
    calls = []

    def cost(sh):
        return float(sum(abs((a or 256) - b) for a, b in zip(sh, target))) + 1.0

    def cb(ptr, _u):
        v = [ptr[i] for i in range(3)]
        calls.append(v)
        return cost(v)

    best = (I32 * 3)()
    bc = C.c_double(cost([0, 0, 0]))
    fn = B.mt_share_cost_fn(cb)
    assert B.load().mt_search_cu_share(3, 256, 2, fn, None, best, C.byref(bc)) == 0
    ocalls = []
    oshare, ocost = S.cu_share_descent(3, 256, 2, lambda sh: (ocalls.append(list(sh)) or cost(sh)), cost([0, 0, 0]))
    assert [best[i] for i in range(3)] == oshare == [64, 160, 32]
    assert bc.value == ocost and calls == ocalls


def test_cu_share_descent_from_a_start_vector():
    target = [32, 160, 64]

    def cost(sh):
        return float(sum(abs((a or 256) - b) for a, b in zip(sh, target))) + 1.0

    start = [64, 96, 96]
    best = (I32 * 3)(*start)
    bc = C.c_double(cost(start))
    calls, ocalls = [], []
    fn = B.mt_share_cost_fn(lambda ptr, _u: (calls.append([ptr[i] for i in range(3)]) or cost(calls[-1])))
    assert B.load().mt_search_cu_share(3, 256, 1, fn, None, best, C.byref(bc)) == 0
    oshare, ocost = S.cu_share_descent(3, 256, 1, lambda sh: (ocalls.append(list(sh)) or cost(sh)), cost(start), start)
    assert [best[i] for i in range(3)] == oshare == target
    assert bc.value == ocost == 1.0 and calls == ocalls
    bad = (I32 * 3)(64, 300, 0)
    assert B.load().mt_search_cu_share(3, 256, 1, fn, None, bad, C.byref(bc)) != 0


def test_proportional_cu_share():
    lib = B.load()

    def host(w, cus=256):
        out = (I32 * len(w))()
        assert lib.mt_proportional_cu_share(len(w), cus, (C.c_double * len(w))(*w), out) == 0
        return [out[i] for i in range(len(w))]

    # hand-worked: 5 spare eighths, quotas 1.163 / 1.954 / 1.883 -> floors 1,1,1, the two left go to tenants 1 and 2
    assert host([147.0, 247.0, 238.0]) == [64, 96, 96] == S.proportional_shares([147.0, 247.0, 238.0], 256)
    assert host([1.0, 1.0]) == [128, 128]
    assert host([3.0, 1.0]) == [192, 64]     # 6 spare eighths, quotas 4.5 / 1.5: tie on the remainder, lower index first
    assert host([0.0, 0.0, 0.0]) == [96, 96, 64] == S.proportional_shares([0.0, 0.0, 0.0], 256)
    assert host([1.0] * 8) == [32] * 8
    assert host([5.0] * 12) == [32] * 12 == S.proportional_shares([5.0] * 12, 256)
    rng = np.random.default_rng(5)
    for _ in range(200):
        n = int(rng.integers(1, 9))
        w = [float(x) for x in rng.uniform(0.0, 10.0, n)]
        sh = host(w)
        assert sh == S.proportional_shares(w, 256)
        assert sum(sh) == 256 and min(sh) >= 32 and all(v % 32 == 0 for v in sh)
        for i in range(n):                                       # monotone: a heavier tenant never gets less
            for j in range(n):
                if w[i] > w[j]:
                    assert sh[i] >= sh[j]
    assert lib.mt_proportional_cu_share(3, 256, (C.c_double * 3)(1.0, -1.0, 1.0), (I32 * 3)()) != 0


def test_wave_priority_descent_matches_oracle_and_finds_a_separable_optimum():
    # a separable cost with a known minimum: the descent must land on it in one round and stop after the next one
    target = [3, 0, -1, 2]

    def cost(pr):
        return float(sum((a - b) ** 2 for a, b in zip(pr, target))) + 0.5

    for start in ([0, 0, 0, 0], [-1, 3, 2, 1]):
        best = (I32 * 4)(*start)
        bc = C.c_double(cost(start))
        calls, ocalls = [], []
        fn = B.mt_share_cost_fn(lambda ptr, _u: (calls.append([ptr[i] for i in range(4)]) or cost(calls[-1])))
        assert B.load().mt_search_wave_priority(4, 5, fn, None, best, C.byref(bc)) == 0
        oprio, ocost = S.wave_priority_descent(4, 5, lambda pr: (ocalls.append(list(pr)) or cost(pr)), cost(start), start)
        assert [best[i] for i in range(4)] == oprio == target
        assert bc.value == ocost == 0.5 and calls == ocalls
        assert len(calls) <= 2 * 4 * 5                      # one improving round, one round without change, then stop
    # a cost that never improves keeps the start vector and evaluates one round only
    best = (I32 * 2)(1, 2)
    bc = C.c_double(1.0)
    n = []
    fn = B.mt_share_cost_fn(lambda ptr, _u: (n.append(1) or 2.0))
    assert B.load().mt_search_wave_priority(2, 3, fn, None, best, C.byref(bc)) == 0
    assert [best[0], best[1]] == [1, 2] and bc.value == 1.0 and len(n) == 8
    bad = (I32 * 2)(0, 4)
    assert B.load().mt_search_wave_priority(2, 1, fn, None, bad, C.byref(bc)) != 0


@pytest.mark.parametrize("h,w,c,k,resident", [
    (80, 102, 128, 256, False), (128, 64, 128, 256, False), (128, 80, 256, 64, False), (128, 81, 256, 64, False), (250, 200, 256, 512, False),
    (128, 80, 64, 256, False), (10241, 1, 64, 256, False), (13333, 3, 64, 256, False), (200, 200, 64, 256, True), (200, 200, 64, 64, True),
    (450, 450, 128, 128, False)])
def test_1x1_layers_take_the_resident_filter_kernel_in_its_pixel_range(h, w, c, k, resident):
    g = GraphBuilder("t", "bf16", 1, h, w, c)
    g.conv(0, k, 1)
    m = api.Model(g.done())
    name = m.op_form(0).name.decode()
    assert (name == "igemm_resident_filters") == resident, name
    assert resident or name.startswith("tile_") or name.startswith("ring_")
    m.close()


def test_a_unit_holds_as_many_walking_workgroups_as_their_launches_count_on():
    """Launches cut to a share of the units count on as many workgroups per unit as the LDS holds, three at most: registers have to leave room for
    them.  None of these kernels keeps scalars in vector registers (the loads to LDS take theirs without the compiler's wait states)."""
    walking = {name: k for name, k in code_objects.kernels().items() if "_walk_kernel" in name}
    assert len(walking) == 30
    for name, k in walking.items():
        assert code_objects.held_by_registers(k) >= min(3, 160 * 1024 // k[".group_segment_fixed_size"]), name
        assert k[".sgpr_spill_count"] == 0 and k[".vgpr_spill_count"] == 0, name


def test_loads_to_lds_keep_their_distance_from_vector_instructions_that_write_scalars():
    """The tile kernels' loads to LDS are inline assembly, in which the compiler does not add the five wait states that a load needs after a
    vector instruction has written a scalar register it reads.  Shown on small listings, then in every kernel of the library."""
    load = (8, "buffer_load_dwordx4", ["v4", "s[20:23]", "s14 offen lds"])
    end = (16, "s_endpgm", [""])
    for op, early in ((("v_readlane_b32", ["s22", "v1", "3"]), True), (("v_readfirstlane_b32", ["s14", "v1"]), True), (("v_readlane_b32", ["m0", "v1", "3"]), True),
                      (("v_add_co_u32_e64", ["v2", "s[14:15]", "v1", "v3"]), True), (("v_readlane_b32", ["s24", "v1", "3"]), False), (("s_mov_b32", ["s22", "s1"]), False)):
        assert bool(code_objects.early_lds_loads([(0, *op), (4, "s_nop", ["3"]), load, end])) == early, op
        assert not code_objects.early_lds_loads([(0, *op), (4, "s_nop", ["4"]), load, end])
    # behind the jump back to the head of a loop
    loop = [(0, "s_nop", ["4"]), load, (16, "v_readlane_b32", ["s14", "v1", "3"]), (24, "s_cbranch_scc1", ["65531"]), (28, "s_endpgm", [""])]
    assert code_objects.early_lds_loads(loop)
    n = 0
    for name, code in code_objects.listings():
        n += sum(1 for _, m, ops in code if m.startswith("buffer_load") and ops[-1].endswith(" lds"))
        assert not code_objects.early_lds_loads(code), name
    assert n > 1000


def test_operands_are_loaded_as_global_memory():
    """A generic load may be to LDS: it counts among those as well, and waits that go by counts wait for all that is under way."""
    n = 0
    for name, code in code_objects.listings():
        n += 1
        assert not [hex(a) for a, m, _ in code if m.startswith("flat_")], name
    assert n > 250


def test_tiles_with_filters_in_registers_wait_for_one_stage():
    """In the loop over the reduction a wave waits for the filters that it multiplies next; those of the stages behind them stay under way."""
    n = 0
    for name, code in code_objects.listings():
        m = re.search(r"tile_(?:walk_|pair_)?kernelI(?:DF16_|NS_4bf16E)Li(128ELi64ELi4|64ELi64ELi2)ELi1ELi(\d)ELi(\d)ELi(\d)ELi\dEE", name)
        if not m:
            continue
        bn, wn = map(int, m[1].split("ELi")[::2])
        wk, kd, nbuf = int(m[2]), int(m[3]), int(m[4])
        loop = code_objects.staging_loop(code)
        waits = [int(re.search(r"vmcnt\((\d+)\)", o[0])[1]) for (_, w, o), (_, after, _) in zip(loop, loop[1:])
                 if w == "s_waitcnt" and "vmcnt" in o[0] and after != "s_barrier"]
        requested = (nbuf - 1) * (kd * 4 // wk) * (bn // wn // 32)
        assert waits and min(waits) == requested - 1, (name, waits)
        n += 1
    assert n >= 30


def test_kernels_end_with_their_results_in_memory():
    """Packets between dependent launches release nothing, so every store of an operator's kernel goes through to memory (sc1) and no wave
    ends before its stores have arrived there.  Shown on small listings, then in every kernel of the library but the probes."""
    through, held = (8, "buffer_store_dwordx4", ["v[0:3]", "v4", "s[20:23]", "0 offen sc1"]), (8, "global_store_dword", ["v1", "v2", "s[4:5]"])
    wait, end = (16, "s_waitcnt", ["vmcnt(0) lgkmcnt(0)"]), (28, "s_endpgm", [""])
    assert not code_objects.held_back_stores([through, wait, end])
    assert code_objects.held_back_stores([held, wait, end]) and code_objects.held_back_stores([through, end])
    assert code_objects.held_back_stores([through, (16, "s_waitcnt", ["vmcnt(1)"]), end])
    # a way round the wait
    assert code_objects.held_back_stores([through, (12, "s_cbranch_execz", ["2"]), wait, (20, "s_nop", ["0"]), (24, "s_nop", ["0"]), end])
    n = 0
    for name, code in code_objects.listings():
        if any(p in name for p in ("peak_", "probe_kernel", "arrive_kernel", "fill_u32_kernel")) or "_kernel" not in name:
            continue
        n += 1
        assert any("store" in m and "sc1" in ops[-1] for _, m, ops in code), name
        assert not code_objects.held_back_stores(code), name
    assert n > 250


@pytest.mark.parametrize("win,stride,k", [(7, 2, 64), (7, 2, 32), (3, 1, 64), (3, 2, 32)])
def test_a_unit_holds_as_many_first_layer_workgroups_as_their_grids_count_on(win, stride, k):
    """The grids of first layers, also those cut to a share of the units, are a number of workgroups per unit that registers and LDS have room for."""
    g = GraphBuilder("t", "f16", 64, 224, 224, 3)
    g.conv(0, k, win, stride, win // 2)
    m = api.Model(g.done())
    per_unit = m.op_info(0).grid_blocks / 256
    m.close()
    forms = [kern for name, kern in code_objects.kernels().items() if "11stem_kernel" in name and "Li%dELi%dELi" % (win, win) in name and "Li%dELb" % (k // 32) in name]
    assert len(forms) == 4                               # two types, aligned and general
    for kern in forms:
        assert per_unit <= code_objects.held_by_registers(kern) and per_unit * kern[".group_segment_fixed_size"] <= 160 * 1024


@pytest.mark.parametrize("kernel,form", [
    ("void mt::ring_patch_kernel<mt::bf16, 2, 4>(mt::OpArgs)", "ring_32x16"),
    ("void mt::ring_patch_kernel<float, 1, 8>(mt::OpArgs)", "ring_16x16"),
    ("_ZN2mt21ring_patch_pair_kernelINS_4bf16ELi1ELi8EEEvNS_10OpArgsPairE", "ring_16x16"),
    ("void mt::ring_kernel<_Float16, 16, 8, 2, 1>(mt::OpArgs)", "ring_16x16"),
    ("void mt::patch_kernel<mt::bf16, 64, 64, 2, 1, 4, 9, 192>(mt::OpArgs)", "patch_64x64"),
    ("void mt::tile_walk_kernel<mt::bf16, 128, 64, 4, 1, 1, 1, 3, 0>(mt::OpArgs)", "tile_128x64"),
])
def test_kernels_of_a_trace_are_grouped_by_their_form(kernel, form):
    assert report._family_of(kernel) == form
