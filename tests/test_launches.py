"""Routes and workspaces of the library's calls, from the launches that they make on a machine without a GPU (launches.py)."""
import random

import launches
import pytest


def _layer(rng, odd):
    """A layer of any of the settings that vq_gemv knows; odd: of an odd width."""
    v, k = rng.choice([(6, 4096), (6, 4096), (6, 3000), (12, 4096), (8, 256), (8, 65536), (4, 256), (2, 16), (5, 37)])
    out = round(2 ** rng.uniform(4, 14))
    inp = round(2 ** rng.uniform(6, 14.2)) // 2 * 2 + odd
    outliers = 4 * rng.randint(1, 10) if rng.random() < 0.3 else 0
    orientation = rng.randint(0, 1)
    vectors = (inp - outliers) // (1 if orientation else v)
    return dict(out_features=out, in_features=inp, v=v, k=k, k_res=rng.choice([0, 0, k, min(k, 256)]), n_outlier_cols=outliers, orientation=orientation,
                group_vectors=rng.choice([0, 0, 0, max(8, vectors // rng.randint(2, 16) // 8 * 8)]), col_perm=rng.random() < 0.3)


def _inside(call, answer):
    """The sums and the copy of the activations that an answer's kernels write lie in the workspace."""
    for launch in answer["launches"]:
        words, end = launch["words"], launches.WORKSPACE + answer["lent"]
        if "finish" in launch["name"]:
            part, part_xs, slots, batch, out = words[:5]
            assert launches.WORKSPACE <= part and part + slots * batch * out * 4 <= part_xs and part_xs + slots * 64 <= end, (call, launch)
        if "gather_cols" in launch["name"]:
            to, pitch = words[4:6]
            assert launches.WORKSPACE <= to and to + call["rows"] * pitch * 2 <= end, (call, launch)


@pytest.mark.parametrize("odd", [1, 0])
def test_gemv_stays_inside_its_workspace(odd):
    """A workspace of the size asked for, one byte less, one asked for more rows: with activations that can be taken as they are and others."""
    rng = random.Random(odd)
    calls = []
    for _ in range(700):
        layer, rows = _layer(rng, odd), rng.choice([1, 2, 3, 4, 5, 8, 16])
        inp = layer["in_features"]
        for pitch, x in ((inp + odd, 0), ((inp + 7) // 8 * 8, 0), (inp + 3, 2)):
            one = dict(entry="gemv_with_workspace", layer=layer, rows=rows, pitch=pitch, x=launches.X + x, workspace="asked")
            calls += [one, dict(one, asked_for_rows=rng.randint(rows, 16))]
    # two tables of vectors down the outputs and more activations than fit LDS beside them, in as many blocks as compute units: no parts, and once
    # the size of a copy that was not made passed for that of the sums
    for rows, out in ((4, 14336), (8, 14336), (16, 14336), (2, 30000)):
        layer = dict(out_features=out, in_features=15873, k_res=4096, orientation=1)
        calls += [dict(entry="gemv_with_workspace", layer=layer, rows=rows, pitch=pitch, workspace="asked", asked_for_rows=asked)
                  for pitch in (15880, 15873) for asked in (rows, 16)]
    answers = launches.run(calls)
    smaller = [dict(call, workspace=answer["asked"] - 256) for call, answer in zip(calls, answers) if answer["asked"] > 256]
    with_sums = 0
    for call, answer in list(zip(calls, answers)) + list(zip(smaller, launches.run(smaller))):
        assert answer["status"] == 0 and answer["launches"]
        _inside(call, answer)
        with_sums += any("finish" in launch["name"] for launch in answer["launches"])
    assert with_sums > 300


@pytest.mark.parametrize("permuted", [False, True])
@pytest.mark.parametrize("out,inp,numbers,more", [
    (3520, 6587, (2, 4, 16), {}), (4096, 4097, (16,), {}), (2048, 8193, (2, 4, 16), dict(k_res=4096)), (2048, 8193, (2, 4, 16), dict(k_res=256, n_outlier_cols=40)),
    (4096, 4097, (2, 4, 16), dict(group_vectors=256)),
])
def test_gemv_of_odd_rows_down_the_outputs_in_parts(out, inp, numbers, more, permuted):
    """The workspace of an odd width takes the copy of the activations, where there is one, and the same parts as the next even width."""
    calls = []
    for rows in numbers:
        for width, pitch in ((inp, inp), (inp, inp + 1), (inp + 1, inp + 1)):
            layer = dict(out_features=out, in_features=width, orientation=1, col_perm=permuted, **more)
            calls.append(dict(entry="gemv_with_workspace", layer=layer, rows=rows, pitch=pitch, workspace="asked"))
    answers = launches.run(calls)
    for call, answer in zip(calls, answers):
        _inside(call, answer)
    for i in range(0, len(answers), 3):
        copied, even_pitch, even = [[(launch["name"], launch["grid"]) for launch in answer["launches"] if "gather" not in launch["name"]] for answer in answers[i:i + 3]]
        assert copied == even and even_pitch == even
        assert any("finish" in name for name, _ in even)
        assert answers[i]["launches"][0]["name"] == "gather_cols_kernel" and (answers[i + 1]["launches"][0]["name"] == "gather_cols_kernel") == permuted


@pytest.mark.parametrize("entry,out,inp,rows,more,kernel", [
    ("gemv", 7214, 14999, 4, {}, "gemv_lds"), ("gemv", 550, 3667, 16, {}, "gemv_v8"), ("gemv", 550, 367, 16, {}, "gemv_lds"),
    ("gemv", 16166, 97, 4, dict(group_vectors=8), "gemv_lds"), ("gemv", 10676, 1249, 5, dict(group_vectors=16), "gemv_v8"),
    ("gemv_with_workspace", 10740, 689, 4, dict(group_vectors=40), "gemv_lds"), ("gemv_with_workspace", 2346, 5353, 1, dict(group_vectors=48), "gemv_v8"),
    ("gemv", 5198, 113, 16, dict(k=65536), "gemv_generic"), ("gemv", 5198, 113, 1, dict(k=65536), "gemv_v8"), ("gemv", 1472, 297, 4, dict(k=65536, k_res=0), "gemv_v8"), ("gemv", 50, 7, 1, dict(k=65536), "gemv_generic"),
])
def test_gemv_v8_rows_that_begin_anywhere(entry, out, inp, rows, more, kernel):
    """Each side of the lines between the lookups through L2 and the kernels that take such rows otherwise."""
    layer = dict(dict(out_features=out, in_features=inp, v=8, k=256, k_res=256), **more)
    answer, = launches.run([dict(entry=entry, rows=rows, workspace="asked" if entry != "gemv" else None, layer=layer, pitch=inp)])
    assert answer["status"] == 0
    assert all(launch["name"].startswith((kernel, "gemv_groups_finish")) for launch in answer["launches"]), answer


@pytest.mark.parametrize("entry,out,inp,rows,pitch,more,kernel", [
    ("gemv_with_workspace", 76, 15648, 4, 15648, {}, "gemv_groups_finish"), ("gemv_with_workspace", 44, 11397, 4, 11400, dict(n_outlier_cols=32), "gemv_groups_finish"),
    ("gemv_with_workspace", 184, 13424, 3, 13424, dict(k_res=4096), "gemv_groups_finish"), ("gemv_with_workspace", 2213, 5096, 1, 5096, {}, "gemv_down_v6"),
    ("gemv", 12798, 816, 1, 816, dict(k_res=256), "gemv_down_mfma"), ("gemv", 2670, 1144, 1, 1144, dict(k_res=256), "gemv_down_v6"),
    ("gemv", 61, 10331, 8, 10331, dict(k_res=4096), "gemv_down_lds"), ("gemv", 61, 10331, 1, 10331, dict(k_res=4096), "gemv_down_v6"),
    ("gemv", 13521, 366, 2, 369, dict(n_outlier_cols=20), "gemv_down_lds"), ("gemv", 13521, 366, 2, 369, {}, "gemv_down_v6"),
    ("gemv", 876, 138, 1, 138, dict(k_res=256, group_vectors=8), "gemv_down_kernel"), ("gemv", 876, 1380, 1, 1384, dict(k_res=256, group_vectors=200), "gemv_down_mfma"),
])
def test_gemv_down_takes_the_faster_kernel(entry, out, inp, rows, pitch, more, kernel):
    """Each side of the lines between the kernels for vectors down the outputs, v = 6."""
    layer = dict(dict(out_features=out, in_features=inp, orientation=1), **more)
    answer, = launches.run([dict(entry=entry, rows=rows, pitch=pitch, x=launches.X + (2 if pitch % 8 else 0), workspace="asked" if entry != "gemv" else None, layer=layer)])
    assert answer["status"] == 0 and answer["launches"][-1]["name"].startswith(kernel), answer


@pytest.mark.parametrize("out,inp,rows,more,copied", [
    (12461, 193, 1, {}, False), (3589, 557, 1, {}, False), (1735, 1089, 1, {}, True), (2759, 513, 1, dict(k_res=4096), True), (2759, 735, 2, {}, True), (2759, 335, 2, {}, False), (12201, 289, 10, dict(k_res=4096), True),
    (9609, 173, 2, {}, False), (12996, 2263, 2, dict(group_vectors=24), False), (12996, 2263, 3, dict(group_vectors=24), True),
    (12996, 2263, 4, dict(group_vectors=24, n_outlier_cols=4), False), (12996, 2263, 6, dict(group_vectors=24, n_outlier_cols=4), True),
    (2843, 2455, 4, dict(group_vectors=24, k_res=4096), False), (2843, 2455, 5, dict(group_vectors=24, k_res=4096), True),
    (8181, 3129, 2, dict(group_vectors=104, k_res=256), True), (2836, 27149, 2, dict(group_vectors=1136), True), (2068, 26017, 4, dict(group_vectors=1088, k_res=4096), True),
    (3200, 26733, 4, dict(group_vectors=1104, n_outlier_cols=268), True), (9098, 1467, 3, dict(group_vectors=16, n_outlier_cols=16), False),
    (4526, 25701, 3, dict(group_vectors=1432, n_outlier_cols=256), True),
])
@pytest.mark.parametrize("permuted", [False, True])
def test_gemv_of_an_odd_width_made_even(out, inp, rows, more, copied, permuted):
    """Each side of the lines between the kernels of even widths, on a copy, and those that keep a table in LDS at a time."""
    layer = dict(dict(out_features=out, in_features=inp, col_perm=permuted), **more)
    answer, = launches.run([dict(entry="gemv_with_workspace", layer=layer, rows=rows, pitch=inp, workspace="asked")])
    names = [launch["name"] for launch in answer["launches"]]
    assert answer["status"] == 0 and any(name.startswith("gemv_v6") for name in names) == copied and (not copied or names[0] == "gather_cols_kernel"), names


@pytest.mark.parametrize("out,inp,rows,more,products", [
    (6399, 1052, 1, {}, False), (12213, 4395, 1, {}, False), (5859, 10344, 1, {}, True), (5859, 10344, 2, {}, False), (4096, 4096, 1, dict(k_res=4096), True),
    (637, 3640, 1, dict(group_vectors=80), False), (1700, 4096, 1, dict(group_vectors=88), True), (637, 3640, 1, dict(group_vectors=32), True),
    (637, 3640, 1, dict(group_vectors=80, k_res=4096), True), (2164, 3903, 2, dict(group_vectors=48), False), (2164, 3903, 2, dict(group_vectors=16), True),
    (4096, 4096, 2, dict(group_vectors=48), True),
])
def test_gemv_from_tables_of_products_where_they_pay(out, inp, rows, more, products):
    """Each side of the lines between tables of products and the kernels that look entries up, v = 12."""
    layer = dict(dict(out_features=out, in_features=inp, v=12), **more)
    answer, = launches.run([dict(entry="gemv_with_workspace", layer=layer, rows=rows, pitch=(inp + 7) // 8 * 8, workspace="asked")])
    assert answer["status"] == 0 and answer["launches"][0]["name"].startswith("gemv_products") == products, answer


def test_gemm_default_asks_for_the_sums_that_it_writes():
    """Beside the restored matrix only the sums of a product that is cut: 8 MiB more once stood there whatever the tokens."""
    rng = random.Random(5)
    calls = [dict(entry="gemm_default", rows=200, workspace="asked", layer=dict(out_features=700, in_features=640))]
    for _ in range(400):
        v, k = rng.choice([(6, 4096), (12, 4096), (8, 65536), (4, 256)])
        layer = dict(out_features=round(2 ** rng.uniform(6, 13.2)), in_features=round(2 ** rng.uniform(3, 10)) * 8 + 256, v=v, k=k, k_res=rng.choice([0, 0, 256]),
                     orientation=rng.randint(0, 1), col_perm=rng.random() < 0.3)
        calls.append(dict(entry="gemm_default", rows=round(2 ** rng.uniform(4.1, 11)), workspace="asked", layer=layer))
    answers = launches.run(calls)
    more = launches.run([dict(call, workspace=answer["asked"] + (8 << 20)) for call, answer in zip(calls, answers)])
    least = launches.run([dict(call, workspace="least") for call in calls])
    whole = cut = 0
    for call, answer, with_more, with_less in zip(calls, answers, more, least):
        names = [launch["name"] for launch in answer["launches"]]
        assert answer["status"] == 0 and (answer["launches"] == with_more["launches"] or not any("gemm_dense" in launch["name"] for launch in with_more["launches"])), call
        if "gemm_dense_finish_kernel" in names:
            cut += 1
            # without that room the same route, not cut
            assert with_less["lent"] < answer["lent"] and [name.split("<")[0] for name in names[:-1]] == [launch["name"].split("<")[0] for launch in with_less["launches"]]
        elif any(name.startswith("gemm_dense_kernel") for name in names):
            whole += 1
            assert with_less == answer
            d, tokens = call["layer"], call["rows"]
            matrices = 2 if d.get("k_res") else 1
            assert answer["asked"] <= matrices * (d["out_features"] * d["in_features"] * 2 + 256) + tokens * (4 + d["in_features"] * 2 * d.get("col_perm", 0)) + 512, call
    assert whole > 100 and cut > 30


@pytest.mark.parametrize("out,inp,rows,more", [
    (2872, 3616, 1, dict(group_vectors=16, col_perm=True)), (5315, 936, 2, dict(group_vectors=8, col_perm=True)),
    (7812, 592, 2, dict(group_vectors=8, k_res=4096, n_outlier_cols=16, col_perm=True)), (1024, 4096, 1, dict(group_vectors=88, k_res=4096)),
    (5859, 10344, 1, {}),
])
def test_gemv_with_less_than_it_asks_for_is_gemv(out, inp, rows, more):
    """Tables of products take a part of a workspace that other kernels ask more of; with no more than that part the call is vq_gemv."""
    layer = dict(dict(out_features=out, in_features=inp, v=12), **more)
    call = dict(entry="gemv_with_workspace", layer=layer, rows=rows, pitch=inp)
    enough, plain = launches.run([dict(call, workspace="asked"), dict(call, entry="gemv")])
    assert enough["launches"][0]["name"].startswith("gemv_products")
    less, = launches.run([dict(call, workspace=enough["asked"] - 256)])
    assert [launch["name"] for launch in less["launches"]] == [launch["name"] for launch in plain["launches"]]


def test_gemv_borrows_only_what_its_rows_use():
    """gemv() without a workspace: none for tables of products that only fewer rows take; with v = 6 and an odd width what a workspace is good for."""
    wide = dict(out_features=11008, in_features=4096, v=12, k_res=4096)
    calls = [dict(entry="gemv_with_workspace", layer=wide, rows=rows, pitch=4096, workspace="lent") for rows in (1, 2, 16)]
    calls += [dict(entry="gemv_with_workspace", layer=dict(out_features=128, in_features=28672, v=12), rows=16, pitch=28672, workspace="lent")]
    rng = random.Random(9)
    for _ in range(300):
        layer = dict(_layer(rng, 1), v=6, k=rng.choice([4096, 256]), k_res=rng.choice([0, 256, 4096]), col_perm=False)
        calls.append(dict(entry="gemv_with_workspace", layer=layer, rows=rng.randint(1, 16), workspace="lent", pitch=layer["in_features"]))
    one, two, sixteen, narrow, *odd = launches.run(calls)
    assert one["lent"] and one["launches"][0]["name"].startswith("gemv_products") and not two["lent"] and not sixteen["lent"] and narrow["lent"]
    plain = launches.run([dict(call, entry="gemv", workspace=None) for call in calls[4:]])
    asked = launches.run([dict(call, workspace="asked") for call in calls[4:]])
    assert [answer["launches"] for answer in odd] == [answer["launches"] for answer in asked]
    unused = [call for call, answer, without in zip(calls[4:], odd, plain) if answer["lent"] and answer["launches"] == without["launches"]]
    # (of some layers of few vectors the size is asked for, for activations that begin elsewhere)
    assert sum(answer["lent"] > 0 for answer in odd) > 100 and len(unused) < 20


@pytest.mark.parametrize("out,inp,rows,more,streams", [
    (11008, 4096, 8, {}, 8), (11008, 4096, 9, {}, 16), (11008, 4096, 2, dict(k_res=4096), 8), (4096, 4096, 4, {}, 4), (4096, 4096, 5, {}, 8), (14080, 4096, 4, {}, 16),
    (95, 1282, 7, dict(k_res=256), 8), (3001, 1030, 4, dict(k_res=4096), 4), (9605, 1300, 2, {}, 8), (512, 256, 4, dict(k_res=4096), 16),
])
def test_gemv_down_folds_of_the_columns(out, inp, rows, more, streams):
    """How many index streams a workgroup takes of a layer whose vectors run down the outputs."""
    answer, = launches.run([dict(entry="gemv", rows=rows, pitch=inp + inp % 2, layer=dict(out_features=out, in_features=inp, orientation=1, **more))])
    grids = [launch["grid"] for launch in answer["launches"] if launch["name"].startswith("gemv_down_mfma")]
    assert [list(grid)[0] for grid in grids] == [-(-(-(-out // 6)) // streams)], answer


@pytest.mark.parametrize("rows", [1, 2, 4])
def test_gemv_of_rows_far_apart_keeps_its_kernel(rows):
    """Rows of activations, or of results, more than 2^31 elements apart: the kernel for small tables as for any others."""
    layer = dict(out_features=256, in_features=384, k=256)
    near, far = launches.run([dict(entry="gemv", rows=rows, layer=layer, pitch=pitch) for pitch in (384, (1 << 31) + 8)], switches="rows=0")
    assert near["status"] == 0 and far["launches"] == near["launches"] and near["launches"][0]["name"].startswith("gemv_lds_window_kernel")


@pytest.mark.parametrize("out,inp,rows,more,used", [
    (11008, 4096, 4, {}, False), (4096, 4097, 8, dict(col_perm=True), False), (1811, 3052, 3, {}, True), (7614, 7226, 5, {}, True), (7614, 7226, 6, {}, False),
    (515, 3900, 3, dict(v=2, k=16), False), (131, 4098, 4, dict(v=4, k=256), False), (131, 3500, 8, dict(v=6, k=256), False), (515, 3900, 12, dict(v=2, k=16), True),
    (130, 10000, 4, dict(v=8, k=65536, orientation=0), False), (130, 10000, 8, dict(v=8, k=65536, orientation=0), True), (14336, 512, 16, {}, False),
])
def test_gemv_in_folds_of_the_columns_uses_no_workspace(out, inp, rows, more, used):
    """Folds need no sums of parts: such rows are lent none, and run the same kernel with any workspace and
    without."""
    layer = dict(dict(out_features=out, in_features=inp, orientation=1), **more)
    call = dict(entry="gemv_with_workspace", layer=layer, rows=rows, pitch=inp)
    asked, lent, generous, none = launches.run([dict(call, workspace="asked"), dict(call, workspace="lent"), dict(call, workspace=16 << 20), dict(call, entry="gemv")])
    copy = (rows * (inp + 7) // 8 * 8 * 2 + 255) // 256 * 256 if layer.get("col_perm") else 0
    assert asked["launches"] == generous["launches"] and any("finish" in launch["name"] for launch in asked["launches"]) == used
    if not used:
        assert lent["lent"] <= copy + 256 and (copy or none["launches"] == asked["launches"])
        fewer = [0] + [answer["asked"] for answer in launches.run([dict(call, rows=r, workspace="asked") for r in range(1, rows)])]
        assert layer.get("v", 6) == 6 and layer.get("k", 4096) == 4096 or asked["asked"] == max(fewer)


def test_gemv_asks_for_what_fewer_rows_use():
    """A loop may lend its calls the workspace of the largest number of rows."""
    rng = random.Random(12)
    calls = []
    for _ in range(60):
        layer = dict(_layer(rng, rng.randint(0, 1)), orientation=1, group_vectors=0)
        calls += [dict(entry="gemv_with_workspace", layer=layer, rows=rows, workspace="asked") for rows in range(1, 17)]
    sizes = [answer["asked"] for answer in launches.run(calls)]
    assert sum(size > 0 for size in sizes) > 300
    for i in range(0, len(sizes), 16):
        assert sizes[i:i + 16] == sorted(sizes[i:i + 16]), calls[i]


@pytest.mark.parametrize("out,inp,v,k,more,orientation,rows,streams", [
    (700, 900, 8, 65536, {}, 1, 3, 4), (701, 333, 8, 65536, {}, 1, 8, 8), (130, 10001, 8, 65536, {}, 0, 4, 4), (1001, 3205, 8, 65536, {}, 0, 7, 8),
    (301, 1700, 12, 4096, dict(k_res=4096), 1, 4, 4), (301, 505, 12, 4096, dict(k_res=4096, n_outlier_cols=24), 1, 6, 8),
    (77, 9509, 12, 4096, dict(k_res=4096), 0, 2, 4), (900, 3300, 12, 4096, dict(k_res=4096, n_outlier_cols=40), 0, 5, 8),
    (131, 4099, 4, 256, {}, 1, 4, 4), (2003, 700, 4, 256, {}, 1, 8, 8), (130, 3209, 4, 256, {}, 0, 4, 8), (1003, 6001, 4, 256, {}, 0, 8, 8),
    (515, 3900, 2, 16, {}, 1, 1, 4), (3001, 1001, 2, 16, {}, 1, 8, 8), (333, 1035, 2, 16, {}, 0, 3, 8),
    (131, 4099, 6, 256, {}, 1, 4, 4), (131, 777, 6, 256, {}, 1, 8, 8), (1002, 3461, 6, 256, {}, 0, 4, 8),
])
def test_gemv_rows_folds_of_the_columns(out, inp, v, k, more, orientation, rows, streams):
    """How many index streams a workgroup takes of the layers and rows whose results test_gemv_rows_folds compares, with the workspace of the size asked for and without."""
    layer = dict(out_features=out, in_features=inp, v=v, k=k, orientation=orientation, **more)
    call = dict(entry="gemv", rows=rows, pitch=(inp + 7) // 8 * 8 + 8, layer=layer)
    count = -(-out // v) if orientation else out
    plain, asked = launches.run([call, dict(call, entry="gemv_with_workspace", workspace="asked")], switches="rows=1")
    assert [launch["grid"][0] for launch in plain["launches"]] == [-(-count // streams)] and plain["launches"][0]["name"].startswith("gemv_rows_kernel")
    names = [launch["name"].split("<")[0] for launch in asked["launches"]]
    assert "gemv_rows_kernel" in names and (asked["launches"] == plain["launches"] or names[-1] == "gemv_groups_finish_kernel" or names[0] == "gather_cols_kernel")
