"""The C-ABI boundary on the host: exported symbols and argument validation (no GPU work is enqueued)."""
import ctypes
import os
import re

import pytest

import paper_2409_17066_amd as vq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "vq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(vq_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = vq.load()
    names = _declared_functions()
    assert set(names) == set(vq.EXPORTED)
    for n in names:
        assert getattr(lib, n) is not None
        assert callable(getattr(vq, n))        # the binding carries the same names


def test_version_and_status_strings():
    assert vq.vq_version() >= 100
    texts = {vq.vq_status_string(s) for s in range(0, -7, -1)}
    assert len(texts) == 7 and vq.vq_status_string(-99) == "unknown status"


def _desc(**kw):
    d = vq.vq_layer_desc(ctypes.sizeof(vq.vq_layer_desc), 8, 30, 6, 256, 0, 0, 0, 0,
                         0x1000, None, None, 0x2000, 16, None, 0, None, 0, None, None)
    for k, v in kw.items():
        setattr(d, k, v)
    return d


def test_valid_descriptor_passes():
    assert vq.vq_validate(_desc()) == vq.VQ_OK
    assert vq.vq_validate(_desc(k_res=16, codebook_res=0x3000, idx_res=0x4000, idx_res_row_stride=16)) == vq.VQ_OK
    assert vq.vq_validate(_desc(n_outlier_cols=8, v_out=4, k_out=16, codebook_out=0x3000, idx_out=0x4000,
                                idx_out_row_stride=16)) == vq.VQ_OK


def test_vectors_down_the_output_dimension_in_the_descriptor():
    assert vq.vq_validate(_desc(orientation=1, idx_row_stride=32)) == vq.VQ_OK
    # outlier columns need not be a multiple of v_out there
    assert vq.vq_validate(_desc(orientation=1, idx_row_stride=32, n_outlier_cols=7, v_out=4, k_out=16, codebook_out=0x3000,
                                idx_out=0x4000, idx_out_row_stride=16)) == vq.VQ_OK


def test_codebook_groups_in_the_descriptor():
    assert vq.vq_validate(_desc(group_vectors=2)) == vq.VQ_OK               # 5 vectors: groups of 2, 2, 1
    assert vq.vq_validate(_desc(group_vectors=1000)) == vq.VQ_OK            # one group
    # the layout that ends with `bias` is still taken, as a layer with one group (whatever follows it in memory)
    old = vq.vq_layer_desc.group_vectors.offset
    assert vq.vq_validate(_desc(struct_size=old, group_vectors=-5)) == vq.VQ_OK


@pytest.mark.parametrize("kw,status", [
    (dict(struct_size=4), vq.VQ_ERR_SHAPE),
    (dict(group_vectors=-1), vq.VQ_ERR_SHAPE),
    (dict(orientation=2), vq.VQ_ERR_SHAPE), (dict(orientation=-1), vq.VQ_ERR_SHAPE),
    (dict(orientation=1, idx_row_stride=16), vq.VQ_ERR_SHAPE),          # 30 indices of 8 bits a stream need 30 bytes
    (dict(out_features=0), vq.VQ_ERR_SHAPE),
    (dict(in_features=0), vq.VQ_ERR_SHAPE),
    (dict(v=0), vq.VQ_ERR_SHAPE), (dict(v=17), vq.VQ_ERR_SHAPE),
    (dict(k=1), vq.VQ_ERR_SHAPE), (dict(k=65537), vq.VQ_ERR_SHAPE),
    (dict(k_res=1), vq.VQ_ERR_SHAPE),
    (dict(codebook=None), vq.VQ_ERR_NULL), (dict(idx=None), vq.VQ_ERR_NULL),
    (dict(codebook=0x1008), vq.VQ_ERR_ALIGNMENT), (dict(idx=0x2004), vq.VQ_ERR_ALIGNMENT),
    (dict(idx_row_stride=0), vq.VQ_ERR_SHAPE),            # 5 vectors x 8 bits need 5 bytes
    (dict(idx_row_stride=24), vq.VQ_ERR_ALIGNMENT),
    (dict(k_res=16), vq.VQ_ERR_NULL),
    (dict(k_res=16, codebook_res=0x3000, idx_res=0x4000, idx_res_row_stride=0), vq.VQ_ERR_SHAPE),
    (dict(n_outlier_cols=7, v_out=4, k_out=16, codebook_out=0x3000, idx_out=0x4000, idx_out_row_stride=16), vq.VQ_ERR_SHAPE),
    (dict(n_outlier_cols=32, v_out=4, k_out=16, codebook_out=0x3000, idx_out=0x4000, idx_out_row_stride=16), vq.VQ_ERR_SHAPE),
    (dict(n_outlier_cols=8, v_out=4, k_out=16), vq.VQ_ERR_NULL),
    (dict(scale=0x5001), vq.VQ_ERR_ALIGNMENT),
])
def test_invalid_descriptors(kw, status):
    assert vq.vq_validate(_desc(**kw)) == status


def test_entry_points_reject_bad_arguments_before_any_launch():
    d = _desc()
    assert vq.vq_validate(None) == vq.VQ_ERR_NULL
    assert vq.vq_dequant(None, 0x9000, 30) == vq.VQ_ERR_NULL
    assert vq.vq_dequant(d, None, 30) == vq.VQ_ERR_NULL
    assert vq.vq_dequant(d, 0x9000, 29) == vq.VQ_ERR_SHAPE
    assert vq.vq_dequant(d, 0x9001, 30) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_gemv(d, None, 30, 1, 0x9000, 8) == vq.VQ_ERR_NULL
    assert vq.vq_gemv(d, 0x8000, 30, 0, 0x9000, 8) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv(d, 0x8000, 30, 17, 0x9000, 8) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv(d, 0x8000, 28, 1, 0x9000, 8) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv(d, 0x8000, 30, 1, 0x9000, 7) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv(d, 0x8001, 30, 1, 0x9000, 8) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_gemv(d, 0x8000, 30, 1, 0x9001, 8) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_gemm(d, 0x8000, 32, 0, 0x9000, 8) == vq.VQ_ERR_SHAPE        # empty token batch
    assert vq.vq_gemm(d, 0x8000, 30, 4, 0x9000, 8) == vq.VQ_ERR_ALIGNMENT    # ldx not a multiple of 8
    assert vq.vq_gemm(d, 0x8008, 32, 4, 0x9000, 8) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_gemm(d, None, 32, 4, 0x9000, 8) == vq.VQ_ERR_NULL
    assert vq.vq_gemm_workspace_bytes(_desc(v=0), 4) == 0


def test_gemv_multi_rejects_bad_arguments_before_any_launch():
    d, e = _desc(), _desc(out_features=5)
    ok = dict(x_ptr=0x8000, ldx=30, batch=1, y_ptrs=[0x9000, 0xA000], ldys=[8, 5])
    assert vq.vq_gemv_multi([d, e], **dict(ok, x_ptr=None)) == vq.VQ_ERR_NULL
    assert vq.vq_gemv_multi([d, e], **dict(ok, y_ptrs=[0x9000, None])) == vq.VQ_ERR_NULL
    assert vq.vq_gemv_multi([d, e], **dict(ok, batch=0)) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv_multi([d, e], **dict(ok, batch=17)) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv_multi([d, e], **dict(ok, ldys=[8, 4])) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv_multi([d, e], **dict(ok, ldx=29)) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv_multi([d, e], **dict(ok, y_ptrs=[0x9000, 0xA001])) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_gemv_multi([d, _desc(in_features=36, idx_row_stride=16)], **ok) == vq.VQ_ERR_SHAPE     # not the same activations
    assert vq.vq_gemv_multi([d, _desc(v=0)], **ok) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv_multi([d] * 9, 0x8000, 30, 1, [0x9000] * 9, [8] * 9) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv_multi([], 0x8000, 30, 1, [], []) == vq.VQ_ERR_SHAPE


def test_gemv_with_workspace_rejects_bad_arguments_before_any_launch():
    d = _desc()
    assert vq.vq_gemv_workspace_bytes(d, 4) == 0                       # one group: no kernel would use a workspace
    assert vq.vq_gemv_workspace_bytes(_desc(v=0), 4) == 0
    assert vq.vq_gemv_with_workspace(d, None, 30, 1, 0x9000, 8) == vq.VQ_ERR_NULL
    assert vq.vq_gemv_with_workspace(d, 0x8000, 30, 17, 0x9000, 8) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemv_with_workspace(d, 0x8000, 30, 1, 0x9001, 8) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_gemv_with_workspace(d, 0x8000, 30, 1, 0x9000, 8, 0xA010, 4096) == vq.VQ_ERR_ALIGNMENT
    big = _desc(in_features=6 * 64, idx_row_stride=96, v=6, k=4096, group_vectors=16)
    assert vq.vq_gemv_workspace_bytes(big, 2) >= 4 * (2 * 8 + 16) * 4   # 4 groups x (2 tokens x 8 rows + 16 activation sums)
    # groups that do not start on a dword of the index stream: not the matrix-core kernel's, but the kernel that keeps one table
    # in LDS at a time takes a group per workgroup too (6 groups x (2 x 8 + 16) sums)
    assert vq.vq_gemv_workspace_bytes(_desc(in_features=6 * 64, idx_row_stride=96, v=6, k=4096, group_vectors=12), 2) >= 6 * (2 * 8 + 16) * 4
    assert vq.vq_gemv_workspace_bytes(_desc(in_features=5 * 64, idx_row_stride=96, v=5, k=4096, group_vectors=12), 2) == 0    # no kernel of v = 5 uses one


# (layer, rows): what vq_gemv_static_workspace takes, and of what size at most
FIT_THE_STATIC_WORKSPACE = [
    # 67 codebook groups that the kernel walks by itself (more workgroups than the chip has room for): no workspace at all
    (dict(out_features=28672, in_features=4288 * 4, v=4, k=256, group_vectors=64), 16, 0),
    (dict(out_features=4096, in_features=28672, v=4, k=256, group_vectors=72), 16, 0),
    (dict(out_features=27520, in_features=56038, v=12, k=4096, k_res=4096, group_vectors=704, orientation=1), 4, 0),
    # rows of an odd width whose copy alone would take more; the same where a column permutation asks for nearly all of it
    (dict(out_features=256, in_features=(1 << 20) + 1, v=6, k=256), 16, 1 << 24),
    (dict(out_features=1544, in_features=516012, v=2, k=16, orientation=1, col_perm=0x10000), 16, 1 << 24),
    # sixteen codebook groups whose sums fit, and would not with a seventeenth set of sums for the outlier columns
    (dict(out_features=16000, in_features=16 * 48 + 40, v=6, k=4096, n_outlier_cols=40, v_out=4, k_out=8192, group_vectors=8), 16, 1 << 24),
]


@pytest.mark.parametrize("layer,batch,most", FIT_THE_STATIC_WORKSPACE)
def test_no_more_workspace_than_the_library_has_where_none_was_needed(layer, batch, most):
    """vq_gemv_static_workspace refuses a layer whose vq_gemv_workspace_bytes exceeds its array: a kernel that does without, or
    with less, must not ask for more."""
    import vq_synth as s
    f = dict(layer, out=layer["out_features"], inp=layer["in_features"], n=layer.get("n_outlier_cols", 0))
    main = f["inp"] - f["n"] if f.get("orientation") else -(-(f["inp"] - f["n"]) // f["v"])
    d = _desc(**layer, idx_row_stride=s.row_stride_bytes(main, s.index_bits(f["k"])))
    if f.get("k_res"):
        d.codebook_res, d.idx_res, d.idx_res_row_stride = 0x10000, 0x10000, s.row_stride_bytes(main, s.index_bits(f["k_res"]))
    if f["n"]:
        d.codebook_out, d.idx_out, d.idx_out_row_stride = 0x10000, 0x10000, s.row_stride_bytes(f["n"] // 4, s.index_bits(f["k_out"]))
    assert vq.vq_validate(d) == vq.VQ_OK
    assert vq.vq_gemv_workspace_bytes(d, batch) <= min(most, vq.VQ_GEMV_STATIC_WORKSPACE_BYTES)


def test_gemv_workspace_for_vectors_down_the_output_dimension():
    """Orientation 1 on the matrix cores cuts the columns into parts when a workspace is there: asked for from two rows
    on (one row stays on the kernel that needs none), sized parts x (rows x tokens + 16) floats, parts >= 2."""
    d = _desc(orientation=1, out_features=96, in_features=1024, idx_row_stride=1536, v=6, k=4096)
    assert vq.vq_validate(d) == vq.VQ_OK
    assert vq.vq_gemv_workspace_bytes(d, 1) == 0
    for batch in (2, 5, 16):
        need = vq.vq_gemv_workspace_bytes(d, batch)
        assert need >= 2 * (batch * 96 + 16) * 4 and need % 256 == 0, batch
    # streams too short to cut (a part needs a 32-column window per wave), odd numbers of outlier columns: no workspace
    assert vq.vq_gemv_workspace_bytes(_desc(orientation=1, out_features=96, in_features=256, idx_row_stride=384, v=6, k=4096), 4) == 0
    odd = _desc(orientation=1, out_features=96, in_features=1024 + 7, idx_row_stride=1536, v=6, k=4096, n_outlier_cols=7, v_out=4, k_out=16,
                codebook_out=0x3000, idx_out=0x4000, idx_out_row_stride=16)
    assert vq.vq_validate(odd) == vq.VQ_OK and vq.vq_gemv_workspace_bytes(odd, 4) == 0
    # codebook groups are parts by themselves, from one row on
    grouped = _desc(orientation=1, out_features=96, in_features=1024, idx_row_stride=1536, v=6, k=4096, group_vectors=256)
    assert vq.vq_gemv_workspace_bytes(grouped, 1) >= 4 * (96 + 16) * 4
    # so is a row too long for the one-row kernel's LDS (28672 activations beside two 64 KB tables)
    long_rows = _desc(orientation=1, out_features=96, in_features=28672, idx_row_stride=43008, v=6, k=4096, k_res=4096,
                      codebook_res=0x5000, idx_res=0x6000, idx_res_row_stride=43008)
    assert vq.vq_validate(long_rows) == vq.VQ_OK
    assert vq.vq_gemv_workspace_bytes(long_rows, 1) >= 2 * (96 + 16) * 4


def test_assign_rejects_bad_arguments_before_any_launch():
    ok = dict(W_ptr=0x8000, B_ptr=None, ld=30, rows=8, cols=30, codebook_ptr=0x1000, v=6, k=256, idx_ptr=0x2000, idx_row_stride=16)
    assert vq.vq_assign(**dict(ok, W_ptr=None)) == vq.VQ_ERR_NULL
    assert vq.vq_assign(**dict(ok, codebook_ptr=None)) == vq.VQ_ERR_NULL
    assert vq.vq_assign(**dict(ok, idx_ptr=None)) == vq.VQ_ERR_NULL
    for bad in (dict(rows=0), dict(cols=0), dict(ld=29), dict(v=0), dict(v=17), dict(k=1), dict(k=65537)):
        assert vq.vq_assign(**dict(ok, **bad)) == vq.VQ_ERR_SHAPE, bad
    assert vq.vq_assign(**dict(ok, cols=30, k=4096, idx_row_stride=0)) == vq.VQ_ERR_SHAPE       # 5 x 12 bits need 8 bytes
    assert vq.vq_assign(**dict(ok, W_ptr=0x8001)) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_assign(**dict(ok, B_ptr=0x8001)) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_assign(**dict(ok, idx_ptr=0x2008)) == vq.VQ_ERR_ALIGNMENT
    assert vq.vq_assign(**dict(ok, idx_row_stride=24)) == vq.VQ_ERR_ALIGNMENT


def test_assign_down_rejects_bad_arguments_before_any_launch():
    ok = dict(W_ptr=0x8000, B_ptr=None, ld=30, rows=8, cols=30, codebook_ptr=0x1000, v=6, k=256, idx_ptr=0x2000, idx_row_stride=32)
    assert vq.vq_assign_down(**dict(ok, W_ptr=None)) == vq.VQ_ERR_NULL
    for bad in (dict(rows=0), dict(cols=0), dict(ld=29), dict(v=17), dict(k=1)):
        assert vq.vq_assign_down(**dict(ok, **bad)) == vq.VQ_ERR_SHAPE, bad
    assert vq.vq_assign_down(**dict(ok, idx_row_stride=16)) == vq.VQ_ERR_SHAPE         # 30 indices of 8 bits a stream
    assert vq.vq_assign_down(**dict(ok, idx_ptr=0x2004)) == vq.VQ_ERR_ALIGNMENT


def test_binding_has_no_cpu_fallback():
    src = open(os.path.join(ROOT, "paper_2409_17066_amd", "__init__.py")).read()
    assert "oracle" not in src.replace("no CPU fallback", "")


def test_default_workspace_of_gemm_has_room_for_W_only_where_it_is_rounded_anyway():
    def default(tokens, **kw):
        d = _desc(**kw)
        assert vq.vq_validate(d) == vq.VQ_OK
        return vq.vq_gemm_default_workspace_bytes(d, tokens), vq.vq_gemm_fast_workspace_bytes(d, tokens), vq.vq_gemv_workspace_bytes(d, min(tokens, 16))
    v6 = dict(out_features=11008, in_features=4096, v=6, k=4096, idx_row_stride=1040)
    for tokens in (65, 509):                                    # the kernel that restores on the fly: rounded in any case
        got, fast, rows = default(tokens, **v6)
        assert got == fast == 11008 * 4096 * 2
    for tokens in (9, 32, 48):                                  # vq_gemv's kernels
        got, fast, rows = default(tokens, **v6)
        assert got == rows == 0
    res = dict(codebook_res=0x3000, idx_res=0x4000, idx_res_row_stride=1040, k_res=4096)
    for kw, matrices in ((dict(v6, group_vectors=176), 1), (dict(v6, group_vectors=176, **res), 2)):      # codebook groups
        assert default(9, **kw)[0] == default(9, **kw)[2]
        for tokens in (100, 509):                               # ... centroids, and a sum a token
            got, fast, rows = default(tokens, **kw)
            assert got == matrices * fast + (tokens * 4 + 255) // 256 * 256
    down = dict(out_features=11008, in_features=4096, v=6, k=4096, idx_row_stride=6144, orientation=1)
    got, fast, rows = default(16, **down)
    assert got == rows
    assert default(128, **down)[0] == fast + 512 and default(129, **down)[0] == fast
    v12 = dict(out_features=11008, in_features=4096, v=12, k=4096, idx_row_stride=528)
    assert [default(t, **v12)[0] == default(t, **v12)[2] for t in (16, 32, 33)] == [True, True, False]
    assert default(9, **dict(v6, col_perm=0x1000))[0] == default(9, **dict(v6, col_perm=0x1000))[1]      # the generic tile kernel
    assert vq.vq_gemm_default_workspace_bytes(_desc(v=0), 4) == 0
    wide = dict(in_features=8192, v=8, k=65536, idx_row_stride=2048)                # 256 MiB, and more
    assert default(100, **dict(wide, out_features=16384))[0] == 1 << 28 and default(100, **dict(wide, out_features=16385))[0] == 0
    assert default(100, **dict(v6, out_features=20000, group_vectors=176, **res))[0] < 1 << 25      # (two matrices of 156 MiB)
    assert vq.vq_gemm_default(_desc(), None, 32, 9, 0x9000, 8) == vq.VQ_ERR_NULL
    assert vq.vq_gemm_default(_desc(), 0x8000, 32, 0, 0x9000, 8) == vq.VQ_ERR_SHAPE
    assert vq.vq_gemm_default(_desc(), 0x8008, 32, 9, 0x9000, 8) == vq.VQ_ERR_ALIGNMENT


@pytest.mark.parametrize("out_features", [32000, 53248])
def test_gemv_workspace_of_layers_whose_rows_leave_no_room_for_a_table_a_slot(out_features):
    """v = 12 with two tables of 4096 in eight codebook groups, one and two rows: a slot is a group where LDS has no room for the row
    sums of twice the rows, and the workspace is that of the eight groups."""
    columns = 28672
    vectors = -(-columns // 12)
    stride = (vectors * 12 + 127) // 128 * 16
    d = _desc(out_features=out_features, in_features=columns, v=12, k=4096, k_res=4096, codebook_res=0x3000, idx_row_stride=stride,
              idx_res=0x4000, idx_res_row_stride=stride, group_vectors=-(-vectors // 64) * 8)
    for batch in (1, 2):
        assert vq.vq_gemv_workspace_bytes(d, batch) == (8 * (batch * out_features + 16) * 4 + 255) // 256 * 256


@pytest.mark.parametrize("perm", [None, 0x5000])
@pytest.mark.parametrize("v,k,columns", [(12, 4096, 1024), (4, 256, 4096), (2, 16, 771)])
@pytest.mark.parametrize("groups", [2, 5, 8])
def test_gemv_workspace_of_more_rows_holds_that_of_fewer(perm, v, k, columns, groups):
    """A loop lends the workspace of its largest batch to every call.  One and two rows of a layer with two tables a group take a slot a
    table: where the workspace of more rows holds a slot a group for them, it holds those too."""
    vectors = -(-columns // v)
    stride = (vectors * (k - 1).bit_length() + 127) // 128 * 16
    d = _desc(out_features=512, in_features=columns, v=v, k=k, k_res=k, codebook_res=0x3000, idx_row_stride=stride, idx_res=0x4000,
              idx_res_row_stride=stride, group_vectors=-(-vectors // (8 * groups)) * 8, col_perm=perm)
    sizes = [vq.vq_gemv_workspace_bytes(d, batch) for batch in range(1, 17)]
    assert sizes[0] > 0
    for rows in (1, 2):
        head = (rows * ((columns + 7) // 8 * 8) * 2 + 255) // 256 * 256 if perm else 0
        a_slot_a_group = head + (groups * (rows * 512 + 16) * 4 + 255) // 256 * 256
        assert all(size >= sizes[rows - 1] for size in sizes[rows:] if size >= a_slot_a_group)
    assert sizes[2] >= sizes[1]
