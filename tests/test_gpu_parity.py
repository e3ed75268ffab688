"""GPU parity: the HIP library through its C ABI against the CPU oracle, element by element."""
import numpy as np
import pytest

import oracle
import vq_synth as s
from cases import SMALL, MULTI, small_layer, multi_layers, lent

pytestmark = pytest.mark.gpu

TOL = 1e-2        # max |y - y_ref| <= TOL * RMS(y_ref): the stated bar for GEMV and GEMM


def _check_matmul(y_gpu, y_ref, what):
    y = y_gpu.float().cpu().numpy().astype(np.float64)
    rms = np.sqrt((y_ref ** 2).mean())
    err = np.abs(y - y_ref).max()
    assert np.isfinite(y).all(), what
    assert err <= TOL * rms, "%s: max abs err %.3e > %.0e * rms %.3e" % (what, err, TOL, rms)


@pytest.mark.parametrize("name", list(SMALL))
@pytest.mark.parametrize("pad", [8, 16, 24])
def test_dequant_leaves_the_padding_of_aligned_rows_alone(gpu_lib, name, pad):
    """Leading dimensions that keep every row 16-byte aligned (the layouts the kernels with 16-byte stores take): the
    logical columns bit-exact, the columns [in_features, ldw) still holding the caller's sentinel."""
    import torch
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    ldw = (L.in_features + 7) // 8 * 8 + pad
    W = torch.full((L.out_features, ldw), -3.5, dtype=torch.float16, device="cuda")
    rc = gpu_lib.vq_dequant(dl.desc, W.data_ptr(), ldw, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    got = W.cpu().numpy()
    want = oracle.dequant(L, L.in_features)
    assert np.array_equal(got[:, :L.in_features].view(np.uint16), want.view(np.uint16)), name
    assert (got[:, L.in_features:] == np.float16(-3.5)).all(), name


@pytest.mark.parametrize("name", list(SMALL))
def test_dequant_bit_exact_small(gpu_lib, name):
    import torch
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    for ldw in (L.in_features, L.in_features + 11):
        W = gpu_lib.dequant(dl, ldw)
        torch.cuda.synchronize()
        want = oracle.dequant(L, ldw)
        assert np.array_equal(W.cpu().numpy().view(np.uint16), want.view(np.uint16)), name


@pytest.mark.parametrize("name", list(SMALL))
@pytest.mark.parametrize("batch", [1, 2, 3, 4, 8, 16])
@pytest.mark.parametrize("kernel", ["auto", "m", "d"])
def test_gemv_small(gpu_lib, monkeypatch, name, batch, kernel):
    """Every batch through the default dispatch, then with the matrix-core kernel and the dot-product kernels forced
    (layers they do not take fall through to the generic kernel)."""
    import torch
    if kernel != "auto":
        monkeypatch.setenv("VQ_SWITCHES", "gemv=" + kernel)
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(300, L, batch)
    y = gpu_lib.gemv(dl, torch.from_numpy(x).cuda())
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x), "%s batch %d" % (name, batch))


# (the restore-then-multiply route exists for layers whose in_features is a multiple of 256: only those get its cases)
GEMM_CASES = [(name, ws) for name in SMALL for ws in (None, "none", "fast", "fast, 256 x 256 tiles")
              if ws in (None, "none") or SMALL[name]["in_features"] % 256 == 0]


@pytest.mark.parametrize("name,workspace", GEMM_CASES)
@pytest.mark.parametrize("tokens", [1, 37, 130, 300])
def test_gemm_small(gpu_lib, monkeypatch, name, tokens, workspace):
    """By default, without a workspace (weights restored on the fly) and with the one that lets vq_gemm restore W once (that
    route forced: by itself the library leaves small token counts to vq_gemv's kernels where those are faster), the dense product in
    its smallest and its largest tiles."""
    import torch
    if workspace not in (None, "none"):
        monkeypatch.setenv("VQ_SWITCHES", "gemm=w,dense=" + ("1" if "256" in workspace else "0"))      # its smallest and its largest tiles
        workspace = "fast"
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    if workspace == "fast":
        assert gpu_lib.vq_gemm_fast_workspace_bytes(dl.desc, tokens) > 0
    x = s.make_activations(300, L, tokens)
    ldx = (L.in_features + 7) // 8 * 8
    X = torch.zeros((tokens, ldx), dtype=torch.float16, device="cuda")
    X[:, : L.in_features] = torch.from_numpy(x).cuda()
    if ldx > L.in_features:
        X[:, L.in_features:] = float("nan")           # padding of the caller's buffer must never be read into the sum
    Y = gpu_lib.gemm(dl, X, workspace=lent(workspace))
    torch.cuda.synchronize()
    _check_matmul(Y, oracle.gemm(L, x), "%s tokens %d workspace %s" % (name, tokens, workspace))


@pytest.mark.parametrize("tokens,out_features,in_features,more", [
    (33, 64, 1544, {}), (65, 130, 2056, dict(permute=True)), (17, 67, 3400, dict(k_res=200)), (129, 1000, 4104, dict(orientation=1)),
    (326, 977, 5296, {}), (385, 2482, 7192, {}), (40, 300, 520, {}), (64, 512, 512, {}),
])
def test_gemm_columns_in_parts(gpu_lib, tokens, out_features, in_features, more):
    """Products of few tiles and many columns, the columns cut into parts of whole steps, the last one ragged (64 x 64, 64 x 128 and 128 x 128 tiles; the
    last two shapes are not cut); with room for the restored matrix alone they are not.  Workspace filled with NaN patterns, guarded behind."""
    import torch
    L = s.make_layer(8400, "parts", out_features, in_features, 8, 300, **more)
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(8400, L, tokens)
    X = torch.full((tokens, in_features + 8), float("nan"), dtype=torch.float16, device="cuda")
    X[:, :in_features] = torch.from_numpy(x).cuda()
    need = gpu_lib.vq_gemm_fast_workspace_bytes(dl.desc, tokens)
    assert need <= gpu_lib.vq_gemm_fast_workspace_bytes(dl.desc, 4 * tokens)      # (the workspace of more tokens does for fewer)
    matrix = (tokens * in_features * 2 + 255) // 256 * 256 * bool(more.get("permute")) + out_features * in_features * 2
    rows = np.unique(np.linspace(0, out_features - 1, 130).astype(np.int32))
    ref = oracle.gemm(L, x, rows=rows)
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for size in (need, matrix):
        ws[:] = 0xFF
        Y = torch.full((tokens, out_features + 3), 7.0, dtype=torch.float16, device="cuda")
        assert gpu_lib.vq_gemm(dl.desc, X.data_ptr(), X.stride(0), tokens, Y.data_ptr(), Y.stride(0), ws.data_ptr(), size, stream) == 0
        torch.cuda.synchronize()
        _check_matmul(Y[:, torch.from_numpy(rows.astype(np.int64)).cuda()], ref, "%d tokens, workspace of %d bytes" % (tokens, size))
        assert torch.isfinite(Y).all() and (Y[:, out_features:] == 7.0).all() and (ws[size:] == 0xFF).all()


@pytest.mark.parametrize("tokens,out_features,in_features,v,k,more", [
    (44, 333, 4104, 4, 256, {}), (79, 130, 5000, 6, 300, dict(group_vectors=400)), (95, 650, 5128, 6, 300, dict(k_res=256, group_vectors=100)),
    (64, 257, 5000, 12, 300, dict(k_res=300, orientation=1, group_vectors=999, n_outlier_cols=40, v_out=4, k_out=300)),
    (326, 977, 5296, 4, 256, {}),
])
def test_gemm_by_default_with_columns_in_parts(gpu_lib, tokens, out_features, in_features, v, k, more):
    """The same with the centroids in W, and those of a residual table in a second matrix behind it: scale, bias and the rows' sums come in with
    the parts.  With less room the columns stay whole."""
    import torch
    L = s.make_layer(8500, "parts", out_features, in_features, v, k, **more)
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(8500, L, tokens)
    X = torch.from_numpy(x).cuda()
    need = gpu_lib.vq_gemm_default_workspace_bytes(dl.desc, tokens)
    rows = np.unique(np.linspace(0, out_features - 1, 130).astype(np.int32))
    ref = oracle.gemm(L, x, rows=rows)
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    for size in (need, need - 256, max(need - (8 << 20), 0)):
        ws[:] = 0xFF
        Y = torch.full((tokens, out_features + 3), 7.0, dtype=torch.float16, device="cuda")
        rc = gpu_lib.vq_gemm_default(dl.desc, X.data_ptr(), X.stride(0), tokens, Y.data_ptr(), Y.stride(0), ws.data_ptr(), size, torch.cuda.current_stream().cuda_stream)
        assert rc == 0
        torch.cuda.synchronize()
        _check_matmul(Y[:, torch.from_numpy(rows.astype(np.int64)).cuda()], ref, "%d tokens, workspace of %d bytes" % (tokens, size))
        assert torch.isfinite(Y).all() and (Y[:, out_features:] == 7.0).all() and (ws[size:] == 0xFF).all()


DENSE_SHAPES = [(1, 1, 8), (17, 300, 520), (64, 64, 64), (65, 129, 120), (128, 192, 192), (191, 257, 1032), (256, 256, 128), (300, 513, 136), (513, 768, 320)]


@pytest.mark.parametrize("tokens,out_features,in_features", DENSE_SHAPES)
@pytest.mark.parametrize("tiles", ["auto", "smallest", "largest"])
def test_gemm_dense_tile_edges(gpu_lib, monkeypatch, tokens, out_features, in_features, tiles):
    """The dense product of the restore-then-multiply route around the edges of its tiles (64 to 256 tokens and channels) and
    steps (64 columns; the last one may hold as few as 8), NaN in the padding of X and a sentinel in the padding of Y."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "gemm=w" + {"auto": "", "smallest": ",dense=0", "largest": ",dense=1"}[tiles])
    L = s.make_layer(7, "dense", out_features, in_features, v=4, k=16)
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(300, L, tokens)
    X = torch.full((tokens, in_features + 8), float("nan"), dtype=torch.float16, device="cuda")
    X[:, :in_features] = torch.from_numpy(x).cuda()
    Y = torch.full((tokens, out_features + 3), 7.0, dtype=torch.float16, device="cuda")
    gpu_lib.gemm(dl, X, out=Y, workspace="fast")
    torch.cuda.synchronize()
    _check_matmul(Y[:, :out_features], oracle.gemm(L, x), "%s %s" % ((tokens, out_features, in_features), tiles))
    assert (Y[:, out_features:] == 7.0).all()


@pytest.mark.parametrize("kind", range(2, 6))
@pytest.mark.parametrize("tokens,out_features,in_features", [(1, 1, 8), (193, 257, 200), (192, 256, 128), (400, 600, 1032)])
def test_gemm_dense_tile_kinds(gpu_lib, monkeypatch, tokens, out_features, in_features, kind):
    """The tiles between the largest and the smallest, each forced: less than a tile, one row, channel and chunk of columns past a tile,
    exactly one tile, several; with fewer steps than stages, and as centroids as well (scale and bias after the sum)."""
    import torch
    for route, setting in (("w", dict(v=4, k=16)), ("c", dict(v=6, k=256, k_res=256))):
        monkeypatch.setenv("VQ_SWITCHES", "gemm=%s,dense=%d" % (route, kind))
        L = s.make_layer(8, "kinds", out_features, in_features, **setting)
        x = s.make_activations(301, L, tokens)
        X = torch.full((tokens, in_features + 8), float("nan"), dtype=torch.float16, device="cuda")
        X[:, :in_features] = torch.from_numpy(x).cuda()
        Y = torch.full((tokens, out_features + 3), 7.0, dtype=torch.float16, device="cuda")
        gpu_lib.gemm(gpu_lib.DeviceLayer(L), X, out=Y, workspace="fast" if route == "w" else None)
        torch.cuda.synchronize()
        _check_matmul(Y[:, :out_features], oracle.gemm(L, x), "%s %s %s" % ((tokens, out_features, in_features), route, kind))
        assert (Y[:, out_features:] == 7.0).all()


@pytest.mark.parametrize("name", list(SMALL))
@pytest.mark.parametrize("tokens", [9, 37, 300])
def test_gemm_without_workspace(gpu_lib, name, tokens):
    """An empty workspace tensor: the routes that never write W to memory."""
    import torch
    L = small_layer(name)
    x = s.make_activations(300, L, tokens)
    X = torch.full((tokens, (L.in_features + 7) // 8 * 8), float("nan"), dtype=torch.float16, device="cuda")
    X[:, : L.in_features] = torch.from_numpy(x).cuda()
    Y = gpu_lib.gemm(gpu_lib.DeviceLayer(L), X, workspace=lent("none"))
    torch.cuda.synchronize()
    _check_matmul(Y, oracle.gemm(L, x), "%s tokens %d" % (name, tokens))


ROWS_LAYERS = {
    "v2": dict(out_features=65, in_features=1000, v=2, k=16), "v2_odd": dict(out_features=17, in_features=333, v=2, k=13),
    "v4": dict(out_features=4200, in_features=130, v=4, k=256), "v4_12bit": dict(out_features=33, in_features=515, v=4, k=4096),
    "v6_outliers": dict(out_features=100, in_features=2054, v=6, k=256, n_outlier_cols=12, v_out=4, k_out=4096),
    "v8": dict(out_features=49, in_features=700, v=8, k=200), "v8_12bit": dict(out_features=48, in_features=264, v=8, k=4096, k_res=4096),
    "v8_16bit": dict(out_features=40, in_features=1023, v=8, k=65536), "v8_16bit_many": dict(out_features=4201, in_features=72, v=8, k=65000),
    "v12": dict(out_features=31, in_features=4100, v=12, k=4096, k_res=3000), "v12_tiny": dict(out_features=1, in_features=5, v=12, k=4000),
    "v12_many": dict(out_features=9000, in_features=60, v=12, k=4096, k_res=4096),
    "v12_groups": dict(out_features=70, in_features=2300, v=12, k=4096, k_res=4096, n_outlier_cols=44, v_out=4, k_out=8192, group_vectors=40),
    "v12_permuted": dict(out_features=50, in_features=1201, v=12, k=4096, k_res=4096, n_outlier_cols=8, v_out=4, k_out=500, permute=True),
    "v4_bare": dict(out_features=60, in_features=600, v=4, k=256, with_scale=False, with_bias=False),
}


def _unrounded_weights(gpu_lib, L):
    """scale * (main + residual) + bias in binary64: what the products multiply with before anything is rounded.  (A layer without
    residual, scale and bias restores to its centroids, exactly.)"""
    import copy
    parts = []
    for codebook, idx, k in ((L.codebook, L.idx, L.k),) + (((L.codebook_res, L.idx_res, L.k_res),) if L.k_res else ()):
        P = copy.copy(L)
        P.codebook, P.idx, P.k, P.codebook_res, P.idx_res, P.k_res, P.scale, P.bias = codebook, idx, k, None, None, 0, None, None
        D = gpu_lib.dequant(gpu_lib.DeviceLayer(P)).double()
        if parts and L.n_outlier_cols:
            D[:, : L.n_outlier_cols] = 0.0
        parts.append(D)
    scale, bias = (torch_double(a) for a in (L.scale, L.bias))
    return scale[:, None] * sum(parts) + bias[:, None]


def torch_double(a):
    import torch
    return torch.from_numpy(a.astype(np.float64)).cuda()


@pytest.mark.parametrize("scaled", [(True, False), (False, True), (False, False)])
@pytest.mark.parametrize("tiles", [0, 1, 5])
def test_gemm_centroids_without_scale_or_bias(gpu_lib, monkeypatch, scaled, tiles):
    """The centroids' product, whose last step applies scale and bias to the sums, of layers that lack one or both of them."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "gemm=c,dense=%d" % tiles)
    L = s.make_layer(9, "unscaled", 333, 520, v=6, k=256, k_res=256)
    L.scale, L.bias = L.scale if scaled[0] else None, L.bias if scaled[1] else None
    x = s.make_activations(302, L, 131)
    Y = gpu_lib.gemm(gpu_lib.DeviceLayer(L), torch.from_numpy(x).cuda())
    torch.cuda.synchronize()
    _check_matmul(Y, oracle.gemm(L, x), "scale %s, bias %s" % scaled)


HOLD_THE_WEIGHTS = {            # layers and token counts that vq_gemm without a workspace computes from unrounded weights
    "v6, 64 tokens": (dict(out_features=512, in_features=1536, v=6, k=4096), 64),
    "v6, no room for tiles": (dict(out_features=512, in_features=1536, v=6, k=4096, k_res=4096), 100),
    "v6 groups": (dict(out_features=512, in_features=1536, v=6, k=4096, group_vectors=64), 300),
    "v6 groups, residual": (dict(out_features=513, in_features=1544, v=6, k=4096, k_res=256, group_vectors=64), 300),
    "v6, odd outlier columns, residual": (dict(out_features=700, in_features=1600, v=6, k=4096, k_res=4096, n_outlier_cols=28, v_out=4, k_out=4096), 513),
    "v6, ragged width": (dict(out_features=3000, in_features=2056, v=6, k=4096), 200),
    "v6, odd width": (dict(out_features=512, in_features=1541, v=6, k=4096), 100),
    "orientation 1": (dict(out_features=384, in_features=1600, v=6, k=4096, orientation=1), 128),
    "orientation 1, residual, outliers": (dict(out_features=3001, in_features=2056, v=6, k=4096, k_res=256, orientation=1, n_outlier_cols=7, v_out=4, k_out=300), 127),
    "v8": (dict(out_features=3000, in_features=2048, v=8, k=256, k_res=256), 120),
    "v4": (dict(out_features=512, in_features=1600, v=4, k=256), 32),
    "v12": (dict(out_features=512, in_features=1536, v=12, k=4096, k_res=4096), 17),
}


@pytest.mark.parametrize("name", list(HOLD_THE_WEIGHTS))
def test_gemm_by_default_rounds_no_weights_that_it_would_not_round_without_a_workspace(gpu_lib, name):
    """The relative error (2-norm, against unrounded weights) of the default call against that of an empty workspace.  Rounding
    every result to binary16 gives about 2^-12 / sqrt(3) * 1.4 = 2e-4; weights rounded as well add as much in quadrature, 1.4 times
    the error, so 1.1 tells the two apart at 2^17 results."""
    import torch
    kw, tokens = HOLD_THE_WEIGHTS[name]
    kw = dict(kw)
    L = s.make_layer(61, "hold", kw.pop("out_features"), kw.pop("in_features"), kw.pop("v"), kw.pop("k"), kw.pop("k_res", 0), **kw)
    dl = gpu_lib.DeviceLayer(L)
    x = torch.from_numpy(s.make_activations(300, L, tokens)).cuda()
    X = torch.full((tokens, (L.in_features + 7) // 8 * 8 + 8), float("nan"), dtype=torch.float16, device="cuda")
    X[:, : L.in_features] = x
    want = x.double() @ _unrounded_weights(gpu_lib, L).T.contiguous()

    def error(workspace):
        Y = gpu_lib.gemm(dl, X, workspace=workspace).double()
        return float((Y - want).norm() / want.norm())
    by_default, without, restored = error(None), error(lent("none")), error("fast")
    print("%s: default %.3g, without %.3g, fast %.3g" % (name, by_default, without, restored))
    assert by_default <= 1.1 * without


@pytest.mark.parametrize("name", [n for n in SMALL if SMALL[n]["in_features"] % 8 == 0 and not SMALL[n].get("permute")])
@pytest.mark.parametrize("tokens,tiles", [(9, "smallest"), (65, "auto"), (130, "largest"), (257, "largest"), (300, "smallest")])
def test_gemm_from_restored_centroids(gpu_lib, monkeypatch, name, tokens, tiles):
    """Centroids restored into one or two matrices, scale and bias applied to the sums, forced for every layer: around the edges of
    the tiles and of the step from one matrix to the other, with NaN in the padding of X, a sentinel in that of Y, and a workspace
    full of NaN."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "gemm=c" + {"auto": "", "smallest": ",dense=0", "largest": ",dense=1"}[tiles])
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    need = gpu_lib.vq_gemm_default_workspace_bytes(dl.desc, tokens)
    matrices = 0 if L.k_res > 4096 else 2 if L.k_res else 1
    assert need >= matrices * L.out_features * L.in_features * 2 + tokens * 4 or not matrices
    x = s.make_activations(300, L, tokens)
    X = torch.full((tokens, L.in_features + 8), float("nan"), dtype=torch.float16, device="cuda")
    X[:, : L.in_features] = torch.from_numpy(x).cuda()
    Y = torch.full((tokens, L.out_features + 3), 7.0, dtype=torch.float16, device="cuda")
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    rc = gpu_lib.vq_gemm_default(dl.desc, X.data_ptr(), X.stride(0), tokens, Y.data_ptr(), Y.stride(0), ws.data_ptr(), need, torch.cuda.current_stream().cuda_stream)
    assert rc == gpu_lib.VQ_OK
    torch.cuda.synchronize()
    _check_matmul(Y[:, : L.out_features], oracle.gemm(L, x), "%s tokens %d" % (name, tokens))
    assert (Y[:, L.out_features:] == 7.0).all() and (ws[need:] == 0xFF).all()


@pytest.mark.parametrize("out_features,refused", [(16384, False), (8192, True)])
def test_gemm_by_default_borrows_256_mib_at_most(gpu_lib, out_features, refused):
    """W of 16384 x 8448 takes 264 MiB: the call goes without.  And one whose workspace (132 MiB) the allocator refuses does so too."""
    import torch
    L = s.make_layer(62, "large", out_features, 8448, 8, 65536)
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(300, L, 64)
    X = torch.from_numpy(x).cuda()
    Y = gpu_lib.gemm(dl, X, workspace=lent("none"))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    if refused:                                # (the segments that other tests left have holes: filled, so that it needs a new one)
        reserved = torch.cuda.memory_reserved()
        while torch.cuda.memory_reserved() == reserved:
            held.append(torch.empty(100 << 20, dtype=torch.uint8, device="cuda"))
        held.pop()
        torch.cuda.empty_cache()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    if refused:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (8 << 20)) / torch.cuda.get_device_properties(0).total_memory)
    try:
        got = gpu_lib.gemm(dl, X)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.cuda.max_memory_allocated() - before < 32 << 20
    assert torch.equal(got, Y)
    rows = np.arange(0, out_features, 64).astype(np.int32)
    _check_matmul(got[:, torch.from_numpy(rows.astype(np.int64)).cuda()], oracle.gemm(L, x, rows=rows), "%d outputs" % out_features)


@pytest.mark.parametrize("workspace", ["none", "fast"])
@pytest.mark.parametrize("batch", [1, 3, 16])
@pytest.mark.parametrize("orientation", [0, 1])
@pytest.mark.parametrize("name", list(ROWS_LAYERS))
def test_gemv_rows(gpu_lib, monkeypatch, name, orientation, batch, workspace):
    """The matrix-core kernel for layers looked up entry by entry: ragged rows, streams, steps and groups, with NaN in the padding
    of x and a sentinel in that of y."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "rows=1")
    kw = dict(ROWS_LAYERS[name], orientation=orientation)
    if orientation and kw.get("group_vectors"):
        kw["group_vectors"] = 600
    L = s.make_layer(60 + list(ROWS_LAYERS).index(name), name, kw.pop("out_features"), kw.pop("in_features"), kw.pop("v"), kw.pop("k"), **kw)
    x = s.make_activations(300, L, batch)
    X = torch.full((batch, L.in_features + 4), float("nan"), dtype=torch.float16, device="cuda")
    X[:, : L.in_features] = torch.from_numpy(x).cuda()
    Y = torch.full((batch, L.out_features + 3), 7.0, dtype=torch.float16, device="cuda")
    gpu_lib.gemv(gpu_lib.DeviceLayer(L), X, out=Y, workspace=lent(workspace))
    torch.cuda.synchronize()
    _check_matmul(Y[:, : L.out_features], oracle.gemv(L, x), "%s orientation %d batch %d workspace %s" % (name, orientation, batch, workspace))
    assert (Y[:, L.out_features:] == 7.0).all()


V6_GEMM = ["v6_gemm_plain", "v6_gemm_res8", "v6_gemm_res12", "single_row", "v6_exact_fit", "v6_gemm_outlier32", "v6_gemm_outlier48",
           "v6_gemm_outlier16_res12"]


@pytest.mark.parametrize("name", V6_GEMM)
@pytest.mark.parametrize("tokens", [1, 37, 130, 300, 700])
def test_gemm_v6_on_the_fly(gpu_lib, monkeypatch, name, tokens):
    """The kernel that restores v = 6 layers from tables in LDS, forced for every token count (by itself vq_gemm takes it
    without a workspace from 65 tokens on), with NaN in the padding of X and a sentinel in the padding of Y."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "gemm=6")
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(300, L, tokens)
    X = torch.full((tokens, L.in_features + 8), float("nan"), dtype=torch.float16, device="cuda")
    X[:, : L.in_features] = torch.from_numpy(x).cuda()
    Y = torch.full((tokens, L.out_features + 3), 7.0, dtype=torch.float16, device="cuda")
    gpu_lib.gemm(dl, X, out=Y, workspace=lent("none"))
    torch.cuda.synchronize()
    _check_matmul(Y[:, : L.out_features], oracle.gemm(L, x), "%s tokens %d on the fly" % (name, tokens))
    assert (Y[:, L.out_features:] == 7.0).all()


@pytest.mark.parametrize("kernel", ["auto", "m", "d"])
@pytest.mark.parametrize("batch", [1, 4, 5, 16])
@pytest.mark.parametrize("name,pad_x,pad_y", [("v6_res256_outlier", 10, 6), ("v6_k4096_res4096", 2, 1), ("v6_passes", 6, 3)])
def test_gemv_strided_buffers_and_untouched_padding(gpu_lib, monkeypatch, name, pad_x, pad_y, batch, kernel):
    """Row strides larger than the rows, NaN in the caller's padding (it must never reach a sum), sentinel values
    in the output padding (they must survive); odd output strides take the kernels' narrow store paths."""
    import torch
    if kernel != "auto":
        monkeypatch.setenv("VQ_SWITCHES", "gemv=" + kernel)
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(300, L, batch)
    xb = torch.full((batch, L.in_features + pad_x), float("nan"), dtype=torch.float16, device="cuda")
    xb[:, : L.in_features] = torch.from_numpy(x).cuda()
    yb = torch.full((batch, L.out_features + pad_y), 7.0, dtype=torch.float16, device="cuda")
    gpu_lib.gemv(dl, xb, out=yb)
    torch.cuda.synchronize()
    _check_matmul(yb[:, : L.out_features], oracle.gemv(L, x), "strided %s batch %d" % (name, batch))
    assert (yb[:, L.out_features:] == 7.0).all()


def test_unit_activation_reads_back_a_column(gpu_lib):
    import torch
    L = small_layer("v6_res256_outlier")
    dl = gpu_lib.DeviceLayer(L)
    W = oracle.dequant(L).astype(np.float64)
    cols = [0, 5, 23, 24, 29, 30, 1205, 1206]
    for c0 in range(0, len(cols), 4):
        x = np.zeros((4, L.in_features), dtype=np.float16)
        for t, c in enumerate(cols[c0:c0 + 4]):
            x[t, c] = 1.0
        y = gpu_lib.gemv(dl, torch.from_numpy(x).cuda()).float().cpu().numpy()
        for t, c in enumerate(cols[c0:c0 + 4]):
            assert np.allclose(y[t], W[:, c], rtol=2e-3, atol=1e-7)


@pytest.mark.parametrize("batch", [1, 4, 16])
def test_runs_are_deterministic(gpu_lib, batch):
    import torch
    L = small_layer("v6_k4096_res4096")
    dl = gpu_lib.DeviceLayer(L)
    x = torch.from_numpy(s.make_activations(300, L, batch)).cuda()
    a = gpu_lib.gemv(dl, x).clone()
    for _ in range(3):
        assert torch.equal(gpu_lib.gemv(dl, x), a)


def test_non_default_stream(gpu_lib):
    import torch
    L = small_layer("v6_k4096")
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(300, L, 1)
    xs = torch.from_numpy(x).cuda()
    torch.cuda.synchronize()
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        y = gpu_lib.gemv(dl, xs)
    st.synchronize()
    _check_matmul(y, oracle.gemv(L, x), "side stream")


FUSED_SETS = ("qkv_v6", "gate_up_res12", "res8_outlier_pair", "many_rows", "eight_layers")
DOWN_FUSED_SETS = ("down_qkv", "down_gate_up_res12_outlier", "down_res8_many_streams")      # orientation 1: the same body for every batch


@pytest.mark.parametrize("name", list(MULTI))
@pytest.mark.parametrize("batch", [1, 3, 16])
def test_gemv_multi(gpu_lib, monkeypatch, name, batch):
    """Several layers on the same activations in one call: each output against the oracle's product for that layer,
    for more than one row bit-identical to the matrix-core kernel on the layer alone, and padding between output rows
    left alone."""
    import torch
    layers = multi_layers(name)
    dls = [gpu_lib.DeviceLayer(L) for L in layers]
    x_np = s.make_activations(400, layers[0], batch)
    x = torch.from_numpy(x_np).cuda()
    pad = 3
    outs = [torch.full((batch, L.out_features + pad), -7.0, dtype=torch.float16, device="cuda") for L in layers]
    ys = gpu_lib.gemv_multi(dls, x, outs=[o[:, :L.out_features] for o, L in zip(outs, layers)])
    torch.cuda.synchronize()
    monkeypatch.setenv("VQ_SWITCHES", "gemv=m")
    for L, dl, y, o in zip(layers, dls, ys, outs):
        _check_matmul(y, oracle.gemv(L, x_np), "%s / %s batch %d" % (name, L.name, batch))
        assert (o[:, L.out_features:] == -7.0).all()
        alone = gpu_lib.gemv(dl, x)
        torch.cuda.synchronize()
        if (name in FUSED_SETS and batch > 1) or name in DOWN_FUSED_SETS:       # one row runs the dot-product body, whose split (and so its summation
            assert torch.equal(alone, y), L.name   # order) depends on the rows per workgroup; the others go one by one


@pytest.mark.parametrize("name", FUSED_SETS)
def test_gemv_multi_single_row_with_the_matrix_core_body(gpu_lib, monkeypatch, name):
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "gemv=m")
    layers = multi_layers(name)
    dls = [gpu_lib.DeviceLayer(L) for L in layers]
    x_np = s.make_activations(400, layers[0], 1)
    ys = gpu_lib.gemv_multi(dls, torch.from_numpy(x_np).cuda())
    torch.cuda.synchronize()
    for L, y in zip(layers, ys):
        _check_matmul(y, oracle.gemv(L, x_np), "%s / %s" % (name, L.name))


def test_gemv_multi_one_by_one_matches_fused(gpu_lib, monkeypatch):
    import torch
    layers = multi_layers("qkv_v6")
    dls = [gpu_lib.DeviceLayer(L) for L in layers]
    x = torch.from_numpy(s.make_activations(400, layers[0], 4)).cuda()
    fused = [y.clone() for y in gpu_lib.gemv_multi(dls, x)]
    monkeypatch.setenv("VQ_SWITCHES", "multi=0,gemv=m")
    apart = gpu_lib.gemv_multi(dls, x)
    torch.cuda.synchronize()
    for a, b in zip(fused, apart):
        assert torch.equal(a, b)


GROUPED_FAST = [n for n, kw in SMALL.items() if kw.get("group_vectors", 0) % 8 == 0 and kw.get("group_vectors", 0) > 0 and kw["v"] == 6]


@pytest.mark.parametrize("name", GROUPED_FAST)
@pytest.mark.parametrize("batch", [1, 4, 16])
def test_gemv_groups_with_workspace(gpu_lib, monkeypatch, name, batch):
    """Layers with codebook groups when the caller lends a workspace: one group per workgroup, then the sum over groups.
    Against the oracle, and against the route without a workspace (same per-group sums, added in the same order)."""
    import torch
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
    if L.in_features % 2:
        assert need == 0                # not a layer of the fast kernels: no workspace route
        return
    assert need >= L.n_groups * batch * L.out_features * 4
    x_np = s.make_activations(300, L, batch)
    x = torch.from_numpy(x_np).cuda()
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")       # NaN patterns: nothing may be read before it is written
    y = gpu_lib.gemv(dl, x, workspace=ws[:need])
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x_np), "%s batch %d with workspace" % (name, batch))
    assert (ws[need:] == 0xFF).all()
    small = gpu_lib.gemv(dl, x, workspace=ws[:need - 256])                         # too small: the plain route
    plain = gpu_lib.gemv(dl, x)
    torch.cuda.synchronize()
    assert torch.equal(small, plain)
    _check_matmul(plain, oracle.gemv(L, x_np), "%s batch %d" % (name, batch))


LDS_SLOTS = ["lds_v12_groups_res_outlier", "lds_v12_groups_perm", "lds_v4_k256_groups", "down_lds_v12_groups_outlier", "down_lds_v12_odd_groups"]


@pytest.mark.parametrize("name", LDS_SLOTS)
@pytest.mark.parametrize("batch", [1, 3, 4, 7, 16])
def test_gemv_lds_table_slots_with_workspace(gpu_lib, name, batch):
    """The layers of the LDS-table pass kernel with two codebook groups or more when the caller lends a workspace: a group per
    workgroup and the outlier columns in workgroups of their own, from three rows on the kernel for any number of rows in parts, then
    the sum over the groups.  Workspace filled with NaN patterns beforehand, guarded behind; too small a workspace is the plain route."""
    import torch
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
    assert need >= L.n_groups * batch * L.out_features * 4
    x_np = s.make_activations(300, L, batch)
    x = torch.from_numpy(x_np).cuda()
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    y = gpu_lib.gemv(dl, x, workspace=ws[:need])
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x_np), "%s batch %d with workspace" % (name, batch))
    assert (ws[need:] == 0xFF).all()
    small = gpu_lib.gemv(dl, x, workspace=ws[:need - 256])
    plain = gpu_lib.gemv(dl, x)
    torch.cuda.synchronize()
    assert torch.equal(small, plain)


@pytest.mark.parametrize("groups", [2, 8, 9])
@pytest.mark.parametrize("permuted", [False, True])
@pytest.mark.parametrize("v,k,k_res", [(12, 4096, 4000), (4, 256, 200)])
def test_gemv_lds_table_slots_with_two_tables(gpu_lib, groups, permuted, v, k, k_res):
    """Layers with a residual table: up to eight groups a slot is one table, more and it is a group; one launch gathers permuted
    columns by itself.  Ragged ends: rows that fill no round, a last group of fewer vectors, columns cut off within a vector."""
    import torch
    per = 16 if groups < 9 else 8
    cols = 40 + v * (per * groups - 3) - 1
    L = s.make_layer(310, "slots", 611, cols + cols % 2, v, k, k_res, n_outlier_cols=40, v_out=4, k_out=5000, group_vectors=per, permute=permuted)
    assert L.n_groups == groups
    dl = gpu_lib.DeviceLayer(L)
    for batch in (1, 2):
        x_np = s.make_activations(310, L, batch)
        need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
        ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        y = gpu_lib.gemv(dl, torch.from_numpy(x_np).cuda(), workspace=ws[:need])
        torch.cuda.synchronize()
        _check_matmul(y, oracle.gemv(L, x_np), "v %d, %d groups, permuted %s, batch %d" % (v, groups, permuted, batch))
        assert (ws[need:] == 0xFF).all()


@pytest.mark.parametrize("permuted", [False, True])
@pytest.mark.parametrize("batch,lent_for", [(1, 3), (2, 3), (1, 4), (4, 4)])
def test_gemv_lds_table_slots_with_the_workspace_of_other_rows(gpu_lib, permuted, batch, lent_for):
    """Two tables a group: one and two rows take a table a slot, more another kernel, whose workspace has to do for fewer rows as well, and
    for four rows of an odd width, which go to a group a slot.  That the workspace is made use of: its first sums are written."""
    import torch
    groups, v = 4, 12
    L = s.make_layer(312, "slots", 611, v * (16 * groups - 3) - 1, v, 4096, 4000, group_vectors=16, permute=permuted)
    assert L.n_groups == groups and L.in_features % 2 == 1
    dl = gpu_lib.DeviceLayer(L)
    x_np = s.make_activations(312, L, batch)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, lent_for)
    head = (batch * ((L.in_features + 7) // 8 * 8) * 2 + 255) // 256 * 256 if permuted else 0
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    y = gpu_lib.gemv(dl, torch.from_numpy(x_np).cuda(), workspace=ws[:need])
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x_np), "permuted %s, batch %d, lent for %d" % (permuted, batch, lent_for))
    assert (ws[need:] == 0xFF).all()
    if not permuted or batch < 4:                     # (four gathered rows have an even width again)
        assert torch.isfinite(ws[head : head + groups * batch * L.out_features * 4].view(torch.float32)).all()


@pytest.mark.parametrize("out,inp,setting,batch", [
    (300, 1918, dict(k_res=4096, group_vectors=40), 1),             # a group a workgroup: activations straight into the operands
    (300, 1918, dict(k_res=4096, group_vectors=40), 4),
    (300, 1918, dict(k_res=256, group_vectors=40), 4),             # moved there
    (300, 766, dict(), 5),
    (4100, 8004, dict(), 3),                                       # long rows, few of them: straight into the operands again
    (8200, 8010, dict(), 5),
])
def test_gemv_of_infinite_activations(gpu_lib, out, inp, setting, batch):
    """An infinite activation at either end of a vector makes every output infinite, where no table and no bias has a negative or zero value:
    what is loaded beside a vector never meets the zeros that its entries are padded with."""
    import torch
    L = s.make_layer(313, "infinite", out, inp, 6, 4096, **setting)
    L.codebook, L.bias = np.maximum(np.abs(L.codebook), np.float16(1e-3)), np.maximum(np.abs(L.bias), np.float16(1e-3))
    if L.codebook_res is not None:
        L.codebook_res = np.maximum(np.abs(L.codebook_res), np.float16(1e-3))
    dl = gpu_lib.DeviceLayer(L)
    x = torch.from_numpy(s.make_activations(313, L, batch)).cuda()
    ws = torch.empty((gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch),), dtype=torch.uint8, device="cuda")
    for column in (6, 7, 11, inp // 2 // 6 * 6, inp - 1):
        z = x.clone()
        z[batch - 1, column] = float("inf")
        y = gpu_lib.gemv(dl, z, workspace=ws)
        assert (y[batch - 1] == float("inf")).all(), column
        assert torch.isfinite(y[: batch - 1]).all(), column


@pytest.mark.parametrize("out,k_res", [(300, 0), (4000, 4096), (300, 256)])
@pytest.mark.parametrize("batch", [1, 2])
def test_gemv_of_an_infinite_entry_that_no_index_names(gpu_lib, out, k_res, batch):
    """480 vectors a row, whole lanes of four, five, six or eight: the lanes behind them add nothing to a row, whatever entry they look up."""
    import torch
    L = s.make_layer(320, "entry", out, 2880, 6, 4096, k_res)
    L.codebook[0] = np.inf
    bits = np.unpackbits(L.idx, axis=1, bitorder="little")
    bits[:, 0:480 * 12:12] = 1                           # odd indices
    L.idx = np.packbits(bits, axis=1, bitorder="little")
    x_np = s.make_activations(320, L, batch)
    y = gpu_lib.gemv(gpu_lib.DeviceLayer(L), torch.from_numpy(x_np).cuda())
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x_np), "batch %d" % batch)


@pytest.mark.parametrize("outs,inp,outliers", [
    ((4100,), 8004, 0),                    # two blocks of rows a chunk: up to three activation rows straight into the operands
    ((8200,), 8010, 0),                    # three: up to five
    ((12290,), 8002, 8),                   # four, and outlier columns
    ((3000, 1500, 700), 8006, 0),
    ((9000, 3300), 9998, 4),
])
def test_gemv_of_few_long_rows(gpu_lib, outs, inp, outliers):
    """The matrix-core kernel's operands hold the same values whichever way they are loaded: a row's outputs are the same bits beside any number
    of other rows, and a few of them those of the oracle."""
    import torch
    layers = [s.make_layer(314 + i, "long", out, inp, 6, 4096, 0, outliers, 4 if outliers else 0, 4096 if outliers else 0) for i, out in enumerate(outs)]
    dls = [gpu_lib.DeviceLayer(L) for L in layers]
    x_np = s.make_activations(314, layers[0], 7)
    x = torch.from_numpy(x_np).cuda()
    run = (lambda z: gpu_lib.gemv_multi(dls, z)) if len(dls) > 1 else (lambda z: [gpu_lib.gemv(dls[0], z)])
    seven = run(x)
    for L, y in zip(layers, seven):
        rows = np.array([0, 17, L.out_features // 2, L.out_features - 1], dtype=np.int32)
        _check_matmul(y[:, torch.from_numpy(rows.astype(np.int64)).cuda()], oracle.gemm(L, x_np, rows=rows), "%d x %d" % (L.out_features, inp))
    for batch in (2, 3, 4, 5, 6):
        for y, few in zip(seven, run(x[:batch].contiguous())):
            assert torch.equal(few.view(torch.int16), y[:batch].view(torch.int16)), batch


PERMUTED = [n for n in SMALL if n.startswith("perm_")]


@pytest.mark.parametrize("name", PERMUTED)
@pytest.mark.parametrize("batch", [1, 2, 5, 16])
def test_gemv_permuted_columns_with_workspace(gpu_lib, name, batch):
    """Sec. 3.2.3: stored column order a permutation of the layer's.  With a workspace the activations are gathered into it
    first and the layer's usual kernels run; one row of a short-row v = 6 layer is gathered inside the kernel instead and
    asks for no workspace.  Also through the library's own static workspace."""
    import torch
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
    in_kernel = batch == 1 and L.v == 6 and L.orientation == 0 and not L.group_vectors and L.in_features % 2 == 0 and L.in_features < 16384
    assert (need == 0) == in_kernel, (name, batch, need)
    x_np = s.make_activations(300, L, batch)
    x = torch.full((batch, L.in_features + 4), float("nan"), dtype=torch.float16, device="cuda")
    x[:, : L.in_features] = torch.from_numpy(x_np).cuda()
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    y = gpu_lib.gemv(dl, x, workspace=ws[:need] if need else ws[:256])
    torch.cuda.synchronize()
    ref = oracle.gemv(L, x_np)
    _check_matmul(y, ref, "%s batch %d with workspace" % (name, batch))
    assert (ws[need:] == 0xFF).all()
    y2 = torch.empty_like(y)
    rc = gpu_lib.vq_gemv_static_workspace(dl.desc, x.data_ptr(), x.stride(0), batch, y2.data_ptr(), y2.stride(0), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    plain = gpu_lib.gemv(dl, x, workspace=lent("none"))       # no workspace: gathered in the kernel, or the generic kernels
    torch.cuda.synchronize()
    _check_matmul(plain, ref, "%s batch %d" % (name, batch))


@pytest.mark.parametrize("orientation", [0, 1])
@pytest.mark.parametrize("pitch", [0, 3])
@pytest.mark.parametrize("out_features,in_features", [(1023, 1030), (1024, 6), (1025, 1031), (1026, 8), (1027, 4096), (1030, 10240), (1030, 10241), (2048, 33)])
def test_dequant_moves_columns_of_several_rows(gpu_lib, out_features, in_features, pitch, orientation):
    """Permuted columns of one row to a workgroup and of four, a last one of fewer, rows at any half, columns past the last eight: bit for bit
    what the layer restores in stored order, at its columns; nothing beyond them."""
    import copy
    import torch
    L = s.make_layer(8300, "moved", out_features, in_features, 6, 300, orientation=orientation, permute=True)
    stored = copy.copy(L)
    stored.col_perm = None
    want = gpu_lib.dequant(gpu_lib.DeviceLayer(stored))
    dl = gpu_lib.DeviceLayer(L)
    W = torch.full((out_features, in_features + pitch), -3.5, dtype=torch.float16, device="cuda")
    assert gpu_lib.vq_dequant(dl.desc, W.data_ptr(), W.stride(0), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(W[:, torch.from_numpy(np.asarray(L.col_perm)).long().cuda()].view(torch.int16), want.view(torch.int16))
    assert (W[:, in_features:] == -3.5).all()


@pytest.mark.parametrize("name", PERMUTED)
def test_dequant_permuted_columns_by_the_scattering_kernels(gpu_lib, monkeypatch, name):
    """The generic kernels, which store every value at its column themselves (rows too long for LDS take them)."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "dequant=g")
    L = small_layer(name)
    W = gpu_lib.dequant(gpu_lib.DeviceLayer(L), L.in_features + 5)
    torch.cuda.synchronize()
    assert np.array_equal(W.cpu().numpy().view(np.uint16), oracle.dequant(L, L.in_features + 5).view(np.uint16)), name


@pytest.mark.parametrize("orientation", [0, 1])
@pytest.mark.parametrize("out_features,in_features,v,k,more", [
    (3, 24, 6, 4096, {}), (65, 513, 6, 256, dict(k_res=200)), (515, 1030, 6, 4096, dict(k_res=4096)), (66, 3077, 2, 16, dict(k_res=16)),
    (1030, 520, 4, 256, {}), (130, 2056, 4, 4096, dict(k_res=3001, group_vectors=129)), (40, 9000, 8, 4096, dict(k_res=4096)),
    (96, 600, 8, 65536, {}), (1040, 5000, 8, 65536, {}), (64, 520, 8, 65536, dict(k_res=300, group_vectors=31)), (64, 512, 8, 200, dict(k_res=65536)),
    (70, 1029, 12, 4096, dict(k_res=4096)), (70, 1029, 12, 4096, dict(k_res=2722)), (600, 1500, 12, 4096, dict(k_res=4096, group_vectors=41)),
    (133, 1207, 6, 4096, dict(k_res=256, n_outlier_cols=28, v_out=4, k_out=4096)), (133, 1207, 12, 4000, dict(n_outlier_cols=12, v_out=4, k_out=9, group_vectors=300)),
])
def test_dequant_tables_edges(gpu_lib, out_features, in_features, v, k, more, orientation):
    """Runs that end with a row or a group, groups that begin anywhere, residual tables in LDS, split and in memory, W at any half."""
    import torch
    L = s.make_layer(8200, "edges", out_features, in_features, v, k, orientation=orientation, **more)
    dl, want = gpu_lib.DeviceLayer(L), oracle.dequant(L).view(np.uint16)
    for offset, ldw in ((0, (in_features + 7) // 8 * 8 + 8), (1, in_features)):
        buf = torch.full((out_features * ldw + offset + 8,), 3.0, dtype=torch.float16, device="cuda")
        assert gpu_lib.vq_dequant(dl.desc, buf.data_ptr() + 2 * offset, ldw, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        W = got[offset: offset + out_features * ldw].reshape(out_features, ldw)
        assert np.array_equal(W[:, :in_features].view(np.uint16), want), offset
        assert (W[:, in_features:] == 3.0).all() and (got[:offset] == 3.0).all() and (got[offset + out_features * ldw:] == 3.0).all()


@pytest.mark.parametrize("out_features,in_features,v,k,more", [
    (6001, 1159, 6, 4096, {}), (9000, 772, 6, 4096, dict(k_res=256)), (12500, 770, 6, 4096, dict(k_res=4096, group_vectors=64)), (20000, 390, 6, 256, {}),
    (7000, 1540, 4, 256, {}), (4100, 2050, 8, 65536, {}), (4000, 1540, 12, 4096, dict(k_res=4096)), (10000, 768, 2, 16, {}),
    (8203, 16390, 6, 4096, dict(n_outlier_cols=8, v_out=4, k_out=4096)), (8203, 16390, 4, 256, {}), (8203, 16416, 6, 256, dict(orientation=1)),
    (8203, 16390, 4, 256, dict(orientation=1)),
])
@pytest.mark.parametrize("scale", [True, False])
def test_dequant_waves_with_several_turns(gpu_lib, out_features, in_features, v, k, more, scale):
    """Layers of which a wave restores two runs and more, in turn from two sets of registers, and (the last four: W of more than
    256 MiB) with stores past the caches; with and without scale and bias."""
    import torch
    if not scale and out_features * in_features > 1 << 27:
        pytest.skip("once is enough for the largest")
    L = s.make_layer(8300, "turns", out_features, in_features, v, k, **more)
    if not scale:
        L.scale = L.bias = None
    ldw = in_features + (0 if in_features > 16000 else 2)         # (down the outputs past the caches only with rows on 64 bytes)
    W = gpu_lib.dequant(gpu_lib.DeviceLayer(L), ldw)
    torch.cuda.synchronize()
    assert np.array_equal(W.cpu().numpy().view(np.uint16), oracle.dequant(L, ldw).view(np.uint16))


@pytest.mark.parametrize("name", ["lds_v12_two_tables", "lds_v12_groups_res_outlier", "down_lds_v12_two_tables", "down_lds_v12_odd_groups"])
def test_dequant_two_tables_beyond_lds_in_two_passes(gpu_lib, monkeypatch, name):
    """Two tables that do not fit LDS together: by default the last third of the residual entries comes from memory; dequant=g, the
    generic kernels, read all tables there.  Both bit for bit."""
    import torch
    L = small_layer(name)
    want = oracle.dequant(L, L.in_features + 6).view(np.uint16)
    for switch in (None, "dequant=g"):
        if switch:
            monkeypatch.setenv("VQ_SWITCHES", switch)
        W = gpu_lib.dequant(gpu_lib.DeviceLayer(L), L.in_features + 6)
        torch.cuda.synchronize()
        assert np.array_equal(W.cpu().numpy().view(np.uint16), want), (name, switch)


def test_permuted_unit_activation_reads_back_the_layers_column(gpu_lib):
    """x = e_t returns column t of the LAYER (not of the stored order), outlier columns included."""
    import torch
    L = small_layer("perm_v6_res8_outlier")
    dl = gpu_lib.DeviceLayer(L)
    W = oracle.dequant(L).astype(np.float64)
    cols = [int(L.col_perm[0]), int(L.col_perm[23]), int(L.col_perm[24]), int(L.col_perm[1207]), 0, 1207]
    for ws in ("none", "fast"):
        for t in cols:
            x = np.zeros((2, L.in_features), dtype=np.float16)
            x[0, t] = 1.0
            x[1, t] = -2.0
            y = gpu_lib.gemv(dl, torch.from_numpy(x).cuda(), workspace=lent(ws)).float().cpu().numpy()
            assert np.allclose(y[0], W[:, t], rtol=2e-3, atol=1e-7) and np.allclose(y[1], -2.0 * W[:, t], rtol=2e-3, atol=1e-7)


def test_permutation_entries_outside_the_row_are_ignored(gpu_lib):
    """The library does not check that col_perm is a permutation: an entry outside [0, in_features) must neither be
    read nor written through.  Such a stored column then contributes nothing, which is the same layer with a zero
    activation there."""
    import torch
    L = small_layer("perm_v6_res8_outlier")
    x_np = s.make_activations(300, L, 3)
    bad = [5, 30, 700]                                  # stored columns whose entries go out of range
    ref_x = x_np.copy()
    ref_x[:, L.col_perm[bad]] = 0
    ref = oracle.gemv(L, ref_x)
    want_W = oracle.dequant(L)
    M = small_layer("perm_v6_res8_outlier")
    M.col_perm = L.col_perm.copy()
    M.col_perm[bad] = [-1, L.in_features, 2 ** 31 - 1]
    dl = gpu_lib.DeviceLayer(M)
    x = torch.from_numpy(x_np).cuda()
    for ws in ("none", "fast"):
        for batch in (1, 3):
            y = gpu_lib.gemv(dl, x[:batch], workspace=lent(ws))
            torch.cuda.synchronize()
            _check_matmul(y, ref[:batch], "out-of-range entries, batch %d, workspace %s" % (batch, ws))
    W = torch.full((M.out_features, M.in_features + 8), -3.5, dtype=torch.float16, device="cuda")
    assert gpu_lib.vq_dequant(dl.desc, W.data_ptr(), W.stride(0), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    got = W.cpu().numpy()
    keep = np.setdiff1d(np.arange(M.in_features), L.col_perm[bad])
    assert np.array_equal(got[:, keep].view(np.uint16), want_W[:, keep].view(np.uint16))
    assert (got[:, M.in_features:] == np.float16(-3.5)).all()


def test_gemv_multi_with_permuted_layers(gpu_lib):
    """Layers with a column permutation of their own run one after the other: same results as single calls."""
    import torch
    a, b = small_layer("perm_v6_k4096"), small_layer("v6_k4096")
    dls = [gpu_lib.DeviceLayer(a), gpu_lib.DeviceLayer(b)]
    for batch in (1, 4):
        x_np = s.make_activations(300, a, batch)
        ys = gpu_lib.gemv_multi(dls, torch.from_numpy(x_np).cuda())
        torch.cuda.synchronize()
        for L, y in zip((a, b), ys):
            _check_matmul(y, oracle.gemv(L, x_np), "multi with a permuted layer, batch %d" % batch)


def test_gemv_workspace_is_not_asked_for_without_groups(gpu_lib):
    for name in ("v6_k4096", "v8_k65536", "grp_v6_unaligned", "grp_odd"):
        dl = gpu_lib.DeviceLayer(small_layer(name))
        assert gpu_lib.vq_gemv_workspace_bytes(dl.desc, 4) == 0, name


NATIVE_PLAIN = [n for n, kw in SMALL.items() if n.startswith("down_fast") and not kw.get("group_vectors") and kw.get("n_outlier_cols", 0) % 2 == 0]


@pytest.mark.parametrize("name", NATIVE_PLAIN)
@pytest.mark.parametrize("batch", [2, 3, 6, 16])
def test_gemv_native_orientation_column_parts_with_workspace(gpu_lib, name, batch):
    """Vectors down the output dimension, one codebook group, two rows or more: with a workspace the matrix-core kernel
    cuts the columns into parts that run side by side and a second kernel adds them up."""
    import torch
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
    if L.in_features - L.n_outlier_cols < 2 * 8 * 32 or L.out_features > 16 * 6 * 128:
        assert need == 0, name          # a part needs a window of 32 columns per wave; more blocks of 16 streams than half the chip need no parts
        return
    assert need >= 2 * batch * L.out_features * 4, name
    x_np = s.make_activations(300, L, batch)
    x = torch.from_numpy(x_np).cuda()
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    y = gpu_lib.gemv(dl, x, workspace=ws[:need])
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x_np), "%s batch %d with workspace" % (name, batch))
    assert (ws[need:] == 0xFF).all()
    need1 = gpu_lib.vq_gemv_workspace_bytes(dl.desc, 1)
    if name != "down_fast_long_rows_res12":
        assert need1 == 0                # a single row stays on the kernel that needs none
        return
    # ... unless the row is too long for that kernel's LDS beside the tables: then one row runs in column parts as well,
    # and without a workspace on the matrix-core kernel alone
    assert need1 >= 2 * L.out_features * 4
    for workspace in (ws[:need1], None):
        y1 = gpu_lib.gemv(dl, x[:1], workspace=workspace)
        torch.cuda.synchronize()
        _check_matmul(y1, oracle.gemv(L, x_np[:1]), "%s one row, workspace %s" % (name, workspace is not None))


@pytest.mark.parametrize("workspace", ["none", "fast"])
@pytest.mark.parametrize("batch", [1, 3, 5, 16])
@pytest.mark.parametrize("name,pad_x,pad_y", [("down_fast_res12", 8, 1), ("down_fast_outlier", 24, 6), ("down_fast_parts", 16, 3),
                                               ("down_fast_groups_outlier_tall", 8, 5),
                                               ("down_v6", 1, 3)])       # 391 columns: the last row ends inside a dword
def test_native_orientation_strided_buffers_and_untouched_padding(gpu_lib, name, pad_x, pad_y, batch, workspace):
    """Vectors down the output dimension, fast kernels (row stride of x a multiple of 8): NaN in the caller's padding of x
    must never reach a sum, and sentinels in the padding of y must survive; with and without the workspace route."""
    import torch
    L = small_layer(name)
    dl = gpu_lib.DeviceLayer(L)
    x = s.make_activations(300, L, batch)
    xb = torch.full((batch, L.in_features + pad_x), float("nan"), dtype=torch.float16, device="cuda")
    xb[:, : L.in_features] = torch.from_numpy(x).cuda()
    yb = torch.full((batch, L.out_features + pad_y), 7.0, dtype=torch.float16, device="cuda")
    gpu_lib.gemv(dl, xb, out=yb, workspace=lent(workspace))
    torch.cuda.synchronize()
    _check_matmul(yb[:, : L.out_features], oracle.gemv(L, x), "strided %s batch %d workspace %s" % (name, batch, workspace))
    assert (yb[:, L.out_features:] == 7.0).all()


@pytest.mark.parametrize("seed", range(12))
def test_eight_component_layers_random_shapes(gpu_lib, seed):
    """Layers of 8-component vectors in both orientations with random sizes, table sizes (8- and 16-bit indices), residual
    tables and codebook groups: vq_dequant bit for bit, vq_gemv on padded buffers (NaN in x's padding, sentinels in y's)."""
    import torch
    rng = np.random.default_rng(4321 + seed)
    orientation = seed % 2
    out, P = int(rng.integers(1, 1500)), int(rng.integers(1, 700))
    k = int(rng.choice([65536, 256, 40000, 200, 17]))
    kw = {}
    r = int(rng.integers(0, 3))
    if r == 1:
        kw["k_res"] = int(rng.choice([256, 100]))
    if r == 2:
        kw["k_res"] = int(rng.choice([65536, 5000]))
    if rng.integers(0, 3) == 0:
        kw["group_vectors"] = int(rng.integers(1, max(2, P)))
    in_features = P * 8 if orientation == 0 else int(rng.integers(1, 3000))
    L = s.make_layer(9200 + seed, "v8_random_%d" % seed, out, in_features, 8, k, orientation=orientation, **kw)
    dl = gpu_lib.DeviceLayer(L)
    W = gpu_lib.dequant(dl)
    torch.cuda.synchronize()
    assert np.array_equal(W.cpu().numpy().view(np.uint16), oracle.dequant(L).view(np.uint16)), (out, in_features, k, kw)
    for batch in (1, 2, int(rng.integers(3, 17))):
        x = s.make_activations(9200 + seed, L, batch)
        xb = torch.full((batch, (in_features + 7) // 8 * 8 + 8), float("nan"), dtype=torch.float16, device="cuda")
        xb[:, :in_features] = torch.from_numpy(x).cuda()
        yb = torch.full((batch, out + 3), 7.0, dtype=torch.float16, device="cuda")
        for workspace in ("none", None):
            yb.fill_(7.0)
            gpu_lib.gemv(dl, xb, out=yb, workspace=lent(workspace))
            torch.cuda.synchronize()
            _check_matmul(yb[:, :out], oracle.gemv(L, x), "v = 8, orientation %d, %d x %d, k %d, %s, batch %d" % (orientation, out, in_features, k, kw, batch))
            assert (yb[:, out:] == 7.0).all()


@pytest.mark.parametrize("seed", range(48))
def test_lds_table_kernels_random_shapes(gpu_lib, seed):
    """The (v, index width) pairs of the LDS-table kernels, in both orientations, with random sizes, table sizes, residual
    tables of the same index width, codebook groups, outlier columns of v = 4 (up to 13 index bits) and permutations: vq_dequant bit for bit (W with a
    padded, sentinel-filled pitch), vq_gemv on padded buffers (NaN in x's padding, sentinels in y's), vq_gemm with the
    restore-then-multiply workspace where the layer has one."""
    import torch
    rng = np.random.default_rng(97531 + seed)
    v, bits = [(2, 4), (4, 8), (6, 8), (8, 8), (4, 12), (8, 12), (12, 12), (6, 12)][seed % 8]
    k = int(rng.integers(2 ** (bits - 1) + 1, 2 ** bits + 1))
    out = int(rng.integers(1, 6000)) if seed % 3 == 0 else int(rng.integers(1, 700))
    orientation = 1 if seed >= 24 else 0               # (the second half: vectors down the output dimension, any number of outlier columns)
    n_out = (4 if orientation == 0 else 1) * int(rng.integers(0, 12)) if rng.integers(0, 2) else 0
    in_features = n_out + int(rng.integers(1, 2600))
    kw = {}
    if rng.integers(0, 2):
        kw["k_res"] = int(rng.integers(2 ** (bits - 1) + 1, 2 ** bits + 1))
    if n_out:
        kw.update(n_outlier_cols=n_out, v_out=4, k_out=int(rng.choice([8192, 4096, 300, 5000])))
    P = -(-(in_features - n_out) // v) if orientation == 0 else in_features - n_out
    if rng.integers(0, 2):
        kw["group_vectors"] = int(rng.integers(max(1, P // 17), P + 1))
    if rng.integers(0, 3) == 0:
        kw["permute"] = True
    if orientation:
        kw["orientation"] = 1
    what = "v %d, %d-bit, %d x %d, k %d, %s" % (v, bits, out, in_features, k, kw)
    L = s.make_layer(9300 + seed, "lds_random_%d" % seed, out, in_features, v, k, **kw)
    dl = gpu_lib.DeviceLayer(L)
    ldw = in_features + int(rng.choice([0, 2, 5, 8]))
    W = torch.full((out, ldw), 3.0, dtype=torch.float16, device="cuda")
    assert gpu_lib.vq_dequant(dl.desc, W.data_ptr(), ldw, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert np.array_equal(W[:, :in_features].cpu().numpy().view(np.uint16), oracle.dequant(L).view(np.uint16)), what
    assert (W[:, in_features:] == 3.0).all(), what
    for batch in (1, 2, 4, int(rng.integers(3, 17))):
        x = s.make_activations(9300 + seed, L, batch)
        xb = torch.full((batch, (in_features + 7) // 8 * 8 + 8), float("nan"), dtype=torch.float16, device="cuda")
        xb[:, :in_features] = torch.from_numpy(x).cuda()
        yb = torch.full((batch, out + 3), 7.0, dtype=torch.float16, device="cuda")
        ref = oracle.gemv(L, x)
        for workspace in ("none", "fast"):   # (with a workspace: a codebook group or the outlier columns per workgroup, then a sum)
            yb.fill_(7.0)
            gpu_lib.gemv(dl, xb, out=yb, workspace=lent(workspace))
            torch.cuda.synchronize()
            _check_matmul(yb[:, :out], ref, what + ", batch %d, workspace %s" % (batch, workspace))
            assert (yb[:, out:] == 7.0).all()
    if in_features % 256 == 0:
        x = s.make_activations(9300 + seed, L, 70)
        Y = gpu_lib.gemm(dl, torch.from_numpy(x).cuda(), workspace="fast")
        torch.cuda.synchronize()
        _check_matmul(Y, oracle.gemm(L, x), what + ", 70 tokens")


@pytest.mark.parametrize("out_features,in_features,more", [
    (1, 13, {}), (65, 100, dict(k_res=4096)), (611, 2003, dict(k_res=4000)), (1030, 96 * 3, dict(k_res=2722, group_vectors=8)),
    (4099, 205, {}), (333, 28675, dict(k_res=4096)), (1025, 40 + 12 * 181 - 1, dict(k_res=4096, group_vectors=48, n_outlier_cols=40, v_out=4, k_out=5000)),
    (9001, 772, dict(n_outlier_cols=4, v_out=4, k_out=8192)), (61, 1600, dict(n_outlier_cols=404, v_out=4, k_out=4097)), (130, 1301, dict(k_res=4096, group_vectors=40, n_outlier_cols=12, v_out=4, k_out=9)),
])
@pytest.mark.parametrize("k", [4096, 2050])
@pytest.mark.parametrize("permuted", [False, True])
def test_gemv_from_tables_of_products(gpu_lib, monkeypatch, out_features, in_features, more, k, permuted):
    """One and two rows of layers of twelve-element vectors with a workspace: rows and runs of positions that fill no workgroup, octets cut off by a
    group's or the row's end, tables that are not full, outlier columns, activation rows of any pitch."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "products=1")
    L = s.make_layer(313, "products", out_features, in_features, 12, k, permute=permuted, **more)
    dl = gpu_lib.DeviceLayer(L)
    for batch, pitch in ((1, in_features), (2, in_features), (2, in_features + 3)):
        x_np = s.make_activations(313, L, batch)
        x = torch.full((batch, pitch), float("nan"), dtype=torch.float16, device="cuda")
        x[:, :in_features] = torch.from_numpy(x_np)
        need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
        ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
        y = gpu_lib.gemv(dl, x[:, :in_features], workspace=ws[:need])
        torch.cuda.synchronize()
        _check_matmul(y, oracle.gemv(L, x_np), "batch %d" % batch)
        assert (ws[need:] == 0xFF).all() and (ws[:4] != 0xFF).any()


def test_tables_of_products_keep_what_is_no_number_where_it_belongs(gpu_lib, monkeypatch):
    """An infinite activation reaches every output, an infinite entry those that name it, and neither a neighbour in the same instruction."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "products=1")
    L = s.make_layer(314, "products", 200, 24 * 12, 12, 4096, 4096)
    x_np = s.make_activations(314, L, 1)
    L.codebook[1::2, 3] = np.inf                       # the odd entries; then no index but even ones, save in the first row
    bits = np.unpackbits(L.idx, axis=1, bitorder="little")
    bits[1:, 0:24 * 12:12] = 0
    bits[0, 0:24 * 12:12] = 1
    L.idx = np.packbits(bits, axis=1, bitorder="little")
    dl = gpu_lib.DeviceLayer(L)
    x = torch.from_numpy(x_np).cuda()
    ws = torch.empty(gpu_lib.vq_gemv_workspace_bytes(dl.desc, 1), dtype=torch.uint8, device="cuda")
    y = gpu_lib.gemv(dl, x, workspace=ws).float().cpu()[0]
    assert not torch.isfinite(y[0]) and torch.isfinite(y[1:]).all()
    x[0, 30] = float("inf")
    y = gpu_lib.gemv(dl, x, workspace=ws).float().cpu()[0]
    assert not torch.isfinite(y).any()


@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("last", [1, 7, 8, 11, 12])
def test_tables_of_products_drop_what_lies_past_the_row(gpu_lib, monkeypatch, last, batch):
    """Entries that are infinite past the elements of a row that its last vector has, named by that vector alone; in both tables, in a group of its own."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "products=1")
    inp = 12 * 57 + last
    L = s.make_layer(321, "products", 200, inp, 12, 4096, 4096, group_vectors=40)
    L.codebook[1::2, last:] = np.inf
    L.codebook_res[1::2, last:] = -np.inf
    for stream in ("idx", "idx_res"):
        bits = np.unpackbits(getattr(L, stream), axis=1, bitorder="little")
        bits[:, 0:58 * 12:12] = 0
        bits[::2, 57 * 12] = 1                           # every second row's last vector
        setattr(L, stream, np.packbits(bits, axis=1, bitorder="little"))
    x_np = s.make_activations(321, L, batch)
    dl = gpu_lib.DeviceLayer(L)
    ws = torch.empty(gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch), dtype=torch.uint8, device="cuda")
    y = gpu_lib.gemv(dl, torch.from_numpy(x_np).cuda(), workspace=ws)
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x_np), "%d of twelve" % last)


@pytest.mark.parametrize("out_features,in_features,k_res", [(3000, 16390, 0), (1000, 9001, 4096), (100, 300, 256), (97, 1000, 0)])
@pytest.mark.parametrize("batch", [1, 2, 3, 4, 16])
def test_gemv_down_routes(gpu_lib, out_features, in_features, k_res, batch):
    """Vectors down the outputs: one row in column parts, few rows on either kernel, parts left out where they do not pay; streams and columns
    that fill no block, part or window."""
    import torch
    L = s.make_layer(315, "down", out_features, in_features, 6, 4096, k_res, orientation=1)
    dl = gpu_lib.DeviceLayer(L)
    pitch = (in_features + 7) // 8 * 8
    x_np = s.make_activations(315, L, batch)
    x = torch.full((batch, pitch), float("nan"), dtype=torch.float16, device="cuda")
    x[:, :in_features] = torch.from_numpy(x_np)
    ref = oracle.gemv(L, x_np)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    for y in (gpu_lib.gemv(dl, x[:, :in_features], workspace=ws[:need] if need else None), gpu_lib.gemv(dl, x[:, :in_features])):
        torch.cuda.synchronize()
        _check_matmul(y, ref, "batch %d" % batch)
    assert (ws[need:] == 0xFF).all()


@pytest.mark.parametrize("out_features,in_features,more,batch", [
    (4115, 9008, {}, 3), (4115, 9402, dict(k_res=4096), 16), (500, 12140, dict(k_res=256, n_outlier_cols=120, v_out=4, k_out=4096), 5),
    (1001, 7900, dict(k_res=4096, n_outlier_cols=8, v_out=4, k_out=4096), 9), (1100, 10300, {}, 13), (17, 12011 * 2, dict(permute=True), 3),
])
def test_gemv_column_parts(gpu_lib, out_features, in_features, more, batch):
    """Rows of v = 6 vectors in parts of the columns, added up by a second kernel: parts that end within a step of the waves, a last block of few
    rows, outlier columns with the first part, columns gathered first."""
    import torch
    L = s.make_layer(316, "parts", out_features, in_features, 6, 4096, **more)
    dl = gpu_lib.DeviceLayer(L)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
    assert need >= 2 * (batch * out_features + 16) * 4
    x_np = s.make_activations(316, L, batch)
    x = torch.from_numpy(x_np).cuda()
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    y = gpu_lib.gemv(dl, x, workspace=ws[:need])
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x_np), "batch %d" % batch)
    assert (ws[need:] == 0xFF).all() and (ws[:need] != 0xFF).any()


@pytest.mark.parametrize("out_features,in_features,more", [
    (1030, 1203, {}), (700, 1801, dict(k_res=4096)), (640, 1403, dict(k_res=256, n_outlier_cols=16, v_out=4, k_out=4096)), (1300, 1211, dict(group_vectors=48)),
    (770, 1201, dict(permute=True)), (1030, 1206, dict(orientation=1)), (6000, 901, dict(orientation=1, k_res=4096)),
    (4000, 1202, dict(orientation=1, k_res=256, n_outlier_cols=10, v_out=4, k_out=4096)), (4000, 1203, dict(orientation=1, n_outlier_cols=9, v_out=4, k_out=4096)),
    (4004, 1205, dict(orientation=1, group_vectors=304)),
])
@pytest.mark.parametrize("batch", [1, 2, 5, 16])
def test_gemv_rows_of_any_width(gpu_lib, out_features, in_features, more, batch):
    """v = 6 / 12-bit layers of widths that are no multiples of eight, rows that begin at any half: taken as they are or from a copy."""
    import torch
    L = s.make_layer(317, "width", out_features, in_features, 6, 4096, **more)
    dl = gpu_lib.DeviceLayer(L)
    x_np = s.make_activations(317, L, batch)
    ref = oracle.gemv(L, x_np)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, batch)
    ws = torch.full((need + 256,), 0xFF, dtype=torch.uint8, device="cuda")
    for pitch, offset in ((in_features, 0), (in_features + 3, 1)):
        x = torch.full((batch * pitch + 8,), float("nan"), dtype=torch.float16, device="cuda")
        rows = x[offset: offset + batch * pitch].view(batch, pitch)[:, :in_features]
        rows.copy_(torch.from_numpy(x_np))
        for y in (gpu_lib.gemv(dl, rows, workspace=ws[:need] if need else None), gpu_lib.gemv(dl, rows)):
            torch.cuda.synchronize()
            _check_matmul(y, ref, "batch %d, pitch %d" % (batch, pitch))
    assert (ws[need:] == 0xFF).all()


@pytest.mark.parametrize("rows,lent_for", [(4, 4), (5, 16)])
def test_gemv_of_odd_rows_without_parts_leaves_the_workspace_alone(gpu_lib, rows, lent_for):
    """As many blocks of streams as compute units, and a row that does not fit LDS beside two tables: the activations are taken as they are, there are
    no parts, and the workspace, which has the size of a copy, is not written."""
    import torch
    L = s.make_layer(319, "blocks", 12391, 15873, 6, 4096, 4096, orientation=1)
    dl = gpu_lib.DeviceLayer(L)
    x_np = s.make_activations(319, L, rows)
    x = torch.full((rows, 15880), float("nan"), dtype=torch.float16, device="cuda")
    x[:, :15873] = torch.from_numpy(x_np)
    need = gpu_lib.vq_gemv_workspace_bytes(dl.desc, lent_for)
    ws = torch.full((need + (4 << 20),), 0xFF, dtype=torch.uint8, device="cuda")
    y = gpu_lib.gemv(dl, x[:, :15873], workspace=ws[:need])
    torch.cuda.synchronize()
    _check_matmul(y, oracle.gemv(L, x_np), "%d rows" % rows)
    assert (ws == 0xFF).all()


@pytest.mark.parametrize("in_features,k,k_res,group_vectors", [(9, 65536, 0, 0), (1203, 65536, 300, 0), (1030, 200, 65536, 31), (2051, 256, 256, 0)])
@pytest.mark.parametrize("batch", [1, 2, 5])
def test_gemv_v8_rows_of_any_width(gpu_lib, in_features, k, k_res, group_vectors, batch):
    """Vectors of eight along rows of any width that begin at any half."""
    import torch
    L = s.make_layer(318, "v8", 70, in_features, 8, k, k_res, group_vectors=group_vectors)
    dl = gpu_lib.DeviceLayer(L)
    x_np = s.make_activations(318, L, batch)
    for pitch, offset in ((in_features, 0), (in_features + 3, 1)):
        x = torch.full((batch * pitch + 8,), float("nan"), dtype=torch.float16, device="cuda")
        rows = x[offset: offset + batch * pitch].view(batch, pitch)[:, :in_features]
        rows.copy_(torch.from_numpy(x_np))
        y = gpu_lib.gemv(dl, rows)
        torch.cuda.synchronize()
        _check_matmul(y, oracle.gemv(L, x_np), "batch %d, pitch %d" % (batch, pitch))


@pytest.mark.parametrize("last", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("batch", [1, 2, 8])
def test_gemv_v8_last_vector_of_any_length(gpu_lib, last, batch):
    """Rows that begin at any half, their last vector short of any number of elements: it meets the row's last eight activations.  Neither entries that
    are infinite past the row nor an infinite activation of the vector before, which one row of the batch has, reach what they are not part of."""
    import torch
    inp = 8 * 70 + last
    L = s.make_layer(322, "v8", 70, inp, 8, 65536, 256)
    L.codebook[: 65535, last:] = np.inf
    L.idx.view(np.uint16)[:, :70] = 65535                # the last vector alone names them
    L.idx.view(np.uint16)[:, 70] %= 65535
    L.codebook[65535] = np.abs(L.codebook[65535]) + np.float16(0.01)
    L.codebook_res = np.abs(L.codebook_res)
    x_np = s.make_activations(322, L, batch)
    want = oracle.gemv(L, x_np)
    pitch = inp + 3
    x = torch.full((batch * pitch + 8,), float("nan"), dtype=torch.float16, device="cuda")
    rows = x[1: 1 + batch * pitch].view(batch, pitch)[:, :inp]
    rows.copy_(torch.from_numpy(x_np))
    dl = gpu_lib.DeviceLayer(L)
    _check_matmul(gpu_lib.gemv(dl, rows), want, "%d of eight" % last)
    L.bias = None
    rows[batch - 1, 8 * 70 - 1] = float("inf")
    y = gpu_lib.gemv(gpu_lib.DeviceLayer(L), rows).float()
    torch.cuda.synchronize()
    assert torch.isinf(y[batch - 1]).all() and torch.isfinite(y[: batch - 1]).all()


@pytest.mark.parametrize("out_features,in_features,batch,more", [
    (37, 70, 12, {}), (37, 1190, 16, {}), (4101, 203 * 2, 13, {}), (4101, 3074, 16, {}), (10242, 390, 14, {}), (15003, 70, 15, {}), (20000, 202, 16, {}),
    (37, 390, 15, dict(k_res=4096)), (1001, 1540, 13, dict(k_res=256)), (40, 9010, 12, dict(k_res=4096)),
    (61, 1030, 16, dict(k_res=256, n_outlier_cols=24, v_out=4, k_out=4096)),
    (4101, 390, 3, dict(k_res=4096)), (9999, 202, 5, dict(k_res=256)), (8197, 66, 3, {}),
])
def test_gemv_activations_through_lds_and_short_blocks(gpu_lib, out_features, in_features, batch, more):
    """Rows of v = 6 vectors on the matrix cores: one to five blocks of rows a workgroup, the last of them short, activations through LDS from the rows on
    that each number of blocks takes, one and several passes of the waves, the last of them of part of a wave; rows of y that several
    workgroups share none of, by 8-byte stores and by single ones."""
    import torch
    L = s.make_layer(317, "short", out_features, in_features, 6, 4096, **more)
    dl = gpu_lib.DeviceLayer(L)
    x_np = s.make_activations(317, L, batch)
    ref = oracle.gemv(L, x_np)
    x = torch.from_numpy(x_np).cuda()
    for pad in (0, 3):
        y = torch.full((batch, out_features + pad), 7.0, dtype=torch.float16, device="cuda")
        gpu_lib.gemv(dl, x, out=y)
        torch.cuda.synchronize()
        _check_matmul(y[:, :out_features], ref, "pad %d" % pad)
        assert (y[:, out_features:] == 7.0).all()
    if "n_outlier_cols" not in more:
        second = s.make_layer(318, "second", 333, in_features, 6, 4096, **more)
        ya, yb = gpu_lib.gemv_multi([dl, gpu_lib.DeviceLayer(second)], x)
        torch.cuda.synchronize()
        _check_matmul(ya, ref, "first of two")
        _check_matmul(yb, oracle.gemv(second, x_np), "second of two")


@pytest.mark.parametrize("out_features,in_features,more,batch", [
    (37, 1300, {}, 4), (1501, 2018, {}, 3), (3001, 1030, dict(k_res=4096), 4), (95, 1282, dict(k_res=256), 1), (49, 2000, dict(k_res=4096, n_outlier_cols=24, v_out=4, k_out=4096), 2),
    (3100, 1500, {}, 8), (9605, 1300, {}, 2), (9700, 1160, dict(k_res=4096), 5), (71, 1345, dict(k_res=256, n_outlier_cols=10, v_out=4, k_out=4096), 7),
])
def test_gemv_down_folds(gpu_lib, monkeypatch, out_features, in_features, more, batch):
    """Vectors down the outputs, two and four folds of the columns in one instruction: blocks of eight and four streams, the last one short, and windows of
    which some folds lie past the columns, where they meet the next stream's indices: its entries, infinite ones, are that stream's alone."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "gemv=m")
    L = s.make_layer(323, "folds", out_features, in_features, 6, 4096, orientation=1, **more)
    L.codebook[1::2] = np.inf
    bits = np.unpackbits(L.idx, axis=1, bitorder="little")
    bits[:, 0 : L.vectors_per_row * 12 : 12] = 0
    bits[1, 0] = 1                                       # one odd index, the first of the second stream
    L.idx = np.packbits(bits, axis=1, bitorder="little")
    pitch = (in_features + 7) // 8 * 8 + 8
    x_np = s.make_activations(323, L, batch)
    x = torch.full((batch, pitch), float("nan"), dtype=torch.float16, device="cuda")
    x[:, :in_features] = torch.from_numpy(x_np)
    dl, second = gpu_lib.DeviceLayer(L), s.make_layer(324, "second", 100, in_features, 6, 4096, orientation=1, **more)
    rows = np.r_[0:6, 12:out_features]
    ref = oracle.gemv(L, x_np)[:, rows]
    y = gpu_lib.gemv(dl, x[:, :in_features])
    ya, yb = gpu_lib.gemv_multi([dl, gpu_lib.DeviceLayer(second)], x[:, :in_features])
    torch.cuda.synchronize()
    for what, one in (("alone", y), ("first of two", ya)):
        assert not torch.isfinite(one[:, 6:12]).any()
        _check_matmul(one[:, rows], ref, what)
    _check_matmul(yb, oracle.gemv(second, x_np), "second of two")


@pytest.mark.parametrize("out_features,in_features,v,k,more,orientation,batch", [
    (700, 900, 8, 65536, {}, 1, 3), (701, 333, 8, 65536, {}, 1, 8), (130, 10001, 8, 65536, {}, 0, 4), (1001, 3205, 8, 65536, {}, 0, 7),
    (301, 1700, 12, 4096, dict(k_res=4096), 1, 4), (301, 505, 12, 4096, dict(k_res=4096, n_outlier_cols=24, v_out=4, k_out=4096), 1, 6),
    (77, 9509, 12, 4096, dict(k_res=4096), 0, 2), (900, 3300, 12, 4096, dict(k_res=4096, n_outlier_cols=40, v_out=4, k_out=4096), 0, 5),
    (131, 4099, 4, 256, {}, 1, 4), (2003, 700, 4, 256, {}, 1, 8), (130, 3209, 4, 256, {}, 0, 4), (1003, 6001, 4, 256, {}, 0, 8),
    (515, 3900, 2, 16, {}, 1, 1), (3001, 1001, 2, 16, {}, 1, 8), (333, 1035, 2, 16, {}, 0, 3),
    (131, 4099, 6, 256, {}, 1, 4), (131, 777, 6, 256, {}, 1, 8), (1002, 3461, 6, 256, {}, 0, 4),
])
def test_gemv_rows_folds(gpu_lib, monkeypatch, out_features, in_features, v, k, more, orientation, batch):
    """Two and four folds of the columns, with and without a workspace: short last blocks, folds that lie past the columns, outlier columns of several folds,
    rows followed by what is no number."""
    import torch
    monkeypatch.setenv("VQ_SWITCHES", "rows=1")
    L = s.make_layer(325, "folds", out_features, in_features, v, k, orientation=orientation, **more)
    pitch = (in_features + 7) // 8 * 8 + 8
    x_np = s.make_activations(325, L, batch)
    x = torch.full((batch, pitch), float("nan"), dtype=torch.float16, device="cuda")
    x[:, :in_features] = torch.from_numpy(x_np)
    dl = gpu_lib.DeviceLayer(L)
    ref = oracle.gemv(L, x_np)
    for workspace in (torch.empty(0, dtype=torch.uint8, device="cuda"), "fast"):
        y = gpu_lib.gemv(dl, x[:, :in_features], workspace=workspace)
        torch.cuda.synchronize()
        _check_matmul(y, ref, "workspace %s" % (workspace if isinstance(workspace, str) else None))
