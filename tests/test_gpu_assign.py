"""GPU parity of vq_assign (nearest-centroid assignment, Eq. 2 / residual stage of Sec. 3.2.2) through the C ABI:
the packed index streams bit for bit against the oracle's indices packed by the input generator's packer."""
import numpy as np
import pytest

import oracle
import vq_synth as s

pytestmark = pytest.mark.gpu

# rows, cols, v, k: ragged last vectors, several lanes' segments per row, partly filled workgroups, a table walked in
# LDS chunks (k = 65536), k not a power of two, cols < v
CASES = {
    "v6_k4096_ragged": (70, 391, 6, 4096),
    "v6_k256_exact": (256, 384, 6, 256),
    "v8_k65536_chunks": (33, 520, 8, 65536),
    "v4_k4096": (50, 1200, 4, 4096),
    "v5_k37": (37, 203, 5, 37),
    "v1_k2": (9, 77, 1, 2),
    "v16_k300": (33, 530, 16, 300),
    "v12_k4096": (20, 600, 12, 4096),
    "v6_k3000_many_rows": (3000, 390, 6, 3000),
    "one_short_vector": (5, 4, 6, 64),
    "v7_long_rows": (3, 9000, 7, 512),
}


def _inputs(name, with_base):
    rows, cols, v, k = CASES[name]
    seed = 7000 + list(CASES).index(name)
    ld = cols + 5
    W = s.to_fp16(s.normal(seed, rows * ld, 0.02)).reshape(rows, ld)
    C = s.to_fp16(s.normal(seed + 100, k * v, 0.02)).reshape(k, v)
    B = s.to_fp16(s.normal(seed + 200, rows * ld, 0.015)).reshape(rows, ld) if with_base else None
    return W, C, B, cols


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("with_base", [False, True])
def test_assign_bit_exact(gpu_lib, name, with_base):
    import torch
    W, C, B, cols = _inputs(name, with_base)
    k, v = C.shape
    idx = gpu_lib.assign(torch.from_numpy(W).cuda(), torch.from_numpy(C).cuda(),
                         base=torch.from_numpy(B).cuda() if with_base else None, cols=cols)
    torch.cuda.synchronize()
    want = oracle.assign(W, C, base=B, cols=cols)
    bits = oracle.index_bits(k)
    packed = s.pack_indices(want, bits, idx.shape[1])
    got = idx.cpu().numpy()
    if not np.array_equal(got, packed):
        mine = np.stack([oracle.unpack_row(got[o], bits, want.shape[1]) for o in range(got.shape[0])])
        bad = np.argwhere(mine != want)
        raise AssertionError("%s: %d of %d indices differ, first at %s: %d vs %d" %
                             (name, len(bad), want.size, bad[0], mine[tuple(bad[0])], want[tuple(bad[0])]))


def test_assign_leaves_the_rest_of_the_stride_alone(gpu_lib):
    import torch
    W, C, _, cols = _inputs("v6_k4096_ragged", False)
    P = -(-cols // 6)
    used = -(-P * 12 // 32) * 4
    stride = (used + 15) // 16 * 16 + 32
    idx = torch.full((W.shape[0], stride), 0xAB, dtype=torch.uint8, device="cuda")
    Wd, Cd = torch.from_numpy(W).cuda(), torch.from_numpy(C).cuda()
    rc = gpu_lib.vq_assign(Wd.data_ptr(), None, W.shape[1], W.shape[0], cols, Cd.data_ptr(), 6, 4096, idx.data_ptr(), stride,
                           torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0
    got = idx.cpu().numpy()
    assert (got[:, used:] == 0xAB).all()
    assert np.array_equal(got[:, :used], s.pack_indices(oracle.assign(W, C, cols=cols), 12, used))


def test_encode_then_decode_on_the_gpu(gpu_lib):
    """Two stages (Sec. 3.2.2) on the device, then vq_dequant: the oracle restores the same matrix from the same streams,
    and the second stage lowers the error."""
    import torch
    L = s.make_layer(7100, "enc", 64, 600, 6, 4096, k_res=256, with_scale=False, with_bias=False)
    W = s.to_fp16(s.normal(7101, 64 * 600, 0.02)).reshape(64, 600)
    Wd, Cd, Crd = (torch.from_numpy(a).cuda() for a in (W, L.codebook, L.codebook_res))
    idx = gpu_lib.assign(Wd, Cd)
    L.idx = idx.cpu().numpy()
    plain = s.VQLayer("stage1", 64, 600, 6, 4096)
    plain.codebook, plain.idx = L.codebook, L.idx
    stage1 = gpu_lib.dequant(gpu_lib.DeviceLayer(plain))
    idx_res = gpu_lib.assign(Wd, Crd, base=stage1)
    L.idx_res = idx_res.cpu().numpy()
    both = gpu_lib.dequant(gpu_lib.DeviceLayer(L))
    torch.cuda.synchronize()
    assert np.array_equal(both.cpu().numpy().view(np.uint16), oracle.dequant(L).view(np.uint16))
    e1 = ((W.astype(np.float64) - stage1.cpu().numpy().astype(np.float64)) ** 2).sum()
    e2 = ((W.astype(np.float64) - both.cpu().numpy().astype(np.float64)) ** 2).sum()
    assert e2 < e1


def test_assign_at_the_headline_size_on_sampled_rows(gpu_lib):
    """The 11008 x 4096 layer against its own 4096 x 6 table: every row on the GPU, sampled rows through the oracle."""
    import torch
    _, L = next(s.config_layers(1))
    W = s.to_fp16(s.normal(7200, L.out_features * L.in_features, 0.02)).reshape(L.out_features, L.in_features)
    idx = gpu_lib.assign(torch.from_numpy(W).cuda(), torch.from_numpy(L.codebook).cuda())
    torch.cuda.synchronize()
    rows = [0, 1, 4095, 7777, 11006, 11007]
    want = oracle.assign(W[rows], L.codebook)
    assert np.array_equal(idx.cpu().numpy()[rows], s.pack_indices(want, 12, idx.shape[1]))


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("with_base", [False, True])
def test_assign_down_bit_exact(gpu_lib, name, with_base):
    """The paper's own vectors (v consecutive rows of a column): index streams per block of rows, bit for bit."""
    import torch
    W, C, B, cols = _inputs(name, with_base)
    k, v = C.shape
    idx = gpu_lib.assign(torch.from_numpy(W).cuda(), torch.from_numpy(C).cuda(),
                         base=torch.from_numpy(B).cuda() if with_base else None, cols=cols, orientation=1)
    torch.cuda.synchronize()
    want = oracle.assign(W, C, base=B, cols=cols, orientation=1)
    assert idx.shape[0] == want.shape[0] == -(-W.shape[0] // v)
    assert np.array_equal(idx.cpu().numpy(), s.pack_indices(want, oracle.index_bits(k), idx.shape[1])), name


def test_encode_then_decode_in_the_papers_orientation(gpu_lib):
    import torch
    L = s.make_layer(7300, "enc_down", 70, 600, 6, 4096, with_scale=False, with_bias=False, orientation=1)
    W = s.to_fp16(s.normal(7301, 70 * 600, 0.02)).reshape(70, 600)
    idx = gpu_lib.assign(torch.from_numpy(W).cuda(), torch.from_numpy(L.codebook).cuda(), orientation=1)
    L.idx = idx.cpu().numpy()
    What = gpu_lib.dequant(gpu_lib.DeviceLayer(L))
    torch.cuda.synchronize()
    assert np.array_equal(What.cpu().numpy().view(np.uint16), oracle.dequant(L).view(np.uint16))
    # every restored vector is the nearest centroid of its block of rows: re-encoding returns the same streams
    again = gpu_lib.assign(What, torch.from_numpy(L.codebook).cuda(), orientation=1)
    torch.cuda.synchronize()
    assert torch.equal(again, idx)


# rows, cols, v, k, base, values: the matrix-core screening at its edges -- one block of 32 centroids more or less, the last
# chunk of a table, the vector lengths at which operands change their layout, both tile counts a wave takes, and values that
# its rounding bounds have to hold for
SCREEN = {
    "k63_vector_alus": (40, 600, 6, 63, False, "normal"),
    "k64": (40, 600, 6, 64, False, "normal"),
    "k65_one_row_past_a_block": (40, 600, 6, 65, True, "normal"),
    "k4095": (20, 606, 6, 4095, False, "normal"),
    "k4097_second_chunk_of_one": (9, 603, 6, 4097, False, "normal"),
    "v7_base_two_instructions": (33, 700, 7, 300, True, "normal"),
    "v13_base_longest": (20, 650, 13, 1000, True, "normal"),
    "v14_vector_alus": (20, 650, 14, 300, False, "normal"),
    "many_vectors": (1100, 1000, 2, 64, False, "normal"),
    "many_vectors_base_v8": (2100, 1003, 8, 64, True, "normal"),
    "equal_entries": (60, 600, 6, 512, False, "ties"),
    "equal_entries_base": (60, 600, 6, 512, True, "ties"),
    "nearly_equal_entries": (60, 600, 6, 512, False, "close"),
    "nearly_equal_entries_base_v12": (60, 600, 12, 512, True, "close"),
    "nearly_equal_entries_over_magnitudes": (60, 600, 12, 512, True, "spread close"),
    "subnormal_values": (40, 600, 6, 256, False, "tiny"),
    "subnormal_values_base": (40, 600, 8, 256, True, "tiny"),
    "values_near_the_top": (40, 600, 6, 256, False, "huge"),
    "spread_over_magnitudes": (60, 600, 6, 1024, False, "spread"),
    "spread_over_magnitudes_base": (60, 600, 12, 1024, True, "spread"),
}


@pytest.mark.parametrize("name", list(SCREEN))
def test_assign_screening_edges(gpu_lib, name):
    import torch
    rows, cols, v, k, with_base, values = SCREEN[name]
    seed = 7300 + list(SCREEN).index(name)
    scale = {"tiny": 2e-6, "huge": 9000.0}.get(values, 0.02)
    W, C, B = (s.normal(seed + 100 * i, n, scale) for i, n in enumerate((rows * cols, k * v, rows * cols)))
    if "spread" in values:
        W, C, B = (a * np.exp(2.0 * s.normal(seed + 100 * i + 50, a.size, 1.0)) for i, a in enumerate((W, C, B)))
    W, C = s.to_fp16(W).reshape(rows, cols), s.to_fp16(C).reshape(k, v)
    if values == "ties":
        C[k // 2:] = C[: k - k // 2][::-1]
    if "close" in values:              # the second half differs from the first by one unit in the last place of one element
        C[k // 2:] = C[: k - k // 2]
        C[k // 2:, 0] = np.nextafter(C[k // 2:, 0], np.float16(1))
    B = s.to_fp16(B).reshape(rows, cols) if with_base else None
    for orientation in (0, 1):
        idx = gpu_lib.assign(torch.from_numpy(W).cuda(), torch.from_numpy(C).cuda(), base=torch.from_numpy(B).cuda() if with_base else None,
                             orientation=orientation)
        torch.cuda.synchronize()
        want = oracle.assign(W, C, base=B, orientation=orientation)
        assert np.array_equal(idx.cpu().numpy(), s.pack_indices(want, oracle.index_bits(k), idx.shape[1])), (name, orientation)


# v, k, base, values, table starts at an odd address: waves that hold two tiles of vectors (more than 131072 vectors), whose lanes look
# after one vector each, in blocks of 16 and (k >= 4096) 32 centroids, with tables of one chunk and of several, in both operand layouts
TWO_TILES = {
    "v6_k4096": (6, 4096, False, "normal", False),
    "v6_k4095_blocks_of_16": (6, 4095, False, "normal", False),
    "v6_k4097_second_chunk_of_one": (6, 4097, False, "normal", False),
    "v8_k8200_odd_table": (8, 8200, False, "normal", True),
    "v12_k4160_base": (12, 4160, True, "normal", False),
    "v1_k64": (1, 64, False, "normal", False),
    "v6_k64_base_odd_table": (6, 64, True, "normal", True),
    "v7_k100_base": (7, 100, True, "normal", False),
    "v9_k300": (9, 300, False, "normal", False),
    "v13_k4096_base": (13, 4096, True, "normal", False),
    "v6_k4096_ties": (6, 4096, True, "ties", False),
    "v12_k256_subnormal": (12, 256, False, "tiny", False),
    "v6_k256_not_finite": (6, 256, False, "not finite", False),
}


@pytest.mark.parametrize("name", list(TWO_TILES))
def test_assign_two_tiles_a_wave(gpu_lib, name):
    """Sampled rows (blocks of rows) of a large matrix, bit for bit: an index has no tolerance."""
    import torch
    v, k, with_base, values, odd = TWO_TILES[name]
    rows, cols, seed = 905, 150 * v + (1 if v > 1 else 0), 7500 + list(TWO_TILES).index(name)
    scale = 2e-6 if values == "tiny" else 0.02
    W, C, B = (s.to_fp16(s.normal(seed + 100 * i, n, scale)) for i, n in enumerate((rows * cols, k * v, rows * cols)))
    W, C, B = W.reshape(rows, cols), C.reshape(k, v), B.reshape(rows, cols) if with_base else None
    if values == "ties":
        C[k // 2:] = C[: k - k // 2][::-1]
    if values == "not finite":                                 # (a vector without a distance below infinity takes the first entry)
        C[5, 2], W[0, 7], W[450, 100], W[904, 200] = np.inf, np.inf, np.nan, -np.inf
    room = torch.zeros(k * v + 1, dtype=torch.float16, device="cuda")
    Cd = room[1:] if odd else room[:-1]
    Cd = Cd.view(k, v).copy_(torch.from_numpy(C))
    Wd, Bd = torch.from_numpy(W).cuda(), torch.from_numpy(B).cuda() if with_base else None
    for orientation in (0, 1):
        idx = gpu_lib.assign(Wd, Cd, base=Bd, orientation=orientation)
        torch.cuda.synchronize()
        got = idx.cpu().numpy()
        for at in (0, 450, 904) if orientation == 0 else (0, 450 // v, 904 // v):
            part = slice(at, at + 1) if orientation == 0 else slice(at * v, min(rows, at * v + v))
            with np.errstate(all="ignore"):
                want = oracle.assign(W[part], C, base=B[part] if with_base else None, orientation=orientation)
            assert np.array_equal(got[at:at + 1], s.pack_indices(want, oracle.index_bits(k), idx.shape[1])), (name, orientation, at)


@pytest.mark.parametrize("v,k", [(3, 5000), (5, 4097), (6, 4300), (8, 8192), (12, 4700), (13, 5000), (6, 4096), (6, 130), (8, 384)])
@pytest.mark.parametrize("with_base", [False, True])
def test_assign_of_cut_off_vectors_of_one_element(gpu_lib, v, k, with_base):
    """Among scalars many entries are about as near, so that every distance is computed: tables whose shares do not fill the steps of that
    loop, elements loaded one by one and in whole entries, entries twice in the table."""
    import torch
    rows, cols = 3 * v + 1, 40 * v + 1
    W, C, B = (s.to_fp16(s.normal(7700 + 10 * v + i, n, 0.02)) for i, n in enumerate((rows * cols, k * v, rows * cols)))
    W, C, B = W.reshape(rows, cols), C.reshape(k, v), B.reshape(rows, cols) if with_base else None
    C[k - 20:] = C[:20]
    for orientation in (0, 1):
        idx = gpu_lib.assign(torch.from_numpy(W).cuda(), torch.from_numpy(C).cuda(), base=torch.from_numpy(B).cuda() if with_base else None,
                             orientation=orientation)
        torch.cuda.synchronize()
        want = oracle.assign(W, C, base=B, orientation=orientation)
        assert np.array_equal(idx.cpu().numpy(), s.pack_indices(want, oracle.index_bits(k), idx.shape[1])), (v, k, orientation)


@pytest.mark.parametrize("rows,cols,v,k", [(37, 390, 6, 4096), (13, 3, 6, 300), (700, 4096, 6, 256), (19, 77, 2, 16), (9, 200, 16, 300), (21, 130, 8, 65536), (5, 128, 4, 256)])
@pytest.mark.parametrize("orientation", [0, 1])
def test_assign_fills_the_whole_stride_of_a_buffer_of_its_own(gpu_lib, rows, cols, v, k, orientation):
    """Streams of no, one, two and three dwords of padding, cut-off vectors whose dword two launches share, each of the three kernels; the buffer is one
    that the allocator hands out again."""
    import torch
    W = torch.from_numpy(s.to_fp16(s.normal(7300, rows * cols, 0.02)).reshape(rows, cols)).cuda()
    C = torch.from_numpy(s.to_fp16(s.normal(7301, k * v, 0.02)).reshape(k, v)).cuda()
    want = gpu_lib.assign(W, C, cols=cols, orientation=orientation).cpu()
    used = torch.full(want.shape, 0xFF, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    del used
    got = gpu_lib.assign(W, C, orientation=orientation)
    torch.cuda.synchronize()
    assert torch.equal(got.cpu(), want)
